// Softmax attention for gfx950 on 16-bit tensors (element type E: bf16, or f16 = IEEE half) with fp32 accumulation: forward with an online softmax, and a
// deterministic two-kernel backward (no float atomics).  Causal (decoder: position i sees j <= i) or unmasked
// (encoder: every position sees its whole sequence; only keys past the end of a ragged last tile are masked).
//
// All three kernels are built the same way.  A wavefront owns 32-position blocks of one (sequence, head) and
// lane l owns position l%32 of a block, so every softmax statistic and row sum is lane-local (only the two
// lane halves of a position exchange a value, with one 32-lane swap).  That works because the score tile is
// produced transposed - the tile that is streamed through LDS (keys in the forward and the dQ kernel, queries
// in the dK/dV kernel) is the MFMA's first operand - and the v_mfma_f32_32x32x16 result layout (lane = column,
// 4 consecutive rows per register group) is, after conversion to bf16, directly a valid second operand for the
// next MFMA: its K index is a permutation of the streamed positions, and the first operand of that MFMA is
// read from the streamed tile with the same permutation by the transposing LDS read.  Tiles go from global
// memory straight into LDS (buffer_load ... lds), as stored; nothing is transposed in registers or copied.
//
//   forward      S^T = K Q^T ; P^T = softmax ; O^T += V^T P^T              streams K, V
//   dQ kernel    S^T = K Q^T ; dP^T = V dO^T ; dS^T ; dQ^T += K^T dS^T      streams K, V
//   dK/dV kernel S = Q K^T ; dP = dO V^T ; dV^T += dO^T P ; dK^T += Q^T dS  streams Q, dO
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <type_traits>

#include "attention16.h"
#include "kernels.h"

// The forward kernel's restart loop keeps one requested unroll from being applied in the optimizer's loop pass
// (everything is unrolled later: no array ends up indexed at run time, no scratch memory is used).
#pragma clang diagnostic ignored "-Wpass-failed"

namespace lga {

namespace {

// Tiles that are filled by DMA keep their rows at a padded pitch instead of an XOR swizzle, so that every
// MFMA operand address is one per-lane base plus a compile-time offset (swizzled addresses each need
// their own register, and the compiler keeps them all live across the key loop).
//   pitch_rd<DH>  rows read with ds_read_b128 (lane = row): 16 bytes of padding rotate the banks row by row
//   pitch_tr<DH>  rows read with the transposing ds_read_b64_tr_b16, one pass of which covers 4 consecutive
//                 rows x 64 bytes: power-of-two row sizes get 64 bytes of padding, the others already stagger
template <int DH> constexpr int pitch_rd() { return DH + 8; }
template <int DH> constexpr int pitch_tr() { return (DH == 64 || DH == 128) ? DH + 32 : DH; }

// Per-lane part of the address of a transposed operand read from a NATURAL tile [position][pitch]:
// within each group of 16 lanes, lane i passes the address of 4 consecutive values and receives, with lane
// i pointing at (row i/4, columns 4 (i%4) ..+3), column i of rows 0..3.
template <int PITCH> __device__ __forceinline__ int tr_lane_off(int lane) {
    const int i = lane & 15;
    return (4 * (lane >> 5) + (i >> 2)) * PITCH + 16 * ((lane >> 4) & 1) + 4 * (i & 3);
}
// MFMA first operand "row n = 32 c + lrow of the transposed tile, k element e <-> streamed position
// 16 kk + 8 (e/4) + 4 half + e%4" (the permutation that matches a 32x32 MFMA result used as second operand).
// base = tile + tr_lane_off(lane).
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
template <int PITCH, class E> __device__ __forceinline__ x8<E> frag_nat_tr(const E *base, int c, int kk) {
    // Issued as inline assembly: the compiler makes the builtin form wait for every outstanding
    // direct-to-LDS load first (it cannot tell which LDS bytes those write), which would serialise the
    // tile prefetch.  The price: the compiler does not count these reads in lgkmcnt, so wait_tr_reads()
    // must stand between them and their first use.
    const uint32_t addr = (uint32_t)(uintptr_t)base;        // low 32 bits of a generic LDS pointer = LDS address
    u32x2 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "i"((16 * kk * PITCH + 32 * c) * 2));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "i"(((16 * kk + 8) * PITCH + 32 * c) * 2));
    const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(x8<E>, v);
}
// DMA of a ROWS x DH tile (global row pitch gp2 bytes) into LDS rows of PITCH elements.  The tile is
// ROWS * (PITCH / 8) slots of 16 bytes, filled 64 at a time; instruction j covers slots [64 j, 64 j + 64).
// Slots that are padding get the poison offset, and rows at or beyond nvalid lie outside the buffer's range (zeros either way).
template <int ROWS, int DH, int PITCH> struct TileDma {
    static constexpr int SLOTS = PITCH / 8;                 // per row
    static constexpr int NI = (ROWS * SLOTS + 63) / 64;     // instructions that carry data
    static constexpr int NJ = (NI + 3) / 4;                 // per wavefront (4 wavefronts): every wavefront issues NJ,
                                                            // so that "all but the newest tile" is one vmcnt value
    static constexpr int ELEMS = NJ * 4 * 512;              // LDS elements to reserve: 4 NJ instructions of 1 KB
    int off[NJ], pitch2, row2;
    // dh <= DH: the head size in memory; columns from dh on are padding like the rest of the pitch
    __device__ __forceinline__ void init(int wave, int lane, int gp2, int dh) {
        pitch2 = gp2;
        row2 = dh * 2;
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const int slot = (i * 4 + wave) * 64 + lane, r = slot / SLOTS, pc = slot % SLOTS;
            off[i] = pc < dh / 8 && r < ROWS ? r * gp2 + (pc << 4) : kBufPoison;
        }
    }
    // src, dst: tiles of 16-bit elements of either format
    __device__ __forceinline__ void issue(const void *src, void *dst, int nvalid, int wave) const {
        const int rows = min(nvalid, ROWS);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src, rows > 0 ? (rows - 1) * pitch2 + row2 : 0);
#pragma unroll
        for (int i = 0; i < NJ; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(static_cast<char *>(dst) + (i * 4 + wave) * 1024), 16, off[i], 0, 0, 0);
    }
};

// S^T tiles live in ordinary registers: the exponentials read them, and the builtin's results would be in accumulation registers, a
// move apart from any other instruction.  Two such products in a row on one tile are separated by what stands between the
// statements; a result is read only behind at least two other matrix instructions, or the wait states below.
template <class E> __device__ __forceinline__ void mfma_scores(x8<E> a, x8<E> b, f32x16 &c, bool first);
#define LGA_MFMA_SCORES(E, name)                                                                                                              \
    template <> __device__ __forceinline__ void mfma_scores<E>(x8<E> a, x8<E> b, f32x16 &c, bool first) {                                     \
        const i32x4 ai = __builtin_bit_cast(i32x4, a), bi = __builtin_bit_cast(i32x4, b);                                                     \
        if (first) asm volatile(name " %0, %1, %2, 0" : "=&v"(c) : "v"(ai), "v"(bi));                                                         \
        else asm volatile(name " %0, %1, %2, %0" : "+v"(c) : "v"(ai), "v"(bi));                                                               \
    }
LGA_MFMA_SCORES(bf16, "v_mfma_f32_32x32x16_bf16")
LGA_MFMA_SCORES(f16, "v_mfma_f32_32x32x16_f16")
#undef LGA_MFMA_SCORES
// s_waitcnt immediate: all LDS reads returned, at most n loads in flight
constexpr int wait_loads(int n) { return 0x0070 | (n & 15) | (n >> 4 << 14); }

// ============================================================================================
// Forward.  One workgroup per (sequence, head, block of 128 U queries), see block_of(); rank 0 = the last block.
//
// A wavefront owns 32 U queries as U sub-blocks of 32, so every K and V operand it reads from LDS feeds U MFMAs.
// Key tiles of 64 (K and V as stored, rows of DH) stream from global memory straight into one of three
// LDS stages; one barrier per tile publishes it.  V^T operands come from the natural V tile through the
// transposing LDS read.
template <int DH, int U, class E>
__global__ __launch_bounds__(256, 1) void attn_fwd_kernel(const E *__restrict__ qkv, E *__restrict__ out,
                                                       float *__restrict__ lse, AttnShape sh) {
    constexpr int KT = 64;                 // keys per streamed tile
    constexpr int NK = DH / 16, NC = DH / 32;
    constexpr int NU = 2 * U;              // units of 32 keys x 32 queries per tile and wavefront
    constexpr int QW = 32 * U;             // queries per wavefront
    constexpr int PK = pitch_rd<DH>(), PV = pitch_tr<DH>();    // LDS row pitches of the K and V tiles
    typedef TileDma<KT, DH, PK> DmaK;
    typedef TileDma<KT, DH, PV> DmaV;
    constexpr int STAGE = DmaK::ELEMS + DmaV::ELEMS;            // elements per stage: K tile, then V tile
    constexpr int NSTAGE = 3, LOADS = DmaK::NJ + DmaV::NJ;
    // tiles requested ahead of the one that is published: with U = 2 all reads of the tile before it are done by then
    constexpr int AHEAD = U == 2 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);

    const int qblocks = (sh.s + 4 * QW - 1) / (4 * QW);
    int bh, rank;
    block_of(sh, qblocks, bh, rank);
    const int qb = qblocks - 1 - rank;
    const int h = bh % sh.heads, b = bh / sh.heads;
    const int dh = sh.dh;                           // head size in memory: a multiple of 8, DH - 24 <= dh <= DH
    const int d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const E *seq = qkv + (size_t)b * sh.s * pitch + (size_t)h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, half = lane >> 5;
    const int qw0 = (qb * 4 + wave) * QW;           // first query of this wavefront
    const bool causal = sh.causal != 0;
    // Last visible key of sub-block u's lanes = vis_u(u) + vis_lane + 4 half: the query itself, or the end of the sequence.
    const int vis_lane = (causal ? lrow : 0) - 4 * half;
    auto vis_u = [&](int u) { return causal ? qw0 + 32 * u : sh.s - 1; };

    x8<E> qf[U][NK];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = qw0 + 32 * u + lrow;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) qf[u][ks] = frag_global(seq + (size_t)q * pitch, ks, half, q < sh.s, dh);
    }
    // Softmax reference per query, in the log2 domain.  It is FIXED once the query's first 32 keys are seen
    // (p = 2^(score - m_ref) is then exact up to a common factor that the final division removes), so the
    // output accumulators are never rescaled - they live in accumulation registers that only MFMAs touch.
    // A probability far above 1 must still fit the format P is rounded to for the second product - bf16 reaches
    // as far as fp32, IEEE half ends at 65504 - and a probability is never larger than its row's running sum.  So a
    // lane whose sum reaches kSumLimit makes the whole workgroup start over, with its query's reference raised
    // by what its sum asks for (to a sum of about 2^kTargetLog2), or by kRefStep if the sum overflowed fp32.  The
    // other queries keep theirs, and come to the same sums again: a result does not depend on which queries share a workgroup.
    // On ordinary activations bf16 never restarts; half precision does when the keys beyond the first 32 score
    // some 15 (log2 units) higher, which wide layers do reach.  The number of attempts is bounded, so that scores
    // that are infinite or not numbers end in a non-finite output instead of an endless loop.
    constexpr float kSumLimit = std::is_same<E, f16>::value ? 6.0e4f : 1.0e30f;
    constexpr float kRefStep = 64.f, kTargetLog2 = 8.f;
    // Half precision starts 6 units above the best of the first 32 scores: its probabilities then have 22 units of
    // headroom instead of 16, which at the score spread of wide layers saves most restarts, and keys more than 8
    // units below that best score become denormal (still exact to 2^-25 of the row's largest terms).
    constexpr float kRefBias = std::is_same<E, f16>::value ? 6.f : 0.f;
    constexpr int kMaxAttempts = 6;
    f32x16 oacc[U][NC];
    float m_ref[U], l_run[U];
    const float c2 = rsqrtf((float)dh) * kLog2e;
    // Plain (not volatile) so that the compiler keeps it an LDS access, which waits for no global load; the
    // barriers' memory clobbers make every read after them a fresh one.
    __shared__ int restart_flag[1];
    if (threadIdx.x == 0) restart_flag[0] = 0;

    // ---- tile loader ------------------------------------------------------------------------
    DmaK dk;
    DmaV dv;
    dk.init(wave, lane, (int)(pitch * 2), dh);
    dv.init(wave, lane, (int)(pitch * 2), dh);
    const int kend = causal ? min(sh.s, (qb + 1) * 4 * QW) : sh.s;  // keys needed by this block: [0, kend)
    const int ntiles = (kend + KT - 1) / KT;
    auto dma_tile = [&](int t, int stage) __attribute__((always_inline)) {
        if (t >= ntiles) return;
        E *Ks = lds + stage * STAGE, *Vs = Ks + DmaK::ELEMS;
        dk.issue(seq + (size_t)t * KT * pitch + d, Ks, sh.s - t * KT, wave);
        dv.issue(seq + (size_t)t * KT * pitch + 2 * d, Vs, sh.s - t * KT, wave);
    };
    const int koff = lrow * PK + 8 * half;              // per-lane part of a K operand's address
    const int voff = tr_lane_off<PV>(lane);             // ... and of a V^T operand's

    // ---- the pipeline over units ----------------------------------------------------------------
    // A unit is 32 keys x 32 queries, n = U kb + u of a tile: S = NK MFMAs, the exponentials (VALU), P V = 2 NC MFMAs.  A phase per unit:
    //     MFMA   P V of the unit before it, then S of the unit behind it
    //     VALU   its exponentials
    // across tiles, a share of the exponentials behind every MFMA: a wavefront issues in order, and two MFMAs in a row keep the
    // VALU waiting for the first.  One set of K and one of V^T operand registers: each is read again, for the next key
    // block, right behind the last MFMA that uses it, so that a read is half a phase and more ahead of its use.  The issue
    // order is pinned (sched_barrier).  Units of one tile only, groups of 2 to 4 MFMAs between groups of exponentials and scores in
    // accumulation registers took 4590 cycles a tile of 64 queries x 64 keys x 128, of which 2048 are MFMAs; now 3700, at a lower clock: the
    // board's power binds (8100 x 16 heads x 128: 348 -> 302 us, 1024 x 384 x 64: 114 -> 103, 2048 x 32 x 128 unmasked 106 -> 94).
    x8<E> kf[NK], vf[2 * NC];
    u32x4 pf[2][2];                                // P operands of a unit and of the one before it
    f32x16 st[2];                                  // scores of a unit and of the one behind it
    float pr[16];
    constexpr int NM = NK + 2 * NC;                // MFMAs of a phase
    constexpr int FIRST = NM >= 8 ? 2 : 1;         // the exponentials begin behind this many, when the scores have left the matrix pipe
    auto read_k = [&](const E *Ks, int kb, int ks) __attribute__((always_inline)) {
        kf[ks] = *reinterpret_cast<const x8<E> *>(Ks + kb * 32 * PK + 16 * ks);
    };
    auto element = [&](int n, int e, int k0, bool masked) __attribute__((always_inline)) {
        const int u = n % U;
        float p = __builtin_amdgcn_exp2f(fmaf(st[n & 1][e], c2, -m_ref[u]));
        // key of score register r is visible iff 8 (r / 4) + r % 4 <= qrel
        if (masked && 8 * (e >> 2) + (e & 3) > vis_u(u) + vis_lane - (k0 + 32 * (n / U))) p = 0.f;
        pr[e] = p;
    };
    auto finish = [&](int n, int e) __attribute__((always_inline)) {       // into the row's sum and, in pairs, the operand
        l_run[n % U] += pr[e];
        if (e & 1) {
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            typedef E x2 __attribute__((ext_vector_type(2)));
            const f32x2 two = {pr[e - 1], pr[e]};
            pf[n & 1][e >> 3][(e >> 1) & 3] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, x2));
        }
    };
    // wait for this wavefront's part of the oldest tile in flight (`newer`: a younger one is in flight too),
    // then a bare s_barrier - a __syncthreads() fence would wait for the younger tile as well.  After it tile t is
    // published, and everyone's reads before it have returned: tile t + AHEAD may overwrite what they read.
    auto publish = [&](int t, int stage) __attribute__((always_inline)) {
        if (t >= ntiles) return;
        if (t + AHEAD - 1 < ntiles && AHEAD > 1)
            __builtin_amdgcn_s_waitcnt(wait_loads((AHEAD - 1) * LOADS));
        else
            __builtin_amdgcn_s_waitcnt(wait_loads(0));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        dma_tile(t + AHEAD, stage + AHEAD >= NSTAGE ? stage + AHEAD - NSTAGE : stage + AHEAD);
    };
    // Phase n of tile t, in stage `stage`.  LAST: the wavefront's last tile (masked, no scores of a tile behind it).
    auto phase = [&](auto n_c, auto last_c, int t, int stage) __attribute__((always_inline)) {
        constexpr int n = decltype(n_c)::value;
        constexpr bool LAST = decltype(last_c)::value;
        constexpr int u2 = U == 1 ? 0 : (n + 1) & 1;                    // sub-block of the units before and behind
        constexpr bool kScores = !LAST || n + 1 < NU;                   // of the unit behind
        constexpr bool kNextK = u2 == U - 1 && (!LAST || n + 2 < NU);   // K operands of unit n + 2 to be read
        constexpr bool kNextV = n % U == 0;                             // V^T operands of unit n to be read
        constexpr bool kPublish = n == NU - 2;                          // before the first reads of tile t + 1
        constexpr int kPubAt = NK >= 8 ? 1 : 0;                         // behind this score MFMA: the V^T reads just before it return meanwhile
        const E *Vs = lds + stage * STAGE + DmaK::ELEMS + voff;
        const int nstage = stage == NSTAGE - 1 ? 0 : stage + 1;
        const E *Kn = lds + (n + 2 < NU ? stage : nstage) * STAGE + koff;
        const int k0 = t * KT;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            if (i < 2 * NC) {
                oacc[u2][i % NC] = MFMA(vf[i], __builtin_bit_cast(x8<E>, pf[(n + 1) & 1][i / NC]), oacc[u2][i % NC]);
                if (kNextV) vf[i] = frag_nat_tr<PV>(Vs, i % NC, 2 * (n / U) + i / NC);
            } else if (kScores) {
                const int ks = i - 2 * NC;
                mfma_scores<E>(kf[ks], qf[u2][ks], st[(n + 1) & 1], ks == 0);
                if (kPublish && ks == kPubAt) {
                    __builtin_amdgcn_sched_barrier(0);
                    publish(t + 1, nstage);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (kNextK) {
                    constexpr int from = kPublish ? kPubAt : 0;         // reads begin behind this MFMA and end with the last one
                    if (ks >= from) {
#pragma unroll
                        for (int r = (ks - from) * NK / (NK - from); r < (ks - from + 1) * NK / (NK - from); ++r) read_k(Kn, ((n + 2) / U) & 1, r);
                    }
                }
            }
            if (i >= FIRST) {
#pragma unroll
                for (int e = (i - FIRST) * 16 / (NM - FIRST); e < (i - FIRST + 1) * 16 / (NM - FIRST); ++e) {
                    element(n, e, k0, LAST);
                    if (e > 0) finish(n, e - 1);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        finish(n, 15);
        // (K reads issued behind the V^T reads may still be under way)
        if constexpr (kNextV) wait_tr_reads<kNextK ? NK : 0>(vf);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto tile = [&](auto last_c, int t, int stage) __attribute__((always_inline)) {
        phase(std::integral_constant<int, 0>{}, last_c, t, stage);
        phase(std::integral_constant<int, 1>{}, last_c, t, stage);
        if constexpr (NU == 4) {
            phase(std::integral_constant<int, 2>{}, last_c, t, stage);
            phase(std::integral_constant<int, 3>{}, last_c, t, stage);
        }
    };

    // This wavefront's tiles before its last one are fully visible to it; the last one is the diagonal one, or the ragged end of the sequence.
    const int nfull = causal ? min(qw0 / KT, ntiles - 1) : ntiles - 1;
    for (int attempt = 1;; ++attempt) {
        const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            l_run[u] = 0.f;
#pragma unroll
            for (int c = 0; c < NC; ++c) oacc[u][c] = zero16;
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) dma_tile(i, i);
        publish(0, 0);
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) read_k(lds + koff, 0, ks);
        if (attempt == 1) {
            // First attempt: the scores of each query's first 32 keys fix its softmax reference (key 0 is
            // visible to every query; for the first queries of the sequence these keys are partly masked).
#pragma unroll
            for (int u = 0; u < U; ++u) {
                f32x16 first = MFMA(kf[0], qf[u][0], zero16);
#pragma unroll
                for (int ks = 1; ks < NK; ++ks) first = MFMA(kf[ks], qf[u][ks], first);
                const int qrel = vis_u(u) + vis_lane;
                float raw = -INFINITY;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + (r & 3) <= qrel) raw = fmaxf(raw, first[r]);
                m_ref[u] = fmaxf(raw, __shfl_xor(raw, 32, 64)) * c2 + kRefBias;
            }
        }
        // into the pipeline: unit 0's scores, a product of zeros in place of the unit before it, K operands of unit 1
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) mfma_scores<E>(kf[ks], qf[0][ks], st[0], ks == 0);
        if constexpr (U == 1) {
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) read_k(lds + koff, 1, ks);
        }
#pragma unroll
        for (int i = 0; i < 2 * NC; ++i) vf[i] = __builtin_bit_cast(x8<E>, u32x4{0, 0, 0, 0});
        pf[1][0] = pf[1][1] = u32x4{0, 0, 0, 0};
        int stage = 0, t = 0;
        for (; t < nfull; ++t, stage = stage == NSTAGE - 1 ? 0 : stage + 1) tile(std::false_type{}, t, stage);
        tile(std::true_type{}, t, stage);
#pragma unroll
        for (int i = 0; i < 2 * NC; ++i)
            oacc[U - 1][i % NC] = MFMA(vf[i], __builtin_bit_cast(x8<E>, pf[1][i / NC]), oacc[U - 1][i % NC]);
        // other wavefronts' tiles behind this one's last
        for (t += 2, stage = (stage + 2) % NSTAGE; t < ntiles; ++t, stage = stage == NSTAGE - 1 ? 0 : stage + 1) publish(t, stage);
        // overflow guard: a sum this large means that some score was far above the reference (sums only grow, and keep what is not a number)
        bool over = false;
#pragma unroll
        for (int u = 0; u < U; ++u) over = over || !(l_run[u] < kSumLimit);
        if (__any(over)) restart_flag[0] = 1;
        __syncthreads();
        if (!restart_flag[0] || attempt == kMaxAttempts) break;
        // start over with larger references
        __syncthreads();
        if (threadIdx.x == 0) restart_flag[0] = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float other = __shfl_xor(l_run[u], 32, 64), l_tot = l_run[u] + other;      // both lanes of a query see the same sums
            if (!(l_run[u] < kSumLimit) || !(other < kSumLimit)) m_ref[u] += l_tot < 3.0e38f ? ceilf(__log2f(l_tot)) - kTargetLog2 : kRefStep;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = qw0 + 32 * u + lrow;
        const float l_tot = l_run[u] + __shfl_xor(l_run[u], 32, 64);
        if (q < sh.s) {
            const float inv = 1.0f / l_tot;
            E *orow = out + ((size_t)b * sh.s + q) * d + (size_t)h * dh;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    x4<E> o;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = (E)(oacc[u][c][4 * g + i] * inv);
                    if (c * 32 + 8 * g + 4 * half < dh) *reinterpret_cast<x4<E> *>(orow + c * 32 + 8 * g + 4 * half) = o;
                }
            if (half == 0) lse[((size_t)b * sh.heads + h) * sh.s + q] = fmaf(m_ref[u], kLn2, logf(l_tot));
        }
    }
}

// ============================================================================================
// delta of every row, from whole 16-byte pieces: a thread multiplies one piece of out and dout (both [tokens][heads * dh], so that
// consecutive (token, head) items are consecutive runs of dh elements), one thread per item adds its dh / 8 products in order.  Only where the
// dQ kernel cannot take delta itself because it would read O from memory that it writes dQ to (see delta_apart).
template <class E>
__global__ __launch_bounds__(256) void attn_delta_kernel(const E *out, const E *dout, float *delta, AttnShape sh, int items_per_block) {
    __shared__ float part[256];
    const int pieces = sh.dh / 8, tid = threadIdx.x;
    const size_t items = (size_t)sh.n_seq * sh.s * sh.heads, item0 = (size_t)blockIdx.x * items_per_block;
    float sum = 0.f;
    if (tid < items_per_block * pieces && item0 + tid / pieces < items) {
        const x8<E> o = *reinterpret_cast<const x8<E> *>(out + (item0 * pieces + tid) * 8);
        const x8<E> g = *reinterpret_cast<const x8<E> *>(dout + (item0 * pieces + tid) * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += (float)o[i] * (float)g[i];
    }
    part[tid] = sum;
    __syncthreads();
    if (tid < items_per_block && item0 + tid < items) {
        float all = 0.f;
        for (int c = 0; c < pieces; ++c) all += part[tid * pieces + c];
        const size_t item = item0 + tid, token = item / sh.heads;
        delta[((token / sh.s) * sh.heads + item % sh.heads) * sh.s + token % sh.s] = all;
    }
}

// ============================================================================================
// dQ.  One workgroup per (sequence, head, block of 128 queries), see block_of(); rank 0 = the last block.
//
// A wavefront owns 32 queries (Q and dO operands in registers); key tiles of 64 (K and V as stored) stream
// from global memory straight into one of two LDS stages while the other is multiplied, one barrier per
// tile.  K^T operands come from the natural K tile through the transposing LDS read.  Two workgroups per
// CU, so that one's MFMAs run under the other's VALU work - which needs tiles of DH elements per row, swizzled: with padded rows
// the two stages take 90 KB at DH = 128 and only one workgroup fits (16 heads x 8100 positions x 128, causal: 485 us; now 395, and no
// bank conflicts instead of a quarter of the LDS cycles; 384 x 1024 x 64: 121 -> 108).
// OWN: delta is this kernel's to make, from out; otherwise it is there already (a test of out in the kernel instead: 1 - 2 % at 64 channels).
template <int DH, int OCC, bool OWN, class E>
__global__ __launch_bounds__(256, OCC) void attn_bwd_dq_kernel(const E *__restrict__ qkv, const E *__restrict__ out,
                                                          const float *__restrict__ lse, float *__restrict__ delta,
                                                          const E *__restrict__ dout, E *__restrict__ dqkv,
                                                          AttnShape sh) {
    constexpr int KT = 64;
    constexpr int NK = DH / 16, NC = DH / 32;
    typedef TileDmaSw<KT, DH> Dma;
    constexpr int TILE = Dma::ELEMS, STAGE = 2 * TILE;          // K tile, then V tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);

    const int qblocks = (sh.s + 127) / 128;
    int bh, rank;
    block_of(sh, qblocks, bh, rank);
    const int qb = qblocks - 1 - rank;
    const int h = bh % sh.heads, b = bh / sh.heads;
    const int dh = sh.dh;                           // head size in memory, <= DH
    const int d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const E *seq = qkv + (size_t)b * sh.s * pitch + (size_t)h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, half = lane >> 5;
    const int qw0 = qb * 128 + wave * 32;
    const int q = qw0 + lrow;
    const bool qvalid = q < sh.s;

    Dma dma;                                                    // K and V rows have the same pitch
    dma.init(wave, lane, (int)(pitch * 2), dh);
    auto dma_tile = [&](int k0, int stage) {
        E *Ks = lds + stage * STAGE;
        dma.issue(seq + (size_t)k0 * pitch + d, Ks, sh.s - k0, wave);
        dma.issue(seq + (size_t)k0 * pitch + 2 * d, Ks + TILE, sh.s - k0, wave);
    };
    x8<E> qf[NK], dof[NK];
    float lse2, dl;
    {
        // (A uniform base and a row each: an index over b and q together is kept up to the store of dQ, which at 128 channels spilled.)
        const size_t seq0 = (size_t)b * sh.s * d + (size_t)h * dh, row = (size_t)q * d;
        const size_t stat = ((size_t)b * sh.heads + h) * sh.s;
        x8<E> of[NK];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            if constexpr (OWN) of[ks] = frag_global(out + seq0 + row, ks, half, qvalid, dh);
            dof[ks] = frag_global(dout + seq0 + row, ks, half, qvalid, dh);
        }
        lse2 = qvalid ? (lse + stat)[q] : 0.f;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) qf[ks] = frag_global(seq + (size_t)q * pitch, ks, half, qvalid, dh);
        dma_tile(0, 0);                                         // (on its way before anything is waited for)
        if constexpr (OWN) {
            dl = row_delta<NK, E>(dof, of);
            if (qvalid && half == 0) (delta + stat)[q] = dl;
        } else dl = qvalid ? (delta + stat)[q] : 0.f;
        lse2 = qvalid ? lse2 * kLog2e : INFINITY;               // invalid rows: p = exp2(-inf) = 0
    }
    const float scale = rsqrtf((float)dh);
    const float c2 = scale * kLog2e;

    f32x16 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
    // From 128 channels on the registers hold neither all row operands of a block nor a second copy of the read addresses.  Left to itself
    // the compiler spilled 7 of them inside this loop, reloaded them behind the next tile's loads and so waited for those
    // before the first product: 4 heads x 4096 x 128, one workgroup on a compute unit, 138 us; 104 without (32 heads x 2048, two on each:
    // 86 and 73).  Below 128 there is room, and the reads in one go are the faster ones (32 channels: 54 us, 57 in this form).
    constexpr bool TIGHT = DH >= 128;
    std::conditional_t<TIGHT, BothStages<DH, STAGE * 2>, BothAddr<DH>> ad;
    if constexpr (TIGHT) ad.init(lds, lane);
    else ad.init(lane);

    const bool causal = sh.causal != 0;
    const int kend = causal ? min(sh.s, qb * 128 + 128) : sh.s;
    int stage = 0;
    auto next_stage = [&]() __attribute__((always_inline)) {
        stage ^= 1;
        if constexpr (TIGHT) ad.move(stage != 0);
    };
    for (int k0 = 0; k0 < kend; k0 += KT, next_stage()) {
        // this wavefront's part of tile k0 has landed and its LDS reads of the previous tile have returned; after
        // the barrier the tile is published and the other stage is free for the next one
        __builtin_amdgcn_s_waitcnt(0x0070);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (k0 + KT < kend) dma_tile(k0 + KT, stage ^ 1);
        if (causal && k0 > qw0 + 31) continue;     // whole tile is in this wavefront's future
        const E *Ks = lds + stage * STAGE, *Vs = Ks + TILE;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int kbs = k0 + 32 * kb;          // first key of this block of 32
            // in the future of all 32 queries (both are multiples of 32), or past the end of the sequence
            if (causal ? kbs > qw0 : kbs >= sh.s) continue;
            // last visible key of this lane's query, relative to the block: the query itself, or the end of the sequence
            const int klast = causal ? qw0 + lrow - kbs : sh.s - 1 - kbs;
            constexpr int AHEAD = 4, SLOTS = TIGHT ? AHEAD + 2 : NK;
            x8<E> kf[SLOTS], vfr[SLOTS], ktf[2 * NC];
            f32x16 st, dpt;
            auto load = [&](int ks, int i) __attribute__((always_inline)) {
                if constexpr (TIGHT) {
                    kf[i] = ad.template nat<E>(0, kb, ks);
                    vfr[i] = ad.template nat<E>(TILE * 2, kb, ks);
                } else {
                    kf[i] = ad.nat(Ks, kb, ks);
                    vfr[i] = ad.nat(Vs, kb, ks);
                }
            };
            auto multiply = [&](int ks, int i) __attribute__((always_inline)) {
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                st = MFMA(kf[i], qf[ks], ks == 0 ? zero : st);
                dpt = MFMA(vfr[i], dof[ks], ks == 0 ? zero : dpt);
            };
            if constexpr (TIGHT) {
                products_ahead<NK, AHEAD>(load, multiply);
            } else {
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) load(ks, ks);
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) multiply(ks, ks);
            }
            // the K^T operands take over the registers of the K and V operands; their latency passes under the
            // exponentials
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if constexpr (TIGHT) ktf[kk * NC + c] = ad.template tr<E>(0, c, 2 * kb + kk);
                    else ktf[kk * NC + c] = ad.tr(Ks, c, 2 * kb + kk);
                }
            __builtin_amdgcn_sched_barrier(0);
            if (causal ? kbs == qw0 : kbs + 32 > sh.s) {     // the diagonal block, or the ragged last one: masked keys
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float p = __builtin_amdgcn_exp2f(fmaf(st[r], c2, -lse2));
                    if (8 * (r >> 2) + 4 * half + (r & 3) > klast) p = 0.f;
                    st[r] = p * (dpt[r] - dl);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) st[r] = __builtin_amdgcn_exp2f(fmaf(st[r], c2, -lse2)) * (dpt[r] - dl);
            }
            wait_tr_reads(ktf);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const x8<E> dsf = pack16<E>(st, kk);
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] = MFMA(ktf[kk * NC + c], dsf, acc[c]);
            }
        }
    }
    if (qvalid) {
        E *orow = dqkv + ((size_t)b * sh.s + q) * pitch + (size_t)h * dh;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                x4<E> o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = (E)(acc[c][4 * g + i] * scale);
                if (c * 32 + 8 * g + 4 * half < dh) *reinterpret_cast<x4<E> *>(orow + c * 32 + 8 * g + 4 * half) = o;
            }
    }
}


// ============================================================================================
// dK, dV.  One workgroup per (sequence, head, block of 128 keys), see block_of(); rank = key block index (with the
// causal mask the first key block has the most queries).
//
// A wavefront owns 32 keys (K and V operands in registers, dK and dV accumulators); query tiles of 64 (Q and
// dO as stored) stream from global memory straight into one of three LDS stages, one barrier per tile.  Every
// tile is read both ways: rows for S = Q K^T and dP = dO V^T, transposed for dV^T += dO^T P and dK^T += Q^T dS.
// With the causal mask the first two query tiles of a key block contain its diagonal (masked, partly skipped); all
// later ones - without the mask, all tiles from the start of the sequence - are fully visible and go through a loop
// without tests (rows past the end of the sequence are zero and carry zero statistics: they add nothing).
// Up to 64 channels two workgroups share a compute unit, and the register budget says so: with a budget for one, scores and dP came out of
// the products in accumulation registers, 32 moves a unit (1024 x 384 x 64: 175 -> 164 us, 1024 x 48 x 64: 32 -> 29.6).
// LDS stages; four where the loop over fully visible tiles is pipelined across units
template <int DH> constexpr int dkv_stages() { return DH == 96 || DH == 128 ? 4 : 3; }
template <int DH, class E>
__global__ __launch_bounds__(256, DH <= 64 ? 2 : 1) void attn_bwd_dkv_kernel(const E *__restrict__ qkv, const float *__restrict__ lse,
                                                              const float *__restrict__ delta,
                                                              const E *__restrict__ dout, E *__restrict__ dqkv,
                                                              AttnShape sh) {
    constexpr int QT = 64, NST = dkv_stages<DH>();
    constexpr int NK = DH / 16, NC = DH / 32;
    typedef TileDmaSw<QT, DH> Dma;
    constexpr int TILE = Dma::ELEMS, STAGE = 2 * TILE;          // Q tile, then dO tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);
    float *lse_s = reinterpret_cast<float *>(lds + NST * STAGE);     // [NST][QT]  log-sum-exp, log2 domain, negated
    float *dl_s = lse_s + NST * QT;                                  // [NST][QT]  delta, negated

    int bh, kb128;
    block_of(sh, (sh.s + 127) / 128, bh, kb128);
    const int h = bh % sh.heads, b = bh / sh.heads;
    const int dh = sh.dh;                           // head size in memory, <= DH
    const int d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const E *seq = qkv + (size_t)b * sh.s * pitch + (size_t)h * dh;
    const E *doseq = dout + (size_t)b * sh.s * d + (size_t)h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, half = lane >> 5;
    const int kw0 = kb128 * 128 + wave * 32;        // first key of this wavefront
    const int key = kw0 + lrow;
    const bool kvalid = key < sh.s;

    x8<E> kf[NK], vf[NK];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        kf[ks] = frag_global(seq + (size_t)key * pitch + d, ks, half, kvalid, dh);
        vf[ks] = frag_global(seq + (size_t)key * pitch + 2 * d, ks, half, kvalid, dh);
    }
    const float scale = rsqrtf((float)dh);
    const float c2 = scale * kLog2e;
    const size_t stat0 = ((size_t)b * sh.heads + h) * sh.s;

    f32x16 dk[NC], dv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) dk[c][r] = dv[c][r] = 0.f;

    Dma dq_, do_;
    dq_.init(wave, lane, (int)(pitch * 2), dh);
    do_.init(wave, lane, d * 2, dh);
    BothAddr<DH> ad;
    ad.init(lane);
    const bool causal = sh.causal != 0;
    // Tile t holds queries [qbeg + 64 t, +64); with the causal mask, queries before the key block see none of its keys.  Its row statistics go through registers: wavefront 0 fetches the
    // log-sum-exps, wavefront 1 the deltas, one tile ahead of the tile data, and they are stored to LDS before
    // the barrier that publishes the tile.
    const int qbeg = causal ? kb128 * 128 : 0;
    const int ntiles = (sh.s - qbeg + QT - 1) / QT;
    auto dma_tile = [&](int t, int stage) {
        const int q0 = qbeg + QT * t;
        dq_.issue(seq + (size_t)q0 * pitch, lds + stage * STAGE, sh.s - q0, wave);
        do_.issue(doseq + (size_t)q0 * d, lds + stage * STAGE + TILE, sh.s - q0, wave);
    };
    // (the value is left as loaded until it is stored a tile later: arithmetic on it here would wait for it, and with it for every tile
    // in flight, at once.  The store still waits for the tiles that are in flight then.)
    auto load_stat = [&](int t) -> float {
        const int qq = min(qbeg + QT * t + lane, sh.s - 1);
        return wave == 0 ? lse[stat0 + qq] : delta[stat0 + qq];
    };
    auto store_stat = [&](int t, int stage, float v) {
        const bool in = qbeg + QT * t + lane < sh.s;
        if (wave == 0) lse_s[stage * QT + lane] = in ? -v * kLog2e : 0.f;
        if (wave == 1) dl_s[stage * QT + lane] = in ? -v : 0.f;
    };

    // A unit is 32 keys x 32 queries: query rows [32 u, 32 u + 32) of the tile in `stage`, first query qs.  Its steps:
    x8<E> qn[NK], don[NK];                         // row operands (Q, dO) of a unit
    x8<E> dot[2 * NC], qt[2 * NC];                 // transposed operands
    x8<E> pf[2], dsf[2];                           // P and dS as operands
    auto read_rows = [&](int stage, int u, int ks) {
        qn[ks] = ad.nat(lds + stage * STAGE, u, ks);
        don[ks] = ad.nat(lds + stage * STAGE + TILE, u, ks);
    };
    auto read_tr = [&](int stage, int u, int j) {  // j = kk NC + c
        dot[j] = ad.tr(lds + stage * STAGE + TILE, j % NC, 2 * u + j / NC);
        qt[j] = ad.tr(lds + stage * STAGE, j % NC, 2 * u + j / NC);
    };
    // S = Q K^T and dP - delta = dO V^T - delta: the latter starts from the negated deltas of its rows, which saves the subtraction
    auto init_dp = [&](int stage, int u, f32x16 &dp) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 d4 = *reinterpret_cast<const f32x4 *>(dl_s + stage * QT + 32 * u + 8 * g + 4 * half);
#pragma unroll
            for (int i = 0; i < 4; ++i) dp[4 * g + i] = d4[i];
        }
    };
    auto s_dp = [&](int ks, f32x16 &s_, f32x16 &dp) {
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        s_ = MFMA(qn[ks], kf[ks], ks == 0 ? zero : s_);
        dp = MFMA(don[ks], vf[ks], dp);
    };
    auto read_lse = [&](int stage, int u, f32x4 (&l4)[4]) {
#pragma unroll
        for (int g = 0; g < 4; ++g) l4[g] = *reinterpret_cast<const f32x4 *>(lse_s + stage * QT + 32 * u + 8 * g + 4 * half);
    };
    auto softmax = [&](int g, const f32x4 &l4, const f32x16 &s_, const f32x16 &dp, int qs, auto masked_c) {      // quarter g of P and dS
        constexpr bool MASKED = decltype(masked_c)::value;
        float p[4], ds[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = __builtin_amdgcn_exp2f(fmaf(s_[4 * g + i], c2, l4[i]));
            if (MASKED && qs + 8 * g + 4 * half + i < key) p[i] = 0.f;
            ds[i] = p[i] * dp[4 * g + i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pf[g >> 1][4 * (g & 1) + i] = (E)p[i];
            dsf[g >> 1][4 * (g & 1) + i] = (E)ds[i];
        }
    };
    auto dv_dk = [&](int j) {
        dv[j % NC] = MFMA(dot[j], pf[j / NC], dv[j % NC]);
        dk[j % NC] = MFMA(qt[j], dsf[j / NC], dk[j % NC]);
    };
    // all steps of one unit in turn
    auto unit = [&](int stage, int u, int qs, auto masked_c) {
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) read_rows(stage, u, ks);
        f32x16 s_, dp;
        f32x4 l4[4];
        init_dp(stage, u, dp);
        read_lse(stage, u, l4);
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) s_dp(ks, s_, dp);
        // the transposed operands take over the registers of the row operands; their latency passes under the
        // exponentials
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 2 * NC; ++j) read_tr(stage, u, j);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) softmax(g, l4[g], s_, dp, qs, masked_c);
        wait_tr_reads(dot);
        wait_tr_reads(qt);
#pragma unroll
        for (int j = 0; j < 2 * NC; ++j) dv_dk(j);
    };
    // wait for this wavefront's part of the oldest tile in flight (`newer`: a younger one is in flight too),
    // then a bare s_barrier - a __syncthreads() fence would wait for the younger tile as well
    constexpr int kLoadsPerTile = 2 * Dma::NJ;      // upper bound of what a wavefront issues per tile
    static_assert(Dma::NI % 4 == 0 && kLoadsPerTile < 16, "every wavefront issues the same number of loads per tile");
    auto publish = [&](bool newer) {
        if (newer)
            __builtin_amdgcn_s_waitcnt(0x0070 | kLoadsPerTile);
        else
            __builtin_amdgcn_s_waitcnt(0x0070);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // tile t is multiplied while tiles t + 1 and t + 2 are in flight
    float stat = load_stat(0);
    dma_tile(0, 0);
    store_stat(0, 0, stat);
    if (ntiles > 1) {
        stat = load_stat(1);
        dma_tile(1, 1);
    }
    // start of tile t: tile t + 1's statistics go to LDS (the next call's barrier publishes them), tile t is published, tile
    // t + 2 is requested
    auto slot = [&](int t) { return NST == 4 ? t & 3 : t % NST; };
    auto advance = [&](int t) {
        if (t + 1 < ntiles) store_stat(t + 1, slot(t + 1), stat);
        publish(t + 1 < ntiles);
        if (t + 2 < ntiles) {
            stat = load_stat(t + 2);
            dma_tile(t + 2, slot(t + 2));
        }
    };
    // Two loops in sequence rather than one with two kinds of iteration: with two code paths through the
    // MFMAs in one loop the compiler merges their accumulator registers with copies at every iteration.
    int t = 0;
    const int ndiag = causal ? 2 : 0;
    for (; t < ndiag && t < ntiles; ++t) {                      // the diagonal part
        advance(t);
        const int q0 = qbeg + QT * t;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int qs = q0 + 32 * u;
            if (qs + 31 < kw0 || qs >= sh.s) continue;      // all its queries precede this wavefront's keys, or are past the end
            unit(slot(t), u, qs, std::true_type{});
        }
    }
    if constexpr (NST == 4) {
        // Fully visible tiles, one unit's steps spread over its neighbours' (a wavefront is alone on its SIMD: in turn, the LDS reads, the
        // first products, the exponentials and the second products each leave the other units idle - 0.28 of the matrix
        // pipe's cycles at 128 channels):
        //   phase A of unit n   S, dP of unit n + 1  |  P, dS of unit n, its transposed reads
        //   phase B of unit n   dV, dK of unit n     |  row reads of unit n + 2
        // 16 heads x 8100 positions x 128, causal: 3670 -> 2270 cycles a unit (1024 of them matrix instructions), 590 -> 550 us; what is
        // left is the 32 moves a unit out of accumulation registers, LDS waits, the barrier per tile and, in the two wavefronts that
        // carry the statistics, a wait for every tile in flight where they store them.
        // Unit n + 2 may lie in the next tile, which is published in phase B of the tile's first unit; the tile itself is still read
        // in the phases after that, which is what the fourth stage is for.
        if (t < ntiles) {
            f32x16 s0, dp0, s1, dp1;
            f32x4 l4[4];
            auto phase_a = [&](int stage, int u, const f32x16 &s_, const f32x16 &dp, f32x16 &ns, f32x16 &ndp) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
#pragma unroll
                    for (int ks = 0; ks < NK; ++ks)
                        if (ks >= g * NK / 4 && ks < (g + 1) * NK / 4) s_dp(ks, ns, ndp);
                    softmax(g, l4[g], s_, dp, 0, std::false_type{});
#pragma unroll
                    for (int i = 0; i < NK / 2; ++i) {           // one matrix instruction, then its share of the exponentials
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 56 / NK, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < 2 * NC; ++j)             // done by the third quarter: the last one covers their latency
                        if (g < 3 && j >= g * 2 * NC / 3 && j < (g + 1) * 2 * NC / 3) read_tr(stage, u, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // ... and at its end the statistics: the log-sum-exps of unit n + 1, the deltas of unit n + 2
            auto phase_b = [&](int lstage, int lu, int rstage, int ru, f32x16 &rdp, int publish_t) __attribute__((always_inline)) {
                wait_tr_reads(dot);
                wait_tr_reads(qt);
                __builtin_amdgcn_sched_barrier(0);
                dv_dk(0);
                __builtin_amdgcn_sched_barrier(0);
                if (publish_t >= 0 && publish_t < ntiles) advance(publish_t);
#pragma unroll
                for (int j = 1; j < 2 * NC; ++j) {
                    dv_dk(j);
#pragma unroll
                    for (int ks = 0; ks < NK; ++ks)
                        if (ks * (2 * NC - 2) / NK == j - 1) read_rows(rstage, ru, ks);
                    if (j == 2 * NC - 2) read_lse(lstage, lu, l4);
                    if (j == 2 * NC - 1) init_dp(rstage, ru, rdp);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            advance(t);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) read_rows(slot(t), 0, ks);
            init_dp(slot(t), 0, dp0);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) s_dp(ks, s0, dp0);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) read_rows(slot(t), 1, ks);
            read_lse(slot(t), 0, l4);
            init_dp(slot(t), 1, dp1);
            // behind the last tile the products and reads of a tile that does not exist run too, on whatever its stage holds: nothing
            // uses them, and the loop has one path through the matrix instructions
            for (; t < ntiles; ++t) {
                const int cur = slot(t), nxt = slot(t + 1);
                phase_a(cur, 0, s0, dp0, s1, dp1);
                phase_b(cur, 1, nxt, 0, dp0, t + 1);
                phase_a(cur, 1, s1, dp1, s0, dp0);
                phase_b(nxt, 0, nxt, 1, dp1, -1);
            }
        }
    } else {
        for (; t < ntiles; ++t) {                               // fully visible tiles
            advance(t);
            unit(slot(t), 0, 0, std::false_type{});
            unit(slot(t), 1, 0, std::false_type{});
        }
    }
    if (kvalid) {
        E *orow = dqkv + ((size_t)b * sh.s + key) * pitch + (size_t)h * dh;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                x4<E> ok, ov;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ok[i] = (E)(dk[c][4 * g + i] * scale);
                    ov[i] = (E)dv[c][4 * g + i];
                }
                if (c * 32 + 8 * g + 4 * half < dh) {
                    *reinterpret_cast<x4<E> *>(orow + d + c * 32 + 8 * g + 4 * half) = ok;
                    *reinterpret_cast<x4<E> *>(orow + 2 * d + c * 32 + 8 * g + 4 * half) = ov;
                }
            }
    }
}

// Explicit instantiations: the host compiler does not always emit the launch stub of a kernel template from its
// use in the launchers below alone.
#define LGA_INSTANTIATE_KERNELS(DH, OCC, E)                                                                          \
    template __global__ void attn_fwd_kernel<DH, 1, E>(const E *, E *, float *, AttnShape);                          \
    template __global__ void attn_fwd_kernel<DH, 2, E>(const E *, E *, float *, AttnShape);                          \
    template __global__ void attn_bwd_dq_kernel<DH, OCC, true, E>(const E *, const E *, const float *, float *, const E *, E *,  \
                                                                  AttnShape);                                        \
    template __global__ void attn_bwd_dq_kernel<DH, OCC, false, E>(const E *, const E *, const float *, float *, const E *, E *, \
                                                                   AttnShape);                                       \
    template __global__ void attn_bwd_dkv_kernel<DH, E>(const E *, const float *, const float *, const E *, E *,     \
                                                        AttnShape)
#define LGA_INSTANTIATE_TYPE(E)                                                                            \
    template __global__ void attn_delta_kernel<E>(const E *, const E *, float *, AttnShape, int);          \
    LGA_INSTANTIATE_KERNELS(32, 2, E);                                                                     \
    LGA_INSTANTIATE_KERNELS(64, 2, E);                                                                     \
    LGA_INSTANTIATE_KERNELS(96, 2, E);                                                                     \
    LGA_INSTANTIATE_KERNELS(128, 2, E);                                                                    \
    LGA_INSTANTIATE_KERNELS(160, 1, E)
LGA_INSTANTIATE_TYPE(bf16);
LGA_INSTANTIATE_TYPE(f16);
#undef LGA_INSTANTIATE_TYPE
#undef LGA_INSTANTIATE_KERNELS

// Dynamic LDS of the three kernels, in bytes.
// forward: three stages of a 64-key K tile and V tile
template <int DH> constexpr int smem_fwd() {
    return 3 * (TileDma<64, DH, pitch_rd<DH>()>::ELEMS + TileDma<64, DH, pitch_tr<DH>()>::ELEMS) * 2;
}
// dQ: two stages of a 64-key K tile and V tile
template <int DH> constexpr int smem_dq() { return 2 * 2 * 64 * DH * 2; }
// dK/dV: three or four stages of a Q tile, a dO tile and the row statistics
template <int DH> constexpr int smem_dkv() { return dkv_stages<DH>() * (2 * 64 * DH * 2 + 2 * 64 * 4); }
template <int DH> constexpr int occ_dq() { return DH <= 128 ? 2 : 1; }     // workgroups per CU the dQ kernel's register budget is set for

// All three kernels use more dynamic LDS than a launch may ask for by default: raise the limit of every
// instantiation.  Called once, outside any launch path (see attn_prepare_kernels).
template <int DH, class E> hipError_t raise_lds_limits() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_fwd_kernel<DH, 1, E>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem_fwd<DH>());
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_fwd_kernel<DH, 2, E>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem_fwd<DH>());
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_bwd_dq_kernel<DH, occ_dq<DH>(), true, E>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem_dq<DH>());
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_bwd_dq_kernel<DH, occ_dq<DH>(), false, E>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem_dq<DH>());
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_bwd_dkv_kernel<DH, E>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem_dkv<DH>());
    return e;
}
template <class E> hipError_t raise_lds_limits_all() {
    hipError_t e = raise_lds_limits<32, E>();
    if (e == hipSuccess) e = raise_lds_limits<64, E>();
    if (e == hipSuccess) e = raise_lds_limits<96, E>();
    if (e == hipSuccess) e = raise_lds_limits<128, E>();
    if (e == hipSuccess) e = raise_lds_limits<160, E>();
    return e;
}

template <int DH, class E> void fwd_dh(const E *qkv, E *out, float *lse, AttnShape sh, hipStream_t s) {
    const int U = attn_fwd_subblocks(sh);
    dim3 grid((unsigned)(sh.n_seq * sh.heads) * ((sh.s + 128 * U - 1) / (128 * U)));
    char name[64];
    snprintf(name, sizeof(name), "attn_fwd_kernel<%d, %d>", DH, U);
    const double pairs = (double)sh.n_seq * sh.heads * sh.s * sh.s * (sh.causal ? 0.5 : 1.0);      // visible (query, key) pairs
    const double act = (double)sh.n_seq * sh.s * sh.heads * sh.dh * 2.0;      // bytes of one [tokens, d] bf16 tensor
    ProfScope scope(name, 4.0 * pairs * sh.dh, 4.0 * act, s);
    hipLaunchKernelGGL((U == 1 ? attn_fwd_kernel<DH, 1, E> : attn_fwd_kernel<DH, 2, E>), grid, dim3(256), smem_fwd<DH>(), s, qkv, out, lse, sh);
}
template <int DH, class E>
void bwd_dh(const E *qkv, const E *out, const float *lse, float *delta, const E *dout, E *dqkv, AttnShape sh,
            hipStream_t s) {
    dim3 grid((unsigned)(sh.n_seq * sh.heads) * ((sh.s + 127) / 128));
    char name[64];
    const double pairs = (double)sh.n_seq * sh.heads * sh.s * sh.s * (sh.causal ? 0.5 : 1.0);
    const double act = (double)sh.n_seq * sh.s * sh.heads * sh.dh * 2.0;
    {
        snprintf(name, sizeof(name), "attn_bwd_dq_kernel<%d>", DH);
        ProfScope scope(name, 6.0 * pairs * sh.dh, 6.0 * act, s);
        const auto kernel = out ? attn_bwd_dq_kernel<DH, occ_dq<DH>(), true, E> : attn_bwd_dq_kernel<DH, occ_dq<DH>(), false, E>;
        hipLaunchKernelGGL(kernel, grid, dim3(256), smem_dq<DH>(), s, qkv, out, lse, delta, dout, dqkv, sh);
    }
    {
        snprintf(name, sizeof(name), "attn_bwd_dkv_kernel<%d>", DH);
        ProfScope scope(name, 8.0 * pairs * sh.dh, 6.0 * act, s);
        hipLaunchKernelGGL((attn_bwd_dkv_kernel<DH, E>), grid, dim3(256), smem_dkv<DH>(), s, qkv, lse, delta, dout, dqkv, sh);
    }
}

}  // namespace

// Query sub-blocks per wavefront of the forward kernel, by what the workgroups take on 256 compute units.  One sub-block instead of two makes
// them half as long, but reads the LDS operands for half the products: 8100 x 16 heads x 128 355 us against 302, 1024 x 384 x 64 107
// against 103 - and few workgroups leave compute units idle behind the longest: 1024 x 48 x 64 (192 blocks of 256) 18.8 against 25.6,
// 1000 x 56 x 152 (224) 39 against 45, 128 x 2 x 64 6.0 against 7.8.  With the causal mask a workgroup is half as long as the longest on
// average.  (Either form adds up a row in the same order and starts over with the same references: the results are the same.)
// Nor where a sequence of 129 to 256 queries is one workgroup, and would be two in more than a round: the second is short and takes its fixed part all the
// same (12 x 137 x 12 x 112 causal 14.9 with one sub-block, 12.4 with two; 6 x 132 x 24 x 128 15.0, 12.7; 4 x 153 x 88 x 48 unmasked 16.6, 14.2; 13 of 14
// such shapes 2 to 37 % more, one 1 % less); but with the mask and up to 64 channels, where several share a compute unit, 210 x 162 x 48 8.3
// against 10.7, 216 x 319 x 32 8.8 against 11.9.
// Never more of the short workgroups than a launch holds, 2^32 work items, beyond which it runs a part of them and reports nothing.
int attn_fwd_subblocks(const AttnShape &sh) {
    const double one = sh.dh <= 64 ? 0.52 : 0.6;             // of what a workgroup with two takes
    const double heads = (double)sh.n_seq * sh.heads;
    if (heads * ((sh.s + 127) / 128) * 256.0 >= 4294967296.0) return 2;
    if (sh.s > 128 && sh.s <= 256 && heads > 128.0 && (sh.dh > 64 || !sh.causal)) return 2;
    auto time = [&](int u, double each) {
        const double work = heads * ((sh.s + 128 * u - 1) / (128 * u)) / 256.0;
        return each * std::max(1.0, sh.causal ? 0.5 * work : std::ceil(work));
    };
    return time(1, one) < time(2, 1.0) ? 1 : 2;
}

// Head sizes 32, 64, 96, 128, 160 have kernels; any other multiple of 8 up to 160 runs in the next larger one with
// its extra columns read as zeros and not written.
bool attn_bf16_supports(int dh) { return dh >= 8 && dh <= 160 && dh % 8 == 0; }
static int padded_dh(int dh) { return (dh + 31) / 32 * 32; }

hipError_t attn_prepare_kernels() {
    hipError_t e = raise_lds_limits_all<bf16>();
    if (e == hipSuccess) e = raise_lds_limits_all<f16>();
    return e;
}

template <class E> void launch_attn_fwd_mfma(const E *qkv, E *out, float *lse, AttnShape sh, hipStream_t s) {
    if (sh.n_seq == 0 || sh.s == 0) return;
    if (!attn_bf16_supports(sh.dh)) {
        launch_attn_fwd_simple<E>(qkv, out, lse, sh, s);
        return;
    }
    (void)prepare_kernels();
    switch (padded_dh(sh.dh)) {
        case 32: fwd_dh<32, E>(qkv, out, lse, sh, s); break;
        case 64: fwd_dh<64, E>(qkv, out, lse, sh, s); break;
        case 96: fwd_dh<96, E>(qkv, out, lse, sh, s); break;
        case 128: fwd_dh<128, E>(qkv, out, lse, sh, s); break;
        case 160: fwd_dh<160, E>(qkv, out, lse, sh, s); break;
    }
}

template <class E> const E *delta_apart(const E *out, const E *dout, const E *dqkv, float *delta, AttnShape sh, hipStream_t s) {
    const size_t n = (size_t)sh.n_seq * sh.s * sh.heads * sh.dh;
    if (out + n <= dqkv || dqkv + 3 * n <= out) return out;
    const size_t items = n / sh.dh;
    const int items_per_block = 256 / (sh.dh / 8);                  // dh is a multiple of 8, at most 320
    ProfScope scope("attn_delta_kernel", 2.0 * n, 4.0 * n, s);
    hipLaunchKernelGGL(attn_delta_kernel<E>, dim3((unsigned)((items + items_per_block - 1) / items_per_block)), dim3(256), 0, s, out, dout, delta, sh,
                       items_per_block);
    return nullptr;
}

template <class E>
void launch_attn_bwd_mfma(const E *qkv, const E *out, const float *lse, const E *dout, E *dqkv,
                          float *delta, AttnShape sh, hipStream_t s) {
    if (sh.n_seq == 0 || sh.s == 0) return;
    if (!attn_bf16_supports(sh.dh)) {
        launch_attn_bwd_simple<E>(qkv, out, lse, dout, dqkv, delta, sh, s);
        return;
    }
    (void)prepare_kernels();
    out = delta_apart<E>(out, dout, dqkv, delta, sh, s);
    switch (padded_dh(sh.dh)) {
        case 32: bwd_dh<32, E>(qkv, out, lse, delta, dout, dqkv, sh, s); break;
        case 64: bwd_dh<64, E>(qkv, out, lse, delta, dout, dqkv, sh, s); break;
        case 96: bwd_dh<96, E>(qkv, out, lse, delta, dout, dqkv, sh, s); break;
        case 128: bwd_dh<128, E>(qkv, out, lse, delta, dout, dqkv, sh, s); break;
        case 160: bwd_dh<160, E>(qkv, out, lse, delta, dout, dqkv, sh, s); break;
    }
}

#define LGA_INSTANTIATE_ATTN(E)                                                                          \
    template const E *delta_apart<E>(const E *, const E *, const E *, float *, AttnShape, hipStream_t);    \
    template void launch_attn_fwd_mfma<E>(const E *, E *, float *, AttnShape, hipStream_t);               \
    template void launch_attn_bwd_mfma<E>(const E *, const E *, const float *, const E *, E *, float *, \
                                          AttnShape, hipStream_t)
LGA_INSTANTIATE_ATTN(bf16);
LGA_INSTANTIATE_ATTN(f16);
#undef LGA_INSTANTIATE_ATTN

}  // namespace lga
