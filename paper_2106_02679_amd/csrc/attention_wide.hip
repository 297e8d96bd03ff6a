// Softmax attention for head sizes above 160 and up to 320 (the X_[x] family: 216 for X_108, 320 for X_160) on 16-bit tensors, in
// the manner of the kernels for smaller heads: 32 positions per wavefront, score blocks produced transposed so that a lane owns one
// position, tiles straight into LDS and read both ways.
//
// dS = P (dP - delta) / sqrt(d_h) is rounded to half precision with the factor in it: without, it leaves that format's range at
// gradients sqrt(d_h) times smaller.  bfloat16 has the range, and the factor goes into the finished sums (as a multiplication per score
// it would cost the joint dK/dV kernel 8 %).
//
// What differs is what a wavefront's registers hold.  Forward: 32 queries instead of 64 (one accumulator block of 32 x DH); the softmax
// reference moves only when a score exceeds it by kLazy, so that the accumulators are rescaled in a few tiles of a row.  dQ:
// one wavefront per SIMD.  dK/dV: operands and both accumulators of 32 keys fit up to 224 channels; beyond, the kernel runs twice,
// once per result (the scores are computed in both: 5 products instead of 4).  Tiles are 32 positions long.
//
// Against the path through memory that served these heads (batched GEMMs with fp32 score matrices and two row kernels, 12 s^2
// bytes per head), causal, forward / backward in us: 2 x 54 heads x 1728 x 216: 869 / 1922 -> 209 / 749; 80 x 2560 x 320: 1330 /
// 3575 -> 560 / 1755; 32 x 2048 x 256 in half precision: 332 / 744 -> 110 / 371.
#include <cstdio>
#include <type_traits>

#include "attention16.h"
#include "kernels.h"

namespace lga {

namespace {

// wait for all but the newest `newer` loads and for this wavefront's LDS reads, then a bare s_barrier (a fence would wait for every load)
template <int NEWER> __device__ __forceinline__ void publish_tile(bool newer) {
    constexpr int kWait = 0x0070 | (NEWER & 15) | (NEWER >> 4 << 14);
    if (newer) __builtin_amdgcn_s_waitcnt(kWait);
    else __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ f32x16 zero16() { return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; }

// far enough ahead for the LDS latency with four wavefronts reading
constexpr int kAhead = 6, kSlots = kAhead + 2;
template <int NK, class L, class M> __device__ __forceinline__ void products(L load, M multiply) { products_ahead<NK, kAhead>(load, multiply); }

template <class E> constexpr bool scale_first() { return std::is_same<E, f16>::value; }

constexpr int kTile = 32;
// two workgroups per compute unit where registers and LDS (two stages) allow it, else one with three stages
template <int DH> constexpr int fwd_occ() { return DH <= 224 ? 2 : 1; }
template <int DH> constexpr int fwd_stages() { return fwd_occ<DH>() == 2 ? 2 : 3; }
template <int DH> constexpr int stage_elems() { return 2 * TileDmaSw<kTile, DH>::ELEMS; }

// ---- forward: one workgroup per (sequence, head, 128 queries) ------------------------------------------------------------------
template <int DH, class E>
__global__ __launch_bounds__(256, fwd_occ<DH>()) void attn_wide_fwd_kernel(const E *__restrict__ qkv, E *__restrict__ out,
                                                                           float *__restrict__ lse, AttnShape sh) {
    constexpr int NK = DH / 16, NC = DH / 32, NST = fwd_stages<DH>();
    typedef TileDmaSw<kTile, DH> Dma;
    constexpr int TILE = Dma::ELEMS, STAGE = 2 * TILE;          // K tile, then V tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);
    const int qblocks = (sh.s + 127) / 128;
    int bh, rank;
    block_of(sh, qblocks, bh, rank);
    const int qb = qblocks - 1 - rank, h = bh % sh.heads, b = bh / sh.heads, dh = sh.dh, d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const E *seq = qkv + (size_t)b * sh.s * pitch + (size_t)h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, half = lane >> 5;
    const int qw0 = qb * 128 + wave * 32, q = qw0 + lrow;
    const bool causal = sh.causal != 0;

    x8<E> qf[NK];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) qf[ks] = frag_global(seq + (size_t)q * pitch, ks, half, q < sh.s, dh);
    f32x16 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = zero16();
    // p = 2^(score - m_ref) stays below 2^kLazy, inside either format's range, and the common factor leaves with the final division
    constexpr float kLazy = 8.f;
    float m_ref = -INFINITY, l_run = 0.f;
    const float c2 = rsqrtf((float)dh) * kLog2e;

    Dma dma;
    dma.init(wave, lane, (int)(pitch * 2), dh);
    auto dma_tile = [&](int k0, int stage) {
        E *Ks = lds + stage * STAGE;
        dma.issue(seq + (size_t)k0 * pitch + d, Ks, sh.s - k0, wave);
        dma.issue(seq + (size_t)k0 * pitch + 2 * d, Ks + TILE, sh.s - k0, wave);
    };
    BothAddr<DH> ad;
    ad.init(lane);
    const int kend = causal ? min(sh.s, qb * 128 + 128) : sh.s;
    dma_tile(0, 0);
    if (NST > 2 && kTile < kend) dma_tile(kTile, 1);
    auto tile = [&](int k0, int stage, auto masked_c) {
        const E *Ks = lds + stage * STAGE, *Vs = Ks + TILE;
        f32x16 st = zero16();
        x8<E> kf[kSlots];
        products<NK>([&](int ks, int i) { kf[i] = ad.nat(Ks, 0, ks); }, [&](int ks, int i) { st = MFMA(kf[i], qf[ks], st); });
        x8<E> v0[NC], v1[NC];                                    // V^T operands of the tile's two halves; their latency passes under the softmax
        auto read_v0 = [&]() {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < NC; ++c) v0[c] = ad.tr(Vs, c, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (DH <= 256) read_v0();
        const bool MASKED = masked_c;                             // the diagonal part, or the ragged last tile
        const int klast = (causal ? q : sh.s - 1) - k0 - 4 * half;           // register r is visible iff 8 (r / 4) + r % 4 <= klast
        float top = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (MASKED && 8 * (r >> 2) + (r & 3) > klast) st[r] = -INFINITY;
            top = fmaxf(top, st[r]);
        }
        top = fmaxf(top, __shfl_xor(top, 32, 64)) * c2;
        if (__any(top > m_ref + kLazy)) {
            const float m = fmaxf(m_ref, top);
            const float scale = m == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_ref - m);
            l_run *= scale;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[c][r] *= scale;
            m_ref = m;
        }
        if constexpr (DH > 256) read_v0();                       // (there is no room for them beside the accumulators before)
        const float ref = m_ref == -INFINITY ? 0.f : m_ref;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            st[r] = __builtin_amdgcn_exp2f(fmaf(st[r], c2, -ref));
            l_run += st[r];
        }
        const x8<E> p0 = pack16<E>(st, 0), p1 = pack16<E>(st, 1);
        wait_tr_reads(v0);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            acc[c] = MFMA(v0[c], p0, acc[c]);
            v1[c] = ad.tr(Vs, c, 1);                             // (into the registers that fall free)
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_tr_reads(v1);
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = MFMA(v1[c], p1, acc[c]);
    };
    // Two loops in sequence, the second for the tiles that some wavefront masks or leaves out: with two paths through the matrix
    // instructions in one loop, the accumulators are copied at every iteration (dQ at 216: 498 -> 392 us; this kernel at 256: 130 ->
    // 110).  Beyond 256 channels both loops' registers do not fit beside each other and one loop is faster (320: 520 against 789).
    const int kfull = DH > 256 ? 0 : causal ? qb * 128 : sh.s / kTile * kTile;
    int stage = 0, k0 = 0;
    auto advance = [&]() {
        publish_tile<2 * Dma::NJ>(NST > 2 && k0 + kTile < kend);
        const int ahead = k0 + (NST - 1) * kTile;
        if (ahead < kend) dma_tile(ahead, stage == 0 ? NST - 1 : stage - 1);
    };
    for (; k0 < kfull; k0 += kTile, stage = stage == NST - 1 ? 0 : stage + 1) {
        advance();
        tile(k0, stage, std::false_type{});
    }
    for (; k0 < kend; k0 += kTile, stage = stage == NST - 1 ? 0 : stage + 1) {
        advance();
        if (causal && k0 > qw0) continue;
        if constexpr (DH > 256) tile(k0, stage, causal ? k0 == qw0 : k0 + kTile > sh.s);
        else tile(k0, stage, std::true_type{});
    }
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    if (q >= sh.s) return;
    const float inv = 1.0f / l_tot;
    E *orow = out + ((size_t)b * sh.s + q) * d + (size_t)h * dh;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            x4<E> o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (E)(acc[c][4 * g + i] * inv);
            if (c * 32 + 8 * g + 4 * half < dh) *reinterpret_cast<x4<E> *>(orow + c * 32 + 8 * g + 4 * half) = o;
        }
    if (half == 0) lse[((size_t)b * sh.heads + h) * sh.s + q] = m_ref * kLn2 + logf(l_tot);
}

// ---- dQ: one workgroup per (sequence, head, 128 queries); OWN: it makes delta, too, from out; otherwise delta is there ----------
template <int DH, bool OWN, class E>
__global__ __launch_bounds__(256, 1) void attn_wide_dq_kernel(const E *__restrict__ qkv, const E *__restrict__ out,
                                                              const float *__restrict__ lse, float *__restrict__ delta,
                                                              const E *__restrict__ dout, E *__restrict__ dqkv, AttnShape sh) {
    constexpr int NK = DH / 16, NC = DH / 32, NST = 3;
    typedef TileDmaSw<kTile, DH> Dma;
    constexpr int TILE = Dma::ELEMS, STAGE = 2 * TILE;          // K tile, then V tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);
    const int qblocks = (sh.s + 127) / 128;
    int bh, rank;
    block_of(sh, qblocks, bh, rank);
    const int qb = qblocks - 1 - rank, h = bh % sh.heads, b = bh / sh.heads, dh = sh.dh, d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const E *seq = qkv + (size_t)b * sh.s * pitch + (size_t)h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, half = lane >> 5;
    const int qw0 = qb * 128 + wave * 32, q = qw0 + lrow;
    const bool qvalid = q < sh.s, causal = sh.causal != 0;

    Dma dma;
    dma.init(wave, lane, (int)(pitch * 2), dh);
    auto dma_tile = [&](int k0, int stage) {
        E *Ks = lds + stage * STAGE;
        dma.issue(seq + (size_t)k0 * pitch + d, Ks, sh.s - k0, wave);
        dma.issue(seq + (size_t)k0 * pitch + 2 * d, Ks + TILE, sh.s - k0, wave);
    };
    const int kend = causal ? min(sh.s, qb * 128 + 128) : sh.s;
    const float scale = rsqrtf((float)dh), c2 = scale * kLog2e;
    const float at_end = scale_first<E>() ? 1.f : scale;
    x8<E> qf[NK], dof[NK];
    const size_t row = ((size_t)b * sh.s + q) * d + (size_t)h * dh, stat = ((size_t)b * sh.heads + h) * sh.s + q;
    float lse2, dl;
    {
        x8<E> of[NK];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            if constexpr (OWN) of[ks] = frag_global(out + row, ks, half, qvalid, dh);
            dof[ks] = frag_global(dout + row, ks, half, qvalid, dh);
        }
        lse2 = qvalid ? lse[stat] : 0.f;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) qf[ks] = frag_global(seq + (size_t)q * pitch, ks, half, qvalid, dh);
        dma_tile(0, 0);                                         // (on their way before anything is waited for)
        if (kTile < kend) dma_tile(kTile, 1);
        if constexpr (OWN) {
            dl = row_delta<NK, E>(dof, of);
            if (qvalid && half == 0) delta[stat] = dl;
        } else dl = qvalid ? delta[stat] : 0.f;
        if constexpr (scale_first<E>()) dl *= scale;
        lse2 = qvalid ? lse2 * kLog2e : INFINITY;               // invalid rows: p = exp2(-inf) = 0
    }
    f32x16 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = zero16();

    BothAddr<DH> ad;
    ad.init(lane);
    auto tile = [&](int k0, int stage, auto masked_c) {
        const E *Ks = lds + stage * STAGE, *Vs = Ks + TILE;
        f32x16 st = zero16(), dpt = zero16();
        // S first, then dP with the exponentials of S between its products: alone on its SIMD, a wavefront overlaps only what it issues
        // next to each other
        x8<E> kf[kSlots], k0t[NC], k1t[NC];
        products<NK>([&](int ks, int i) { kf[i] = ad.nat(Ks, 0, ks); }, [&](int ks, int i) { st = MFMA(kf[i], qf[ks], st); });
        constexpr bool MASKED = decltype(masked_c)::value;        // the diagonal part, or the ragged last tile
        const int klast = (causal ? q : sh.s - 1) - k0 - 4 * half;
        products<NK>([&](int ks, int i) { kf[i] = ad.nat(Vs, 0, ks); },
                     [&](int ks, int i) {
                         dpt = MFMA(kf[i], dof[ks], dpt);
#pragma unroll
                         for (int r = ks * 16 / NK; r < (ks + 1) * 16 / NK; ++r) {
                             st[r] = __builtin_amdgcn_exp2f(fmaf(st[r], c2, -lse2));
                             if (MASKED && 8 * (r >> 2) + (r & 3) > klast) st[r] = 0.f;
                         }
                     });
#pragma unroll
        for (int c = 0; c < NC; ++c) k0t[c] = ad.tr(Ks, c, 0);   // K^T operands
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] *= scale_first<E>() ? fmaf(dpt[r], scale, -dl) : dpt[r] - dl;
        const x8<E> ds0 = pack16<E>(st, 0), ds1 = pack16<E>(st, 1);
        wait_tr_reads(k0t);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            acc[c] = MFMA(k0t[c], ds0, acc[c]);
            k1t[c] = ad.tr(Ks, c, 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_tr_reads(k1t);
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = MFMA(k1t[c], ds1, acc[c]);
    };
    const int kfull = causal ? qb * 128 : sh.s / kTile * kTile;         // two loops: see the forward kernel
    int stage = 0, k0 = 0;
    auto advance = [&]() {
        publish_tile<2 * Dma::NJ>(k0 + kTile < kend);
        if (k0 + 2 * kTile < kend) dma_tile(k0 + 2 * kTile, stage == 0 ? NST - 1 : stage - 1);
    };
    for (; k0 < kfull; k0 += kTile, stage = stage == NST - 1 ? 0 : stage + 1) {
        advance();
        tile(k0, stage, std::false_type{});
    }
    for (; k0 < kend; k0 += kTile, stage = stage == NST - 1 ? 0 : stage + 1) {
        advance();
        if (!causal || k0 <= qw0) tile(k0, stage, std::true_type{});
    }
    if (!qvalid) return;
    E *orow = dqkv + ((size_t)b * sh.s + q) * pitch + (size_t)h * dh;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            x4<E> o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (E)(acc[c][4 * g + i] * at_end);
            if (c * 32 + 8 * g + 4 * half < dh) *reinterpret_cast<x4<E> *>(orow + c * 32 + 8 * g + 4 * half) = o;
        }
}

// ---- dK, dV: one workgroup per (sequence, head, 128 keys) ----------------------------------------------------------------------------
enum WideResult : int { kBoth = 0, kOnlyDV = 1, kOnlyDK = 2 };

// up to 224 channels one run gives both results
template <int DH> constexpr bool dkv_in_one_run() { return DH <= 224; }

template <int DH, int WHAT, class E>
__global__ __launch_bounds__(256, 1) void attn_wide_dkv_kernel(const E *__restrict__ qkv, const float *__restrict__ lse,
                                                               const float *__restrict__ delta, const E *__restrict__ dout,
                                                               E *__restrict__ dqkv, AttnShape sh) {
    constexpr bool DV = WHAT != kOnlyDK, DK = WHAT != kOnlyDV;
    constexpr int NK = DH / 16, NC = DH / 32, NST = 3;
    typedef TileDmaSw<kTile, DH> Dma;
    constexpr int TILE = Dma::ELEMS, STAGE = 2 * TILE;          // Q tile, then dO tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);
    float *stat_s = reinterpret_cast<float *>(lds + NST * STAGE);    // [3][64]: 32 log-sum-exps (log2 domain) and 32 deltas, negated

    int bh, kb128;
    block_of(sh, (sh.s + 127) / 128, bh, kb128);
    const int h = bh % sh.heads, b = bh / sh.heads, dh = sh.dh, d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const E *seq = qkv + (size_t)b * sh.s * pitch + (size_t)h * dh, *doseq = dout + (size_t)b * sh.s * d + (size_t)h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, half = lane >> 5;
    const int kw0 = kb128 * 128 + wave * 32, key = kw0 + lrow;
    const bool kvalid = key < sh.s, causal = sh.causal != 0;

    x8<E> kf[NK], vf[DK ? NK : 1];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        kf[ks] = frag_global(seq + (size_t)key * pitch + d, ks, half, kvalid, dh);
        if constexpr (DK) vf[ks] = frag_global(seq + (size_t)key * pitch + 2 * d, ks, half, kvalid, dh);
    }
    const float scale = rsqrtf((float)dh), c2 = scale * kLog2e;
    const size_t stat0 = ((size_t)b * sh.heads + h) * sh.s;
    f32x16 dk[DK ? NC : 1], dv[DV ? NC : 1];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if constexpr (DK) dk[c] = zero16();
        if constexpr (DV) dv[c] = zero16();
    }

    Dma dq_, do_;
    dq_.init(wave, lane, (int)(pitch * 2), dh);
    do_.init(wave, lane, d * 2, dh);
    BothAddr<DH> ad;
    ad.init(lane);
    const int qbeg = causal ? kb128 * 128 : 0;                  // with the causal mask, queries before the key block see none of its keys
    const int ntiles = (sh.s - qbeg + kTile - 1) / kTile;
    auto dma_tile = [&](int t) {
        const int q0 = qbeg + kTile * t;
        E *Qs = lds + t % NST * STAGE;
        dq_.issue(seq + (size_t)q0 * pitch, Qs, sh.s - q0, wave);
        do_.issue(doseq + (size_t)q0 * d, Qs + TILE, sh.s - q0, wave);
    };
    // wavefront 0 carries the statistics of the tile after next (left as loaded: arithmetic on them would wait for the load)
    auto load_stat = [&](int t) -> float {
        const int qq = min(qbeg + kTile * t + lrow, sh.s - 1);
        return half == 0 ? lse[stat0 + qq] : delta[stat0 + qq];
    };
    auto store_stat = [&](int t, float v) {
        if (wave == 0) stat_s[t % 3 * 64 + lane] = qbeg + kTile * t + lrow >= sh.s ? 0.f : half == 0 ? -v * kLog2e : -v;
    };
    // tile t + 1's statistics are stored while tile t's are read: the stage they take was read before the last barrier
    float stat = load_stat(0);
    dma_tile(0);
    store_stat(0, stat);
    if (ntiles > 1) {
        stat = load_stat(1);
        dma_tile(1);
    }
    auto advance = [&](int t) {
        if (t + 1 < ntiles) store_stat(t + 1, stat);
        publish_tile<2 * Dma::NJ>(t + 1 < ntiles);
        if (t + 2 < ntiles) {
            stat = load_stat(t + 2);
            dma_tile(t + 2);
        }
    };
    auto unit = [&](int t, auto masked_c) {
        constexpr bool MASKED = decltype(masked_c)::value;
        const E *Qs = lds + t % NST * STAGE, *dOs = Qs + TILE;
        const float *ss = stat_s + t % 3 * 64 + 4 * half;
        f32x16 s_ = zero16(), dp = s_;
        f32x4 l4[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            l4[g] = *reinterpret_cast<const f32x4 *>(ss + 8 * g);
            if constexpr (DK) {
                const f32x4 d4 = *reinterpret_cast<const f32x4 *>(ss + 32 + 8 * g);       // dP - delta comes out of the products
#pragma unroll
                for (int i = 0; i < 4; ++i) dp[4 * g + i] = d4[i];
            }
        }
        x8<E> qn[kSlots], t0[NC], t1[NC], u0[NC], u1[NC];             // row operands; transposed dO and Q
        f32x16 pr;
        auto probability = [&](int r) {
            pr[r] = __builtin_amdgcn_exp2f(fmaf(s_[r], c2, l4[r >> 2][r & 3]));
            if (MASKED && qbeg + kTile * t + 8 * (r >> 2) + 4 * half + (r & 3) < key) pr[r] = 0.f;
        };
        products<NK>([&](int ks, int i) { qn[i] = ad.nat(Qs, 0, ks); }, [&](int ks, int i) { s_ = MFMA(qn[i], kf[ks], s_); });
        if constexpr (DK)                                        // the exponentials between the products of dP
            products<NK>([&](int ks, int i) { qn[i] = ad.nat(dOs, 0, ks); },
                         [&](int ks, int i) {
                             dp = MFMA(qn[i], vf[ks], dp);
#pragma unroll
                             for (int r = ks * 16 / NK; r < (ks + 1) * 16 / NK; ++r) probability(r);
                         });
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (DV) t0[c] = ad.tr(dOs, c, 0);
            if constexpr (DK) u0[c] = ad.tr(Qs, c, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if constexpr (!DK) probability(r);
            else s_[r] = scale_first<E>() ? pr[r] * scale * dp[r] : pr[r] * dp[r];
        }
        const x8<E> p0 = pack16<E>(pr, 0), p1 = pack16<E>(pr, 1);
        x8<E> s0 = p0, s1 = p1;
        if constexpr (DK) {
            s0 = pack16<E>(s_, 0);
            s1 = pack16<E>(s_, 1);
        }
        if constexpr (DV) wait_tr_reads(t0);
        if constexpr (DK) wait_tr_reads(u0);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (DV) {
                dv[c] = MFMA(t0[c], p0, dv[c]);
                t1[c] = ad.tr(dOs, c, 1);
            }
            if constexpr (DK) {
                dk[c] = MFMA(u0[c], s0, dk[c]);
                u1[c] = ad.tr(Qs, c, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (DV) wait_tr_reads(t1);
        if constexpr (DK) wait_tr_reads(u1);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (DV) dv[c] = MFMA(t1[c], p1, dv[c]);
            if constexpr (DK) dk[c] = MFMA(u1[c], s1, dk[c]);
        }
    };
    // two loops in sequence: with two paths through the matrix instructions in one, their accumulators are copied at every iteration
    int t = 0;
    for (; t < (causal ? 4 : 0) && t < ntiles; ++t) {           // the diagonal part
        advance(t);
        if (qbeg + kTile * t < kw0) continue;                    // all its queries precede this wavefront's keys
        unit(t, std::true_type{});
    }
    for (; t < ntiles; ++t) {
        advance(t);
        unit(t, std::false_type{});
    }
    if (!kvalid) return;
    E *orow = dqkv + ((size_t)b * sh.s + key) * pitch + (size_t)h * dh;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = c * 32 + 8 * g + 4 * half;
            if (col >= dh) continue;
            x4<E> o;
            if constexpr (DK) {
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = (E)(dk[c][4 * g + i] * (scale_first<E>() ? 1.f : scale));
                *reinterpret_cast<x4<E> *>(orow + d + col) = o;
            }
            if constexpr (DV) {
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = (E)dv[c][4 * g + i];
                *reinterpret_cast<x4<E> *>(orow + 2 * d + col) = o;
            }
        }
}

// Explicit instantiations: the host compiler does not always find a kernel template from its use in the launchers below alone.
#define LGA_WIDE_KERNELS(DH, E)                                                                                  \
    template __global__ void attn_wide_fwd_kernel<DH, E>(const E *, E *, float *, AttnShape);                   \
    template __global__ void attn_wide_dq_kernel<DH, true, E>(const E *, const E *, const float *, float *, const E *, E *, AttnShape); \
    template __global__ void attn_wide_dq_kernel<DH, false, E>(const E *, const E *, const float *, float *, const E *, E *, AttnShape)
#define LGA_WIDE_DKV(DH, WHAT, E) \
    template __global__ void attn_wide_dkv_kernel<DH, WHAT, E>(const E *, const float *, const float *, const E *, E *, AttnShape)
#define LGA_WIDE_TYPE(E)          \
    LGA_WIDE_KERNELS(192, E);     \
    LGA_WIDE_KERNELS(224, E);     \
    LGA_WIDE_KERNELS(256, E);     \
    LGA_WIDE_KERNELS(320, E);     \
    LGA_WIDE_DKV(192, kBoth, E);   \
    LGA_WIDE_DKV(224, kBoth, E); \
    LGA_WIDE_DKV(256, kOnlyDV, E); \
    LGA_WIDE_DKV(256, kOnlyDK, E); \
    LGA_WIDE_DKV(320, kOnlyDV, E); \
    LGA_WIDE_DKV(320, kOnlyDK, E)
LGA_WIDE_TYPE(bf16);
LGA_WIDE_TYPE(f16);
#undef LGA_WIDE_TYPE
#undef LGA_WIDE_DKV
#undef LGA_WIDE_KERNELS

template <int DH> constexpr int smem_fwd() { return fwd_stages<DH>() * stage_elems<DH>() * 2; }
template <int DH> constexpr int smem_dq() { return 3 * stage_elems<DH>() * 2; }
template <int DH> constexpr int smem_dkv() { return 3 * stage_elems<DH>() * 2 + 3 * 64 * 4; }

template <class K> hipError_t raise(K kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}
template <int DH, class E> hipError_t raise_dh() {
    hipError_t e = raise(attn_wide_fwd_kernel<DH, E>, smem_fwd<DH>());
    auto next = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    next(raise(attn_wide_dq_kernel<DH, true, E>, smem_dq<DH>()));
    next(raise(attn_wide_dq_kernel<DH, false, E>, smem_dq<DH>()));
    if constexpr (dkv_in_one_run<DH>()) {
        next(raise(attn_wide_dkv_kernel<DH, kBoth, E>, smem_dkv<DH>()));
    } else {
        next(raise(attn_wide_dkv_kernel<DH, kOnlyDV, E>, smem_dkv<DH>()));
        next(raise(attn_wide_dkv_kernel<DH, kOnlyDK, E>, smem_dkv<DH>()));
    }
    return e;
}
template <class E> hipError_t raise_type() {
    hipError_t e = raise_dh<192, E>();
    if (e == hipSuccess) e = raise_dh<224, E>();
    if (e == hipSuccess) e = raise_dh<256, E>();
    if (e == hipSuccess) e = raise_dh<320, E>();
    return e;
}

template <int DH, class E> void fwd_dh(const E *qkv, E *out, float *lse, AttnShape sh, hipStream_t s) {
    const dim3 grid((unsigned)(sh.n_seq * sh.heads) * ((sh.s + 127) / 128));
    char name[64];
    snprintf(name, sizeof(name), "attn_wide_fwd_kernel<%d>", DH);
    const double pairs = (double)sh.n_seq * sh.heads * sh.s * sh.s * (sh.causal ? 0.5 : 1.0), act = (double)sh.n_seq * sh.s * sh.heads * sh.dh * 2.0;
    ProfScope scope(name, 4.0 * pairs * sh.dh, 4.0 * act, s);
    hipLaunchKernelGGL((attn_wide_fwd_kernel<DH, E>), grid, dim3(256), smem_fwd<DH>(), s, qkv, out, lse, sh);
}
template <int DH, class E>
void bwd_dh(const E *qkv, const E *out, const float *lse, float *delta, const E *dout, E *dqkv, AttnShape sh, hipStream_t s) {
    const dim3 grid((unsigned)(sh.n_seq * sh.heads) * ((sh.s + 127) / 128));
    char name[64];
    const double pairs = (double)sh.n_seq * sh.heads * sh.s * sh.s * (sh.causal ? 0.5 : 1.0), act = (double)sh.n_seq * sh.s * sh.heads * sh.dh * 2.0;
    {
        snprintf(name, sizeof(name), "attn_wide_dq_kernel<%d>", DH);
        ProfScope scope(name, 6.0 * pairs * sh.dh, 6.0 * act, s);
        const auto kernel = out ? attn_wide_dq_kernel<DH, true, E> : attn_wide_dq_kernel<DH, false, E>;
        hipLaunchKernelGGL(kernel, grid, dim3(256), smem_dq<DH>(), s, qkv, out, lse, delta, dout, dqkv, sh);
    }
    snprintf(name, sizeof(name), "attn_wide_dkv_kernel<%d>", DH);
    ProfScope scope(name, (dkv_in_one_run<DH>() ? 8.0 : 10.0) * pairs * sh.dh, 6.0 * act, s);
    if constexpr (dkv_in_one_run<DH>()) {
        hipLaunchKernelGGL((attn_wide_dkv_kernel<DH, kBoth, E>), grid, dim3(256), smem_dkv<DH>(), s, qkv, lse, delta, dout, dqkv, sh);
    } else {
        hipLaunchKernelGGL((attn_wide_dkv_kernel<DH, kOnlyDV, E>), grid, dim3(256), smem_dkv<DH>(), s, qkv, lse, delta, dout, dqkv, sh);
        hipLaunchKernelGGL((attn_wide_dkv_kernel<DH, kOnlyDK, E>), grid, dim3(256), smem_dkv<DH>(), s, qkv, lse, delta, dout, dqkv, sh);
    }
}

}  // namespace

bool attn_wide_supports(int dh) { return dh > 160 && dh <= 320 && dh % 8 == 0; }

hipError_t attn_wide_prepare_kernels() {
    hipError_t e = raise_type<bf16>();
    if (e == hipSuccess) e = raise_type<f16>();
    return e;
}

template <class E> void launch_attn_fwd_wide(const E *qkv, E *out, float *lse, AttnShape sh, hipStream_t s) {
    if (sh.n_seq == 0 || sh.s == 0) return;
    (void)prepare_kernels();
    if (sh.dh <= 192) fwd_dh<192, E>(qkv, out, lse, sh, s);
    else if (sh.dh <= 224) fwd_dh<224, E>(qkv, out, lse, sh, s);
    else if (sh.dh <= 256) fwd_dh<256, E>(qkv, out, lse, sh, s);
    else fwd_dh<320, E>(qkv, out, lse, sh, s);
}
template <class E>
void launch_attn_bwd_wide(const E *qkv, const E *out, const float *lse, const E *dout, E *dqkv, float *delta, AttnShape sh, hipStream_t s) {
    if (sh.n_seq == 0 || sh.s == 0) return;
    (void)prepare_kernels();
    out = delta_apart<E>(out, dout, dqkv, delta, sh, s);
    if (sh.dh <= 192) bwd_dh<192, E>(qkv, out, lse, delta, dout, dqkv, sh, s);
    else if (sh.dh <= 224) bwd_dh<224, E>(qkv, out, lse, delta, dout, dqkv, sh, s);
    else if (sh.dh <= 256) bwd_dh<256, E>(qkv, out, lse, delta, dout, dqkv, sh, s);
    else bwd_dh<320, E>(qkv, out, lse, delta, dout, dqkv, sh, s);
}
#define LGA_INSTANTIATE_WIDE(E)                                                                        \
    template void launch_attn_fwd_wide<E>(const E *, E *, float *, AttnShape, hipStream_t);             \
    template void launch_attn_bwd_wide<E>(const E *, const E *, const float *, const E *, E *, float *, \
                                          AttnShape, hipStream_t)
LGA_INSTANTIATE_WIDE(bf16);
LGA_INSTANTIATE_WIDE(f16);
#undef LGA_INSTANTIATE_WIDE

}  // namespace lga
