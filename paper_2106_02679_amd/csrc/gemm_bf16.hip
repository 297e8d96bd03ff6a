// 16-bit MFMA GEMMs for gfx950, fp32 accumulate: C[M,N] = sum_k A(m,k) B(k,n) + epilogue.
// Every kernel here takes the element type E as its last template argument: bf16 (the default 16-bit mode, from
// which the kernels have their names) or f16 (IEEE half); the two differ in the matrix instruction and in the
// conversions of the epilogues, nothing else.
//
// The three GEMM families of a transformer layer (appendix C.1: each is 2 flop per token per parameter)
//   forward          Y[t,out]  = X[t,in]  W[in,out]
//   input gradient   dX[t,in]  = dY[t,out] W[in,out]^T
//   weight gradient  dW[in,out] (+)= X[t,in]^T dY[t,out]      K = tokens of the micro-batch group
// The layer stack runs the first two with BOTH operands k-contiguous (it keeps a transposed 16-bit copy of every weight
// matrix), the third with both as stored, [k][in] and [k][out], where it is large enough for 256 x 256 tiles, and on transposed
// copies otherwise.  All of these are served by gemm_bf16_dma_kernel: 256 threads = 4 wavefronts (2x2) on a 256x256x64 tile - or
// 256x192, 256x128 where those fill the last round of tiles better -, v_mfma_f32_16x16x32_bf16, tiles moved global -> LDS without passing
// through registers.
//
// Most problems with fewer than 128 tiles of 256x256 go to gemm_small.hip.
//
// gemm_bf16_kernel is the register-staged predecessor and still serves the other operand layouts of
// the op-level API and of the GEMM-built attention: both operands sit in LDS k-contiguous
// (8 chunks of 16 B per row, XOR-swizzled against bank conflicts), so every MFMA operand is one 16-byte
// LDS read; an operand that is not k-contiguous in HBM is transposed in registers (8x8 blocks of 16-bit
// values) on its way from global memory to LDS; two LDS stages; the global loads of tile k+1 are in
// flight while tile k is multiplied.
//
// Common to both: the MFMA is issued with the B tile as its first operand so that each lane ends up with
// 4 consecutive n of one row m (row-major stores of 8 bytes (bf16) or 16 bytes (fp32) per lane, epilogues
// fused); workgroup ids are remapped so that each XCD (ids are dealt round-robin over the 8 XCDs) works on
// a contiguous range of tiles, walked in groups of 8 tile-rows for L2 reuse - or, in the direct-to-LDS kernel on
// tile grids made of whole 16 x 16 blocks, so that all XCDs work on one such block at a time.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

#include "gemm16.h"
#include "kernels.h"

namespace lga {

namespace {


__device__ __forceinline__ int swz(int row) { return ((row >> 1) ^ (row >> 4)) & 7; }

// LDS tile: rows x 64 bf16, row pitch 128 B, chunk c of row r stored at chunk c ^ swz(r).
__device__ __forceinline__ int lds_off(int row, int chunk) { return row * BK + ((chunk ^ swz(row)) << 3); }

// 8x8 transpose of 16-bit values held as 8 rows of 4 dwords.  in[r][q] holds (row r, cols 2q, 2q+1);
// out[c][p] holds (col c, rows 2p, 2p+1).
__device__ __forceinline__ void transpose8x8(const u32x4 (&in)[8], u32x4 (&out)[8]) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t x = in[2 * p][q], y = in[2 * p + 1][q];
            out[2 * q][p] = (x & 0xFFFFu) | (y << 16);
            out[2 * q + 1][p] = (x >> 16) | (y & 0xFFFF0000u);
        }
    }
}

// Global -> register staging of one operand tile (ROWS logical rows x 64 k) through buffer loads.
// The buffer resource is re-based to the tile's (row0, k0) origin for every k tile, so per-lane
// offsets stay small and loop-invariant; a lane whose row or k index is out of range gets an
// offset beyond num_records, for which the hardware returns zeros without touching memory.
//   KMAJOR: storage [rows][ld], k contiguous.  Thread t: chunk t%8, rows t/8 + 32*i.
//   else:   storage [k][ld], row index contiguous.  Thread t owns the 8x8 block with rows
//           8*(t%(ROWS/8)).., k 8*(t/(ROWS/8)).., transposed in registers before the LDS store.
template <int ROWS, bool KMAJOR> struct Stager {
    static constexpr int NV = KMAJOR ? ROWS / 32 : 8;
    static constexpr int NOFF = KMAJOR ? NV : 1;
    static_assert(KMAJOR || ROWS <= 256, "one 8x8 block per thread");
    u32x4 v[NV];
    int off[NOFF];       // per-load byte offset inside the tile, or the poison offset for invalid rows
    int ld2;             // leading dimension in bytes

    __device__ __forceinline__ void init(int ld, int row0, int nrows) {
        const int tid = threadIdx.x;
        ld2 = ld * 2;
        if constexpr (KMAJOR) {
            const int voff = (tid >> 3) * ld2 + (tid & 7) * 16;
#pragma unroll
            for (int i = 0; i < NV; ++i) off[i] = (row0 + (tid >> 3) + 32 * i < nrows) ? voff : kBufPoison;
        } else {
            constexpr int CB = ROWS / 8;
            const int r = (tid % CB) * 8, kb = tid / CB;
            off[0] = (tid < ROWS && row0 + r < nrows) ? kb * 8 * ld2 + r * 2 : kBufPoison;
        }
    }

    // base: address of element (row0, k0) of the operand.  Full k tile: no k test.
    __device__ __forceinline__ void load(const void *base) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(base);
        if constexpr (KMAJOR) {
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, off[i], i * 32 * ld2, 0);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, off[0], j * ld2, 0);
        }
    }

    // Last, partial k tile: krem = K - k0 < 64 valid k; the rest reads as zero.
    __device__ __forceinline__ void load_tail(const void *base, int krem) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(base);
        const int tid = threadIdx.x;
        if constexpr (KMAJOR) {
            const int kmask = ((tid & 7) * 8 < krem) ? 0 : kBufPoison;     // OR-ing the poison keeps it out of range
#pragma unroll
            for (int i = 0; i < NV; ++i)
                v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, off[i] | kmask, i * 32 * ld2, 0);
        } else {
            constexpr int CB = ROWS / 8;
            const int kb = tid / CB;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int kmask = (kb * 8 + j < krem) ? 0 : kBufPoison;
                v[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, off[0] | kmask, j * ld2, 0);
            }
        }
    }

    template <class E> __device__ __forceinline__ void store(E *lds) const {
        const int tid = threadIdx.x;
        if constexpr (KMAJOR) {
            const int chunk = tid & 7;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int r = (tid >> 3) + 32 * i;
                *reinterpret_cast<u32x4 *>(lds + lds_off(r, chunk)) = v[i];
            }
        } else {
            constexpr int CB = ROWS / 8;
            if (ROWS >= 256 || tid < ROWS) {
                u32x4 out[8];
                transpose8x8(v, out);
                const int r = (tid % CB) * 8, kb = tid / CB;
#pragma unroll
                for (int c = 0; c < 8; ++c) *reinterpret_cast<u32x4 *>(lds + lds_off(r + c, kb)) = out[c];
            }
        }
    }
};

template <int BM, int BN, bool A_KM, bool B_KM, int EPI, class E>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmParams<E> p, int tiles_m, int tiles_n) {
    constexpr int WM = BM / 2, WN = BN / 2;     // wavefront tile
    constexpr int FM = WM / 32, FN = WN / 32;   // 32x32 MFMA blocks per wavefront
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);
    // stage s: A at s*(BM+BN)*BK, B right after it
    auto As = [&](int s) { return lds + (size_t)s * (BM + BN) * BK; };
    auto Bs = [&](int s) { return lds + (size_t)s * (BM + BN) * BK + BM * BK; };

    // ---- workgroup -> tile, XCD-aware ----------------------------------------------------
    const int ntiles = tiles_m * tiles_n;
    int tile = xcd_contiguous(p.batch > 1 ? ntiles * p.batch : ntiles);      // a batch is ntiles work items per problem
    if (p.batch > 1) select_problem(p, tile, ntiles);
    constexpr int GROUP_M = 8;
    const int group_size = GROUP_M * tiles_n;
    const int gid = tile / group_size;
    const int first_m = gid * GROUP_M;
    const int gsz = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (tile % group_size) % gsz;
    const int tn = (tile % group_size) / gsz;
    const int m0 = tm * BM, n0 = tn * BN;
    if (p.tri == 1 && n0 >= m0 + BM) return;             // whole workgroup: the tile lies above the diagonal

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 31, lhalf = lane >> 5;

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    Stager<BM, A_KM> sa;
    Stager<BN, B_KM> sb;
    sa.init(p.lda, m0, p.M);
    sb.init(p.ldb, n0, p.N);
    // element (row0, k) of each operand: k-major rows advance by 1 per k, the others by ld per k
    const E *a_ptr = A_KM ? p.A + (size_t)m0 * p.lda : p.A + m0;
    const E *b_ptr = B_KM ? p.B + (size_t)n0 * p.ldb : p.B + n0;
    const size_t a_step = A_KM ? (size_t)BK : (size_t)BK * p.lda;
    const size_t b_step = B_KM ? (size_t)BK : (size_t)BK * p.ldb;
    if (p.tri == 2) p.K = min(p.K, m0 + BM);
    if (p.tri == 3) {
        const int skip = min(m0, p.K) / BK;              // whole k tiles before the tile's first row
        a_ptr += skip * a_step;
        b_ptr += skip * b_step;
        p.K -= skip * BK;
    }
    const int nk = (p.K + BK - 1) / BK, nk_full = p.K / BK;
    auto load_tile = [&](int t) {
        if (t < nk_full) {
            sa.load(a_ptr + (size_t)t * a_step);
            sb.load(b_ptr + (size_t)t * b_step);
        } else {
            sa.load_tail(a_ptr + (size_t)t * a_step, p.K - t * BK);
            sb.load_tail(b_ptr + (size_t)t * b_step, p.K - t * BK);
        }
    };

    x8<E> af[2][FM], bf[2][FN];
    auto load_frags = [&](int buf, const E *a_lds, const E *b_lds, int ks) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
            af[buf][i] = *reinterpret_cast<const x8<E> *>(a_lds + lds_off(wm * WM + i * 32 + lrow, 2 * ks + lhalf));
#pragma unroll
        for (int j = 0; j < FN; ++j)
            bf[buf][j] = *reinterpret_cast<const x8<E> *>(b_lds + lds_off(wn * WN + j * 32 + lrow, 2 * ks + lhalf));
    };

    load_tile(0);
    sa.store(As(0));
    sb.store(Bs(0));
    __syncthreads();
    load_frags(0, As(0), Bs(0), 0);

    // MFMAs of one k step for accumulator rows [i0, i1) of the wavefront tile
    auto mfma_rows = [&](int fb, int i0, int i1) {
#pragma unroll
        for (int i = i0; i < i1; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = mfma_32x32x16<E>(bf[fb][j], af[fb][i], acc[i][j]);
    };
    auto mfma_step = [&](int fb) { mfma_rows(fb, 0, FM); };

    // Instruction-mix hints for the scheduler (masks: 0x008 MFMA, 0x020 VMEM read, 0x100 LDS read,
    // 0x200 LDS write): spread the memory instructions of a k step evenly under its MFMAs.  A CU's
    // texture-address unit takes 16 cycles per 16-byte-per-lane load, so the global loads are
    // issued at no more than one per two MFMAs (64 cycles) per wavefront.
    constexpr int NMF = FM * FN, NDR = FM + FN;
    constexpr int NVA = Stager<BM, A_KM>::NV, NVB = Stager<BN, B_KM>::NV;
    constexpr bool kHints = NMF % NDR == 0 && NMF % NVA == 0 && NMF % NVB == 0 && FM % 2 == 0 &&
                            (NMF / 2) % NDR == 0 && (NVA + NVB) % (NMF / 2) == 0;

    int kt = 0;
    // Main loop: the next k tile exists and is full, so the body is straight-line code.
    //   step 0 : MFMAs | global loads of A(kt+1) | LDS reads of step 1's operands
    //   step 1 : MFMAs | global loads of B(kt+1) | LDS reads of step 2's operands
    //   step 2 : MFMAs | LDS reads of step 3's operands
    //   step 3a: first half of the MFMAs | LDS writes of tile kt+1 into the other stage
    //   barrier
    //   step 3b: second half of the MFMAs | LDS reads of tile kt+1's step-0 operands
    for (; kt + 1 < nk_full; ++kt) {
        const int cur = kt & 1;
        const E *a_lds = As(cur), *b_lds = Bs(cur);
        E *a_nxt = As(cur ^ 1), *b_nxt = Bs(cur ^ 1);

        sa.load(a_ptr + (size_t)(kt + 1) * a_step);
        load_frags(1, a_lds, b_lds, 1);
        mfma_step(0);
        if constexpr (kHints) {
#pragma unroll
            for (int i = 0; i < NMF; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (i % (NMF / NVA) == 0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                if (i % (NMF / NDR) == 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        sb.load(b_ptr + (size_t)(kt + 1) * b_step);
        load_frags(0, a_lds, b_lds, 2);
        mfma_step(1);
        if constexpr (kHints) {
#pragma unroll
            for (int i = 0; i < NMF; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (i % (NMF / NVB) == 0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                if (i % (NMF / NDR) == 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        load_frags(1, a_lds, b_lds, 3);
        mfma_step(0);
        if constexpr (kHints) {
#pragma unroll
            for (int i = 0; i < NDR; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, NMF / NDR, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        sa.store(a_nxt);
        sb.store(b_nxt);
        mfma_rows(1, 0, FM / 2);
        if constexpr (kHints) {
#pragma unroll
            for (int i = 0; i < NMF / 2; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x200, (NVA + NVB) / (NMF / 2), 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);

        load_frags(0, a_nxt, b_nxt, 0);
        mfma_rows(1, FM / 2, FM);
        if constexpr (kHints) {
#pragma unroll
            for (int i = 0; i < NDR; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, NMF / 2 / NDR, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // Remaining tiles (the last full one, and a partial one if K is not a multiple of 64).
    for (; kt < nk; ++kt) {
        const int cur = kt & 1;
        const bool more = kt + 1 < nk;
        if (more) load_tile(kt + 1);
        const E *a_lds = As(cur), *b_lds = Bs(cur);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int fb = ks & 1;
            if (ks + 1 < BK / 16) {
                load_frags(fb ^ 1, a_lds, b_lds, ks + 1);
            } else {
                if (more) {
                    sa.store(As(cur ^ 1));
                    sb.store(Bs(cur ^ 1));
                }
                __syncthreads();
                if (more) load_frags(fb ^ 1, As(cur ^ 1), Bs(cur ^ 1), 0);
            }
            mfma_step(fb);
        }
    }

    // ---- epilogue: lane holds row m = lrow, columns n = 8*q + 4*lhalf + (0..3) of each 32x32 block
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = m0 + wm * WM + i * 32 + lrow;
        if (m >= p.M) continue;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + wn * WN + j * 32 + 8 * q + 4 * lhalf;
                if (n >= p.N) continue;
                const float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                epilogue4<EPI, E>(p, m, n, v);
            }
        }
    }
}

// ============================================================================================
// Both operands k-contiguous: global -> LDS without passing through registers.
//
// `buffer_load_dwordx4 ... lds` writes lane L's 16 bytes at (LDS base in M0) + 16 L, so one
// wavefront instruction fills 8 consecutive 128-byte tile rows.  The XOR swizzle of the tile is
// obtained on the global side: lane L, which lands in physical chunk L%8 of row r, fetches logical
// chunk (L%8) ^ swz16(r) of that row.  No staging registers, no LDS store instructions, no waits on
// individual loads: the next k tile streams into the other LDS stage while this one is multiplied,
// and one vmcnt wait + barrier per tile publishes it.
//
// The matrix instruction is v_mfma_f32_16x16x32 (a wavefront's 128 x 128 tile = 8 x 8 blocks of 16 x 16, four
// accumulator registers each), not the 32x32x16 one: same flops per cycle and the same LDS operand bytes per k tile,
// twice the 16-bit operand registers read per flop, but a quarter of the fp32 accumulator registers read and written
// per instruction, half per flop (a 16 x 16 block stays in the pipe for 32 k, a 32 x 32 block for 16) - 0.5 instead of
// 0.625 register bytes per multiply-add.  The chip is power-limited on this kernel, and at the board's limit the
// clock it grants is what that difference in power per cycle buys: measured on a merged weight-gradient shape of
// d = 12288 at sustained load and the same 1.35 kW, the 32x32x16 form of this loop ran at 1.50 GHz (1.37 PFLOP/s) and
// this one runs at 1.65 GHz (1.56 PFLOP/s), both with the matrix pipe busy in 0.9 of the cycles.  For the same reason
// the two products that a block receives per k tile are issued back to back (see `half` in the kernel): the second finds
// the accumulator still in the pipe.

//
// TN: the same loop for operands that are m- and n-contiguous ([k][ld], a weight gradient's activations and output
// gradients as the layer stores them).  An operand tile is then 64 k rows of 256 elements: a DMA instruction fills two of
// its 512-byte rows, and ds_read_b64_tr_b16 transposes on the way to the registers - twice the LDS read instructions of
// half the width.  A wavefront's read covers 8 rows x 32 bytes per cycle, so 32-byte segment g of row r is stored at
// segment g ^ (r & 7): 8 rows, 8 different bank groups.  A lane's 8 k values of a step are rows 4 lq .. + 3 and 16 + 4 lq .. + 3,
// for both operands alike.  The loop runs no slower for it: the four weight gradients of a d = 768 layer over 32768 tokens take 104 us
// each on average, 107 in the k-contiguous form - and the transposing passes before those took 330 us more, at the rate of a copy.
// With the bias gradients' column sums in a pass of their own (99 us; they rode along with the transposes) the layer's backward
// went from 2.26 to 1.93 ms; a training step of a d = 2048 layer over 65536 tokens from 25.0 to 24.0 ms, of a d = 12288 layer
// over 16384 from 160.4 to 158.8.
// It takes a group of weight gradients in one launch, for layers whose matrices do not fill the chip one by one: workgroups are dealt
// to the problems in order, each problem's slices as in a launch of its own.
template <class E, bool TN> using DmaInput = std::conditional_t<TN, GemmGroup<E>, GemmParams<E>>;
template <int BM, int BN, int WGM, int WGN, int EPI, class E, bool TN>
__device__ __forceinline__ void dma_tile_product(const DmaInput<E, TN> &in, int tiles_m, int tiles_n) {
    constexpr int NW = WGM * WGN;                   // wavefronts per workgroup, WGM x WGN over the tile
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / 16, FN = WN / 16;       // 16 x 16 blocks of a wavefront's tile
    constexpr int NIA = BM / (8 * NW), NIB = BN / (8 * NW);     // DMA instructions per wavefront per operand tile
    static_assert(BN <= BM && (!TN || BM == BN), "the operand ring below uses A's slot size for both operands");
    static_assert(BK == 64, "two k steps of 32 per tile");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    E *lds = reinterpret_cast<E *>(smem_raw);
    // LDS is a ring of kSlots operand tiles of BM x BK.  Operand tiles enter it in the order A(0), B(0), A(1),
    // B(1), ...: A(kt) sits in slot (2 kt) mod kSlots and B(kt) in the next one.  Five slots hold two whole k
    // tiles plus half of a third, which is what lets the loads of A(kt+2) start before tile kt is retired.
    constexpr int kSlots = 5;
    constexpr int kSlotElems = BM * BK;
    auto slot = [&](int q) { return lds + q * kSlotElems; };
    auto wrap = [](int q) { return q >= kSlots ? q - kSlots : q; };

    GemmParams<E> p;
    int tile;
    if constexpr (TN) {
        tile = xcd_contiguous(gridDim.x);
        p = select_from_group<BM, BN>(in, tile, tiles_m, tiles_n);
    } else {
        p = in;
        // with a split k range there are ksplit work items per tile, slice-major
        tile = xcd_contiguous(tiles_m * tiles_n * ((EPI == EPI_ACCUM_F32 && p.ksplit > 1) ? p.ksplit : p.batch > 1 ? p.batch : 1));
    }
    const int ntiles = tiles_m * tiles_n;
    if (!TN && p.batch > 1) select_problem(p, tile, ntiles);
    if constexpr (EPI == EPI_ACCUM_F32) {
        if (p.ksplit > 1) {
            // this workgroup multiplies slice z of the k range into partial result z ([M][N], dense)
            const int z = tile / ntiles, k0 = z * p.kchunk;
            tile -= z * ntiles;
            p.A += TN ? (size_t)k0 * p.lda : k0;
            p.B += TN ? (size_t)k0 * p.ldb : k0;
            p.K = min(p.K - k0, p.kchunk);
            p.outf = p.partial + (size_t)z * p.M * p.N;
            p.ldc = p.N;
            p.beta = 0.f;
        }
    }
    constexpr int GROUP_M = 8;
    const int group_size = GROUP_M * tiles_n;
    const int gid = tile / group_size;
    const int first_m = gid * GROUP_M;
    const int gsz = min(tiles_m - first_m, GROUP_M);
    int tm = first_m + (tile % group_size) % gsz;
    int tn = (tile % group_size) / gsz;
    if (p.sblock) {
        // Round r of 256 consecutive workgroup ids is one 16 x 16 block of tiles (blocks walk along n first); XCD
        // x = id mod 8 takes rows 8 (x / 4) .. + 7 and columns 4 (x mod 4) .. + 3 of it.  All 8 XCDs then read the
        // same 16 + 16 operand panels at about the same time, so memory sees each of them once per k step instead of
        // once per XCD or per pass over the other dimension; inside an XCD the footprint is the same 8 x 4 tiles.
        const int pid = blockIdx.x, r = pid >> 8, x = pid & 7, local = (pid >> 3) & 31;
        const int nsn = tiles_n >> 4;
        tm = ((r / nsn) << 4) + ((x >> 2) << 3) + (local & 7);
        tn = ((r % nsn) << 4) + ((x & 3) << 2) + (local >> 3);
    }
    const int m0 = tm * BM, n0 = tn * BN;
    if (!TN && p.tri == 1 && n0 >= m0 + BM) return;      // whole workgroup: the tile lies above the diagonal

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int l16 = lane & 15, lq = lane >> 4;           // lane = 16 lq + l16

    // A lane's part of a 16 x 16 block: column (m) l16, rows (n) 4 lq .. + 3 - the B tile is the instruction's first
    // operand, so a lane ends with 4 consecutive n of one row m of C.
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Loop-invariant per-lane byte offsets of the DMA loads inside an operand tile (or the poison
    // offset for rows beyond the matrix, which the hardware answers with zeros).
    const int lda2 = p.lda * 2, ldb2 = p.ldb * 2;
    // DMA instruction i of a wavefront fills tile rows [(wave NIA + i) 8, + 8): 1 KB of LDS, right behind that of
    // instruction i - 1.  Four consecutive instructions share one LDS base (M0, a scalar write each time it changes)
    // and tell their places apart by the instruction's immediate offset, 1024 (i % 4) - which the hardware adds to the
    // memory address too, so the per-lane offsets have it subtracted.  (A row is at least 128 bytes long here - the
    // launcher sends shorter leading dimensions to the other kernel - so the difference is never negative.)
    // (TN: an instruction fills two rows of 512 bytes, and the launcher sends leading dimensions below 256 elsewhere.)
    auto dma_row = [&](bool is_a, int i) {
        const int instr = wave * (is_a ? NIA : NIB) + i;
        return TN ? instr * 2 + (lane >> 5) : instr * 8 + (lane >> 3);
    };
    int offA[NIA], offB[NIB];
#pragma unroll
    for (int i = 0; i < NIA; ++i) {
        const int r = dma_row(true, i);
        if constexpr (TN) {
            const int chunk = (lane & 31) ^ ((r & 7) << 1);
            offA[i] = (m0 + chunk * 8 < p.M) ? r * lda2 + chunk * 16 - (i & 3) * 1024 : kBufPoison;
        } else offA[i] = (m0 + r < p.M) ? r * lda2 + (((lane & 7) ^ swz16(r)) << 4) - (i & 3) * 1024 : kBufPoison;
    }
#pragma unroll
    for (int i = 0; i < NIB; ++i) {
        const int r = dma_row(false, i);
        if constexpr (TN) {
            const int chunk = (lane & 31) ^ ((r & 7) << 1);
            offB[i] = (n0 + chunk * 8 < p.N) ? r * ldb2 + chunk * 16 - (i & 3) * 1024 : kBufPoison;
        } else offB[i] = (n0 + r < p.N) ? r * ldb2 + (((lane & 7) ^ swz16(r)) << 4) - (i & 3) * 1024 : kBufPoison;
    }
    const E *a_ptr = p.A + (TN ? (size_t)m0 : (size_t)m0 * p.lda);
    const E *b_ptr = p.B + (TN ? (size_t)n0 : (size_t)n0 * p.ldb);
    const size_t a_step = TN ? (size_t)BK * p.lda : BK, b_step = TN ? (size_t)BK * p.ldb : BK;      // elements per k tile
    const int nk = (p.K + BK - 1) / BK, nk_full = p.K / BK;

    typedef __attribute__((address_space(3))) void *lds_ptr;
    // One direct-to-LDS load: instruction i of a wavefront's share of an operand tile into ring slot q.  The LDS base
    // is that of the instruction's group of four; the immediate offset (a literal, hence the switch over a value that
    // is a constant wherever this is called) places it inside the group.
    auto lds_dma = [&](bool is_a, const __amdgpu_buffer_rsrc_t &r, int q, int i, int voff, int soff) {
        E *group = slot(q) + (wave * (is_a ? NIA : NIB) + (i & ~3)) * 8 * BK;
        switch (i & 3) {
            case 0: __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)group, 16, voff, soff, 0, 0); break;
            case 1: __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)group, 16, voff, soff, 1024, 0); break;
            case 2: __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)group, 16, voff, soff, 2048, 0); break;
            default: __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)group, 16, voff, soff, 3072, 0); break;
        }
    };
    // krem < 64 (partial last tile): k chunks at or beyond krem read as zero.
    auto dma_one = [&](bool is_a, int q, int kt, int krem, int i) {
        const __amdgpu_buffer_rsrc_t r = make_rsrc((is_a ? a_ptr : b_ptr) + kt * (is_a ? a_step : b_step));
        int off = is_a ? offA[i] : offB[i];
        if constexpr (TN) {
            if (dma_row(is_a, i) >= krem) off = kBufPoison;
        } else if (krem < BK) off |= ((((lane & 7) ^ swz16(dma_row(is_a, i))) * 8 < krem) ? 0 : kBufPoison);
        lds_dma(is_a, r, q, i, off, 0);
    };
    // MFMA operands of a whole k tile: block f of k step s (32 k each) of A and of B, 128 registers.  A tile is
    // multiplied in two halves of FM/2 A blocks against all FN B blocks, and the two products of a block - k step 0,
    // k step 1 - are issued one right after the other (see `half` below), so both steps' operands of the blocks in
    // work are in registers at once.  The registers are refilled as they fall free: the A blocks of the second half
    // while the first is multiplied, the next tile's first A half while the second is, and the next tile's B
    // blocks column by column behind the second half's walk over them.  Every LDS read is thus at least 18 block
    // pairs (some 580 cycles) ahead of its use, which rides out the LDS latency spikes that the incoming DMA
    // traffic causes.
    x8<E> af[2][FM], bf[2][FN];
    // LDS byte address of an operand chunk.  A lane reads row (block row 0 + l16), logical chunk 4 s + lq of k step
    // s; the swizzle term of that row is l16 >> 1 whatever the block (blocks start at multiples of 16 rows), so the
    // chunk lies at (lane address) ^ (s << 6) plus a compile-time offset for slot and block.
    static_assert(WM % 16 == 0 && WN % 16 == 0, "whole 16 x 16 blocks");
    const int lane_sw = lq ^ (l16 >> 1);
    const int lane_a = ((wm * WM + l16) * BK + lane_sw * 8) * 2;
    const int lane_b = ((wn * WN + l16) * BK + lane_sw * 8) * 2;
    // TN: block f's segment of row r is (8 wm + f) ^ (r & 7), and r & 7 is the lane's whatever the step and half
    const int tn_row = 4 * lq + (l16 >> 2);
    auto tn_lane = [&](int w, int f) { return tn_row * (BM * 2) + w * (WM * 2) + ((f ^ (tn_row & 7)) << 5) + (l16 & 3) * 8; };
    // Rows 4 lq .. + 3 and 16 + 4 lq .. + 3 of column l16 of the block at LDS byte address addr + imm (imm a constant).  In asm: the
    // builtin makes the compiler wait for all direct-to-LDS loads in flight before it.  The result must not be touched before one
    // of the waits below, which name it.
    auto tr_read = [&](int addr, int imm) __attribute__((always_inline)) {
        u32x2 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "i"(imm));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "i"(imm + 16 * BM * 2));
        const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
        return __builtin_bit_cast(x8<E>, v);
    };
    const int lds_base = (int)(uintptr_t)(lds_ptr)smem_raw;
    static_assert(!TN || (WM == 128 && WN == 128), "8 segments per wavefront");
    // operand f of step s (f < FN: B block f, else A block f - FN) of the tile whose A operand is in slot qa
    auto load_frag = [&](int s, int qa, int f) {
        if constexpr (TN) {
            const int step = s * 32 * BM * 2;
            if (f < FN) bf[s][f] = tr_read(lds_base + tn_lane(wn, f) + wrap(qa + 1) * (kSlotElems * 2), step);
            else af[s][f - FN] = tr_read(lds_base + tn_lane(wm, f - FN) + qa * (kSlotElems * 2), step);
            return;
        }
        if (f < FN) {
            const int vb = (lane_b ^ (s << 6)) + wrap(qa + 1) * (kSlotElems * 2);
            bf[s][f] = *reinterpret_cast<const x8<E> *>(smem_raw + vb + f * 16 * BK * 2);
        } else {
            const int g = f - FN, va = (lane_a ^ (s << 6)) + qa * (kSlotElems * 2);
            af[s][g] = *reinterpret_cast<const x8<E> *>(smem_raw + va + g * 16 * BK * 2);
        }
    };
    // The same operation for the unrolled main loop, where the ring slot is a compile-time constant.  A wavefront
    // issues strictly in order and, being alone on its SIMD, has nobody to fill the matrix pipe while it issues
    // anything else: measured (32x32x16 form of this loop), 126 other instructions per k tile made a k tile take 2400
    // cycles where its MFMAs need 2048, 64 of them about 2230.  So the loop keeps nothing but the loads themselves:
    //  - LDS operand reads take their address from one of 12 registers set up once - (lane address ^ step term) for
    //    the two steps, in each of the three 64 KB ranges an immediate offset reaches - plus an immediate offset: no
    //    address arithmetic per read;
    //  - the direct-to-LDS loads use one buffer resource per operand for the whole tile and take the k position from
    //    a scalar offset that advances once per k tile; the LDS destination is a constant.
    // (TN: the swizzle makes one lane address per block, 48 registers.)
    constexpr int kLanes = TN ? FM : 2;
    int pa[kLanes][3], pb[kLanes][3];
#pragma unroll
    for (int v = 0; v < kLanes; ++v)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            pa[v][r] = (TN ? lds_base + tn_lane(wm, v) : lane_a ^ (v << 6)) + r * 65536;
            pb[v][r] = (TN ? lds_base + tn_lane(wn, v) : lane_b ^ (v << 6)) + r * 65536;
            // opaque to the compiler, which would otherwise fold the range into each read's offset and add it back
            // with a VALU instruction per read
            asm volatile("" : "+v"(pa[v][r]), "+v"(pb[v][r]));
        }
    auto load_frag_c = [&](int s, int qa, int f) {           // qa: a constant at every call
        const bool is_b = f < FN;
        const int blk = is_b ? f : f - FN;
        if constexpr (TN) {
            const int at = (is_b ? wrap(qa + 1) : qa) * (kSlotElems * 2) + s * 32 * BM * 2;
            const x8<E> v = tr_read(is_b ? pb[blk][at >> 16] : pa[blk][at >> 16], at & 0xFFFF);
            if (is_b) bf[s][blk] = v;
            else af[s][blk] = v;
            return;
        }
        const int off = (is_b ? wrap(qa + 1) : qa) * (kSlotElems * 2) + blk * 16 * BK * 2;      // below 160 KB
        const unsigned char *src = smem_raw + (is_b ? pb[s][off >> 16] : pa[s][off >> 16]) + (off & 0xFFFF);
        if (is_b) bf[s][blk] = *reinterpret_cast<const x8<E> *>(src);
        else af[s][blk] = *reinterpret_cast<const x8<E> *>(src);
    };
    const __amdgpu_buffer_rsrc_t rsA = make_rsrc(a_ptr), rsB = make_rsrc(b_ptr);
    // TN: where k tile kt + 2 of the main loop begins; a tile's rows reach too far for a scalar offset, so each tile has its resource
    const E *a_run = a_ptr + 2 * a_step, *b_run = b_ptr + 2 * b_step;
    // DMA instruction i of a full k tile of A or B into (constant) ring slot q; koff: byte offset of the k tile in a row
    auto dma_c = [&](bool is_a, int q, int koff, int i) {
        // (two calls: the host pass of the compiler does not take a conditional expression of the resource type)
        const int vo = is_a ? offA[i] : offB[i];
        if constexpr (TN) {
            lds_dma(is_a, make_rsrc(is_a ? a_run : b_run), q, i, vo, 0);
            return;
        }
        if (is_a) lds_dma(true, rsA, q, i, vo, koff);
        else lds_dma(false, rsB, q, i, vo, koff);
    };
    // s_waitcnt immediates (vmcnt in bits 3:0, expcnt 6:4 left at its maximum, lgkmcnt 11:8 = 0): all LDS reads
    // returned and every load landed, or every load but the newest NIA landed.
    constexpr int kWaitVm0 = 0x0070;
    static_assert(NIA < 16, "vmcnt immediate below uses the low four bits only");
    constexpr int kWaitVmA = 0x0070 | NIA;

    // prologue: tile 0 published, tile 1 in flight, tile 0's B blocks and first A half in registers
#pragma unroll
    for (int i = 0; i < NIA; ++i) dma_one(true, 0, 0, p.K, i);
#pragma unroll
    for (int i = 0; i < NIB; ++i) dma_one(false, 1, 0, p.K, i);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    if (nk > 1) {
#pragma unroll
        for (int i = 0; i < NIA; ++i) dma_one(true, 2, 1, p.K - BK, i);
#pragma unroll
        for (int i = 0; i < NIB; ++i) dma_one(false, 3, 1, p.K - BK, i);
    }
#pragma unroll
    for (int f = 0; f < FN + FM / 2; ++f) {
        load_frag(0, 0, f);
        load_frag(1, 0, f);
    }
    // TN: names operands that a wait before it has made valid: A blocks g0 .. g0 + 3 of both steps, B block j of both steps
    auto got_a = [&](int g0) __attribute__((always_inline)) {
        asm volatile("" : "+v"(af[0][g0]), "+v"(af[1][g0]), "+v"(af[0][g0 + 1]), "+v"(af[1][g0 + 1]), "+v"(af[0][g0 + 2]), "+v"(af[1][g0 + 2]),
                          "+v"(af[0][g0 + 3]), "+v"(af[1][g0 + 3]));
    };
    auto got_b = [&](int j) __attribute__((always_inline)) { asm volatile("" : "+v"(bf[0][j]), "+v"(bf[1][j])); };
    // Reads in flight are values the compiler takes for ready: it may copy a register wherever values meet at a loop's edge or leave a loop.
    // So no read is outstanding there: k_tile ends with this wait, and the main loop turns in the middle of a k tile, where
    // the barrier's wait is for every read anyway.
    auto wait_first_half = [&]() __attribute__((always_inline)) {       // what half 0 multiplies
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        got_a(0);
#pragma unroll
        for (int j = 0; j < FN; ++j) got_b(j);
    };
    if constexpr (TN) wait_first_half();

    // Half h of a k tile: A blocks g = 4 h .. 4 h + 3 against all B blocks, column by column (j outer, g inner), and
    // for each block its two products in a row on the same accumulator.  Measured on register operands, a second
    // MFMA on the accumulator of the one just issued costs no cycles and less power than one on another accumulator
    // - the board then grants the clock for it: at the same power, random operands, 2.43 PFLOP/s with strictly
    // adjacent pairs against 2.21 with 64 different accumulators in turn - and in this kernel, on the merged
    // weight-gradient shape of d = 12288 at sustained load, this order gave 1.53 PFLOP/s where the order "all blocks
    // of k step 0, then all of k step 1" gave 1.47 on the same box.
    // Each half also issues its share of the tile's other work, between the pairs and never more than two memory
    // instructions at one place: its 8 direct-to-LDS loads of operand tile `dkt`, one after the first pair of every
    // column; with rd_a, the 8 LDS reads of A blocks ga0 .. ga0 + 3 (both steps) of the tile in slot rqa, after the
    // second and third pair of the first four columns; with rd_b, the two reads of B block j of that tile after the
    // last pair of column j, which was the last use of those registers.
    // The order is pinned (sched_barrier): left to itself the compiler clumps the loads, and a wavefront that issues
    // several in a row right after the barrier, together with the three others, finds the load queue full and
    // stalls with its MFMAs behind it.
    static_assert(NIA == 8 && NIB == FN && FM == 8 && FN >= 4 && FN <= 8, "a load per column of a half or more, four A blocks per half");
    // lean_c: the unrolled main loop's forms of the loads (constant slots; dkt is then the k tile's byte offset)
    auto half = [&](auto lean_c, int h, bool do_dma, bool dma_is_a, int dq, int dkt, int dkrem, bool rd_a, int ga0, bool rd_b,
                    int rqa) __attribute__((always_inline)) {
        constexpr bool LEAN = decltype(lean_c)::value;
#pragma unroll
        for (int pr = 0; pr < 4 * FN; ++pr) {
            const int j = pr >> 2, g = 4 * h + (pr & 3);
            if constexpr (TN && LEAN) {
                // Reads return in order, four a block.  Behind those of column j's B block lie those of the B blocks after it and of
                // the A blocks that this half has asked for so far, 4 (FN - 1 - j) + 4 min(j, FM / 2): fewest in the last
                // column, 4 FM / 2 = 16.  (Behind the A blocks of this half: the last five B blocks'.)
                static_assert(4 * (FM / 2) >= 14 && FN == 8 && FM == 8, "reads behind the ones waited for");
                if (h == 0 && (pr & 3) == 0) {
                    asm volatile("s_waitcnt lgkmcnt(14)" ::: "memory");
                    if (j == 0) got_a(0);
                    got_b(j);
                }
            }
            mfma_16x16x32_acc<E>(bf[0][j], af[0][g], acc[g][j]);
            mfma_16x16x32_acc<E>(bf[1][j], af[1][g], acc[g][j]);
            // loads evenly over the half, one per column where there are as many
            const int nload = dma_is_a ? NIA : NIB, li = (pr * nload + 4 * FN - 1) / (4 * FN);
            if (do_dma && li < nload && li * 4 * FN / nload == pr) {
                if constexpr (LEAN) dma_c(dma_is_a, dq, dkt, li);
                else dma_one(dma_is_a, dq, dkt, dkrem, li);
            }
            if (rd_a && j < 4 && ((pr & 3) == 1 || (pr & 3) == 2)) {
                const int ia = 2 * j + (pr & 3) - 1;                    // 0 .. 7: block ga0 + ia / 2, step ia % 2
                if constexpr (LEAN) load_frag_c(ia & 1, rqa, FN + ga0 + (ia >> 1));
                else load_frag(ia & 1, rqa, FN + ga0 + (ia >> 1));
            }
            if (rd_b && (pr & 3) == 3) {
                if constexpr (LEAN) {
                    load_frag_c(0, rqa, j);
                    load_frag_c(1, rqa, j);
                } else {
                    load_frag(0, rqa, j);
                    load_frag(1, rqa, j);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // One k tile whose A operand is in ring slot qa; its B blocks and first A half are in registers.  STRAIGHT:
    // tiles kt+1 and kt+2 exist and are full, so nothing is tested.
    //   half 0: MFMAs | LDS reads of this tile's second A half | A(kt+2)'s loads, into the free slot
    //   wait for all loads but A(kt+2)'s + barrier: tile kt+1 is published, and nobody reads tile kt's slots
    //   any more
    //   half 1: MFMAs | LDS reads of tile kt+1's first A half and B blocks | B(kt+2)'s loads, into A(kt)'s slot
    auto k_tile = [&](int kt, int qa, auto straight_c) __attribute__((always_inline)) {
        constexpr bool STRAIGHT = decltype(straight_c)::value;
        const bool more1 = STRAIGHT || kt + 1 < nk, more2 = STRAIGHT || kt + 2 < nk;
        const int krem2 = STRAIGHT ? BK : p.K - (kt + 2) * BK;
        const int qa1 = wrap(qa + 2), qa2 = wrap(qa + 4);      // A(kt+1), A(kt+2); B(kt+2) goes to qa

        half(std::false_type{}, 0, more2, true, qa2, kt + 2, krem2, true, FM / 2, false, qa);
        // A bare s_barrier: __syncthreads() would add a fence that waits for every load, A(kt+2)'s included.
        // The LDS reads above must have returned before other wavefronts may overwrite those slots.
        if constexpr (TN) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more2)
            __builtin_amdgcn_s_waitcnt(kWaitVmA);
        else
            __builtin_amdgcn_s_waitcnt(kWaitVm0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (TN) got_a(FM / 2);
        __builtin_amdgcn_sched_barrier(0);
        half(std::false_type{}, 1, more2, false, qa, kt + 2, krem2, more1, 0, more1, qa1);
        if constexpr (TN) wait_first_half();
    };
    // The same k tile for the unrolled main loop, in its two halves: ring slot qa is a constant, tiles kt+1 and kt+2 exist and are
    // full; koff2 is the byte offset of k tile kt+2 within a row.
    auto first_half_c = [&](int qa, int koff2) __attribute__((always_inline)) {
        half(std::true_type{}, 0, true, true, wrap(qa + 4), koff2, BK, true, FM / 2, false, qa);
        __builtin_amdgcn_s_waitcnt(kWaitVmA);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (TN) got_a(FM / 2);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto second_half_c = [&](int qa, int koff2) __attribute__((always_inline)) {
        half(std::true_type{}, 1, true, false, qa, koff2, BK, true, 0, true, wrap(qa + 2));
        if constexpr (TN) {
            a_run += a_step;
            b_run += b_step;
        }
    };
    auto k_tile_c = [&](int qa, int koff2) __attribute__((always_inline)) {
        first_half_c(qa, koff2);
        second_half_c(qa, koff2);
    };
    int kt = 0, qa = 0;
    // Main loop, unrolled over one period of the ring (five k tiles; the slot of A(kt) is 0, 2, 4, 1, 3, 0, ...).
    if constexpr (TN) {
        if (kt + 7 < nk_full) {                              // as below, from the middle of one k tile to the middle of another
            // from here on 64 values in registers of their own, not one zero that the first products' accumulators are copied from
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));
            first_half_c(0, 0);
            for (; kt + 7 < nk_full; kt += 5) {
                second_half_c(0, 0);
                k_tile_c(2, 0);
                k_tile_c(4, 0);
                k_tile_c(1, 0);
                k_tile_c(3, 0);
                first_half_c(0, 0);
            }
            second_half_c(0, 0);
            wait_first_half();
            ++kt;
            qa = 2;
        }
    } else {
        int koff2 = 2 * BK * (int)sizeof(E);
        for (; kt + 6 < nk_full; kt += 5) {
            k_tile_c(0, koff2);
            k_tile_c(2, koff2 + 1 * BK * (int)sizeof(E));
            k_tile_c(4, koff2 + 2 * BK * (int)sizeof(E));
            k_tile_c(1, koff2 + 3 * BK * (int)sizeof(E));
            k_tile_c(3, koff2 + 4 * BK * (int)sizeof(E));
            koff2 += 5 * BK * (int)sizeof(E);
        }
    }
    for (; kt + 2 < nk_full; ++kt, qa = wrap(qa + 2)) k_tile(kt, qa, std::true_type{});      // what is left of the full tiles
    for (; kt < nk; ++kt, qa = wrap(qa + 2)) k_tile(kt, qa, std::false_type{});              // the last tiles, with tests
    // the accumulators' last updates must have left the matrix pipe before anything else reads them (see
    // mfma_16x16x32_acc): twice the longest wait the instruction set asks for after a matrix instruction
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    // ... their spills, too: a value that leaves the registers is this statement's result, not the loop's
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));

    if constexpr (EPI != EPI_ACCUM_F32) {
        // bf16 outputs: a lane holds 4 consecutive n of 64 different (row, column group) places, so storing from
        // the accumulators writes 8-byte runs per row and instruction - partial cache lines that reach memory in
        // pieces (measured with the 32 x 32 blocks: up to 2.3 x the output bytes) and scattered reads of the residual /
        // pre-activation.  Instead each wavefront passes its results, 16 rows at a time, through a private piece of
        // the (now idle) operand ring and stores whole rows: 16 lanes x 16 bytes = 256 contiguous bytes, 4 rows per
        // instruction.
        const auto al16 = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
        const bool wide = ((p.N | p.ldc) & 7) == 0 && al16(p.out) && (EPI != EPI_BIAS_GELU || al16(p.out2)) &&
                          ((EPI != EPI_BIAS_RESID && EPI != EPI_MUL_DGELU) || al16(p.aux)) &&
                          ((EPI != EPI_BIAS && EPI != EPI_BIAS_RESID && EPI != EPI_BIAS_GELU) || al16(p.bias));
        if (wide) {
            constexpr int SP = WN + 4;                                  // staging pitch in floats
            static_assert(NW * 16 * SP * 4 <= 5 * BM * BK * 2, "staging fits in the operand ring");
            // A strip of 16 rows is 2 WN pieces of 8 columns, IT for a lane: piece it x 64 + lane, of row piece / PR.  With 128 columns a lane has the
            // same 8 columns of every row it stores.
            constexpr int PR = WN / 8, IT = 16 * PR / 64, CS = PR == 16 ? 1 : IT;
            static_assert(16 * PR % 64 == 0, "whole pieces");
            auto row_of = [&](int it) { return PR == 16 ? it * 4 + lq : (it * 64 + lane) / PR; };
            auto col_of = [&](int it) { return PR == 16 ? 8 * l16 : (it * 64 + lane) % PR * 8; };
            // The residual / pre-activation values of the whole wavefront tile are requested first - FM x 4 loads of
            // 16 bytes per lane, into registers the main loop no longer needs - so that their latency is paid once,
            // under the staging of the first strip, and not once per strip.
            constexpr bool kReadsAux = EPI == EPI_BIAS_RESID || EPI == EPI_MUL_DGELU;
            x8<E> aux8[kReadsAux ? FM : 1][kReadsAux ? IT : 1];
            // Tiles that lie inside the matrix take a path of their own: a bounds test per row keeps the loads, arithmetic and stores of
            // different rows apart (d = 768 layer over 32768 tokens: GELU 208 -> 201 us, QKV 130 -> 126, W_o 66 -> 64; not the GELU' product, whose
            // registers a second path moves into scratch memory: 258 -> 289).
            const bool inside = EPI != EPI_MUL_DGELU && m0 + BM <= p.M && n0 + BN <= p.N;
            auto request_aux = [&](auto inside_c) __attribute__((always_inline)) {
                if constexpr (kReadsAux) {
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int it = 0; it < IT; ++it) {
                            const int m = m0 + wm * WM + i * 16 + row_of(it), n = n0 + wn * WN + col_of(it);
                            if (decltype(inside_c)::value || (m < p.M && n < p.N)) aux8[i][it] = *reinterpret_cast<const x8<E> *>(p.aux + (size_t)m * p.ldc + n);
                        }
                }
            };
            if constexpr (EPI != EPI_MUL_DGELU) if (inside) request_aux(std::true_type{});
            if (!inside) request_aux(std::false_type{});
            // A lane stores the same 8 columns of every row: their bias values are read once, not once per store (read
            // inside the loop below, each waits out its whole latency between the staging of two strips: 3 us per tile).
            f32x4 bias_lo[CS], bias_hi[CS];
#pragma unroll
            for (int it = 0; it < CS; ++it) {
                bias_lo[it] = bias_hi[it] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU) {
                    const int n = n0 + wn * WN + col_of(it);
                    if (n < p.N) {
                        bias_lo[it] = *reinterpret_cast<const f32x4 *>(p.bias + n);
                        bias_hi[it] = *reinterpret_cast<const f32x4 *>(p.bias + n + 4);
                    }
                }
            }
            __syncthreads();                                            // every wavefront has left the main loop
            float *stage = reinterpret_cast<float *>(smem_raw) + wave * (16 * SP);
            auto stage_strip = [&](int i) {
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    *reinterpret_cast<f32x4 *>(stage + l16 * SP + j * 16 + 4 * lq) = acc[i][j];
            };
            // LDS operations of one wavefront execute in order, so strip i + 1 may be written into the same piece of
            // LDS as soon as the reads of strip i have been ISSUED: its writes then travel under the wait for those
            // reads.  All eight reads of a strip are issued before any of them is used (left inside the bounds test
            // of its row, each pair waited out the LDS latency on its own: 32 times per tile, 3 us of a tile's 5.5).
            // The bias gradient behind a GELU' product is the sum of its columns: each lane adds up its 8 columns over the rows it stores, instead
            // of a pass over the result (32768 x 3072: 44 of the 100 us that a d = 768 layer's four took; 10 here).
            float cols[EPI == EPI_MUL_DGELU ? 8 : 1];
#pragma unroll
            for (float &c : cols) c = 0.f;
            // PRE: GELU's pre-activation is stored
            auto strips = [&](auto inside_c, auto pre_c) __attribute__((always_inline)) {
                constexpr bool INSIDE = decltype(inside_c)::value, PRE = decltype(pre_c)::value;
                stage_strip(0);
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    asm volatile("" ::: "memory");
                    f32x4 lo[IT], hi[IT];
#pragma unroll
                    for (int it = 0; it < IT; ++it) {
                        lo[it] = *reinterpret_cast<const f32x4 *>(stage + row_of(it) * SP + col_of(it));
                        hi[it] = *reinterpret_cast<const f32x4 *>(stage + row_of(it) * SP + col_of(it) + 4);
                    }
                    asm volatile("" ::: "memory");
                    if (i + 1 < FM) stage_strip(i + 1);
                    if constexpr (IT == 4)
                        asm volatile("" : "+v"(lo[0]), "+v"(hi[0]), "+v"(lo[1]), "+v"(hi[1]), "+v"(lo[2]), "+v"(hi[2]), "+v"(lo[3]), "+v"(hi[3]));
                    else if constexpr (IT == 3)
                        asm volatile("" : "+v"(lo[0]), "+v"(hi[0]), "+v"(lo[1]), "+v"(hi[1]), "+v"(lo[2]), "+v"(hi[2]));
                    else
                        asm volatile("" : "+v"(lo[0]), "+v"(hi[0]), "+v"(lo[IT - 1]), "+v"(hi[IT - 1]));
#pragma unroll
                    for (int it = 0; it < IT; ++it) {
                        const int m = m0 + wm * WM + i * 16 + row_of(it), n = n0 + wn * WN + col_of(it);
                        if (INSIDE || (m < p.M && n < p.N)) {
                            x8<E> o8;
                            epilogue8<EPI, PRE, E>(p, m, n, lo[it], hi[it], aux8[kReadsAux ? i : 0][kReadsAux ? it : 0], bias_lo[it % CS],
                                                  bias_hi[it % CS], o8);
                            if (EPI == EPI_MUL_DGELU && PR == 16 && p.colsum) {
#pragma unroll
                                for (int c = 0; c < (EPI == EPI_MUL_DGELU ? 8 : 1); ++c) cols[c] += (float)o8[c];
                            }
                        }
                    }
                }
            };
            auto strips_for = [&](auto inside_c) __attribute__((always_inline)) {
                if constexpr (EPI == EPI_BIAS_GELU) {
                    if (p.out2) strips(inside_c, std::true_type{});
                    else strips(inside_c, std::false_type{});
                } else strips(inside_c, std::false_type{});
            };
            if constexpr (EPI != EPI_MUL_DGELU) if (inside) strips_for(std::true_type{});
            if (!inside) strips_for(std::false_type{});
            if constexpr (EPI == EPI_MUL_DGELU && PR == 16) {
                static_assert(WM == kGemmSumRows, "a wavefront's rows are a chunk");
                if (p.colsum && m0 + wm * WM < p.M) {                    // (uniform)
#pragma unroll
                    for (float &c : cols) c = sum_over_rows_of_16(c);
                    const int n = n0 + wn * WN + 8 * l16;
                    if (lq == 0 && n < p.N) {
                        float *to = p.colsum + (size_t)((m0 + wm * WM) / kGemmSumRows) * 2 * p.N + n;
                        *reinterpret_cast<f32x4 *>(to) = f32x4{cols[0], cols[1], cols[2], cols[3]};
                        *reinterpret_cast<f32x4 *>(to + 4) = f32x4{cols[4], cols[5], cols[6], cols[7]};
                    }
                }
            }
            return;
        }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = m0 + wm * WM + i * 16 + l16;
        if (m >= p.M) continue;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int n = n0 + wn * WN + j * 16 + 4 * lq;
            if (n >= p.N) continue;
            const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            epilogue4<EPI, E>(p, m, n, v);
        }
    }
}

template <int BM, int BN, int WGM, int WGN, int EPI, class E, bool TN>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_dma_kernel(DmaInput<E, TN> in, int tiles_m, int tiles_n) {
    dma_tile_product<BM, BN, WGM, WGN, EPI, E, TN>(in, tiles_m, tiles_n);
}
// The same on tiles of fewer columns (see gemm_narrow_width)
template <int BN, int EPI, class E> __global__ __launch_bounds__(256) void gemm_bf16_narrow_kernel(GemmParams<E> p, int tiles_m, int tiles_n) {
    dma_tile_product<256, BN, 2, 2, EPI, E, false>(p, tiles_m, tiles_n);
}

// Explicit instantiations: the host compiler does not always emit the launch stub of a kernel template from its use
// in the launchers below alone.
#define LGA_INSTANTIATE_DMA(EPI, TN)                                                                                      \
    template __global__ void gemm_bf16_dma_kernel<256, 256, 2, 2, EPI, bf16, TN>(DmaInput<bf16, TN>, int, int);            \
    template __global__ void gemm_bf16_dma_kernel<256, 256, 2, 2, EPI, f16, TN>(DmaInput<f16, TN>, int, int)
#define LGA_INSTANTIATE_NARROW(BN, EPI)                                                      \
    template __global__ void gemm_bf16_narrow_kernel<BN, EPI, bf16>(GemmParams<bf16>, int, int); \
    template __global__ void gemm_bf16_narrow_kernel<BN, EPI, f16>(GemmParams<f16>, int, int)
#define LGA_INSTANTIATE_WIDTHS(EPI)    \
    LGA_INSTANTIATE_DMA(EPI, false);   \
    LGA_INSTANTIATE_NARROW(192, EPI);  \
    LGA_INSTANTIATE_NARROW(128, EPI)
LGA_INSTANTIATE_WIDTHS(EPI_STORE);
LGA_INSTANTIATE_WIDTHS(EPI_BIAS);
LGA_INSTANTIATE_WIDTHS(EPI_BIAS_RESID);
LGA_INSTANTIATE_WIDTHS(EPI_BIAS_GELU);
LGA_INSTANTIATE_WIDTHS(EPI_MUL_DGELU);
LGA_INSTANTIATE_DMA(EPI_ACCUM_F32, false);
LGA_INSTANTIATE_DMA(EPI_ACCUM_F32, true);
#undef LGA_INSTANTIATE_WIDTHS
#undef LGA_INSTANTIATE_NARROW
#undef LGA_INSTANTIATE_DMA

// The kernel that serves a (tile size, layout, epilogue) combination and its dynamic LDS in bytes.
template <int BM, int BN, bool A_KM, bool B_KM, int EPI, class E, bool DMA = A_KM && B_KM> struct KernelFor {
    static constexpr bool kDma = DMA;
    static_assert(!kDma || A_KM == B_KM, "both operands k-contiguous, or neither");
    static_assert(!kDma || BM == 256, "smaller k-contiguous problems: gemm_small.hip");
    static constexpr size_t smem = kDma ? (size_t)5 * BM * BK * sizeof(E)            // the DMA kernel's operand ring
                                        : (size_t)2 * (BM + BN) * BK * sizeof(E);    // two stages of both operands
    static constexpr bool kGroup = kDma && !A_KM;
    static auto get() -> void (*)(DmaInput<E, kGroup>, int, int) {
        if constexpr (kDma && BN < BM) return gemm_bf16_narrow_kernel<BN, EPI, E>;
        else if constexpr (kDma) return gemm_bf16_dma_kernel<BM, BN, 2, 2, EPI, E, !A_KM>;
        else return gemm_bf16_kernel<BM, BN, A_KM, B_KM, EPI, E>;
    }
    // up to 160 KB of dynamic LDS: more than a launch may ask for by default
    static hipError_t raise_lds_limit() {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(get()), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    }
};

template <int BM, int BN, bool A_KM, bool B_KM, int EPI, class E, bool DMA = A_KM && B_KM>
void launch_one(const GemmParams<E> &p, hipStream_t s) {
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    using Kernel = KernelFor<BM, BN, A_KM, B_KM, EPI, E, DMA>;
    const size_t smem = Kernel::smem;
    auto kern = Kernel::get();
    char name[96];
    const char *et = std::is_same<E, bf16>::value ? "bf16" : "f16";       // profile names: gemm_bf16_... or gemm_f16_...
    if (DMA)
        snprintf(name, sizeof(name), "gemm_%s_dma%s_kernel<%d, %d, %d>", et, A_KM ? "" : "_tn", BM, BN, EPI);
    else
        snprintf(name, sizeof(name), "gemm_%s_kernel<%d, %d, %s, %s, %d>", et, BM, BN, A_KM ? "true" : "false",
                 B_KM ? "true" : "false", EPI);
    if (p.batch > 1) {                                       // the products of attention: listed apart from the layer's own
        const size_t len = strlen(name);
        snprintf(name + len, sizeof(name) - len, " (batched)");
    }
    const double mn = (double)p.M * p.N;
    const double out_bytes = EPI == EPI_ACCUM_F32 ? (p.beta != 0.f ? 8.0 : 4.0) : (EPI == EPI_BIAS_GELU && p.out2 ? 4.0 : 2.0);
    const double aux_bytes = (EPI == EPI_BIAS_RESID || EPI == EPI_MUL_DGELU) ? 2.0 : 0.0;
    const double nb = p.batch > 1 ? p.batch : 1;
    ProfScope scope(name, nb * 2.0 * mn * p.K,
                    nb * (2.0 * ((double)p.M * p.K + (double)p.K * p.N) + mn * (out_bytes + aux_bytes)), s);
    const int work = tiles_m * tiles_n * (p.ksplit > 1 ? p.ksplit : p.batch > 1 ? p.batch : 1);
    if constexpr (Kernel::kGroup) {
        GemmGroup<E> one{};
        one.n = 1;
        one.p[0] = p;
        one.p[0].ksplit = std::max(1, p.ksplit);
        hipLaunchKernelGGL(kern, dim3(work), dim3(256), smem, s, one, 0, 0);
    } else {
        hipLaunchKernelGGL(kern, dim3(work), dim3(256), smem, s, p, tiles_m, tiles_n);
    }
}

// out[m, n] = beta * out[m, n] + sum_z partial[z][m][n]; the slices are added in index order (deterministic).
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ partial, int slices, size_t stride,
                                                            float *__restrict__ out, int M, int N, int ldc, float beta) {
    const size_t quads = (size_t)M * (N / 4);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < quads; i += (size_t)gridDim.x * 256) {
        const size_t m = i / (N / 4), n = (i % (N / 4)) * 4;
        f32x4 acc = *reinterpret_cast<const f32x4 *>(partial + m * N + n);
        for (int z = 1; z < slices; ++z) acc += *reinterpret_cast<const f32x4 *>(partial + z * stride + m * N + n);
        float *o = out + m * ldc + n;
        if (beta != 0.f) acc += beta * *reinterpret_cast<const f32x4 *>(o);
        *reinterpret_cast<f32x4 *>(o) = acc;
    }
}

// The same for a group's products whose k range is split, one after the other: outputs without gaps between their rows.
struct SplitkGroup {
    const float *partial[kGemmGroup];
    float *out[kGemmGroup];
    size_t quads[kGemmGroup];
    float beta[kGemmGroup];
    int slices, n;
};
__global__ __launch_bounds__(256) void splitk_reduce_group_kernel(SplitkGroup g, size_t all) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < all; i += (size_t)gridDim.x * 256) {
        int z = 0;
        size_t at = i;
        while (z + 1 < g.n && at >= g.quads[z]) at -= g.quads[z++];
        const f32x4 *partial = reinterpret_cast<const f32x4 *>(g.partial[z]) + at;
        f32x4 acc = *partial;
        for (int k = 1; k < g.slices; ++k) acc += partial[k * g.quads[z]];
        f32x4 *o = reinterpret_cast<f32x4 *>(g.out[z]) + at;
        if (g.beta[z] != 0.f) acc += g.beta[z] * *o;
        *o = acc;
    }
}

// The slices in which the large-tile kernels run a weight gradient: 1 if its tiles alone are enough work, 0 if even slices are not
// (see launch_tiles).
template <class E> int large_tile_slices(const GemmParams<E> &p) {
    const long big = (long)((p.M + 255) / 256) * ((p.N + 255) / 256);
    const int slices = p.batch > 1 || p.K == 0 ? 1 : gemm_splitk_slices(p.M, p.N, p.K);        // (its K = 0 means: of any length)
    const bool fits = slices > 1 && p.partial && (size_t)slices * p.M * p.N <= p.partial_floats && p.N % 4 == 0 && p.ldc % 4 == 0 &&
                      (reinterpret_cast<uintptr_t>(p.outf) & 15) == 0;
    if (fits && (big * slices >= 192 || (p.K >= 10240 && p.K / gemm_small_slices(p.M, p.N, p.K, p.partial_floats) >= 8192))) return slices;
    return big >= 128 ? 1 : 0;
}

template <bool A_KM, bool B_KM, int EPI, class E> void launch_slices(const GemmParams<E> &p, int slices, hipStream_t s) {
    GemmParams<E> q = p;
    q.kchunk = ((p.K + slices - 1) / slices + BK - 1) / BK * BK;
    q.ksplit = (p.K + q.kchunk - 1) / q.kchunk;          // rounding the slice length up may have emptied the last ones
    launch_one<256, 256, A_KM, B_KM, EPI, E, true>(q, s);
    launch_splitk_reduce(p.partial, q.ksplit, p.outf, p.M, p.N, p.ldc, p.beta, s);
}

// What a round of 256 large tiles takes, for the rules that weigh rounds against something else.  Measured between 1.19 us per k tile
// (4096 x 4096 x 1024 .. 4096) and 1.41 (one round of 16384, where the board's power binds; four rounds 1.30), and from 8 (plain store) to 20 us
// (GELU') around them, where a last round, partly empty, has less to wait for; for weight gradients 1.22 to 1.30 and 16 to 20 us.
constexpr double kRoundStep = 1.25, kRound16 = 9.0, kRoundTensor = 3.0, kRoundF32 = 16.5;

// Columns that the large-tile kernel leaves to the small one (0: none).  Its tiles run in rounds of 256, and a last round of a few takes as
// long as a full one; the columns beyond the whole rounds are better off on small tiles where they are few - by what a round takes against
// what the small tiles do: 550 TFLOP/s, at least 0.42 us per 64 k, the way through memory of the rows, which are read a second time, and of
// what the epilogue reads and writes (tensors: 1 to 3 of the output's size) at 3.5 TB/s, and 6 us.  2000 x 17024 x 4256, 536 tiles, with GELU
// 285 -> 243 us; 16384 x 1032 x 4096 159 -> 114.  Not 65280 x 264 x 4096, whose rows are 535 MB: 179, with the columns apart 310.
// Of 220 products of all epilogues none takes more than 2 % longer for it, most of what it applies to 5 - 30 % less.
// Up to four rounds and 65536 rows; of 40 products beyond, columns apart were between 3 % slower and 10 % faster, 2 % on average.
// Either kernel adds up an element's products in the same order.
int peeled_columns(int M, int N, int K, int tensors) {
    const long tm = (M + 255) / 256, tn = (N + 255) / 256, rounds = tm * tn / 256;
    if (rounds < 1 || rounds > 4 || tm * tn % 256 == 0 || tm > 256) return 0;
    const long keep = rounds * 256 / tm;                     // whole columns of tiles that the full rounds hold
    const int rest = N - (int)keep * 256;
    if (keep < 1 || rest <= 0) return 0;
    const double ksteps = (double)K / BK, round = ksteps * kRoundStep + kRound16 + (tensors - 1) * kRoundTensor;
    const double memory = 2e-6 * ((double)M * K + (double)rest * K + (double)tensors * M * rest) / 3.5;
    const double small = std::max({2e-6 * M * rest * K / 550.0, ksteps * 0.42, memory}) + 6.0;
    return small < 0.8 * round ? rest : 0;
}
// Tensors of the output's size that an epilogue reads and writes
template <int EPI, class E> int epilogue_tensors(const GemmParams<E> &p) {
    return 1 + (EPI == EPI_BIAS_RESID || EPI == EPI_MUL_DGELU) + (EPI == EPI_BIAS_GELU && p.out2);
}

// What a product takes in tiles of 256 x width, in us: its rounds of 256 tiles, each k tiles and a prologue and epilogue.  A k tile is the longer the more
// compute units work - they share memory and the power that sets the clock -: the least below half a round, the most in a full one, and
// in full rounds of the narrower tiles more with the length of the k range.  Where an epilogue moves 100 MB and more it takes longer than that
// (32768 x 3072 x 768 with GELU' 266 us for 182, with GELU and its input stored 197 for 164): for comparing widths, not for the time itself.
double tiles_time(int width, long M, long N, int K, double epilogue) {
    struct { double few, all, per_ktile, limit, fixed; } const c = width == 256   ? decltype(c){0.88, 1.25, 0.0, 1.25, 7.0}
                                                                 : width == 192 ? decltype(c){0.68, 0.95, 0.0010, 1.17, 5.7}
                                                                                : decltype(c){0.55, 0.66, 0.0007, 0.85, 4.5};
    const long tiles = (M + 255) / 256 * ((N + width - 1) / width);
    const double kt = (K + BK - 1) / BK, fixed = c.fixed + epilogue * width / 256, part = (double)(tiles % 256) / 256;
    double us = 2.0 + (double)(tiles / 256) * (kt * std::min(c.all + c.per_ktile * kt, c.limit) + fixed);
    if (part > 0.0) us += kt * (c.few + (c.all - c.few) * std::max(0.0, 2.0 * part - 1.0)) + fixed;
    return us;
}

template <bool A_KM, bool B_KM, int EPI, class E> void launch_tiles(const GemmParams<E> &p, hipStream_t s) {
    // Large tiles when they fill the 256 CUs at least about once (the direct-to-LDS kernel is so much faster per
    // tile that a partly idle second round still wins); smaller ones otherwise.
    const long big = (long)((p.M + 255) / 256) * ((p.N + 255) / 256);
    if constexpr (A_KM && B_KM) {
        if constexpr (EPI == EPI_ACCUM_F32) {
            // A weight-gradient GEMM of a narrow layer: few output tiles, very long k.  The k range is cut into slices
            // that run as separate work items of the large-tile kernel and are summed afterwards - where that gives at least
            // 192 work items: with fewer the small tiles are faster (768 x 768 x 8192, 72 items: 36 against 30 us;
            // 768 x 2304 x 8192, 216 items: 43 against 48; 1280 x 3840 x 2048, 150 items: 41 against 32).  Unless one of their
            // workgroups walks over 8192 k and more: 768 x 768 x 16384, 135 items, 40 against 56; 640 x 640 x 16384, 8192 k
            // each in two slices, 39 against 44; 256 x 1024 x 65536 58 against 83 - but x 16384, 4096 k each, 37 against 26.
            const int slices = large_tile_slices(p);
            if (slices > 1) return launch_slices<A_KM, B_KM, EPI, E>(p, slices, s);
        }
        // (the direct-to-LDS loads of the large-tile kernel want rows of at least 128 bytes: see its per-lane load offsets)
        const bool short_rows = p.lda < BK || p.ldb < BK;
        bool large = big >= 128;
        if (p.batch > 1) {
            // many small problems (the products of attention, one per head): enough work items either way, so take the
            // tile size that pads the output less, the large one on a tie
            const double pad256 = (double)big * 65536.0, pad128 = (double)((p.M + 127) / 128) * ((p.N + 127) / 128) * 16384.0;
            large = big * p.batch >= 128 && pad256 <= 1.15 * pad128;
        }
        if constexpr (EPI != EPI_ACCUM_F32) {
            const int width = p.batch > 1 || p.tri || p.colsum || short_rows ? 0 : gemm_narrow_width(p.M, p.N, p.K, EPI, EPI == EPI_BIAS_GELU && p.out2);
            if (width == 192) return launch_one<256, 192, A_KM, B_KM, EPI, E>(p, s);
            if (width == 128) return launch_one<256, 128, A_KM, B_KM, EPI, E>(p, s);
        }
        if (!large || short_rows) return launch_gemm_small<EPI, E>(p, s);
        GemmParams<E> q = p;
        const int rest = EPI == EPI_ACCUM_F32 || p.batch > 1 || p.tri || p.colsum ? 0 : peeled_columns(p.M, p.N, p.K, epilogue_tensors<EPI>(p));
        if (rest > 0) {
            const int n = p.N - rest;
            q.N = rest;
            q.B += (size_t)n * p.ldb;
            q.out += n;
            if (q.out2) q.out2 += n;
            if (q.bias) q.bias += n;
            if (q.aux) q.aux += n;
            launch_gemm_small<EPI, E>(q, s);
            q = p;
            q.N = n;
            launch_one<256, 256, A_KM, B_KM, EPI, E>(q, s);
            return;
        }
        const int tm = (p.M + 255) / 256, tn = (p.N + 255) / 256;
        q.sblock = p.batch <= 1 && tm % 16 == 0 && tn % 16 == 0;     // + 1 % on the weight-gradient shapes of d = 12288
        launch_one<256, 256, A_KM, B_KM, EPI, E>(q, s);
    } else {
        if constexpr (!A_KM && !B_KM && EPI == EPI_ACCUM_F32) {
            // the direct-to-LDS kernel takes a weight gradient's operands as stored, by the same rule; its loads want rows of at
            // least 512 bytes
            const int slices = p.batch > 1 || p.lda < 256 || p.ldb < 256 ? 0 : large_tile_slices(p);
            if (slices > 1) return launch_slices<A_KM, B_KM, EPI, E>(p, slices, s);
            if (slices == 1) {
                GemmParams<E> q = p;
                q.sblock = (p.M + 255) / 256 % 16 == 0 && (p.N + 255) / 256 % 16 == 0;
                return launch_one<256, 256, A_KM, B_KM, EPI, E, true>(q, s);
            }
        }
        const double pad256 = (double)big * 65536.0, pad128 = (double)((p.M + 127) / 128) * ((p.N + 127) / 128) * 16384.0;
        const bool large = p.batch > 1 ? big * p.batch >= 128 && pad256 <= 1.15 * pad128 : big >= 128;
        if (large) launch_one<256, 256, A_KM, B_KM, EPI, E>(p, s);
        else launch_one<128, 128, A_KM, B_KM, EPI, E>(p, s);
    }
}

}  // namespace

void launch_splitk_reduce(const float *partial, int slices, float *out, int M, int N, int ldc, float beta, hipStream_t s) {
    ProfScope scope("splitk_reduce_kernel", (double)slices * M * N, 4.0 * M * N * (slices + (beta != 0.f ? 2.0 : 1.0)), s);
    const size_t quads = (size_t)M * (N / 4);
    const unsigned blocks = (unsigned)std::min<size_t>((quads + 255) / 256, 256 * 16);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(blocks), dim3(256), 0, s, partial, slices, (size_t)M * N, out, M, N, ldc, beta);
}

template <class E> void prepare_gemm_group(GemmGroup<E> &group, const GemmParams<E> *p, int slices) {
    size_t used = 0;
    for (int i = 0; i < group.n; ++i) {
        GemmParams<E> &q = group.p[i];
        q = p[i];
        q.kchunk = slices > 1 ? ((p[i].K + slices - 1) / slices + BK - 1) / BK * BK : p[i].K;
        q.ksplit = slices > 1 ? (p[i].K + q.kchunk - 1) / q.kchunk : 1;
        if (slices > 1) q.partial = p[0].partial + used;
        used += (size_t)slices * p[i].M * p[i].N;
    }
}
template <class E> void launch_splitk_reduce_group(const GemmGroup<E> &group, hipStream_t s) {
    if (group.p[0].ksplit <= 1) return;
    SplitkGroup g{};
    g.n = group.n;
    g.slices = group.p[0].ksplit;
    size_t all = 0;
    double bytes = 0.0;
    for (int i = 0; i < g.n; ++i) {
        const GemmParams<E> &p = group.p[i];
        g.partial[i] = p.partial;
        g.out[i] = p.outf;
        g.quads[i] = (size_t)p.M * p.N / 4;
        g.beta[i] = p.beta;
        all += g.quads[i];
        bytes += 16.0 * g.quads[i] * (g.slices + (p.beta != 0.f ? 2.0 : 1.0));
    }
    ProfScope scope("splitk_reduce_kernel", 4.0 * g.slices * all, bytes, s);
    hipLaunchKernelGGL(splitk_reduce_group_kernel, dim3((unsigned)std::min<size_t>((all + 255) / 256, 256 * 16)), dim3(256), 0, s, g, all);
}
template void prepare_gemm_group<bf16>(GemmGroup<bf16> &, const GemmParams<bf16> *, int);
template void prepare_gemm_group<f16>(GemmGroup<f16> &, const GemmParams<f16> *, int);
template void launch_splitk_reduce_group<bf16>(const GemmGroup<bf16> &, hipStream_t);
template void launch_splitk_reduce_group<f16>(const GemmGroup<f16> &, hipStream_t);

// What weight gradients take in one launch of the large-tile kernel, in us: by what a round of 256 workgroups takes (above) and the way of the slices'
// partial results through memory (4.5 TB/s)
static double group_time(long tiles, double outputs, int slices, int K) {
    return (double)((tiles * slices + 255) / 256) * ((double)(K / slices) / BK * kRoundStep + kRoundF32) + (slices > 1 ? (slices + 1) * outputs * 4.0 / 4.5e6 : 0.0);
}
// Slices of the k range for n weight gradients in one launch, by these times; 0 where that leaves more than a quarter of the chip idle or a workgroup fewer than 16 k
// tiles.  The four matrices of a d = 768 layer over 4096 tokens, 108 tiles: 121 us in four launches of the small kernel behind 38 us of
// transposes, now 58 + 20 us in two slices and 11 us for the bias gradients' column sums.  (With 1.2 and 12 us for a round: 1072 x 2448 over
// 6424 tokens in four slices instead of two 183 us, now 161; 1320 x 1416 over 26240 in five instead of one 550, now 517.)
int gemm_group_slices(const int *M, const int *N, int n, int K) {
    long tiles = 0;
    double outputs = 0.0;
    for (int i = 0; i < n; ++i) {
        if (M[i] < 256 || N[i] < 256) return 0;
        tiles += (long)((M[i] + 255) / 256) * ((N[i] + 255) / 256);
        outputs += (double)M[i] * N[i];
    }
    if (K < 1024) return 0;
    int best = 0;
    double best_us = 0.0;
    for (int s = 1; s <= std::min(32, K / 1024); ++s) {
        if (tiles * s < 192) continue;
        const double us = group_time(tiles, outputs, s, K);
        if (best == 0 || us < best_us) best = s, best_us = us;
    }
    return best;
}

// Matrices that are enough work alone still share a launch where their rounds then fill each other up, by the same times.  Whole, over any k range, from 224
// tiles on: T-NLG's four (289 to 1139 tiles over 4000 tokens, 14 rounds together, 16 apart) 1477 -> 1415 us; d = 2048 over 32768 tokens, W_o and
// W_qkv with 64 and 192 tiles in slices apart, all 768 together, 2207 -> 2144; d = 1664 over 512, three of 140 to 182 tiles, 78 -> 52; d = 3072 over
// 768 269 -> 210.  In slices where that promises 3 %: d = 768, over 8192 tokens three of 27 to 36 tiles 175 -> 110, over 16384 all 108 289 -> 191,
// over 32768 451 -> 388; d = 384 over 11056, three in ten slices, 92 -> 52; d = 1280 over 8704 415 -> 342.  Of 23 layers of widths 256 to 3072 over
// 512 to 34360 tokens (times with the sums of the slices) all take 10 to 47 % less.
bool gemm_stored_group_wins(const int *M, const int *N, int n, int K) {
    long tiles = 0;
    double apart = 0.0, outputs = 0.0;
    for (int i = 0; i < n; ++i) {
        const long mine = (long)((M[i] + 255) / 256) * ((N[i] + 255) / 256);
        tiles += mine;
        outputs += (double)M[i] * N[i];
        apart += group_time(mine, (double)M[i] * N[i], gemm_splitk_slices(M[i], N[i], K), K);
    }
    if (n < 2) return false;
    if (tiles >= 224 && group_time(tiles, outputs, 1, K) < 0.99 * apart) return true;
    const int slices = gemm_group_slices(M, N, n, K);
    return slices > 0 && group_time(tiles, outputs, slices, K) < 0.97 * apart;
}

template <class E> void launch_gemm_stored_group(const GemmParams<E> *p, int n, hipStream_t s) {
    int M[kGemmGroup], N[kGemmGroup];
    size_t outputs = 0;
    for (int i = 0; i < n; ++i) {
        M[i] = p[i].M;
        N[i] = p[i].N;
        outputs += (size_t)M[i] * N[i];
    }
    int slices = std::max(1, gemm_group_slices(M, N, n, p[0].K));
    if (slices > 1 && (!p[0].partial || slices * outputs > p[0].partial_floats)) slices = 1;
    (void)prepare_kernels();
    GemmGroup<E> group{};
    group.n = n;
    prepare_gemm_group(group, p, slices);
    long work = 0;
    double flops = 0.0, bytes = 0.0;
    for (int i = 0; i < n; ++i) {
        const GemmParams<E> &q = group.p[i];
        const double mn = (double)q.M * q.N;
        work += (long)((q.M + 255) / 256) * ((q.N + 255) / 256) * q.ksplit;
        flops += 2.0 * mn * q.K;
        bytes += 2.0 * ((double)q.M * q.K + (double)q.K * q.N) + mn * (q.beta != 0.f ? 8.0 : 4.0);
    }
    {
        char name[96];
        snprintf(name, sizeof(name), "gemm_%s_dma_tn_kernel<256, 256, %d> (grouped)", std::is_same<E, bf16>::value ? "bf16" : "f16", EPI_ACCUM_F32);
        ProfScope scope(name, flops, bytes, s);
        hipLaunchKernelGGL((gemm_bf16_dma_kernel<256, 256, 2, 2, EPI_ACCUM_F32, E, true>), dim3((unsigned)work), dim3(256),
                           (size_t)5 * 256 * BK * sizeof(E), s, group, 0, 0);
    }
    launch_splitk_reduce_group(group, s);
}
template void launch_gemm_stored_group<bf16>(const GemmParams<bf16> *, int, hipStream_t);
template void launch_gemm_stored_group<f16>(const GemmParams<f16> *, int, hipStream_t);

// Weight gradients on transposed operands: those that have enough work for the large tiles by themselves alone, the others together.
template <class E> void launch_gemm_transposed_group(const GemmParams<E> *p, int n, hipStream_t s) {
    GemmParams<E> rest[kGemmGroup];
    int n_rest = 0;
    for (int i = 0; i < n; ++i) {
        const bool whole = p[i].N % 4 == 0 && p[i].ldc == p[i].N;
        if (large_tile_slices(p[i]) > 0 || !whole) (void)launch_gemm_mfma<E>(p[i], true, true, EPI_ACCUM_F32, s);
        else rest[n_rest++] = p[i];
    }
    if (n_rest == 1) (void)launch_gemm_mfma<E>(rest[0], true, true, EPI_ACCUM_F32, s);
    else if (n_rest > 1) {
        (void)prepare_kernels();
        launch_gemm_small_group<E>(rest, n_rest, s);
    }
}
template void launch_gemm_transposed_group<bf16>(const GemmParams<bf16> *, int, hipStream_t);
template void launch_gemm_transposed_group<f16>(const GemmParams<f16> *, int, hipStream_t);

// Whether a product runs on tiles of 256 x 192 or 256 x 128 instead (0: no): the large-tile kernel with fewer columns, the same order of every sum.  Where
// 256 x 256 tiles leave much of their last round empty, narrower ones fill more of it (us, 256 columns / these): 32768 x 768 x 768 45 / 38 with
// 192, 2000 x 4256 x 4256 71 / 62, 4096 x 2304 x 768 20 / 17.6, 38384 x 280 x 1464 64 / 50 with 128; a full round of theirs takes longer for its
// work, 32768 x 2048 x 2048 181 / 214.  By tiles_time, where it promises 3 % and no columns are left to the small kernel (16384 x 1032 x 4096,
// 8 columns apart, 108 / 120); beyond four rounds 7 %, where there is less to fill than the times are off (47888 x 1544 x 5224 with GELU 808 / 882, 59824 x
// 2168 x 200 with a residual 175 / 187); 128 columns up to two rounds, beyond which operands are read too often (43800 x 576 x 2864 175 / 197).
// Fewer than 128 tiles of 256 x 256 belong to the small kernel, unless tiles of 128 columns are at least 144, the k range 704 and its own tiles of 128 x 128
// more than one round: 6424 x 1024 x 4096 (208 of them) 59 / 47, 2000 x 3072 x 3072 (192) 43 / 35, 800 x 5136 x 896 (164) 16 / 13; 2048 x
// 2048 x 2048 (128) 24.0 / 23.7, 880 x 4168 x 4456 (132) 50 / 63, 2080 x 3552 x 576 (252) 13.4 / 13.8, 808 x 4568 x 3336 (252 of the small ones) 38 / 47.
// Of 1200 products of all epilogues 347 take one of them: 12 % less time for these on average, 4 % over all, the worst 3 % more (36880 x 2096 x 1672 with a
// residual).  Of 1400 others 409, six of them 3 to 6 % more, most of these with an A of about the size of the last-level cache that every pass read again, which
// the wider tiles use better: 45928 x 680 x 3128 with GELU, 10 % more on one A, 1 % on six in turn; 23056 x 728 x 6048 4 % more, 5 % less.
int gemm_narrow_width(int M, int N, int K, int epi, bool pre) {
    const long rows = (M + 255) / 256, big = rows * ((N + 255) / 256), narrow = rows * ((N + 127) / 128);
    if (big < 128) return narrow >= 144 && K >= 704 && (long)((M + 127) / 128) * ((N + 127) / 128) > 256 ? 128 : 0;
    const int tensors = 1 + (epi == EPI_BIAS_RESID || epi == EPI_MUL_DGELU) + pre;
    if (peeled_columns(M, N, K, tensors) > 0) return 0;
    const double epilogue = epi == EPI_MUL_DGELU ? 8.0 : epi == EPI_BIAS_GELU ? (pre ? 5.0 : 3.0) : epi == EPI_BIAS_RESID ? 3.0 : epi == EPI_BIAS ? 0.5 : 0.0;
    const double limit = (big > 1024 ? 0.93 : 0.97) * tiles_time(256, M, N, K, epilogue);
    const double with192 = tiles_time(192, M, N, K, epilogue), with128 = narrow <= 512 ? tiles_time(128, M, N, K, epilogue) : with192;
    if (std::min(with192, with128) >= limit) return 0;
    return with128 < with192 ? 128 : 192;
}

bool gemm_takes_stored_operands(int M, int N, int K) {
    if (M < 256 || N < 256) return false;
    GemmParams<bf16> p{};
    p.M = M; p.N = N; p.K = K; p.ldc = N;
    p.partial_floats = SIZE_MAX;                             // the caller provides as much as the slices need
    float probe;
    p.partial = &probe;                                      // (only tested against NULL)
    return large_tile_slices(p) > 0;
}

int gemm_splitk_slices(int M, int N, int K) {
    const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
    if (tiles >= 224) return 1;                              // the output alone occupies the chip
    // Work items = tiles x slices run in rounds of 256 (one per CU).  Take the fewest slices (their partial results
    // are written and read again) whose last round is within a tenth of the best filled one.
    long cap = 32;
    if (K > 0) cap = std::min<long>(cap, K / 1024);          // at least 16 k tiles per slice
    cap = std::max<long>(cap, 1);
    auto fill = [&](long s) { return (double)(tiles * s) / (256.0 * ((tiles * s + 255) / 256)); };
    double best = 0.0;
    for (long s = 1; s <= cap; ++s) best = std::max(best, fill(s));
    for (long s = 1; s <= cap; ++s)
        if (fill(s) >= 0.9 * best) return (int)s;
    return 1;
}

// (The large-tile kernel alone, see launch_tiles.  Columns left to the small one are worth more than the pass over the result: 2000 x 17024 x
// 4256 with GELU' 341 -> 233 + 41 us, the pass 15.)
bool gemm_dgelu_adds_columns(int M, int N, int K) {
    return (long)((M + 255) / 256) * ((N + 255) / 256) >= 128 && K >= BK && peeled_columns(M, N, K, 2) == 0;
}

bool gemm_mfma_supports(bool a_kmajor, bool b_kmajor, Epilogue epi) {
    if (a_kmajor && !b_kmajor) return epi == EPI_STORE || epi == EPI_BIAS || epi == EPI_BIAS_RESID || epi == EPI_BIAS_GELU;
    if (a_kmajor && b_kmajor) return epi >= EPI_STORE && epi <= EPI_ACCUM_F32;
    if (!a_kmajor && !b_kmajor) return epi == EPI_STORE || epi == EPI_ACCUM_F32;
    return false;
}

template <class E>
bool launch_gemm_mfma(const GemmParams<E> &p, bool a_kmajor, bool b_kmajor, Epilogue epi, hipStream_t s) {
    if (!gemm_mfma_supports(a_kmajor, b_kmajor, epi)) return false;
    // the direct-to-LDS loads address an operand tile's 256 rows with 32-bit byte offsets inside a 1 GiB window
    if (p.lda > kGemmMaxLd || p.ldb > kGemmMaxLd) return false;
    if (p.M == 0 || p.N == 0) return true;
    (void)prepare_kernels();
    // The three operand layouts the layer uses; every epilogue is tied to the family that needs it.
    if (a_kmajor && !b_kmajor) {          // forward
        switch (epi) {
            case EPI_BIAS: launch_tiles<true, false, EPI_BIAS, E>(p, s); break;
            case EPI_BIAS_RESID: launch_tiles<true, false, EPI_BIAS_RESID, E>(p, s); break;
            case EPI_BIAS_GELU: launch_tiles<true, false, EPI_BIAS_GELU, E>(p, s); break;
            default: launch_tiles<true, false, EPI_STORE, E>(p, s); break;
        }
    } else if (a_kmajor && b_kmajor) {    // both operands k-contiguous: the layout the layer stack uses
        switch (epi) {
            case EPI_STORE: launch_tiles<true, true, EPI_STORE, E>(p, s); break;
            case EPI_BIAS: launch_tiles<true, true, EPI_BIAS, E>(p, s); break;
            case EPI_BIAS_RESID: launch_tiles<true, true, EPI_BIAS_RESID, E>(p, s); break;
            case EPI_BIAS_GELU: launch_tiles<true, true, EPI_BIAS_GELU, E>(p, s); break;
            case EPI_MUL_DGELU: launch_tiles<true, true, EPI_MUL_DGELU, E>(p, s); break;
            case EPI_ACCUM_F32: launch_tiles<true, true, EPI_ACCUM_F32, E>(p, s); break;
        }
    } else {                              // weight gradient from operands as stored
        if (epi == EPI_ACCUM_F32) launch_tiles<false, false, EPI_ACCUM_F32, E>(p, s);
        else launch_tiles<false, false, EPI_STORE, E>(p, s);
    }
    return true;
}
template bool launch_gemm_mfma<bf16>(const GemmParams<bf16> &, bool, bool, Epilogue, hipStream_t);
template bool launch_gemm_mfma<f16>(const GemmParams<f16> &, bool, bool, Epilogue, hipStream_t);

namespace {
template <bool A_KM, bool B_KM, int EPI, class E> hipError_t raise_pair() {
    hipError_t e = KernelFor<256, 256, A_KM, B_KM, EPI, E>::raise_lds_limit();
    if constexpr (A_KM && B_KM && EPI != EPI_ACCUM_F32) {
        if (e == hipSuccess) e = KernelFor<256, 192, A_KM, B_KM, EPI, E>::raise_lds_limit();
        if (e == hipSuccess) e = KernelFor<256, 128, A_KM, B_KM, EPI, E>::raise_lds_limit();
    }
    if constexpr (!(A_KM && B_KM))
        if (e == hipSuccess) e = KernelFor<128, 128, A_KM, B_KM, EPI, E>::raise_lds_limit();
    return e;
}
template <class E> hipError_t raise_all() {
    hipError_t e = hipSuccess;
    auto next = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    next(raise_pair<true, false, EPI_STORE, E>());
    next(raise_pair<true, false, EPI_BIAS, E>());
    next(raise_pair<true, false, EPI_BIAS_RESID, E>());
    next(raise_pair<true, false, EPI_BIAS_GELU, E>());
    next(raise_pair<true, true, EPI_STORE, E>());
    next(raise_pair<true, true, EPI_BIAS, E>());
    next(raise_pair<true, true, EPI_BIAS_RESID, E>());
    next(raise_pair<true, true, EPI_BIAS_GELU, E>());
    next(raise_pair<true, true, EPI_MUL_DGELU, E>());
    next(raise_pair<true, true, EPI_ACCUM_F32, E>());
    next(raise_pair<false, false, EPI_STORE, E>());
    next(raise_pair<false, false, EPI_ACCUM_F32, E>());
    next(KernelFor<256, 256, false, false, EPI_ACCUM_F32, E, true>::raise_lds_limit());
    return e;
}
}  // namespace

hipError_t gemm_prepare_kernels() {
    hipError_t e = raise_all<bf16>();
    if (e == hipSuccess) e = raise_all<f16>();
    return e;
}

}  // namespace lga
