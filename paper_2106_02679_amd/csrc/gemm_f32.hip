// fp32 GEMM on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: full fp32 products and sums), any shape, any of the
// four operand layouts.
//
// What bounds it at the sizes the fp32 mode is used at (widths of 64 ... 512, a few thousand tokens) is not arithmetic
// but the length of the serial chain over k and the number of compute units that work at all: a weight gradient has
// 4 ... 64 output tiles and contracts over every token of the step.  So
//  - a tile is 64 x 64, multiplied by a group of four wavefronts (one 32 x 32 quadrant each) - or 32 x 64, two wavefronts, where the tiles are few -,
//    32 k per step, the next step's operands on their way from memory while this one is multiplied, one barrier per step;
//  - a workgroup holds KG = 1, 2 or 4 such groups, each of which takes its own part of the k range; their sums meet in
//    LDS at the end, in group order (the result does not depend on scheduling), and every group then writes its
//    share of the tile.  One group alone adds up the same parts in the same order, so that an activation does not depend
//    on how many rows share its launch: the parts follow from K, only the groups from the number of tiles;
//  - where even that leaves compute units idle, the k range is cut into slices over the grid and the partial results
//    are added in slice order by a second kernel (weight gradients of a layer, which come with scratch).
// gemm_f32_dma_kernel serves operands of whole 16-byte pieces in the layouts that the stack uses, gemm_f32_kernel the others; the
// weight gradients of a layer run in one launch.
// Measured (one MI355X, us; gemm_f32_kernel -> gemm_f32_dma_kernel -> vendor library): 2048 x 768 x 256 with bias 17.5 -> 14.4 -> 18.7,
// 4096 x 256 x 1024 31 -> 24 -> 22, 8192 x 512 x 2048 174 -> 144 -> 120; input gradient 2048 x 1024 x 256 17.9 -> 14.2; weight gradient
// 512 x 1536 x 8192 188 -> 135.  The four weight gradients of a 256-wide layer over 2048 tokens: 80 in eight launches, now 41 in one.
#include <algorithm>
#include <type_traits>

#include "gemm16.h"
#include "kernels.h"

namespace lga {

namespace {

constexpr int TN = 64, TK = 32;
// LDS tile: [TK][PITCH], k-major.  A pitch of 66 makes all three accesses conflict-free: the operand read (lanes 0-31 one
// row of k, lanes 32-63 the row 16 further down: 16 * 66 = 32 banks away), the transposing store of a k-contiguous
// operand (8 k quads x 8 rows: (4 c + i) 66 + r = 8 c + r + 2 i modulo 64) and the 8-byte store of the other layout.
constexpr int PITCH = 66;
constexpr int kTileFloats = TK * PITCH;

// One operand's tile: 64 rows (of m or n) x 32 k as 2 x 4 floats per thread of a group of 256.
struct Loader {
    const float *base;       // element (row 0 of the tile, k 0)
    long ld;
    int rows, kend;          // valid rows of the tile; end of this group's k range
    bool kc, vec;            // k contiguous; every aligned group of 4 elements is 16-byte aligned
    int t;                   // thread index inside the group
    f32x4 v[2];

    __device__ __forceinline__ void init(const float *p, int row0, int nrows, long ld_, bool kc_, int kend_, int t_) {
        kc = kc_; ld = ld_; kend = kend_; t = t_;
        rows = min(nrows - row0, 64);
        base = kc ? p + (long)row0 * ld : p + row0;
        vec = (ld & 3) == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0;       // row0 and every k0 are multiples of 4
    }
    __device__ __forceinline__ void load(int k0) {
        if (kc) {
            const int k = k0 + 4 * (t & 7);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = (t >> 3) + 32 * i;
                const float *src = base + (long)r * ld + k;
                if (vec && r < rows && k + 3 < kend) {
                    v[i] = *reinterpret_cast<const f32x4 *>(src);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[i][j] = (r < rows && k + j < kend) ? src[j] : 0.f;
                }
            }
        } else {
            const int r = 4 * (t & 15);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int k = k0 + (t >> 4) + 16 * i;
                const float *src = base + (long)k * ld + r;
                if (vec && k < kend && r + 3 < rows) {
                    v[i] = *reinterpret_cast<const f32x4 *>(src);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[i][j] = (k < kend && r + j < rows) ? src[j] : 0.f;
                }
            }
        }
    }
    __device__ __forceinline__ void store(float *lds) const {
        if (kc) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) lds[(4 * (t & 7) + j) * PITCH + (t >> 3) + 32 * i] = v[i][j];
        } else {
            typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float *dst = lds + ((t >> 4) + 16 * i) * PITCH + 4 * (t & 15);
                *reinterpret_cast<f32x2 *>(dst) = f32x2{v[i][0], v[i][1]};
                *reinterpret_cast<f32x2 *>(dst + 2) = f32x2{v[i][2], v[i][3]};
            }
        }
    }
};

// 4 consecutive n of row m, of which those below N exist.
template <int EPI> __device__ __forceinline__ void epilogue_f32(const GemmParams<float> &p, int m, int n, const f32x4 &a, bool vec) {
    const size_t idx = (size_t)m * p.ldc + n;
    auto one = [&](float acc, size_t at, int col) {
        if constexpr (EPI == EPI_STORE) {
            p.out[at] = acc;
        } else if constexpr (EPI == EPI_BIAS) {
            p.out[at] = acc + p.bias[col];
        } else if constexpr (EPI == EPI_BIAS_RESID) {
            p.out[at] = acc + p.bias[col] + p.aux[at];
        } else if constexpr (EPI == EPI_BIAS_GELU) {
            const float u = acc + p.bias[col];
            if (p.out2) p.out2[at] = u;
            p.out[at] = gelu_f(u);
        } else if constexpr (EPI == EPI_MUL_DGELU) {
            p.out[at] = acc * gelu_grad_f(p.aux[at]);
        } else {
            p.outf[at] = (p.beta == 0.f ? 0.f : p.beta * p.outf[at]) + acc;
        }
    };
    if (vec && n + 3 < p.N) {
        f32x4 o = a;
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU) {
            const f32x4 b = *reinterpret_cast<const f32x4 *>(p.bias + n);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] += b[i];
        }
        if constexpr (EPI == EPI_BIAS_RESID || EPI == EPI_MUL_DGELU) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(p.aux + idx);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = EPI == EPI_MUL_DGELU ? o[i] * gelu_grad_f(x[i]) : o[i] + x[i];
        }
        if constexpr (EPI == EPI_BIAS_GELU) {
            if (p.out2) *reinterpret_cast<f32x4 *>(p.out2 + idx) = o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = gelu_f(o[i]);
        }
        if constexpr (EPI == EPI_ACCUM_F32) {
            if (p.beta != 0.f) {
                const f32x4 old = *reinterpret_cast<const f32x4 *>(p.outf + idx);
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] += p.beta * old[i];
            }
            *reinterpret_cast<f32x4 *>(p.outf + idx) = o;
        } else {
            *reinterpret_cast<f32x4 *>(p.out + idx) = o;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (n + i < p.N) one(a[i], idx + i, n + i);
    }
}

// Which tile and part of the k range a workgroup has.  In: GemmParams, grid (n tiles, m tiles); or GemmGroup, the weight gradients of a layer in
// one launch, a one-dimensional grid over all their tiles and slices of the k range.
struct Place {
    int m0, n0, kbeg, kstop;
};
template <int EPI, int TM, class In> __device__ __forceinline__ Place place_of(const In &in, GemmParams<float> &p, bool &vec_out) {
    if constexpr (std::is_same<In, GemmParams<float>>::value) {
        p = in;
        return Place{(int)blockIdx.y * TM, (int)blockIdx.x * TN, 0, p.K};
    } else {
        int z = 0, item = blockIdx.x;
        for (;; ++z) {
            const int items = ((in.p[z].M + TM - 1) / TM) * ((in.p[z].N + TN - 1) / TN) * in.p[z].ksplit;
            if (z + 1 >= in.n || item < items) break;
            item -= items;
        }
        p = in.p[z];
        const int tiles_m = (p.M + TM - 1) / TM, tiles_n = (p.N + TN - 1) / TN;
        const int slice = item / (tiles_m * tiles_n);
        item -= slice * (tiles_m * tiles_n);
        const int tm = item / tiles_n, tn = item - tm * tiles_n;
        Place at{tm * TM, tn * TN, 0, p.K};
        vec_out = p.ksplit > 1 ? (p.N & 3) == 0 : (p.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(p.outf) & 15) == 0;
        if (p.ksplit > 1) {                     // this slice of the k range, into a partial result of its own ([M][N], dense)
            at.kbeg = slice * p.kchunk;
            at.kstop = min(p.K, at.kbeg + p.kchunk);
            p.outf = p.partial + (size_t)slice * p.M * p.N;
            p.ldc = p.N;
            p.beta = 0.f;
        }
        return at;
    }
}

// The order of a quadrant's sums over its wavefront's steps.  An activation's parts follow from K alone: the parts of a pair, then the
// pairs, whichever group has them.  A weight gradient's sums are folded every four steps, 128 k, however many a group walks over.
template <int EPI, int KG> struct PartSums {
    static constexpr bool FOLD = EPI == EPI_ACCUM_F32, PAIRS = !FOLD && KG < 4;
    f32x16 acc, pair, total;
    int each, left, odd = 0;
    __device__ __forceinline__ explicit PartSums(int part) : each(FOLD ? 4 : part), left(FOLD ? 4 : part) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = pair[r] = total[r] = 0.f;
    }
    __device__ __forceinline__ void step() {
        if (!(FOLD || PAIRS) || --left > 0) return;
        left = each;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            pair[r] += acc[r];
            acc[r] = 0.f;
        }
        if (PAIRS && KG == 1) {
            if (odd) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    total[r] += pair[r];
                    pair[r] = 0.f;
                }
            }
            odd ^= 1;
        }
    }
    __device__ __forceinline__ void finish() {
        if (FOLD || PAIRS) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = total[r] + (pair[r] + acc[r]);
        }
    }
};

// The sums of a wavefront's quadrant leave.  Lane: row m = l32 of it, columns n = 8 q + 4 half + (0 .. 3).
// W: wavefronts of a group
template <int EPI, int KG, int W>
__device__ __forceinline__ void finish_tile(const GemmParams<float> &p, const Place &at, const f32x16 &sum, bool vec_out, float *smem) {
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * W)), wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) % W);
    const int lane = threadIdx.x & 63, wm = wave >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
    const int m = at.m0 + wm * 32 + l32, nq = at.n0 + wn * 32 + 4 * half;
    if constexpr (KG == 1) {
        if (m >= p.M) return;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (nq + 8 * q < p.N) epilogue_f32<EPI>(p, m, nq + 8 * q, f32x4{sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]}, vec_out);
    } else {
        // every group leaves its sums in LDS (nobody reads operands there any more); group g then adds up column quads
        // g, g + KG, ... of all groups, neighbouring groups first
        f32x4 *red = reinterpret_cast<f32x4 *>(smem);
#pragma unroll
        for (int q = 0; q < 4; ++q) red[((group * W + wave) * 4 + q) * 64 + lane] = f32x4{sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]};
        __syncthreads();
        if (m >= p.M) return;
#pragma unroll
        for (int j = 0; j < 4 / KG; ++j) {
            const int q = group + j * KG;
            if (nq + 8 * q >= p.N) continue;
            f32x4 of[KG];
#pragma unroll
            for (int g = 0; g < KG; ++g) of[g] = red[((g * W + wave) * 4 + q) * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) of[0][i] = KG == 4 ? (of[0][i] + of[1][i]) + (of[2 % KG][i] + of[3 % KG][i]) : of[0][i] + of[1][i];
            epilogue_f32<EPI>(p, m, nq + 8 * q, of[0], vec_out);
        }
    }
}

// Block: 256 KG threads.  vec_out: every tensor the epilogue touches takes 16-byte accesses at columns that are multiples of 4.
// log_parts: into 1, 2 or 4 parts the k range is cut for the order of the sums, (0 + 1) + (2 + 3); a group has 1 / KG of them.
template <int EPI, int KG, class In>
__global__ __launch_bounds__(256 * KG) void gemm_f32_kernel(In in, bool a_kc, bool b_kc, bool vec_out, int log_parts) {
    GemmParams<float> p;
    const Place at = place_of<EPI, 64>(in, p, vec_out);
    extern __shared__ __attribute__((aligned(16))) float smem_f32[];
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), t = threadIdx.x & 255;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
    const int m0 = at.m0, n0 = at.n0, kbeg = at.kbeg, kstop = at.kstop;
    // a part of the k range: whole steps, the same number for every part (a group reads zeros where one is empty)
    const int all = (kstop - kbeg + TK - 1) / TK, part = (all + (1 << log_parts) - 1) >> log_parts, each = (part << log_parts) / KG;
    const int steps = KG == 1 ? all : each;
    const int kg0 = kbeg + group * each * TK;
    float *lds = smem_f32 + group * (4 * kTileFloats);           // two stages of A and B

    Loader la, lb;
    la.init(p.A, m0, p.M, p.lda, a_kc, kstop, t);
    lb.init(p.B, n0, p.N, p.ldb, b_kc, kstop, t);
    PartSums<EPI, KG> sums(part);
    f32x16 &acc = sums.acc;

    if (steps > 0) {
        la.load(kg0);
        lb.load(kg0);
        la.store(lds);
        lb.store(lds + kTileFloats);
    }
    __syncthreads();
    for (int s = 0; s < steps; ++s) {
        const float *as = lds + (s & 1) * (2 * kTileFloats), *bs = as + kTileFloats;
        float *nxt = lds + ((s & 1) ^ 1) * (2 * kTileFloats);
        const bool more = s + 1 < steps;
        if (more) {
            la.load(kg0 + (s + 1) * TK);
            lb.load(kg0 + (s + 1) * TK);
        }
        const float *ar = as + half * 16 * PITCH + wm * 32 + l32, *br = bs + half * 16 * PITCH + wn * 32 + l32;
        float av[16], bv[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            av[k] = ar[k * PITCH];
            bv[k] = br[k * PITCH];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[k], av[k], acc, 0, 0, 0);
        if (more) {
            la.store(nxt);
            lb.store(nxt + kTileFloats);
        }
        sums.step();                                             // (behind the stores, which leave the products time to finish)
        __syncthreads();
    }

    sums.finish();
    finish_tile<EPI, KG, 4>(p, at, acc, vec_out, smem_f32);
}

// The same for operands whose rows are whole 16-byte pieces, in the layouts that the stack uses: tiles go from memory to LDS without passing
// through registers, NS stages of 32 k, NS - 1 steps ahead.  A step's chain of latencies - load, LDS store, LDS read - is what bound the
// kernel above (50 - 60 TFLOP/s): here it is one wait for loads issued NS - 1 steps ago, and a k-contiguous operand takes one 16-byte LDS
// read for four matrix instructions.
// In a step of 32 k, instruction j of quad q multiplies k = 8 q + j (lanes 0 - 31) and 8 q + 4 + j (lanes 32 - 63).
// LDS, k-contiguous: rows of 128 bytes, 16-byte chunk c of row r at c ^ ((r >> 1) & 7); otherwise: 32 k rows of 256 bytes (128 for 32 columns), chunk c of
// k row r of 256 bytes at c ^ (r & 4 ? 8 : 0): the two halves of a wavefront read different banks.
template <int EPI, int TM, int KG, int NS, bool A_KC, bool B_KC, class In>
__global__ __launch_bounds__(4 * TM * KG) void gemm_f32_dma_kernel(In in, bool vec_out, int log_parts) {
    constexpr int W = TM / 16;                                   // wavefronts of a group, a quadrant of 32 x 32 each
    GemmParams<float> p;
    const Place at = place_of<EPI, TM>(in, p, vec_out);
    extern __shared__ __attribute__((aligned(16))) float smem_f32[];
    constexpr int kStage = (TM + TN) * TK, NA = TM / 8, NL = (TM + TN) / 8 / W;      // floats of a stage; A's loads; loads of a wavefront per step
    constexpr int kNewer = (NS - 2) * NL;
    static_assert(kNewer < 64, "vmcnt has six bits");
    constexpr int kWaitOlder = 0x0070 | (kNewer & 15) | (kNewer >> 4 << 14);       // s_waitcnt lgkmcnt(0) vmcnt(kNewer)
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * W)), wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) % W);
    const int lane = threadIdx.x & 63, wm = wave >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
    const int all = (at.kstop - at.kbeg + TK - 1) / TK, part = (all + (1 << log_parts) - 1) >> log_parts, each = (part << log_parts) / KG;
    const int steps = KG == 1 ? all : each;
    const int kg0 = at.kbeg + group * each * TK;
    float *ring = smem_f32 + group * NS * kStage;

    // load u = wave NL + i fills 1 KB of the stage, A's tile before B's: 8 rows of a k-contiguous operand; of the other layout 4 k rows (64 wide)
    // or 8 (32 wide)
    const float *base_a = A_KC ? p.A + (size_t)at.m0 * p.lda : p.A + at.m0, *base_b = B_KC ? p.B + (size_t)at.n0 * p.ldb : p.B + at.n0;
    int off[NL], kloc[NL];                                       // byte offset in the tile; first k of the piece
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int u = wave * NL + i;
        const bool is_a = u < NA;
        const int v = is_a ? u : u - NA, ld = is_a ? p.lda : p.ldb, rows = is_a ? p.M - at.m0 : p.N - at.n0;
        if (is_a ? A_KC : B_KC) {
            const int r = v * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            kloc[i] = 4 * c;
            off[i] = r < rows ? r * ld * 4 + c * 16 : kBufPoison;
        } else {
            const int log_row = is_a && TM == 32 ? 3 : 4;        // pieces of a k row
            const int r = (v << (6 - log_row)) + (lane >> log_row), c = (lane & ((1 << log_row) - 1)) ^ (log_row == 4 && (r & 4) ? 8 : 0);
            kloc[i] = r;
            off[i] = 4 * c < rows ? r * ld * 4 + c * 16 : kBufPoison;
        }
    }
    typedef __attribute__((address_space(3))) void *lds_ptr;
    auto load_step = [&](int s) __attribute__((always_inline)) {
        const int k0 = kg0 + s * TK, left = at.kstop - k0;
        float *stage = ring + (s % NS) * kStage + wave * NL * 256;
        // 64 rows: a wavefront loads one operand, A or B; 32: the first of its loads may be A's, the others B's
        const float *one = TM == 64 && wave >= 2 ? base_b + (B_KC ? (size_t)k0 : (size_t)k0 * p.ldb) : base_a + (A_KC ? (size_t)k0 : (size_t)k0 * p.lda);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(left > 0 ? one : base_a);
        const __amdgpu_buffer_rsrc_t rs_b = make_rsrc(left > 0 ? base_b + (B_KC ? (size_t)k0 : (size_t)k0 * p.ldb) : base_b);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int vo = kloc[i] < left ? off[i] : kBufPoison;
            if (TM == 64 || wave * NL + i < NA) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(stage + i * 256), 16, vo, 0, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_b, (lds_ptr)(stage + i * 256), 16, vo, 0, 0, 0);
        }
    };

    PartSums<EPI, KG> sums(part);
    f32x16 &acc = sums.acc;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < steps) load_step(s);
    const int ra = wm * 32 + l32, rb = wn * 32 + l32;
    for (int s = 0; s < steps; ++s) {
        // this wavefront's loads of step s have landed and its LDS reads of step s - 1 have returned; after the barrier the step is
        // published and the stage of step s - 1 is free
        if (NS > 2 && s + NS - 2 < steps) __builtin_amdgcn_s_waitcnt(kWaitOlder);
        else __builtin_amdgcn_s_waitcnt(0x0070);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + NS - 1 < steps) load_step(s + NS - 1);
        if (kg0 + s * TK >= at.kstop) continue;                  // (a group whose share ends before the others')
        const float *as = ring + (s % NS) * kStage, *bs = as + TM * TK;
        f32x4 av[4], bv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (A_KC) av[q] = *reinterpret_cast<const f32x4 *>(as + ra * TK + (((2 * q + half) ^ ((ra >> 1) & 7)) << 2));
            else {
#pragma unroll
                for (int j = 0; j < 4; ++j) av[q][j] = as[(8 * q + 4 * half + j) * TM + (TM == 64 ? ra ^ (half << 5) : ra)];
            }
            if constexpr (B_KC) bv[q] = *reinterpret_cast<const f32x4 *>(bs + rb * TK + (((2 * q + half) ^ ((rb >> 1) & 7)) << 2));
            else {
#pragma unroll
                for (int j = 0; j < 4; ++j) bv[q][j] = bs[(8 * q + 4 * half + j) * 64 + (rb ^ (half << 5))];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[q][j], av[q][j], acc, 0, 0, 0);
        sums.step();
    }
    sums.finish();
    if constexpr (KG > 1) __syncthreads();                       // nobody reads the ring any more
    finish_tile<EPI, KG, W>(p, at, acc, vec_out, smem_f32);
}

constexpr int smem_bytes(int kg) { return kg * 4 * kTileFloats * (int)sizeof(float); }       // 33.8 KB per group; at least the 16 KB per group of the final sum

// Stages of tiles of TM rows: four groups' fill the LDS
constexpr int dma_stages(int tm) { return tm == 64 ? 2 : 3; }
constexpr int dma_smem(int tm, int kg) { return kg * dma_stages(tm) * (tm + TN) * TK * (int)sizeof(float); }       // 32 or 36 KB per group
// The layout that the stack uses with an epilogue
template <int EPI> constexpr bool kDmaA = EPI != EPI_ACCUM_F32;
template <int EPI> constexpr bool kDmaB = EPI == EPI_STORE || EPI == EPI_MUL_DGELU;

// Whether the kernel without staging registers takes a product: by its layout, widths and addresses, never by the number of rows of an
// activation (bits).
template <int EPI> bool dma_takes(const GemmParams<float> &p, bool akc, bool bkc) {
    auto al16 = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
    if (akc != kDmaA<EPI> || bkc != kDmaB<EPI> || !al16(p.A) || !al16(p.B)) return false;
    if (((p.lda | p.ldb) & 3) != 0 || p.lda > kGemmMaxLd || p.ldb > kGemmMaxLd) return false;
    return ((akc ? p.K : p.M) & 3) == 0 && ((bkc ? p.K : p.N) & 3) == 0;
}

// Groups per workgroup.  With staging registers: as many as have at least one step each, while the grid leaves room for their wavefronts.
// Without: four where that leaves every workgroup a compute unit of its own, else two, whose 64 KB let two workgroups share one
// (800 x 480 x 512, 104 tiles: 12.1 with four, 12.9 with two, 16.4 us with one; 3200 x 480 x 256, 400 tiles: 16.3, 14.8, 16.0;
// 12800 x 1536 x 512, 4800 tiles: 211, 197, 222).
template <int EPI, int TM, class In> void launch_dma_f32(const In &in, dim3 grid, int kg, int log_parts, bool vec_out, hipStream_t s) {
    constexpr bool A = kDmaA<EPI>, B = kDmaB<EPI>;
    constexpr int NS = dma_stages(TM);
    if (kg == 4) hipLaunchKernelGGL((gemm_f32_dma_kernel<EPI, TM, 4, NS, A, B, In>), grid, dim3(16 * TM), dma_smem(TM, 4), s, in, vec_out, log_parts);
    else if (kg == 2) hipLaunchKernelGGL((gemm_f32_dma_kernel<EPI, TM, 2, NS, A, B, In>), grid, dim3(8 * TM), dma_smem(TM, 2), s, in, vec_out, log_parts);
    else hipLaunchKernelGGL((gemm_f32_dma_kernel<EPI, TM, 1, NS, A, B, In>), grid, dim3(4 * TM), dma_smem(TM, 1), s, in, vec_out, log_parts);
}
// Tiles of 32 rows where they leave every workgroup a compute unit of its own (work32, grid32), three stages instead of two: half the matrix
// instructions per SIMD and a step more on its way, with the same order of every sum (us): 2048 x 256 x 1024 20.6 -> 13.7, x 256 7.8 -> 5.7,
// 128 x 512 x 2048 36 -> 23, 256 x 192 x 64 4.7 -> 4.3.  With more of them than compute units the larger tiles' better use of what they load wins:
// 2048 x 320 x 960 (320) 20 against 25, 8192 x 512 x 2048 142 against 175.
template <int EPI, class In>
void launch_tiles_f32(const In &in, dim3 grid, long work, dim3 grid32, long work32, int most, bool akc, bool bkc, bool dma, bool vec_out, hipStream_t s) {
    if (dma) {
        const int kg = std::min(most, work > 256 ? 2 : 4);
        const int log_parts = (EPI == EPI_ACCUM_F32 ? kg : most) >> 1;
        if (work32 <= 256) return launch_dma_f32<EPI, 32>(in, grid32, kg, log_parts, vec_out, s);
        return launch_dma_f32<EPI, 64>(in, grid, kg, log_parts, vec_out, s);
    }
    const int kg = work >= 512 ? 1 : most;
    const int log_parts = (EPI == EPI_ACCUM_F32 ? kg : most) >> 1;          // a weight gradient's k range differs with the grouping anyway
    if (kg == 4) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 4, In>), grid, dim3(1024), smem_bytes(4), s, in, akc, bkc, vec_out, log_parts);
    else if (kg == 2) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, In>), grid, dim3(512), smem_bytes(2), s, in, akc, bkc, vec_out, log_parts);
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, 1, In>), grid, dim3(256), smem_bytes(1), s, in, akc, bkc, vec_out, log_parts);
}

template <int EPI> void launch_epi(const GemmParams<float> &p, bool akc, bool bkc, hipStream_t s) {
    const int tm = (p.M + 63) / 64, tn = (p.N + TN - 1) / TN;
    const long tiles = (long)tm * tn;
    auto al16 = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
    const bool vec_out = (p.ldc & 3) == 0 && (EPI == EPI_ACCUM_F32 ? al16(p.outf) : al16(p.out)) && (EPI != EPI_BIAS_GELU || al16(p.out2)) &&
                         ((EPI != EPI_BIAS_RESID && EPI != EPI_MUL_DGELU) || al16(p.aux)) &&
                         ((EPI != EPI_BIAS && EPI != EPI_BIAS_RESID && EPI != EPI_BIAS_GELU) || al16(p.bias));
    const int most = p.K > 2 * TK ? 4 : p.K > TK ? 2 : 1;
    const double mn = (double)p.M * p.N;
    const bool dma = dma_takes<EPI>(p, akc, bkc);
    ProfScope scope(dma ? "gemm_f32_kernel<dma>" : "gemm_f32_kernel", 2.0 * mn * p.K, 4.0 * ((double)p.M * p.K + (double)p.K * p.N + mn), s);
    const int tm32 = (p.M + 31) / 32;
    launch_tiles_f32<EPI>(p, dim3(tn, tm), tiles, dim3(tn, tm32), (long)tm32 * tn, most, akc, bkc, dma, vec_out, s);
}

template <int EPI, class In = GemmParams<float>> hipError_t raise_epi() {
    hipError_t e = hipSuccess;
    auto raise = [&](const void *kernel, int bytes) {
        if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    };
    constexpr bool A = kDmaA<EPI>, B = kDmaB<EPI>;
    raise(reinterpret_cast<const void *>(gemm_f32_kernel<EPI, 4, In>), smem_bytes(4));
    raise(reinterpret_cast<const void *>(gemm_f32_kernel<EPI, 2, In>), smem_bytes(2));
    raise(reinterpret_cast<const void *>(gemm_f32_dma_kernel<EPI, 64, 4, dma_stages(64), A, B, In>), dma_smem(64, 4));
    raise(reinterpret_cast<const void *>(gemm_f32_dma_kernel<EPI, 64, 2, dma_stages(64), A, B, In>), dma_smem(64, 2));
    raise(reinterpret_cast<const void *>(gemm_f32_dma_kernel<EPI, 64, 1, dma_stages(64), A, B, In>), dma_smem(64, 1));
    raise(reinterpret_cast<const void *>(gemm_f32_dma_kernel<EPI, 32, 4, dma_stages(32), A, B, In>), dma_smem(32, 4));
    raise(reinterpret_cast<const void *>(gemm_f32_dma_kernel<EPI, 32, 2, dma_stages(32), A, B, In>), dma_smem(32, 2));
    raise(reinterpret_cast<const void *>(gemm_f32_dma_kernel<EPI, 32, 1, dma_stages(32), A, B, In>), dma_smem(32, 1));
    return e;
}

// The sums of a group's slices, one product after the other; outputs without gaps between their rows.
struct ReduceGroup {
    const float *partial[kGemmGroup];
    float *out[kGemmGroup];
    size_t n[kGemmGroup];
    float beta[kGemmGroup];
    int slices, count;
};
__global__ __launch_bounds__(256) void gemm_f32_reduce_group_kernel(ReduceGroup g, size_t all) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < all; i += (size_t)gridDim.x * 256) {
        int z = 0;
        size_t at = i;
        while (z + 1 < g.count && at >= g.n[z]) at -= g.n[z++];
        float acc = g.partial[z][at];
#pragma unroll 4
        for (int k = 1; k < g.slices; ++k) acc += g.partial[z][k * g.n[z] + at];
        float *o = g.out[z] + at;
        *o = g.beta[z] == 0.f ? acc : g.beta[z] * *o + acc;
    }
}

}  // namespace

// Slices for several weight gradients in one launch, by what they take (192 tiles x 2048: 41 us in one piece, 40 + 5 in two slices,
// 35 + 6 in four): up to 256 workgroups of four groups 2.35 us per 128 k, up to 512 of two groups 2.3 us per 64 k, some us around
// them, and the second kernel with the way of the partial results through memory.
int gemm_f32_group_slices(const int *M, const int *N, int n, int K) {
    long tiles = 0;
    double outputs = 0.0;
    for (int i = 0; i < n; ++i) {
        tiles += (long)((M[i] + 63) / 64) * ((N[i] + TN - 1) / TN);
        outputs += (double)M[i] * N[i];
    }
    int best = 1;
    double best_us = 0.0;
    for (int s = 1; s <= std::min(16, std::max(1, K / 256)); ++s) {
        const long items = tiles * s;
        const double k = (double)K / s, sum = s > 1 ? 4.0 + (s + 1) * outputs * 4.0 / 4.5e6 : 0.0;
        const double us = sum + (items <= 256 ? k / 128.0 * 2.35 + 4.0 : (double)((items + 511) / 512) * (k / 64.0 * 2.3 + 3.0));
        if (s == 1 || us < best_us) best = s, best_us = us;
    }
    return best;
}

// floats of a product's partial results: the next one's begin on a 16-byte boundary
static size_t slices_of_one(int M, int N, int slices) { return ((size_t)slices * M * N + 3) / 4 * 4; }
size_t gemm_f32_group_floats(const int *M, const int *N, int n, int slices) {
    size_t floats = 0;
    for (int i = 0; i < n && slices > 1; ++i) floats += slices_of_one(M[i], N[i], slices);
    return floats;
}

void launch_gemm_f32_group(const GemmParams<float> *p, int n, hipStream_t s) {
    (void)prepare_kernels();
    int M[kGemmGroup], N[kGemmGroup];
    long tiles = 0, tiles32 = 0;
    double flops = 0.0, bytes = 0.0;
    for (int i = 0; i < n; ++i) {
        M[i] = p[i].M;
        N[i] = p[i].N;
        tiles += (long)((M[i] + 63) / 64) * ((N[i] + TN - 1) / TN);
        tiles32 += (long)((M[i] + 31) / 32) * ((N[i] + TN - 1) / TN);
        flops += 2.0 * M[i] * N[i] * p[i].K;
        bytes += 4.0 * ((double)M[i] * p[i].K + (double)p[i].K * N[i] + (double)M[i] * N[i]);
    }
    const int K = p[0].K;
    int slices = gemm_f32_group_slices(M, N, n, K);
    if (!p[0].partial || gemm_f32_group_floats(M, N, n, slices) > p[0].partial_floats) slices = 1;
    const int kchunk = slices > 1 ? ((K + slices - 1) / slices + TK - 1) / TK * TK : K;
    GemmGroup<float> group{};
    ReduceGroup sum{};
    group.n = sum.count = n;
    sum.slices = slices > 1 ? (K + kchunk - 1) / kchunk : 1;
    size_t used = 0, all = 0;
    for (int i = 0; i < n; ++i) {
        GemmParams<float> &q = group.p[i];
        q = p[i];
        q.kchunk = kchunk;
        q.ksplit = sum.slices;
        if (sum.slices > 1) q.partial = p[0].partial + used;
        sum.partial[i] = q.partial;
        sum.out[i] = q.outf;
        sum.n[i] = (size_t)M[i] * N[i];
        sum.beta[i] = q.beta;
        used += slices_of_one(M[i], N[i], sum.slices);
        all += sum.n[i];
    }
    const dim3 grid((unsigned)(tiles * sum.slices));
    const int most = kchunk > 2 * TK ? 4 : kchunk > TK ? 2 : 1;
    bool dma = true;
    for (int i = 0; i < n; ++i) dma = dma && dma_takes<EPI_ACCUM_F32>(p[i], false, false);
    {
        ProfScope scope(dma ? "gemm_f32_kernel<dma> (grouped)" : "gemm_f32_kernel (grouped)", flops, bytes, s);
        launch_tiles_f32<EPI_ACCUM_F32>(group, grid, tiles * sum.slices, dim3((unsigned)(tiles32 * sum.slices)), tiles32 * sum.slices, most, false, false, dma,
                                        false, s);
    }
    if (sum.slices > 1) {
        ProfScope scope("gemm_f32_reduce_kernel", (double)sum.slices * all, 4.0 * all * (sum.slices + (p[0].beta != 0.f ? 2.0 : 1.0)), s);
        hipLaunchKernelGGL(gemm_f32_reduce_group_kernel, dim3((unsigned)std::min<size_t>((all + 255) / 256, 2048)), dim3(256), 0, s, sum, all);
    }
}

hipError_t gemm_f32_prepare_kernels() {
    hipError_t e = raise_epi<EPI_STORE>();
    if (e == hipSuccess) e = raise_epi<EPI_BIAS>();
    if (e == hipSuccess) e = raise_epi<EPI_BIAS_RESID>();
    if (e == hipSuccess) e = raise_epi<EPI_BIAS_GELU>();
    if (e == hipSuccess) e = raise_epi<EPI_MUL_DGELU>();
    if (e == hipSuccess) e = raise_epi<EPI_ACCUM_F32>();
    if (e == hipSuccess) e = raise_epi<EPI_ACCUM_F32, GemmGroup<float>>();
    return e;
}

void launch_gemm_f32(const GemmParams<float> &p, bool a_kmajor, bool b_kmajor, Epilogue epi, hipStream_t s) {
    if (p.M == 0 || p.N == 0) return;
    (void)prepare_kernels();
    switch (epi) {
        case EPI_STORE: launch_epi<EPI_STORE>(p, a_kmajor, b_kmajor, s); break;
        case EPI_BIAS: launch_epi<EPI_BIAS>(p, a_kmajor, b_kmajor, s); break;
        case EPI_BIAS_RESID: launch_epi<EPI_BIAS_RESID>(p, a_kmajor, b_kmajor, s); break;
        case EPI_BIAS_GELU: launch_epi<EPI_BIAS_GELU>(p, a_kmajor, b_kmajor, s); break;
        case EPI_MUL_DGELU: launch_epi<EPI_MUL_DGELU>(p, a_kmajor, b_kmajor, s); break;
        case EPI_ACCUM_F32: launch_epi<EPI_ACCUM_F32>(p, a_kmajor, b_kmajor, s); break;
    }
}

}  // namespace lga
