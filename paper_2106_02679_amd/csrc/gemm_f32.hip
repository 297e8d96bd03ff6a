// fp32 GEMM on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: full fp32 products and sums), any shape, any of the
// four operand layouts.
//
// What bounds it at the sizes the fp32 mode is used at (widths of 64 ... 512, a few thousand tokens) is not arithmetic
// but the length of the serial chain over k and the number of compute units that work at all: a weight gradient has
// 4 ... 64 output tiles and contracts over every token of the step.  So
//  - a tile is 64 x 64, multiplied by a group of four wavefronts (one 32 x 32 quadrant each), 32 k per step, the next
//    step's operands on their way from memory to registers while this one is multiplied, one barrier per step;
//  - a workgroup holds KG = 1, 2 or 4 such groups, each of which takes its own part of the k range; their sums meet in
//    LDS at the end, in group order (the result does not depend on scheduling), and every group then writes its
//    share of the tile.  One group alone adds up the same parts in the same order, so that an activation does not depend
//    on how many rows share its launch: the parts follow from K, only the groups from the number of tiles;
//  - where even that leaves compute units idle, the k range is cut into slices over the grid and the partial results
//    are added in slice order by a second kernel (only with scratch, i.e. for the stack's weight gradients).
// Measured (one MI355X; before: plain FMA on 64 x 64 x 16 tiles, loads waited for at once, no split of k), averages over the
// launches of a step: 256-wide stack of 2048 tokens - weight gradients 440 -> 15 us plus 5 us for the sum of the slices,
// input gradients 116 -> 19, QKV 55 -> 18, first feed-forward with GELU 65 -> 21; 64-wide stack of 256 tokens - 52 -> 9,
// 29 -> 9, 16 -> 5, 17 -> 6 us.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace lga {

namespace {

constexpr int TM = 64, TN = 64, TK = 32;
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
            p.out2[at] = u;
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
            *reinterpret_cast<f32x4 *>(p.out2 + idx) = o;
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

// grid: (n tiles, m tiles, k slices); block: 256 KG threads.  vec_out: every tensor the epilogue touches takes 16-byte accesses
// at columns that are multiples of 4.  log_parts: into 1, 2 or 4 parts the k range is cut for the order of the sums; with KG > 1 KG of them.
template <int EPI, int KG>
__global__ __launch_bounds__(256 * KG) void gemm_f32_kernel(GemmParams<float> p, bool a_kc, bool b_kc, bool vec_out, int log_parts) {
    extern __shared__ __attribute__((aligned(16))) float smem_f32[];
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), t = threadIdx.x & 255;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    int kbeg = 0, kstop = p.K;
    if constexpr (EPI == EPI_ACCUM_F32) {
        if (p.ksplit > 1) {                     // slice blockIdx.z of the k range, into partial result z ([M][N], dense)
            kbeg = blockIdx.z * p.kchunk;
            kstop = min(p.K, kbeg + p.kchunk);
            p.outf = p.partial + (size_t)blockIdx.z * p.M * p.N;
            p.ldc = p.N;
            p.beta = 0.f;
        }
    }
    // a part of the k range: whole steps, the same number for every part; a group has one (and reads zeros if it is empty), or
    // one group has all
    const int all = (kstop - kbeg + TK - 1) / TK, part = KG == 1 ? (all + (1 << log_parts) - 1) >> log_parts : (all + KG - 1) / KG;
    const int steps = KG == 1 ? all : part;
    const int kg0 = kbeg + group * part * TK;
    float *lds = smem_f32 + group * (4 * kTileFloats);           // two stages of A and B

    Loader la, lb;
    la.init(p.A, m0, p.M, p.lda, a_kc, kstop, t);
    lb.init(p.B, n0, p.N, p.ldb, b_kc, kstop, t);
    f32x16 acc, done;                                            // of the part at hand; of the parts before it (KG = 1)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = done[r] = 0.f;
    int left = part;

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
        if (KG == 1 && --left == 0) {                            // end of a part (behind the stores, which leave the products time to finish)
            left = part;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                done[r] += acc[r];
                acc[r] = 0.f;
            }
        }
        __syncthreads();
    }

    // lane: row m = l32 of the quadrant, columns n = 8 q + 4 half + (0 .. 3)
    const int m = m0 + wm * 32 + l32;
    const int nq = n0 + wn * 32 + 4 * half;
    if constexpr (KG == 1) {
        if (m >= p.M) return;
#pragma unroll
        for (int r = 0; r < 16; ++r) done[r] += acc[r];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (nq + 8 * q < p.N) epilogue_f32<EPI>(p, m, nq + 8 * q, f32x4{done[4 * q], done[4 * q + 1], done[4 * q + 2], done[4 * q + 3]}, vec_out);
    } else {
        // every group leaves its sums in LDS (the loop's last barrier has passed); group g then adds up column quads
        // g, g + KG, ... of all groups, in group order
        f32x4 *red = reinterpret_cast<f32x4 *>(smem_f32);
#pragma unroll
        for (int q = 0; q < 4; ++q) red[((group * 4 + wave) * 4 + q) * 64 + lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        __syncthreads();
        if (m >= p.M) return;
#pragma unroll
        for (int j = 0; j < 4 / KG; ++j) {
            const int q = group + j * KG;
            if (nq + 8 * q >= p.N) continue;
            f32x4 sum = red[(wave * 4 + q) * 64 + lane];
#pragma unroll
            for (int g = 1; g < KG; ++g) {
                const f32x4 o = red[((g * 4 + wave) * 4 + q) * 64 + lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[i] += o[i];
            }
            epilogue_f32<EPI>(p, m, nq + 8 * q, sum, vec_out);
        }
    }
}

// out[m, n] = beta * out[m, n] + sum_z partial[z][m][n], the slices in index order
__global__ __launch_bounds__(256) void gemm_f32_reduce_kernel(const float *__restrict__ partial, int slices, float *__restrict__ out,
                                                              int M, int N, int ldc, float beta) {
    const size_t n_all = (size_t)M * N;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_all; i += (size_t)gridDim.x * 256) {
        float acc = partial[i];
#pragma unroll 4
        for (int z = 1; z < slices; ++z) acc += partial[(size_t)z * n_all + i];
        float *o = out + i / N * ldc + i % N;
        *o = beta == 0.f ? acc : beta * *o + acc;
    }
}

constexpr int smem_bytes(int kg) { return kg * 4 * kTileFloats * (int)sizeof(float); }       // 33.8 KB per group; at least the 16 KB per group of the final sum

template <int EPI> void launch_epi(const GemmParams<float> &p, bool akc, bool bkc, hipStream_t s) {
    const int tm = (p.M + TM - 1) / TM, tn = (p.N + TN - 1) / TN;
    const long tiles = (long)tm * tn;
    auto al16 = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
    const bool vec_out = (p.ldc & 3) == 0 && (EPI == EPI_ACCUM_F32 ? al16(p.outf) : al16(p.out)) && (EPI != EPI_BIAS_GELU || al16(p.out2)) &&
                         ((EPI != EPI_BIAS_RESID && EPI != EPI_MUL_DGELU) || al16(p.aux)) &&
                         ((EPI != EPI_BIAS && EPI != EPI_BIAS_RESID && EPI != EPI_BIAS_GELU) || al16(p.bias));
    GemmParams<float> q = p;
    q.ksplit = 1;
    if (EPI == EPI_ACCUM_F32 && p.partial && p.K > 0) {
        const int slices = gemm_f32_slices(p.M, p.N, p.K);
        if (slices > 1 && (size_t)slices * p.M * p.N <= p.partial_floats) {
            q.kchunk = ((p.K + slices - 1) / slices + TK - 1) / TK * TK;
            q.ksplit = (p.K + q.kchunk - 1) / q.kchunk;
        }
    }
    const dim3 grid(tn, tm, q.ksplit);
    const bool vo = q.ksplit > 1 ? (p.N & 3) == 0 && al16(p.partial) : vec_out;
    const int k_each = q.ksplit > 1 ? q.kchunk : p.K;
    // Groups per workgroup: as many as have at least one step each, while the grid leaves room for their wavefronts - a
    // compute unit holds 32 of them, so from 512 tiles on single groups already fill the chip twice.
    const int most = k_each > 2 * TK ? 4 : k_each > TK ? 2 : 1, kg = tiles * q.ksplit >= 512 ? 1 : most;
    const int log_parts = (EPI == EPI_ACCUM_F32 ? kg : most) >> 1;          // a weight gradient's k range differs with the grouping anyway
    {
        const double mn = (double)p.M * p.N;
        ProfScope scope("gemm_f32_kernel", 2.0 * mn * p.K, 4.0 * ((double)p.M * p.K + (double)p.K * p.N + mn), s);
        if (kg == 4) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 4>), grid, dim3(1024), smem_bytes(4), s, q, akc, bkc, vo, log_parts);
        else if (kg == 2) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2>), grid, dim3(512), smem_bytes(2), s, q, akc, bkc, vo, log_parts);
        else hipLaunchKernelGGL((gemm_f32_kernel<EPI, 1>), grid, dim3(256), smem_bytes(1), s, q, akc, bkc, vo, log_parts);
    }
    if (q.ksplit > 1) {
        ProfScope scope("gemm_f32_reduce_kernel", (double)q.ksplit * p.M * p.N, 4.0 * p.M * p.N * (q.ksplit + (p.beta != 0.f ? 2.0 : 1.0)), s);
        const unsigned blocks = (unsigned)std::min<size_t>(((size_t)p.M * p.N + 255) / 256, 2048);
        hipLaunchKernelGGL(gemm_f32_reduce_kernel, dim3(blocks), dim3(256), 0, s, p.partial, q.ksplit, p.outf, p.M, p.N, p.ldc, p.beta);
    }
}

template <int EPI> hipError_t raise_epi() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_f32_kernel<EPI, 4>), hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes(4));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_f32_kernel<EPI, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes(2));
    return e;
}

}  // namespace

// Slices of the k range over the grid: enough for 256 workgroups, each with at least 256 k (two steps for each of its four
// groups - below that the second kernel and the partial results cost more than the shorter chain gives).
int gemm_f32_slices(int M, int N, int K) {
    const long tiles = (long)((M + TM - 1) / TM) * ((N + TN - 1) / TN);
    long cap = 16;
    if (K > 0) cap = std::min<long>(cap, K / 256);
    return (int)std::max<long>(1, std::min<long>(cap, 256 / std::max<long>(1, tiles)));
}

hipError_t gemm_f32_prepare_kernels() {
    hipError_t e = raise_epi<EPI_STORE>();
    if (e == hipSuccess) e = raise_epi<EPI_BIAS>();
    if (e == hipSuccess) e = raise_epi<EPI_BIAS_RESID>();
    if (e == hipSuccess) e = raise_epi<EPI_BIAS_GELU>();
    if (e == hipSuccess) e = raise_epi<EPI_MUL_DGELU>();
    if (e == hipSuccess) e = raise_epi<EPI_ACCUM_F32>();
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
