// HBM-bound kernels of the layer stack: parameter cast, LayerNorm forward / backward, column
// sums (bias and LayerNorm-affine gradients), Adam, counter-based weight fill.
// All arithmetic is fp32; T (float, bf16 or f16) is only the storage type of activations.
#include <climits>
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "row_walk.h"

namespace lga {

namespace {

template <class T> struct VecOf;
template <> struct VecOf<float> { static constexpr int N = 4; };
template <> struct VecOf<bf16> { static constexpr int N = 8; };
template <> struct VecOf<f16> { static constexpr int N = 8; };

template <class T, int N> struct alignas(sizeof(T) * N) Pack { T v[N]; };

template <class T, int N> __device__ __forceinline__ void load_pack(const T *p, float (&out)[N]) {
    if constexpr (N == 1) {
        out[0] = to_f32(p[0]);
    } else {
        const Pack<T, N> t = *reinterpret_cast<const Pack<T, N> *>(p);
#pragma unroll
        for (int i = 0; i < N; ++i) out[i] = to_f32(t.v[i]);
    }
}
template <class T, int N> __device__ __forceinline__ void store_pack(T *p, const float (&in)[N]) {
    if constexpr (N == 1) {
        p[0] = from_f32<T>(in[0]);
    } else {
        Pack<T, N> t;
#pragma unroll
        for (int i = 0; i < N; ++i) t.v[i] = from_f32<T>(in[i]);
        *reinterpret_cast<Pack<T, N> *>(p) = t;
    }
}

constexpr int kLnWave = 4, kLnbWave = 2;

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ------------------------------------------------------------------------------------------
template <class E>
__global__ void cast_kernel(const float *__restrict__ src, E *__restrict__ dst, size_t n, size_t n4) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        const f32x4 v = reinterpret_cast<const f32x4 *>(src)[i];
        x4<E> o;
        o[0] = (E)v[0]; o[1] = (E)v[1]; o[2] = (E)v[2]; o[3] = (E)v[3];
        reinterpret_cast<x4<E> *>(dst)[i] = o;
    }
    for (size_t i = n4 * 4 + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = (E)src[i];
}

// *flag = 1 if any of the n values is not finite.  Every thread that sees one stores the same 1 (plain vector store).
__global__ __launch_bounds__(256) void nonfinite_flag_kernel(const float *__restrict__ g, size_t n, size_t n4,
                                                             int *__restrict__ flag) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        const f32x4 v = reinterpret_cast<const f32x4 *>(g)[i];
        // x - x is 0 for finite x and NaN for infinities and NaNs
        const float t = (v[0] - v[0]) + (v[1] - v[1]) + (v[2] - v[2]) + (v[3] - v[3]);
        bad |= !(t == 0.f);
    }
    for (size_t i = n4 * 4 + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) bad |= !(g[i] - g[i] == 0.f);
    if (bad) *flag = 1;
}

__global__ void fill_const_kernel(float *dst, size_t n, float value) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = value;
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Element i <- std * N(0,1) from a 64-bit mix of (seed, i) and Box-Muller.
__global__ void fill_normal_kernel(float *dst, size_t n, float std, uint64_t seed) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t h = mix64(seed * 0xD1342543DE82EF95ull + i);
        const float u1 = ((float)(uint32_t)(h >> 40) + 1.0f) * (1.0f / 16777217.0f);   // (0, 1)
        const float u2 = (float)(uint32_t)((h >> 8) & 0xFFFFFFu) * (1.0f / 16777216.0f);
        dst[i] = std * sqrtf(-2.0f * __logf(u1)) * __cosf(6.283185307179586f * u2);
    }
}

// ------------------------------------------------------------------------------------------
// LayerNorm forward: one block per row.
template <class T, int V>
__global__ __launch_bounds__(256) void layernorm_fwd_kernel(const T *__restrict__ x, const float *__restrict__ g,
                                                            const float *__restrict__ b, T *__restrict__ y,
                                                            float *__restrict__ mean_out, float *__restrict__ rstd_out,
                                                            int d, float eps) {
    __shared__ float red[16];
    const size_t row = blockIdx.x;
    const T *xr = x + row * (size_t)d;
    T *yr = y + row * (size_t)d;
    float s = 0.f;
    for (int c = threadIdx.x * V; c < d; c += blockDim.x * V) {
        float v[V];
        load_pack<T, V>(xr + c, v);
#pragma unroll
        for (int i = 0; i < V; ++i) s += v[i];
    }
    const float mean = block_sum(s, red) / (float)d;
    float q = 0.f;
    for (int c = threadIdx.x * V; c < d; c += blockDim.x * V) {
        float v[V];
        load_pack<T, V>(xr + c, v);
#pragma unroll
        for (int i = 0; i < V; ++i) q += (v[i] - mean) * (v[i] - mean);
    }
    const float var = block_sum(q, red) / (float)d;
    const float rstd = rsqrtf(var + eps);
    if (threadIdx.x == 0) {
        mean_out[row] = mean;
        rstd_out[row] = rstd;
    }
    for (int c = threadIdx.x * V; c < d; c += blockDim.x * V) {
        float v[V], o[V];
        load_pack<T, V>(xr + c, v);
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] = (v[i] - mean) * rstd * g[c + i] + b[c + i];
        store_pack<T, V>(yr + c, o);
    }
}

// The same with a block walking over many rows and everything it needs more than once in registers: each thread
// keeps its NP packs of the row (one global read of x instead of three) and, if CACHE_GB, its gains and biases (read
// per row they are 8 bytes per element of L2 traffic against 4 bytes of x and y).  Wide rows use large blocks, so
// that a thread holds few packs and many wavefronts fit on a CU.  d <= TH * V * NP.  The forward pass and the
// recompute of the backward pass run the same variant, so they still agree bit for bit.
template <class T, int V, int TH, int NP, bool CACHE_GB>
__global__ __launch_bounds__(TH) void layernorm_fwd_rows_kernel(const T *__restrict__ x, const float *__restrict__ g,
                                                                 const float *__restrict__ b, T *__restrict__ y,
                                                                 float *__restrict__ mean_out, float *__restrict__ rstd_out,
                                                                 int rows, int d, float eps, T *__restrict__ keep) {
    // Two scratch rows used in turn: a sum's barrier also separates the other row's readers from its next writers,
    // so each block-wide sum costs one barrier.
    __shared__ float red[2][16];
    auto sum_all = [&](float v, int which) {
        v = wave_sum(v);
        if ((threadIdx.x & 63) == 0) red[which][threadIdx.x >> 6] = v;
        __syncthreads();
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < TH / 64; ++i) t += red[which][i];
        return t;
    };
    constexpr int NG = CACHE_GB ? NP : 1;
    float gv[NG][V], bv[NG][V];
    if constexpr (CACHE_GB) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
#pragma unroll
                for (int q = 0; q < V / 4; ++q) {
                    float t4[4], u4[4];
                    load_pack<float, 4>(g + c + 4 * q, t4);
                    load_pack<float, 4>(b + c + 4 * q, u4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        gv[p][4 * q + i] = t4[i];
                        bv[p][4 * q + i] = u4[i];
                    }
                }
            }
        }
    }
    // The next row's packs are requested before this row's two block-wide sums, so that loads stay in flight while
    // the block waits at its barriers.
    Pack<T, V> nxt[NP];
    auto request = [&](size_t row) {
        const T *xr = x + row * (size_t)d;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) nxt[p] = *reinterpret_cast<const Pack<T, V> *>(xr + c);
        }
    };
    if (blockIdx.x < (unsigned)rows) request(blockIdx.x);
    for (size_t row = blockIdx.x; row < (size_t)rows; row += gridDim.x) {
        T *yr = y + row * (size_t)d;
        float xv[NP][V];
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    xv[p][i] = to_f32(nxt[p].v[i]);
                    s += xv[p][i];
                }
                if (keep) *reinterpret_cast<Pack<T, V> *>(keep + row * (size_t)d + c) = nxt[p];
            }
        }
        if (row + gridDim.x < (size_t)rows) request(row + gridDim.x);
        const float mean = sum_all(s, 0) / (float)d;
        float q = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
#pragma unroll
                for (int i = 0; i < V; ++i) q += (xv[p][i] - mean) * (xv[p][i] - mean);
            }
        }
        const float var = sum_all(q, 1) / (float)d;
        const float rstd = rsqrtf(var + eps);
        if (threadIdx.x == 0) {
            mean_out[row] = mean;
            rstd_out[row] = rstd;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
                float o[V];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float gi = CACHE_GB ? gv[CACHE_GB ? p : 0][i] : g[c + i];
                    const float bi = CACHE_GB ? bv[CACHE_GB ? p : 0][i] : b[c + i];
                    o[i] = (xv[p][i] - mean) * rstd * gi + bi;
                }
                store_pack<T, V>(yr + c, o);
            }
        }
    }
}

// Narrow rows: a wavefront has a whole row, NP packs a lane, and its sums need no barrier.  In blocks of 256 threads for one row, 96 of
// them work on 768 bf16 elements, and every row costs two barriers (16-bit 32768 x 768: 30 us with the kernel above, 17 with this one;
// 65536 x 256: 51 and 17; 16384 x 1536: 18.5 and 17.3; fp32 8192 x 512: 10.1 and 5.8).  d <= 64 V NP.
template <class T, int V, int NP>
__global__ __launch_bounds__(256) void layernorm_fwd_wave_kernel(const T *__restrict__ x, const float *__restrict__ g, const float *__restrict__ b,
                                                                 T *__restrict__ y, float *__restrict__ mean_out, float *__restrict__ rstd_out,
                                                                 int rows, int d, float eps, T *__restrict__ keep) {
    const int lane = threadIdx.x & 63;
    RowWalk walk(blockIdx.x, gridDim.x, threadIdx.x >> 6, rows);
    Pack<T, V> nxt[NP];
    auto request = [&](int r) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if ((p * 64 + lane) * V < d) nxt[p] = *reinterpret_cast<const Pack<T, V> *>(x + (size_t)r * d + (p * 64 + lane) * V);
    };
    if (walk.valid()) request(walk.row);
    float gv[NP][V], bv[NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int c = (p * 64 + lane) * V;
        if (c < d) {
#pragma unroll
            for (int q = 0; q < V; q += 4) {
                const f32x4 t4 = *reinterpret_cast<const f32x4 *>(g + c + q), u4 = *reinterpret_cast<const f32x4 *>(b + c + q);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gv[p][q + i] = t4[i];
                    bv[p][q + i] = u4[i];
                }
            }
        }
    }
    for (; walk.valid(); walk.advance()) {
        const int row = walk.row;
        float xv[NP][V], s = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < V; ++i) {
                xv[p][i] = (p * 64 + lane) * V < d ? to_f32(nxt[p].v[i]) : 0.f;
                s += xv[p][i];
            }
        if (keep)
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if ((p * 64 + lane) * V < d) *reinterpret_cast<Pack<T, V> *>(keep + (size_t)row * d + (p * 64 + lane) * V) = nxt[p];
        if (walk.has_next()) request(walk.next());
        const float mean = wave_sum(s) / (float)d;
        float q = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if ((p * 64 + lane) * V < d) {
#pragma unroll
                for (int i = 0; i < V; ++i) q += (xv[p][i] - mean) * (xv[p][i] - mean);
            }
        const float rstd = rsqrtf(wave_sum(q) / (float)d + eps);
        if (lane == 0) {
            mean_out[row] = mean;
            rstd_out[row] = rstd;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * 64 + lane) * V;
            if (c < d) {
                float o[V];
#pragma unroll
                for (int i = 0; i < V; ++i) o[i] = (xv[p][i] - mean) * rstd * gv[p][i] + bv[p][i];
                store_pack<T, V>(y + (size_t)row * d + c, o);
            }
        }
    }
}

// LayerNorm backward w.r.t. the input, plus residual: one block per row.
template <class T, int V>
__global__ __launch_bounds__(256) void layernorm_bwd_dx_kernel(const T *__restrict__ dy, const T *__restrict__ x,
                                                               const float *__restrict__ mean,
                                                               const float *__restrict__ rstd,
                                                               const float *__restrict__ g, const T *resid,
                                                               T *dx, int d) {
    __shared__ float red[16];
    const size_t row = blockIdx.x;
    const T *dyr = dy + row * (size_t)d;
    const T *xr = x + row * (size_t)d;
    const T *rr = resid + row * (size_t)d;
    T *dxr = dx + row * (size_t)d;
    const float mu = mean[row], rs = rstd[row];
    float s1 = 0.f, s2 = 0.f;
    for (int c = threadIdx.x * V; c < d; c += blockDim.x * V) {
        float a[V], v[V];
        load_pack<T, V>(dyr + c, a);
        load_pack<T, V>(xr + c, v);
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const float gd = a[i] * g[c + i];
            s1 += gd;
            s2 += gd * (v[i] - mu) * rs;
        }
    }
    s1 = block_sum(s1, red) / (float)d;
    s2 = block_sum(s2, red) / (float)d;
    for (int c = threadIdx.x * V; c < d; c += blockDim.x * V) {
        float a[V], v[V], r[V], o[V];
        load_pack<T, V>(dyr + c, a);
        load_pack<T, V>(xr + c, v);
        load_pack<T, V>(rr + c, r);
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const float xhat = (v[i] - mu) * rs;
            o[i] = r[i] + rs * (a[i] * g[c + i] - s1 - xhat * s2);
        }
        store_pack<T, V>(dxr + c, o);
    }
}

// The same with a block walking over many rows: dy, x and the residual of a row are read once and kept in
// registers, the gains too, the next row is requested before this row's block-wide sums, and the two sums share one
// barrier (two scratch rows used in turn).  d <= TH * V * NP.
// SUMS = 2: every thread also adds up dy and dy * xhat of its columns over the rows its block walks, and the block writes
// them to partial[blockIdx.x][0 / 1][c] - the first pass of the column sums that give the gradients of the LayerNorm
// bias and gain (colsum_final_kernel adds the blocks' rows up in a fixed order), from operands that are in registers anyway.
// SUMS = 4: the same for resid and dx, to more[blockIdx.x][0 / 1][c]: the gradients of the biases behind and in front of the layer's second
// LayerNorm, for which a pass over both cost 0.22 us per MB (450 MB, 100 us).
template <class T, int V, int TH, int NP, int SUMS>
__global__ __launch_bounds__(TH) void layernorm_bwd_dx_rows_kernel(const T *__restrict__ dy, const T *__restrict__ x,
                                                                   const float *__restrict__ mean,
                                                                   const float *__restrict__ rstd,
                                                                   const float *__restrict__ g, const T *resid, T *dx,
                                                                   int rows, int d, float *__restrict__ partial, float *__restrict__ more) {
    __shared__ float red[2][2][16];
    float gv[NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int c = (p * TH + threadIdx.x) * V;
        if (c < d) {
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                float t4[4];
                load_pack<float, 4>(g + c + 4 * q, t4);
#pragma unroll
                for (int i = 0; i < 4; ++i) gv[p][4 * q + i] = t4[i];
            }
        }
    }
    Pack<T, V> na[NP], nx[NP], nr[NP];
    float nmu = 0.f, nrs = 0.f;
    auto request = [&](size_t row) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
                na[p] = *reinterpret_cast<const Pack<T, V> *>(dy + row * (size_t)d + c);
                nx[p] = *reinterpret_cast<const Pack<T, V> *>(x + row * (size_t)d + c);
                nr[p] = *reinterpret_cast<const Pack<T, V> *>(resid + row * (size_t)d + c);
            }
        }
        nmu = mean[row];
        nrs = rstd[row];
    };
    float sums[SUMS ? SUMS : 1][NP][V];
#pragma unroll
    for (int k = 0; k < SUMS; ++k)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < V; ++i) sums[k][p][i] = 0.f;
    if (blockIdx.x < (unsigned)rows) request(blockIdx.x);
    int turn = 0;
    for (size_t row = blockIdx.x; row < (size_t)rows; row += gridDim.x, turn ^= 1) {
        float gd[NP][V], xh[NP][V], r[NP][V];
        const float rs = nrs, mu = nmu;
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float a = to_f32(na[p].v[i]);
                    gd[p][i] = a * gv[p][i];
                    xh[p][i] = (to_f32(nx[p].v[i]) - mu) * rs;
                    r[p][i] = to_f32(nr[p].v[i]);
                    s1 += gd[p][i];
                    s2 += gd[p][i] * xh[p][i];
                    if constexpr (SUMS > 0) {
                        sums[0][p][i] += a;
                        sums[1][p][i] += a * xh[p][i];
                    }
                    if constexpr (SUMS > 2) sums[2][p][i] += r[p][i];
                }
            }
        }
        if (row + gridDim.x < (size_t)rows) request(row + gridDim.x);
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if ((threadIdx.x & 63) == 0) {
            red[turn][0][threadIdx.x >> 6] = s1;
            red[turn][1][threadIdx.x >> 6] = s2;
        }
        __syncthreads();
        float t1 = 0.f, t2 = 0.f;
#pragma unroll
        for (int i = 0; i < TH / 64; ++i) {
            t1 += red[turn][0][i];
            t2 += red[turn][1][i];
        }
        t1 /= (float)d;
        t2 /= (float)d;
        T *dxr = dx + row * (size_t)d;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
                float o[V];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    o[i] = r[p][i] + rs * (gd[p][i] - t1 - xh[p][i] * t2);
                    if constexpr (SUMS > 2) sums[3][p][i] += to_f32(from_f32<T>(o[i]));        // (the values that are stored)
                }
                store_pack<T, V>(dxr + c, o);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < SUMS; ++k) {
        float *to = (k < 2 ? partial : more) + ((size_t)blockIdx.x * 2 + (k & 1)) * d;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * TH + threadIdx.x) * V;
            if (c < d) {
#pragma unroll
                for (int q = 0; q < V; q += 4)          // 16-byte pieces: partial and more are 16-byte aligned, c a multiple of 4
                    *reinterpret_cast<f32x4 *>(to + c + q) = f32x4{sums[k][p][q], sums[k][p][q + 1], sums[k][p][q + 2], sums[k][p][q + 3]};
            }
        }
    }
}

// The same with a row per wavefront (d <= 64 V NP), for the same reason; the four wavefronts' sums meet in LDS at the end.  With the second
// pass of the sums, 16-bit: 32768 x 768 48 us before, 39 now; 65536 x 256 68 and 30.  (Four packs a lane do not leave room for the sums.)
template <class T, int V, int NP, int SUMS>
__global__ __launch_bounds__(256) void layernorm_bwd_dx_wave_kernel(const T *__restrict__ dy, const T *__restrict__ x, const float *__restrict__ mean,
                                                                    const float *__restrict__ rstd, const float *__restrict__ g, const T *resid,
                                                                    T *dx, int rows, int d, float *__restrict__ partial, float *__restrict__ more) {
    __shared__ __attribute__((aligned(16))) float red[4][SUMS ? 64 * V * NP : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    RowWalk walk(blockIdx.x, gridDim.x, wave, rows);
    Pack<T, V> na[NP], nx[NP], nr[NP];
    float nmu = 0.f, nrs = 0.f;
    auto request = [&](int r) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * 64 + lane) * V;
            if (c < d) {
                na[p] = *reinterpret_cast<const Pack<T, V> *>(dy + (size_t)r * d + c);
                nx[p] = *reinterpret_cast<const Pack<T, V> *>(x + (size_t)r * d + c);
                nr[p] = *reinterpret_cast<const Pack<T, V> *>(resid + (size_t)r * d + c);
            }
        }
        nmu = mean[r];
        nrs = rstd[r];
    };
    if (walk.valid()) request(walk.row);
    float gv[NP][V], sums[SUMS ? SUMS : 1][NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int c = (p * 64 + lane) * V;
#pragma unroll
        for (int q = 0; q < V; q += 4) {
            f32x4 t4 = {0.f, 0.f, 0.f, 0.f};
            if (c < d) t4 = *reinterpret_cast<const f32x4 *>(g + c + q);
#pragma unroll
            for (int i = 0; i < 4; ++i) gv[p][q + i] = t4[i];
        }
#pragma unroll
        for (int k = 0; k < SUMS; ++k)
#pragma unroll
            for (int i = 0; i < V; ++i) sums[k][p][i] = 0.f;
    }
    for (; walk.valid(); walk.advance()) {
        const int row = walk.row;
        float gd[NP][V], xh[NP][V], r[NP][V], s1 = 0.f, s2 = 0.f;
        const float mu = nmu, rs = nrs;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if ((p * 64 + lane) * V < d) {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float a = to_f32(na[p].v[i]);
                    gd[p][i] = a * gv[p][i];
                    xh[p][i] = (to_f32(nx[p].v[i]) - mu) * rs;
                    r[p][i] = to_f32(nr[p].v[i]);
                    s1 += gd[p][i];
                    s2 += gd[p][i] * xh[p][i];
                    if constexpr (SUMS > 0) {
                        sums[0][p][i] += a;
                        sums[1][p][i] += a * xh[p][i];
                    }
                    if constexpr (SUMS > 2) sums[2][p][i] += r[p][i];
                }
            }
        }
        if (walk.has_next()) request(walk.next());
        const float t1 = wave_sum(s1) / (float)d, t2 = wave_sum(s2) / (float)d;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = (p * 64 + lane) * V;
            if (c < d) {
                float o[V];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    o[i] = r[p][i] + rs * (gd[p][i] - t1 - xh[p][i] * t2);
                    if constexpr (SUMS > 2) sums[3][p][i] += to_f32(from_f32<T>(o[i]));        // (the values that are stored)
                }
                store_pack<T, V>(dx + (size_t)row * d + c, o);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < SUMS; ++k) {
        if (k) __syncthreads();
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < V; i += 4)
                *reinterpret_cast<f32x4 *>(&red[wave][(p * 64 + lane) * V + i]) = f32x4{sums[k][p][i], sums[k][p][i + 1], sums[k][p][i + 2], sums[k][p][i + 3]};
        __syncthreads();
        float *to = (k < 2 ? partial : more) + ((size_t)blockIdx.x * 2 + (k & 1)) * d;
        for (int c = threadIdx.x; c < d; c += 256) to[c] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
    }
}

// ------------------------------------------------------------------------------------------
// Column sums, pass 1: block (32 column-threads x 8 row-threads) reduces kColsumRows rows of a
// strip of 32*V columns into partial[row_chunk][2][cols].
constexpr int kColsumRows = 128;

// The matrices of one launch of the first pass (a matrix per bias of a layer: four).  N = 1, here and below: a launch for one matrix
// takes its place in it from a two-dimensional grid and the fields of matrix 0 directly, from 48 bytes of arguments and not 200 to 300 (a
// call for one matrix, 4096 x 768 in 16 bits: sums 9.7 us with the others' arguments, 7.6 without; transposed 5.1 and 4.3).
template <class T> struct ColsumInput {
    const T *a, *x;
    const float *mean, *rstd;
    float *partial;
    int rows, cols, ld;
};
template <class T, int N> struct ColsumInputs {
    int first[N];                                          // see matrix_of; unused for N = 1
    ColsumInput<T> m[N];
};
// first: the workgroup that matrix i begins with, INT_MAX behind the last (side by side: one scalar load finds a workgroup's matrix, where a walk
// over the matrices waits for one after the other).  Filled for n matrices by what each takes; returns the workgroups of all.
template <int N, class Blocks> int first_workgroups(int (&first)[N], int n, Blocks blocks_of) {
    int all = 0;
    for (int i = 0; i < N; ++i) {
        first[i] = i < n ? all : INT_MAX;
        if (i < n) all += blocks_of(i);
    }
    return all;
}
template <int N> __device__ __forceinline__ int matrix_of(const int (&first)[N], int &block) {
    int n = 0;
#pragma unroll
    for (int i = 1; i < N; ++i) n += block >= first[i];
    block -= first[n];
    return n;
}

// Whether a thread requests its sixteen rows of a whole chunk before it adds the first (in a loop, some wait out the latency of those before).  Up to 32 MB, what the
// L2 caches hold, the latencies are what the pass takes: the four biases of a layer of width 64 over 256 tokens in fp32 6.6 -> 3.0 us, of width 256 over
// 2048 7.7 -> 4.8, 28620 x 512 in 16 bits 10.2 -> 7.3.  Beyond, so many loads at once are in each other's way: in fp32 22522 x 676 15.2 -> 18.6, 44272 x 304
// 13.5 -> 15.8, 6637 x 6624 28.1 -> 30.4, of 45 sums 2 % more on average; in 16 bits up to 72 MB 2033 x 10216 12.5 -> 14.5, 29951 x 840 14.4 -> 16.4, of 10
// 2 % more; but above that 2 % less on average of 22, 32768 x 768 + 2304 29 -> 24.
template <class T> bool colsum_loads_ahead(double elems) {
    const double mb = sizeof(T) * elems / 1048576.0;
    return mb <= 32.0 || (sizeof(T) == 2 && mb > 72.0);
}

template <class T, int V, bool WITH_XHAT, bool AHEAD, int N>
__global__ __launch_bounds__(256) void colsum_partial_kernel(ColsumInputs<T, N> in) {
    constexpr bool ONE = N == 1;
    __shared__ float red[2][8][32 * V + 1];
    // workgroup -> (matrix, 128-row chunk, 32 V columns), columns fastest
    int n = 0, block = blockIdx.x;
    if constexpr (!ONE) n = matrix_of(in.first, block);
    const T *__restrict__ a = in.m[n].a, *__restrict__ x = in.m[n].x;
    const float *__restrict__ mean = in.m[n].mean, *__restrict__ rstd = in.m[n].rstd;
    const int rows = in.m[n].rows, cols = in.m[n].cols, ld = in.m[n].ld;
    float *__restrict__ partial = in.m[n].partial;
    const int across = (cols + 32 * V - 1) / (32 * V), bx = ONE ? block : block % across, by = ONE ? blockIdx.y : block / across;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int c0 = (bx * 32 + tx) * V;
    const int r0 = by * kColsumRows;
    const int r1 = min(rows, r0 + kColsumRows);
    float s0[V], s1[V];
#pragma unroll
    for (int i = 0; i < V; ++i) s0[i] = s1[i] = 0.f;
    auto add = [&](int r, const float (&av)[V]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < V; ++i) s0[i] += av[i];
        if constexpr (WITH_XHAT) {
            float xv[V];
            load_pack<T, V>(x + (size_t)r * ld + c0, xv);
            const float mu = mean[r], rs = rstd[r];
#pragma unroll
            for (int i = 0; i < V; ++i) s1[i] += av[i] * (xv[i] - mu) * rs;
        }
    };
    if (c0 < cols) {
        if (AHEAD && r1 == r0 + kColsumRows) {
            float av[kColsumRows / 8][V];
#pragma unroll
            for (int k = 0; k < kColsumRows / 8; ++k) load_pack<T, V>(a + (size_t)(r0 + ty + 8 * k) * ld + c0, av[k]);
#pragma unroll
            for (int k = 0; k < kColsumRows / 8; ++k) add(r0 + ty + 8 * k, av[k]);
        } else {
            for (int r = r0 + ty; r < r1; r += 8) {
                float av[V];
                load_pack<T, V>(a + (size_t)r * ld + c0, av);
                add(r, av);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
        red[0][ty][tx * V + i] = s0[i];
        red[1][ty][tx * V + i] = s1[i];
    }
    __syncthreads();
    for (int j = threadIdx.x; j < 32 * V; j += 256) {
        const int c = bx * 32 * V + j;
        if (c >= cols) continue;
        float t0 = 0.f, t1 = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            t0 += red[0][k][j];
            t1 += red[1][k][j];
        }
        partial[((size_t)by * 2 + 0) * cols + c] = t0;
        if constexpr (WITH_XHAT) partial[((size_t)by * 2 + 1) * cols + c] = t1;
    }
}

// Pass 2, for up to kColsumBatch sums in one launch (the four biases and two LayerNorms of a layer).  Block = 32 columns x 32 V
// groups of row chunks, a thread V columns of them: group q adds chunks q, q + 32 V, ... in that order, combined through LDS in group
// order, so the result does not depend on scheduling.  With the partial rows of a kernel that writes one per block (up to 4096)
// a thread's chain of dependent loads and adds is what this pass takes, not its bytes: hence many groups, and eight rows in
// flight per thread.  The six sums of a d = 768 layer over 32768 tokens: 50 us in six launches, 30 in one with a column per thread,
// 21 with four.  A single sum of up to 128 chunks leaves little to split, and a column per thread is faster (16-bit sums with both
// passes, 8192 x 2048: 11.9 us with four, 11.0 with one).  V follows from the widths, lengths and number of sums alone, so their order does.
constexpr int kFinalCols = 32, kFinalThreads = 1024, kFewChunks = 128;

struct ColsumOne {
    ColsumJob job[1];
};
struct ColsumSeveral {
    int first[kColsumBatch];                               // see matrix_of
    ColsumJob job[kColsumBatch];
};

template <int V, class Batch> __global__ __launch_bounds__(kFinalThreads) void colsum_final_kernel(Batch batch) {
    constexpr bool ONE = std::is_same<Batch, ColsumOne>::value;
    constexpr int LANES = kFinalCols / V, GROUPS = kFinalThreads / LANES;
    __shared__ float red[2][GROUPS][kFinalCols + 1];
    int n = 0, block = blockIdx.x;
    if constexpr (!ONE) n = matrix_of(batch.first, block);
    const ColsumJob &job = batch.job[n];
    const int chunks = job.chunks, cols = job.cols;
    const bool two = job.out1 != nullptr;
    typedef float vec __attribute__((ext_vector_type(V)));
    typedef vec loose __attribute__((aligned(4)));         // a caller's scratch: the order of the sums must not depend on its alignment
    {
        const int tx = threadIdx.x % LANES, q = threadIdx.x / LANES;
        const int c = block * kFinalCols + tx * V;
        vec t0 = 0.f, t1 = 0.f;
        if (c < cols) {
            const float *row = job.partial + (size_t)q * 2 * cols + c;      // chunk q; the next of the group lies `step` further
            const size_t step = (size_t)GROUPS * 2 * cols;
            for (int k = q; k < chunks; k += 8 * GROUPS, row += 8 * step) {
                vec a[8], b[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool there = k + i * GROUPS < chunks;
                    a[i] = there ? *reinterpret_cast<const loose *>(row + i * step) : (vec)0.f;
                    b[i] = there && two ? *reinterpret_cast<const loose *>(row + i * step + cols) : (vec)0.f;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    t0 += a[i];
                    t1 += b[i];
                }
            }
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            red[0][q][tx * V + v] = t0[v];
            red[1][q][tx * V + v] = t1[v];
        }
    }
    __syncthreads();
    const int tx = threadIdx.x % kFinalCols, q = threadIdx.x / kFinalCols;
    if constexpr (V > 1) {                                                  // 32 V groups to 32
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            s0 += red[0][q * V + i][tx];
            s1 += red[1][q * V + i][tx];
        }
        __syncthreads();
        red[0][q][tx] = s0;
        red[1][q][tx] = s1;
        __syncthreads();
    }
    const int c = block * kFinalCols + tx;
    if (q < 2 && c < cols && (q == 0 || two)) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) t += red[q][i][tx];
        float *o = q == 0 ? job.out0 : job.out1;
        o[c] = (job.beta == 0.f ? 0.f : job.beta * o[c]) + t;
    }
}

// ------------------------------------------------------------------------------------------
// Adam: streams w, m, v, g once (16 B/param in, 12 B + 2 B out).
struct AdamConsts {
    float beta1, beta2, omb1, omb2, inv_bc1, inv_bc2, lr, eps;
    float grad_mul;        // the gradient is multiplied by this first (1 / loss scale; 1 = no scaling, exact)
};

__device__ __forceinline__ void adam_one(float &w, float &m, float &v, float g, const AdamConsts &c) {
    m = c.beta1 * m + c.omb1 * g;
    v = c.beta2 * v + c.omb2 * g * g;
    const float mh = m * c.inv_bc1;
    const float vh = v * c.inv_bc2;
    w = w - c.lr * mh / (sqrtf(vh) + c.eps);
}

template <class E>
__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ w, float *__restrict__ m,
                                                   float *__restrict__ v, const float *__restrict__ g,
                                                   E *__restrict__ w16, size_t n, size_t n4, AdamConsts c,
                                                   const int *__restrict__ skip) {
    if (skip && *skip) return;          // the gradient held a non-finite value: this update is left out as a whole
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        f32x4 wv = reinterpret_cast<f32x4 *>(w)[i];
        f32x4 mv = reinterpret_cast<f32x4 *>(m)[i];
        f32x4 vv = reinterpret_cast<f32x4 *>(v)[i];
        const f32x4 gv = reinterpret_cast<const f32x4 *>(g)[i];
        float wa[4] = {wv[0], wv[1], wv[2], wv[3]}, ma[4] = {mv[0], mv[1], mv[2], mv[3]};
        float va[4] = {vv[0], vv[1], vv[2], vv[3]};
#pragma unroll
        for (int k = 0; k < 4; ++k) adam_one(wa[k], ma[k], va[k], gv[k] * c.grad_mul, c);
        wv = {wa[0], wa[1], wa[2], wa[3]};
        mv = {ma[0], ma[1], ma[2], ma[3]};
        vv = {va[0], va[1], va[2], va[3]};
        reinterpret_cast<f32x4 *>(w)[i] = wv;
        reinterpret_cast<f32x4 *>(m)[i] = mv;
        reinterpret_cast<f32x4 *>(v)[i] = vv;
        if (w16) {
            x4<E> o;
            o[0] = (E)wa[0]; o[1] = (E)wa[1]; o[2] = (E)wa[2]; o[3] = (E)wa[3];
            reinterpret_cast<x4<E> *>(w16)[i] = o;
        }
    }
    for (size_t i = n4 * 4 + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        float wa = w[i], ma = m[i], va = v[i];
        adam_one(wa, ma, va, g[i] * c.grad_mul, c);
        w[i] = wa; m[i] = ma; v[i] = va;
        if (w16) w16[i] = (E)wa;
    }
}

// The same for a whole layer with both of its 16-bit copies, as stored and each matrix transposed: what one kernel wrote a second read back from memory
// to transpose it (d = 12288: 11.2 + 1.4 ms, now 11.5; d = 2048: 284 + 51 us, now 289; a d = 128 layer's two launches 3.3 + 4.9, now 5.5).  A workgroup has
// a tile of 64 x 64 or 128 x 128 of a matrix, a thread a block of 4 x 4 at a time, with its sixteen loads of 16 bytes in flight; the
// transposed tile leaves through LDS in rows of 128 or 256 bytes.  What lies between the matrices goes by 1024 elements.  For rows of whole
// 128-byte lines in 16 bits: others are written in parts from several workgroups, d = 4256 1617 us where the two kernels take 1339 + 189.  And not for
// layers of some million parameters, whose copies the transposing pass leaves in the caches for the products that come next: d = 768 40 us
// against 36 + 8, but then the input gradients 29.4 us against 27.9.  Of whole steps (us, two kernels / this one): below 2^20 parameters always 1 to 3 % less (1, 2 and
// 4 layers of 64 to 256, 4 of 192 435 / 423); from 2^20 to 2^24 3 % less to 1 % more, left to two kernels (4 layers of 768 over 4096 tokens 2115 / 2098, 2 of 896 in
// micro-batch order over 16384 5187 / 5237); above 8 % less to 1 % more for several layers (6 of 1280 4348 / 4320, 2 of 4096 over 512 5534 / 5222, 2 of
// 1216 832 / 837).  A layer alone, whose copies the very next pass reads, gains from 2^25 on only (512 tokens: 1216 395 / 411, 1536 553 / 580, 1664
// 608 / 611, 1728 663 / 658, 2048 862 / 845; d_ff = d = 3072 931 / 944, over 128 727 / 701).
constexpr size_t kAdamSmall = (size_t)1 << 20, kAdamLarge = (size_t)1 << 24, kAdamLargeAlone = (size_t)1 << 25;
struct AdamRegion {
    size_t at;             // element in the layer's vector
    int rows, cols;        // a matrix [rows][cols]; rows = 0: cols elements of no matrix
};
constexpr int kAdamRegions = 9;
template <class E> struct AdamLayer {
    int first[kAdamRegions];                               // see matrix_of
    AdamRegion region[kAdamRegions];
    float *w, *m, *v;
    const float *g;
    E *w16, *w16t;
};

template <int TILE, class E> __global__ __launch_bounds__(256) void adam_copies_kernel(AdamLayer<E> a, AdamConsts c, const int *__restrict__ skip) {
    if (skip && *skip) return;          // (the copies then stay those of the weights)
    int block = blockIdx.x;
    const AdamRegion t = a.region[matrix_of(a.first, block)];
    auto update = [&](const f32x4 &w, const f32x4 &m, const f32x4 &v, const f32x4 &g, size_t at) __attribute__((always_inline)) {
        float wa[4] = {w[0], w[1], w[2], w[3]}, ma[4] = {m[0], m[1], m[2], m[3]}, va[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
        for (int k = 0; k < 4; ++k) adam_one(wa[k], ma[k], va[k], g[k] * c.grad_mul, c);
        *reinterpret_cast<f32x4 *>(a.w + at) = f32x4{wa[0], wa[1], wa[2], wa[3]};
        *reinterpret_cast<f32x4 *>(a.m + at) = f32x4{ma[0], ma[1], ma[2], ma[3]};
        *reinterpret_cast<f32x4 *>(a.v + at) = f32x4{va[0], va[1], va[2], va[3]};
        x4<E> o;
        o[0] = (E)wa[0]; o[1] = (E)wa[1]; o[2] = (E)wa[2]; o[3] = (E)wa[3];
        *reinterpret_cast<x4<E> *>(a.w16 + at) = o;
        return o;
    };
    if (t.rows == 0) {
        const int i = (block * 256 + threadIdx.x) * 4;
        if (i >= t.cols) return;
        const size_t at = t.at + i;
        update(*reinterpret_cast<const f32x4 *>(a.w + at), *reinterpret_cast<const f32x4 *>(a.m + at), *reinterpret_cast<const f32x4 *>(a.v + at),
               *reinterpret_cast<const f32x4 *>(a.g + at), at);
        return;
    }
    constexpr int P = TILE + 8;                            // pitch: whole 16-byte pieces
    __shared__ __attribute__((aligned(16))) E tile[TILE * P];           // [column][row]
    const int across = (t.cols + TILE - 1) / TILE, r0 = block / across * TILE, c0 = block % across * TILE;
    const int tx = threadIdx.x % (TILE / 4), ty = threadIdx.x / (TILE / 4), col = c0 + 4 * tx;
    constexpr int STEP = 4 * 256 / (TILE / 4);             // rows that the threads cover together
#pragma unroll 1
    for (int r = 4 * ty; r < TILE; r += STEP) {
        if (r0 + r >= t.rows || col >= t.cols) continue;   // (multiples of 8, both)
        const size_t at = t.at + (size_t)(r0 + r) * t.cols + col;
        f32x4 w[4], m[4], v[4], g[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            w[k] = *reinterpret_cast<const f32x4 *>(a.w + at + (size_t)k * t.cols);
            m[k] = *reinterpret_cast<const f32x4 *>(a.m + at + (size_t)k * t.cols);
            v[k] = *reinterpret_cast<const f32x4 *>(a.v + at + (size_t)k * t.cols);
            g[k] = *reinterpret_cast<const f32x4 *>(a.g + at + (size_t)k * t.cols);
        }
        x4<E> o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = update(w[k], m[k], v[k], g[k], at + (size_t)k * t.cols);
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<x4<E> *>(tile + (4 * tx + i) * P + r) = x4<E>{o[0][i], o[1][i], o[2][i], o[3][i]};
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TILE * TILE / 8 / 256; ++k) {
        const int piece = k * 256 + threadIdx.x, cc = piece / (TILE / 8), rr = piece % (TILE / 8) * 8;
        if (c0 + cc < t.cols && r0 + rr < t.rows)
            *reinterpret_cast<x8<E> *>(a.w16t + t.at + (size_t)(c0 + cc) * t.rows + r0 + rr) = *reinterpret_cast<const x8<E> *>(tile + cc * P + rr);
    }
}

// ------------------------------------------------------------------------------------------
// out[c][r] = in[r][c] for 16-bit elements.  A block moves a 128 x 128 tile: each thread loads one
// 8x8 block (16-byte row pieces, lanes along the contiguous direction), transposes it in registers,
// parks it in LDS, and the block then writes whole 256-byte row segments of the output.
constexpr int kTrTile = 128;
constexpr int kTrPitch = kTrTile + 8;     // elements; keeps 16-byte alignment and skews the banks

// One launch moves up to kTransposeBatch matrices (the operands of a layer's weight gradients; its four weight matrices): launched one by
// one, a narrow layer's each take their 4 us.  With partial given the block also adds up its 128 rows of every column it moves
// (as values of format E, in fp32) and writes them to partial[row chunk][0][c] - the first pass of the column sums
// (colsum_partial_kernel's layout, same 128-row chunks), so that the bias gradient costs no pass of its own over a matrix that is being transposed anyway.
struct TransposeSeveral {
    int first[kTransposeBatch];                            // see matrix_of
    TransposeMatrix m[kTransposeBatch];
};
struct TransposeOne {
    TransposeMatrix m[1];
};
template <class E, class Batch> __global__ __launch_bounds__(256) void transpose16_kernel(Batch batch) {
    constexpr bool ONE = std::is_same<Batch, TransposeOne>::value;
    static_assert(kTrTile == kColsumRows, "one transposed tile = one chunk of rows of the column sums");
    __shared__ __attribute__((aligned(16))) uint16_t tile[kTrTile * kTrPitch];     // [c][r]
    int n = 0, block = blockIdx.x;
    if constexpr (!ONE) n = matrix_of(batch.first, block);
    const uint16_t *__restrict__ in = static_cast<const uint16_t *>(batch.m[n].in);
    uint16_t *__restrict__ out = static_cast<uint16_t *>(batch.m[n].out);
    const int R = batch.m[n].R, C = batch.m[n].C;
    const long ldi = batch.m[n].ldi, ldo = batch.m[n].ldo;
    float *__restrict__ partial = batch.m[n].partial;
    const int across = (C + kTrTile - 1) / kTrTile, by = ONE ? blockIdx.y : block / across;
    const int r0 = by * kTrTile, c0 = (ONE ? block : block % across) * kTrTile;
    const int tid = threadIdx.x;
    {
        const int cb = tid & 15, rb = tid >> 4;           // 16 x 16 blocks of 8 x 8
        u32x4 v[8], t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int r = r0 + rb * 8 + j, c = c0 + cb * 8;
            v[j] = u32x4{0, 0, 0, 0};
            if (r < R && c < C) v[j] = *reinterpret_cast<const u32x4 *>(in + (size_t)r * ldi + c);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t x = v[2 * p][q], y = v[2 * p + 1][q];
                t[2 * q][p] = (x & 0xFFFFu) | (y << 16);
                t[2 * q + 1][p] = (x >> 16) | (y & 0xFFFF0000u);
            }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *reinterpret_cast<u32x4 *>(tile + (cb * 8 + i) * kTrPitch + rb * 8) = t[i];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int c = (tid >> 4) + 16 * j, rch = tid & 15;
        const int gc = c0 + c, gr = r0 + rch * 8;
        const u32x4 piece = *reinterpret_cast<const u32x4 *>(tile + c * kTrPitch + rch * 8);
        if (gc < C && gr < R) *reinterpret_cast<u32x4 *>(out + (size_t)gc * ldo + gr) = piece;
        if (partial) {
            // rows beyond R were staged as zeros; the 16 lanes that hold column c's 128 rows are neighbours
            float sum = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t w = piece[q];
                const uint16_t lo = (uint16_t)(w & 0xFFFFu), hi = (uint16_t)(w >> 16);
                sum += to_f32(__builtin_bit_cast(E, lo)) + to_f32(__builtin_bit_cast(E, hi));
            }
            sum = row_of_16_sum(sum);
            if (rch == 0 && gc < C) partial[((size_t)by * 2 + 0) * C + gc] = sum;
        }
    }
}

inline int grid_for(size_t work_items, int block, int max_blocks = 256 * 16) {
    size_t b = (work_items + block - 1) / block;
    if (b < 1) b = 1;
    if (b > (size_t)max_blocks) b = max_blocks;
    return (int)b;
}

}  // namespace

// ==========================================================================================
template <class E> void launch_cast_f32_to_16(const float *src, E *dst, size_t n, hipStream_t s) {
    if (n == 0) return;
    const size_t n4 = (aligned16(src) && (reinterpret_cast<uintptr_t>(dst) & 7u) == 0) ? n / 4 : 0;   // vector part
    ProfScope scope("cast_kernel", 0.0, 6.0 * n, s);
    hipLaunchKernelGGL(cast_kernel<E>, dim3(grid_for(n / 4 + 1, 256)), dim3(256), 0, s, src, dst, n, n4);
}
template void launch_cast_f32_to_16<bf16>(const float *, bf16 *, size_t, hipStream_t);
template void launch_cast_f32_to_16<f16>(const float *, f16 *, size_t, hipStream_t);

void launch_nonfinite_flag(const float *g, size_t n, int *flag, hipStream_t s) {
    if (n == 0) return;
    ProfScope scope("nonfinite_flag_kernel", 0.0, 4.0 * n, s);
    const size_t n4 = aligned16(g) ? n / 4 : 0;
    hipLaunchKernelGGL(nonfinite_flag_kernel, dim3(grid_for(n / 4 + 1, 256, 256 * 8)), dim3(256), 0, s, g, n, n4, flag);
}

void launch_fill_normal(float *dst, size_t n, float std, uint64_t seed, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(fill_normal_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, dst, n, std, seed);
}

void launch_fill_const(float *dst, size_t n, float value, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(fill_const_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, dst, n, value);
}

template <class T>
void launch_layernorm_fwd(const T *x, const float *g, const float *b, T *y, float *mean, float *rstd, int rows,
                          int d, float eps, hipStream_t s, T *keep) {
    if (rows == 0) return;
    constexpr int V = VecOf<T>::N;
    const bool registers = d % V == 0 && aligned16(x) && aligned16(y) && aligned16(g) && aligned16(b) && aligned16(keep) && d <= 1024 * V * 2;
    if (keep && !registers) (void)hipMemcpyAsync(keep, x, (size_t)rows * d * sizeof(T), hipMemcpyDeviceToDevice, s);
    ProfScope scope("layernorm_fwd_kernel", 8.0 * rows * d, (keep && registers ? 3.0 : 2.0) * sizeof(T) * rows * (double)d, s);
    // (rows wider than two packs per thread of a 1024-thread block would leave one block per CU: the one-row-per-block
    // kernel, with its many small blocks, is faster there)
    if (registers) {
        // rows are dealt to a fixed number of blocks (enough to fill every CU), which keep what they reuse in registers
#define LGA_LN_ROWS(TH, NP) \
        hipLaunchKernelGGL((layernorm_fwd_rows_kernel<T, V, TH, NP, true>), dim3((unsigned)std::min(rows, 256 * (2048 / TH))), \
                           dim3(TH), 0, s, x, g, b, y, mean, rstd, rows, d, eps, keep)
#define LGA_LN_WAVE(NP) \
        hipLaunchKernelGGL((layernorm_fwd_wave_kernel<T, V, NP>), dim3((unsigned)row_walk_blocks(rows, 256 * 8)), dim3(256), 0, s, x, g, b, y, \
                           mean, rstd, rows, d, eps, keep)
        const bool wave = d <= kLnWave * 64 * V && row_walk_takes(rows);
        if (wave && d <= 64 * V) LGA_LN_WAVE(1);
        else if (wave && d <= 128 * V) LGA_LN_WAVE(2);
        else if (wave) LGA_LN_WAVE(4);
        else if (d <= 512 * V) LGA_LN_ROWS(512, 1);              // (and narrower rows, more of them than the wavefronts' walk takes)
        else if (d <= 1024 * V) LGA_LN_ROWS(1024, 1);
        else LGA_LN_ROWS(1024, 2);
#undef LGA_LN_ROWS
#undef LGA_LN_WAVE
    } else if (d % V == 0 && aligned16(x) && aligned16(y))
        hipLaunchKernelGGL((layernorm_fwd_kernel<T, V>), dim3(rows), dim3(256), 0, s, x, g, b, y, mean, rstd, d, eps);
    else
        hipLaunchKernelGGL((layernorm_fwd_kernel<T, 1>), dim3(rows), dim3(256), 0, s, x, g, b, y, mean, rstd, d, eps);
}
template void launch_layernorm_fwd<float>(const float *, const float *, const float *, float *, float *, float *, int,
                                          int, float, hipStream_t, float *);
template void launch_layernorm_fwd<bf16>(const bf16 *, const float *, const float *, bf16 *, float *, float *, int,
                                         int, float, hipStream_t, bf16 *);
template void launch_layernorm_fwd<f16>(const f16 *, const float *, const float *, f16 *, float *, float *, int,
                                         int, float, hipStream_t, f16 *);

// whether a row per wavefront
static bool lnb_wave(int rows, int d, int V) { return d <= kLnbWave * 64 * V && row_walk_takes(rows); }
// blocks of the row-walking kernel for `rows` rows of length d (0: that kernel does not serve d)
static int lnb_rows_blocks(int rows, int d, int V) {
    if (d > 1024 * V * 2) return 0;
    if (lnb_wave(rows, d, V)) return row_walk_blocks(rows, 256 * 4);
    const int th = d <= 256 * V ? 256 : d <= 512 * V ? 512 : 1024;
    return std::min(rows, 256 * (2048 / th));
}

size_t layernorm_bwd_partial_floats(int rows, int d) {
    // fused sums: one pair of partial rows per block (only widths one pass of the block covers); else the column sums' own
    const size_t fused = (size_t)std::max(lnb_rows_blocks(rows, d, 4), lnb_rows_blocks(rows, d, 8)) * 2 * (size_t)d;
    return std::max(fused, colsum_partial_floats(rows, d));
}

void launch_colsum_batch(const ColsumBatch &batch, hipStream_t s, bool timed) {
    if (batch.n == 0) return;
    double bytes = 0.0;
    for (int i = 0; i < batch.n; ++i) bytes += (batch.job[i].out1 ? 8.0 : 4.0) * batch.job[i].chunks * batch.job[i].cols;
    ProfScope scope("colsum_final_kernel", 0.25 * bytes, bytes, s, timed);
    bool vec = true;
    for (int i = 0; i < batch.n; ++i) vec &= batch.job[i].cols % 4 == 0;
    int longest = 0;
    for (int i = 0; i < batch.n; ++i) longest = std::max(longest, batch.job[i].chunks);
    vec = vec && (batch.n > 1 || longest > kFewChunks);
    ColsumSeveral all{};
    const dim3 grid((unsigned)first_workgroups(all.first, batch.n, [&](int i) { return (batch.job[i].cols + kFinalCols - 1) / kFinalCols; }));
    const dim3 block(kFinalThreads);
    if (batch.n == 1) {
        const ColsumOne one{{batch.job[0]}};
        if (vec) hipLaunchKernelGGL((colsum_final_kernel<4, ColsumOne>), grid, block, 0, s, one);
        else hipLaunchKernelGGL((colsum_final_kernel<1, ColsumOne>), grid, block, 0, s, one);
    } else {
        std::copy(batch.job, batch.job + batch.n, all.job);
        if (vec) hipLaunchKernelGGL((colsum_final_kernel<4, ColsumSeveral>), grid, block, 0, s, all);
        else hipLaunchKernelGGL((colsum_final_kernel<1, ColsumSeveral>), grid, block, 0, s, all);
    }
}

// The second pass of one sum: with the caller's others, or at once.
static void finish_colsum(ColsumBatch *batch, const float *partial, int chunks, int cols, float beta, float *out0, float *out1, hipStream_t s,
                          bool timed = true) {
    const ColsumJob job{partial, out0, out1, chunks, cols, beta};
    if (batch) {
        batch->job[batch->n++] = job;
        return;
    }
    ColsumBatch one;
    one.job[0] = job;
    one.n = 1;
    launch_colsum_batch(one, s, timed);
}

template <class T>
void launch_layernorm_bwd_dx(const T *dy, const T *x, const float *mean, const float *rstd, const float *g,
                             const T *resid, T *dx, int rows, int d, hipStream_t s, float beta, float *dbeta,
                             float *dgamma, float *partial, ColsumBatch *batch, const BiasSums *biases) {
    constexpr int V = VecOf<T>::N;
    const bool sums = dbeta != nullptr;
    const bool vec = d % V == 0 && aligned16(dy) && aligned16(x) && aligned16(resid) && aligned16(dx);
    const bool rows_kernel = vec && aligned16(g) && d <= 1024 * V * 2;
    // the sums ride along where a thread holds one piece of a row (d <= 1024 V): with two, their 4 V extra registers
    // per thread do not fit beside the row
    const bool fused = sums && rows_kernel && d <= 1024 * V && rows > 0 && aligned16(partial);
    if (sums && !fused) launch_colsum<T>(dy, x, mean, rstd, rows, d, d, beta, dbeta, dgamma, partial, s, true, batch);
    const bool all = fused && biases && aligned16(biases->partial);
    if (biases && !all) launch_colsum<T>(resid, nullptr, nullptr, nullptr, rows, d, d, beta, biases->of_resid, nullptr, biases->partial, s, true, nullptr);
    if (rows == 0) {
        if (biases) launch_colsum<T>(dx, nullptr, nullptr, nullptr, rows, d, d, beta, biases->of_dx, nullptr, biases->partial, s, true, nullptr);
        return;
    }
    {
        ProfScope scope(fused ? "layernorm_bwd_dx_kernel(with sums)" : "layernorm_bwd_dx_kernel", (all ? 20.0 : fused ? 18.0 : 14.0) * rows * d,
                        4.0 * sizeof(T) * rows * (double)d, s);
        const int blocks = lnb_rows_blocks(rows, d, V);
        if (rows_kernel) {
#define LGA_LNB_ROWS(TH, NP, SUMS) \
            hipLaunchKernelGGL((layernorm_bwd_dx_rows_kernel<T, V, TH, NP, SUMS>), dim3((unsigned)blocks), dim3(TH), 0, s, dy, x, \
                               mean, rstd, g, resid, dx, rows, d, partial, all ? biases->partial : nullptr)
#define LGA_LNB_WAVE(NP, SUMS) \
            hipLaunchKernelGGL((layernorm_bwd_dx_wave_kernel<T, V, NP, SUMS>), dim3((unsigned)blocks), dim3(256), 0, s, dy, x, mean, rstd, g, \
                               resid, dx, rows, d, partial, all ? biases->partial : nullptr)
#define LGA_LNB_SUMS(LAUNCH, ...) \
            do { if (all) LAUNCH(__VA_ARGS__, 4); else if (fused) LAUNCH(__VA_ARGS__, 2); else LAUNCH(__VA_ARGS__, 0); } while (0)
            const bool wave = lnb_wave(rows, d, V);
            if (wave && d <= 64 * V) LGA_LNB_SUMS(LGA_LNB_WAVE, 1);
            else if (wave) LGA_LNB_SUMS(LGA_LNB_WAVE, 2);
            else if (d <= 256 * V) LGA_LNB_SUMS(LGA_LNB_ROWS, 256, 1);
            else if (d <= 512 * V) LGA_LNB_SUMS(LGA_LNB_ROWS, 512, 1);
            else if (d <= 1024 * V) LGA_LNB_SUMS(LGA_LNB_ROWS, 1024, 1);
            else LGA_LNB_ROWS(1024, 2, 0);
#undef LGA_LNB_SUMS
#undef LGA_LNB_ROWS
#undef LGA_LNB_WAVE
        } else if (vec)
            hipLaunchKernelGGL((layernorm_bwd_dx_kernel<T, V>), dim3(rows), dim3(256), 0, s, dy, x, mean, rstd, g, resid,
                               dx, d);
        else
            hipLaunchKernelGGL((layernorm_bwd_dx_kernel<T, 1>), dim3(rows), dim3(256), 0, s, dy, x, mean, rstd, g, resid,
                               dx, d);
    }
    if (fused) finish_colsum(batch, partial, lnb_rows_blocks(rows, d, V), d, beta, dbeta, dgamma, s);
    if (all) finish_colsum(batch, biases->partial, lnb_rows_blocks(rows, d, V), d, beta, biases->of_resid, biases->of_dx, s);
    else if (biases) launch_colsum<T>(dx, nullptr, nullptr, nullptr, rows, d, d, beta, biases->of_dx, nullptr, biases->partial, s, true, nullptr);
}
bool layernorm_bwd_adds_biases(int d, int esz) { return d % (16 / esz) == 0 && d <= 1024 * (16 / esz); }
template void launch_layernorm_bwd_dx<float>(const float *, const float *, const float *, const float *,
                                             const float *, const float *, float *, int, int, hipStream_t, float,
                                             float *, float *, float *, ColsumBatch *, const BiasSums *);
template void launch_layernorm_bwd_dx<bf16>(const bf16 *, const bf16 *, const float *, const float *, const float *,
                                            const bf16 *, bf16 *, int, int, hipStream_t, float, float *, float *, float *, ColsumBatch *, const BiasSums *);
template void launch_layernorm_bwd_dx<f16>(const f16 *, const f16 *, const float *, const float *, const float *,
                                            const f16 *, f16 *, int, int, hipStream_t, float, float *, float *, float *, ColsumBatch *, const BiasSums *);

size_t colsum_partial_floats(int rows, int cols) {
    const size_t chunks = ((size_t)rows + kColsumRows - 1) / kColsumRows;
    return (chunks > 0 ? chunks : 1) * 2 * (size_t)cols;
}

template <class T>
void launch_colsum(const T *a, const T *x, const float *mean, const float *rstd, int rows, int cols, int ld,
                   float beta, float *out0, float *out1, float *partial, hipStream_t s, bool timed, ColsumBatch *batch) {
    if (cols == 0) return;
    const ColsumMatrix<T> m{a, x, mean, rstd, out0, out1, partial, rows, cols, ld};
    launch_colsums<T>(&m, 1, beta, s, timed, batch);
}

template <class T> void launch_colsums(const ColsumMatrix<T> *m, int n, float beta, hipStream_t s, bool timed, ColsumBatch *batch) {
    constexpr int VMAX = VecOf<T>::N;
    ColsumInputs<T, 4> in{};
    bool vec = true, xhat = false;
    double elems = 0.0;
    for (int i = 0; i < n; ++i) {
        vec &= m[i].cols % VMAX == 0 && m[i].ld % VMAX == 0 && aligned16(m[i].a) && (m[i].x == nullptr || aligned16(m[i].x));
        xhat |= m[i].out1 != nullptr;
        elems += (double)m[i].rows * m[i].cols;
    }
    int taken = 0;
    for (int i = 0; i < n; ++i)
        if (m[i].rows > 0 && m[i].cols > 0) in.m[taken++] = {m[i].a, m[i].x, m[i].mean, m[i].rstd, m[i].partial, m[i].rows, m[i].cols, m[i].ld};
    const int width = 32 * (vec ? VMAX : 1);
    const int blocks = first_workgroups(in.first, taken, [&](int i) {
        return (in.m[i].rows + kColsumRows - 1) / kColsumRows * ((in.m[i].cols + width - 1) / width);
    });
    if (blocks > 0) {
        ProfScope scope(xhat ? "colsum_partial_kernel(with xhat)" : "colsum_partial_kernel", (xhat ? 4.0 : 1.0) * elems,
                        (xhat ? 2.0 : 1.0) * sizeof(T) * elems, s, timed);
        const int across = (in.m[0].cols + width - 1) / width;
        auto launch = [&](auto v_c, auto xhat_c, auto ahead_c) {
            constexpr int V = decltype(v_c)::value;
            constexpr bool XHAT = decltype(xhat_c)::value, AHEAD = decltype(ahead_c)::value;
            if (taken == 1 && blocks / across <= 65535) {
                const ColsumInputs<T, 1> one{{0}, {in.m[0]}};
                hipLaunchKernelGGL((colsum_partial_kernel<T, V, XHAT, AHEAD, 1>), dim3(across, blocks / across), dim3(256), 0, s, one);
            } else {
                hipLaunchKernelGGL((colsum_partial_kernel<T, V, XHAT, AHEAD, 4>), dim3((unsigned)blocks), dim3(256), 0, s, in);
            }
        };
        typedef std::integral_constant<int, VMAX> Wide;
        typedef std::integral_constant<int, 1> Narrow;
        const bool ahead = colsum_loads_ahead<T>(elems);
        if (vec && xhat) launch(Wide{}, std::true_type{}, std::false_type{});
        else if (vec && ahead) launch(Wide{}, std::false_type{}, std::true_type{});
        else if (vec) launch(Wide{}, std::false_type{}, std::false_type{});
        else if (xhat) launch(Narrow{}, std::true_type{}, std::false_type{});
        else if (ahead) launch(Narrow{}, std::false_type{}, std::true_type{});
        else launch(Narrow{}, std::false_type{}, std::false_type{});
    }
    for (int i = 0; i < n; ++i)
        finish_colsum(batch, m[i].partial, m[i].rows > 0 ? (m[i].rows + kColsumRows - 1) / kColsumRows : 0, m[i].cols, beta, m[i].out0, m[i].out1, s, timed);
}
#define LGA_COLSUM(T)                                                                                                               \
    template void launch_colsum<T>(const T *, const T *, const float *, const float *, int, int, int, float, float *, float *, \
                                   float *, hipStream_t, bool, ColsumBatch *);                                                   \
    template void launch_colsums<T>(const ColsumMatrix<T> *, int, float, hipStream_t, bool, ColsumBatch *)
LGA_COLSUM(float);
LGA_COLSUM(bf16);
LGA_COLSUM(f16);
#undef LGA_COLSUM

template <class E> void launch_transposes(const TransposeMatrix *m, int n, hipStream_t s) {
    TransposeSeveral all{};
    int taken = 0;
    double elems = 0.0;
    bool sums = false;
    for (int i = 0; i < n; ++i) {
        if (m[i].R == 0 || m[i].C == 0) continue;
        all.m[taken++] = m[i];
        elems += (double)m[i].R * m[i].C;
        sums |= m[i].partial != nullptr;
    }
    const int blocks = first_workgroups(all.first, taken, [&](int i) { return ((all.m[i].C + kTrTile - 1) / kTrTile) * ((all.m[i].R + kTrTile - 1) / kTrTile); });
    if (blocks == 0) return;
    ProfScope scope(sums ? "transpose16_kernel(with column sums)" : "transpose16_kernel", sums ? elems : 0.0, 4.0 * elems, s);
    const int across = (all.m[0].C + kTrTile - 1) / kTrTile;
    if (taken == 1 && blocks / across <= 65535) {
        const TransposeOne one{{all.m[0]}};
        hipLaunchKernelGGL((transpose16_kernel<E, TransposeOne>), dim3(across, blocks / across), dim3(256), 0, s, one);
    } else {
        hipLaunchKernelGGL((transpose16_kernel<E, TransposeSeveral>), dim3((unsigned)blocks), dim3(256), 0, s, all);
    }
}
template void launch_transposes<bf16>(const TransposeMatrix *, int, hipStream_t);
template void launch_transposes<f16>(const TransposeMatrix *, int, hipStream_t);

void launch_transpose16(const void *in, void *out, int R, int C, long ldi, long ldo, hipStream_t s) {
    const TransposeMatrix m{in, out, nullptr, ldi, ldo, R, C};
    launch_transposes<bf16>(&m, 1, s);
}

template <class E>
void launch_transpose16_colsum(const E *in, E *out, int R, int C, long ldi, long ldo, float beta, float *out0,
                               float *partial, hipStream_t s) {
    if (C == 0) return;
    const TransposeMatrix m{in, out, partial, ldi, ldo, R, C};
    launch_transposes<E>(&m, 1, s);
    finish_colsum(nullptr, partial, (R + kTrTile - 1) / kTrTile, C, beta, out0, nullptr, s);
}
template void launch_transpose16_colsum<bf16>(const bf16 *, bf16 *, int, int, long, long, float, float *, float *, hipStream_t);
template void launch_transpose16_colsum<f16>(const f16 *, f16 *, int, int, long, long, float, float *, float *, hipStream_t);

void add_colsum(ColsumBatch &batch, const float *partial, int rows, int cols, float beta, float *out0) {
    static_assert(kTrTile == kColsumRows && kGemmSumRows == kColsumRows, "chunks of 128 rows, whichever kernel leaves them");
    finish_colsum(&batch, partial, (rows + kColsumRows - 1) / kColsumRows, cols, beta, out0, nullptr, nullptr);
}

static AdamConsts adam_consts(float lr, float beta1, float beta2, float eps, int step, float grad_mul) {
    AdamConsts c;
    c.beta1 = beta1;
    c.beta2 = beta2;
    c.omb1 = (float)(1.0 - (double)beta1);
    c.omb2 = (float)(1.0 - (double)beta2);
    c.inv_bc1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
    c.inv_bc2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
    c.lr = lr;
    c.eps = eps;
    c.grad_mul = grad_mul;
    return c;
}
template <class E>
void launch_adam(float *w, float *m, float *v, const float *g, E *w16, size_t n, float lr, float beta1, float beta2,
                 float eps, int step, float grad_mul, const int *skip, hipStream_t s) {
    if (n == 0) return;
    const AdamConsts c = adam_consts(lr, beta1, beta2, eps, step, grad_mul);
    ProfScope scope("adam_kernel", 12.0 * n, (w16 ? 30.0 : 28.0) * n, s);
    const bool vec = aligned16(w) && aligned16(m) && aligned16(v) && aligned16(g) &&
                     (reinterpret_cast<uintptr_t>(w16) & 7u) == 0;
    const size_t n4 = vec ? n / 4 : 0;
    hipLaunchKernelGGL(adam_kernel<E>, dim3(grid_for(n / 4 + 1, 256, 256 * 8)), dim3(256), 0, s, w, m, v, g, w16, n, n4,
                       c, skip);
}
template void launch_adam<bf16>(float *, float *, float *, const float *, bf16 *, size_t, float, float, float, float,
                                int, float, const int *, hipStream_t);
template void launch_adam<f16>(float *, float *, float *, const float *, f16 *, size_t, float, float, float, float, int,
                               float, const int *, hipStream_t);


bool adam_writes_copies(int d, int f, size_t n, int layers) {
    return d % 64 == 0 && f % 64 == 0 && (n < kAdamSmall || n >= (layers > 1 ? kAdamLarge : kAdamLargeAlone));
}
template <class E>
void launch_adam_copies(float *w, float *m, float *v, const float *g, E *w16, E *w16t, const AdamMatrix (&matrices)[4], size_t n, float lr, float beta1,
                        float beta2, float eps, int step, float grad_mul, const int *skip, hipStream_t s) {
    AdamLayer<E> a{};
    a.w = w; a.m = m; a.v = v; a.g = g; a.w16 = w16; a.w16t = w16t;
    const int tile = n >= kAdamLarge ? 128 : 64;           // (a d = 2048 layer 289 and 301 us, a d = 128 layer 12.2 and 5.5)
    int regions = 0;
    size_t at = 0;
    auto add = [&](size_t from, int rows, int cols) { a.region[regions++] = {from, rows, cols}; };
    for (const AdamMatrix &t : matrices) {
        if (t.at > at) add(at, 0, (int)(t.at - at));
        add(t.at, t.rows, t.cols);
        at = t.at + (size_t)t.rows * t.cols;
    }
    if (n > at) add(at, 0, (int)(n - at));
    const int blocks = first_workgroups(a.first, regions, [&](int i) {
        const int rows = a.region[i].rows, cols = a.region[i].cols;
        return rows > 0 ? ((rows + tile - 1) / tile) * ((cols + tile - 1) / tile) : (cols + 1023) / 1024;
    });
    ProfScope scope("adam_kernel", 12.0 * n, 32.0 * n, s);
    const auto kernel = tile == 64 ? adam_copies_kernel<64, E> : adam_copies_kernel<128, E>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, adam_consts(lr, beta1, beta2, eps, step, grad_mul), skip);
}
template void launch_adam_copies<bf16>(float *, float *, float *, const float *, bf16 *, bf16 *, const AdamMatrix (&)[4], size_t, float, float, float, float,
                                       int, float, const int *, hipStream_t);
template void launch_adam_copies<f16>(float *, float *, float *, const float *, f16 *, f16 *, const AdamMatrix (&)[4], size_t, float, float, float, float, int,
                                      float, const int *, hipStream_t);

}  // namespace lga
