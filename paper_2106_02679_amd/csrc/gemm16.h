// Device code that the 16-bit GEMM kernels share: buffer resources, epilogues, the choice of a batch's problem.
#pragma once

#include "common.h"

namespace lga {
namespace {

constexpr int BK = 64;           // k elements per stage

constexpr int kBufRange = 0x40000000;          // 1 GiB window; valid offsets are far below it
constexpr int kBufPoison = 0x7FFFFF00;         // always out of range

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, kBufRange, 0x00020000);
}

__device__ __forceinline__ int swz16(int row) { return (row >> 1) & 7; }      // 16 rows of one chunk column -> 8 chunk places x 2 row parities

template <int EPI, class E>
__device__ __forceinline__ void epilogue4(const GemmParams<E> &p, int m, int n, const float (&a)[4]) {
    const size_t idx = (size_t)m * p.ldc + n;
    if constexpr (EPI == EPI_ACCUM_F32) {
        f32x4 o = {a[0], a[1], a[2], a[3]};
        if (p.beta != 0.f) {
            const f32x4 old = *reinterpret_cast<const f32x4 *>(p.outf + idx);
            o += p.beta * old;
        }
        *reinterpret_cast<f32x4 *>(p.outf + idx) = o;
        return;
    } else {
        float r[4] = {a[0], a[1], a[2], a[3]};
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU) {
            const f32x4 b = *reinterpret_cast<const f32x4 *>(p.bias + n);
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] += b[i];
        }
        if constexpr (EPI == EPI_BIAS_RESID) {
            const x4<E> x = *reinterpret_cast<const x4<E> *>(p.aux + idx);
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] += (float)x[i];
        }
        if constexpr (EPI == EPI_MUL_DGELU) {
            const x4<E> u = *reinterpret_cast<const x4<E> *>(p.aux + idx);
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] *= gelu_grad_f((float)u[i]);
        }
        if constexpr (EPI == EPI_BIAS_GELU) {
            x4<E> u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                u[i] = (E)r[i];
                r[i] = gelu_f(r[i]);
            }
            if (p.out2) *reinterpret_cast<x4<E> *>(p.out2 + idx) = u;
        }
        x4<E> o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (E)r[i];
        *reinterpret_cast<x4<E> *>(p.out + idx) = o;
    }
}

// The same for 8 consecutive n of one row, with 16-byte accesses (bf16 outputs only): n, ldc multiples of 8 and
// 16-byte aligned tensors.
// aux8: the 8 values of aux at (m, n .. n + 7) for the two epilogues that read it, and b0, b1: the bias of columns
// n .. n + 7 for the three that add it, both loaded by the caller (ahead of time).  o: the results, too.
// PRE: of EPI_BIAS_GELU, whether the pre-activation is stored (a test per store would keep the stores of a strip apart).
template <int EPI, bool PRE, class E>
__device__ __forceinline__ void epilogue8(const GemmParams<E> &p, int m, int n, const f32x4 &lo, const f32x4 &hi,
                                          const x8<E> &aux8, const f32x4 &b0, const f32x4 &b1, x8<E> &o) {
    static_assert(EPI != EPI_ACCUM_F32, "16-bit outputs only");
    const size_t idx = (size_t)m * p.ldc + n;
    float r[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r[i] += b0[i];
            r[4 + i] += b1[i];
        }
    }
    if constexpr (EPI == EPI_BIAS_RESID) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] += (float)aux8[i];
    }
    if constexpr (EPI == EPI_MUL_DGELU) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] *= gelu_grad_f((float)aux8[i]);
    }
    if constexpr (EPI == EPI_BIAS_GELU) {
        x8<E> u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            u[i] = (E)r[i];
            r[i] = gelu_f(r[i]);
        }
        if constexpr (PRE) *reinterpret_cast<x8<E> *>(p.out2 + idx) = u;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (E)r[i];
    *reinterpret_cast<x8<E> *>(p.out + idx) = o;
}

// Workgroup ids are dealt round-robin over the 8 XCDs: the work item of this workgroup such that each XCD has a contiguous range of them.
__device__ __forceinline__ int xcd_contiguous(int nwork) {
    const int pid = blockIdx.x, xcd = pid & 7, local = pid >> 3;
    const int base = nwork >> 3, rem = nwork & 7;
    return xcd * base + (xcd < rem ? xcd : rem) + local;
}

// Grouped launch: the problem that work item `tile` belongs to, and the item's place in it.
template <int BM, int BN, class E> __device__ __forceinline__ GemmParams<E> select_from_group(const GemmGroup<E> &in, int &tile, int &tiles_m, int &tiles_n) {
    int z = 0;
    for (;;) {
        tiles_m = (in.p[z].M + BM - 1) / BM;
        tiles_n = (in.p[z].N + BN - 1) / BN;
        const int items = tiles_m * tiles_n * in.p[z].ksplit;
        if (z + 1 >= in.n || tile < items) return in.p[z];
        tile -= items;
        ++z;
    }
}

// Batched launch: work item `tile` belongs to problem tile / ntiles; rebase the operands and outputs onto it.
template <class E> __device__ __forceinline__ void select_problem(GemmParams<E> &p, int &tile, int ntiles) {
    const int z = tile / ntiles;
    tile -= z * ntiles;
    p.A += z * p.strideA;
    p.B += z * p.strideB;
    const long long c = z * p.strideC;
    if (p.out) p.out += c;
    if (p.out2) p.out2 += c;
    if (p.outf) p.outf += c;
    if (p.aux) p.aux += c;
}

}  // namespace
}  // namespace lga
