// Softmax attention (causal or unmasked) on fp32 tensors with the fp32 matrix instruction, head sizes up to 128; all scores,
// probabilities and sums in fp32.  Larger heads and sequences of up to 48 positions keep the one-wavefront-per-position kernels.
//
// A wavefront works on 32 positions (queries in the forward and the dQ kernel, keys in the dK/dV kernel) against blocks of 32
// positions of the other kind.  The score block is produced transposed (streamed positions = first operand of the
// instruction), so a lane owns one position l % 32 and its 16 result registers are 16 streamed positions,
// 8 (r / 4) + 4 (l / 32) + r % 4: the softmax is lane-local up to one exchange between the two lane halves, and
// register r is by itself the second operand of the next product, whose first operand is then element [position][channel
// l % 32] of the streamed tensor - one coalesced 4-byte load per lane.  Nothing goes through LDS on the way in: the fp32
// instruction takes 64 cycles, and the rows come from the caches.
//
// What bounds it at the sizes the fp32 mode is used at is the serial chain over the streamed blocks, not arithmetic, so the four
// wavefronts of a workgroup share one block of 32 positions and take every fourth streamed block each; their sums meet in LDS
// in wavefront order (deterministic).  Measured on 8 sequences x 8 heads x 256 positions x 32 without the mask, against
// one wavefront per position with scalar products: forward 114 -> 13 us, dQ 184 -> 17,
// dK/dV 289 -> 21.
#include <type_traits>

#include "kernels.h"

namespace lga {

namespace {

constexpr int kWaves = 4;

// Rows are read through buffer loads based at the first row of a block of 32 positions: a lane whose position or channel does not exist
// gets an offset out of the buffer's range, which the hardware answers with zeros.
constexpr int kRange = 0x40000000, kPoison = 0x7FFFFF00;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_at(const float *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, kRange, 0x00020000);
}
// Channels 8 j + 4 half .. + 3 of the row at byte offset `row` (kPoison: no such row; adding a row's bytes to it leaves it out of range).
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t rs, int row, int j, int half, int dh, bool vec) {
    const int c = 8 * j + 4 * half;
    if (vec) return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (c < dh ? row + 16 * half : kPoison) + 32 * j, 0, 0));
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        v[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (c + i < dh ? row + 16 * half : kPoison) + 32 * j + 4 * i, 0, 0));
    return v;
}
__device__ __forceinline__ f32x16 zero16() { return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; }

template <int DH> struct AttnF32 {
    static constexpr int NJ = DH / 8, NC = DH / 32;
    // C[streamed][own] = sum_c rows[streamed][c] own[c]: `row` is the offset of this lane's streamed row (position l % 32 of the block)
    static __device__ __forceinline__ f32x16 product(__amdgpu_buffer_rsrc_t rs, int row, const f32x4 (&own)[NJ], int half, int dh, bool vec) {
        f32x16 acc = zero16();
        f32x4 f[NJ];
        load_own(f, rs, row, half, dh, vec);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[j][i], own[j][i], acc, 0, 0, 0);
        return acc;
    }
    static __device__ __forceinline__ void load_own(f32x4 (&own)[NJ], __amdgpu_buffer_rsrc_t rs, int row, int half, int dh, bool vec) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) own[j] = load4(rs, row, j, half, dh, vec);
    }
    // acc[channel][own] += sum over the block's 32 streamed positions of base[position][channel] * p[position][own].
    // left: positions of the block inside the sequence.  seen(r): whether this lane's position sees the streamed position of register
    // r; only a masked block asks.  There p is zero where it does not, but 0 * inf is not: a value that must not
    // be seen is kept out of the sums even if it is not finite.
    template <class Seen>
    static __device__ __forceinline__ void accumulate(f32x16 (&acc)[NC], __amdgpu_buffer_rsrc_t rs, int pitch4, int left, int dh, int l32, int half,
                                                      const f32x16 &p, bool masked, Seen seen) {
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) {
            const int c = 32 * cb + l32;
            float a[16];
            bool odd = false;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int pos = 8 * (r >> 2) + 4 * half + (r & 3);
                a[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, pos < left && c < dh ? 4 * half * pitch4 + 4 * c : kPoison,
                                                                                      (8 * (r >> 2) + (r & 3)) * pitch4, 0));
                odd |= !(fabsf(a[r]) < INFINITY);
            }
            if (masked && __any(odd)) {
                for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bool own_half = half == hh, take = seen(8 * (r >> 2) + 4 * hh + (r & 3));
                        const f32x16 t = __builtin_amdgcn_mfma_f32_32x32x2f32(own_half ? a[r] : 0.f, own_half ? p[r] : 0.f, acc[cb], 0, 0, 0);
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[cb][i] = take ? t[i] : acc[cb][i];
                    }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[r], p[r], acc[cb], 0, 0, 0);
            }
        }
    }
    // out_row[c] = mul * sum over the four wavefronts of acc, for the position this lane owns; red: 16 KB of LDS
    static __device__ __forceinline__ void merge_store(const f32x16 (&acc)[NC], float *red, int wave, int lane, float own_mul, float mul,
                                                       float *out_row, bool valid, int dh, bool vec) {
        const int half = lane >> 5;
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[cb][r] * own_mul;
            __syncthreads();
            f32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float t = red[(4 * wave + i) * 64 + lane];
#pragma unroll
                for (int w = 1; w < kWaves; ++w) t += red[(w * 16 + 4 * wave + i) * 64 + lane];
                o[i] = t * mul;
            }
            const int c = 32 * cb + 8 * wave + 4 * half;
            if (!valid || c >= dh) continue;
            if (vec) {
                *reinterpret_cast<f32x4 *>(out_row + c) = o;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c + i < dh) out_row[c + i] = o[i];
            }
        }
    }
};

struct Place {
    int b, h, block;
};
// grid: n_seq * heads * blocks workgroups; with the causal mask the longest blocks (rank 0) are handed out first
__device__ __forceinline__ Place place_of(const AttnShape &sh, int nblocks, bool longest_last) {
    const int bhs = sh.n_seq * sh.heads, bh = blockIdx.x % bhs, rank = blockIdx.x / bhs;
    return Place{bh / sh.heads, bh % sh.heads, longest_last ? nblocks - 1 - rank : rank};
}

template <int DH>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(const float *__restrict__ qkv, float *__restrict__ out, float *__restrict__ lse,
                                                           AttnShape sh, bool vec) {
    typedef AttnF32<DH> A;
    __shared__ float red[kWaves * 16 * 64];
    __shared__ float m_s[kWaves][32], l_s[kWaves][32];
    const int nblocks = (sh.s + 31) / 32;
    const Place at = place_of(sh, nblocks, sh.causal);
    const int dh = sh.dh, d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const float *seq = qkv + (size_t)at.b * sh.s * pitch + (size_t)at.h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, half = lane >> 5;
    const int q = at.block * 32 + l32;
    const int last = sh.causal ? min(q, sh.s - 1) : sh.s - 1;           // last key this lane's query sees
    const float scale = rsqrtf((float)dh);
    f32x4 qf[A::NJ];
    const int pitch4 = 12 * d, row = l32 * pitch4;                      // bytes
    A::load_own(qf, rows_at(seq + (size_t)at.block * 32 * pitch), q < sh.s ? row : kPoison, half, dh, vec);
    f32x16 acc[A::NC];
#pragma unroll
    for (int cb = 0; cb < A::NC; ++cb) acc[cb] = zero16();
    float m = -INFINITY, l = 0.f;
    const int kblocks = sh.causal ? at.block + 1 : nblocks;
    for (int kb = wave; kb < kblocks; kb += kWaves) {
        const int k0 = 32 * kb, key = k0 + l32;
        const bool masked = (sh.causal && kb == at.block) || k0 + 32 > sh.s;
        const float *rows = seq + (size_t)k0 * pitch;
        f32x16 st = A::product(rows_at(rows + d), key < sh.s ? row : kPoison, qf, half, dh, vec);
        float top = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            st[r] *= scale;
            if (masked && k0 + 8 * (r >> 2) + 4 * half + (r & 3) > last) st[r] = -INFINITY;
            top = fmaxf(top, st[r]);
        }
        top = fmaxf(m, fmaxf(top, __shfl_xor(top, 32, 64)));
        const float ref = top == -INFINITY ? 0.f : top;
        const float old = expf(m - ref);
        l *= old;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            st[r] = expf(st[r] - ref);
            l += st[r];
        }
#pragma unroll
        for (int cb = 0; cb < A::NC; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][r] *= old;
        m = top;
        A::accumulate(acc, rows_at(rows + 2 * d), pitch4, sh.s - k0, dh, l32, half, st, masked, [&](int pos) { return k0 + pos <= last; });
    }
    l += __shfl_xor(l, 32, 64);
    if (half == 0) {
        m_s[wave][l32] = m;
        l_s[wave][l32] = l;
    }
    __syncthreads();
    float top = m_s[0][l32];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) top = fmaxf(top, m_s[w][l32]);
    const float ref = top == -INFINITY ? 0.f : top;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += l_s[w][l32] * expf(m_s[w][l32] - ref);
    const bool valid = q < sh.s;
    A::merge_store(acc, red, wave, lane, expf(m - ref), 1.0f / sum, out + ((size_t)at.b * sh.s + q) * d + (size_t)at.h * dh, valid, dh, vec);
    if (wave == 0 && half == 0 && valid) lse[((size_t)at.b * sh.heads + at.h) * sh.s + q] = top + logf(sum);
}

// dQ, and delta = sum_c dO O of every query
template <int DH>
__global__ __launch_bounds__(256) void attn_bwd_dq_f32_kernel(const float *__restrict__ qkv, const float *__restrict__ out,
                                                              const float *__restrict__ lse, const float *__restrict__ dout,
                                                              float *__restrict__ dqkv, float *__restrict__ delta, AttnShape sh, bool vec) {
    typedef AttnF32<DH> A;
    __shared__ float red[kWaves * 16 * 64];
    const int nblocks = (sh.s + 31) / 32;
    const Place at = place_of(sh, nblocks, sh.causal);
    const int dh = sh.dh, d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const float *seq = qkv + (size_t)at.b * sh.s * pitch + (size_t)at.h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, half = lane >> 5;
    const int q = at.block * 32 + l32;
    const bool valid = q < sh.s;
    const int last = sh.causal ? min(q, sh.s - 1) : sh.s - 1;
    const float scale = rsqrtf((float)dh);
    const size_t stat = ((size_t)at.b * sh.heads + at.h) * sh.s + q;
    f32x4 qf[A::NJ], dof[A::NJ];
    const int pitch4 = 12 * d, row = l32 * pitch4, own = valid ? l32 * 4 * d : kPoison;                      // bytes
    const size_t oblock = ((size_t)at.b * sh.s + at.block * 32) * d + (size_t)at.h * dh;
    A::load_own(qf, rows_at(seq + (size_t)at.block * 32 * pitch), valid ? row : kPoison, half, dh, vec);
    A::load_own(dof, rows_at(dout + oblock), own, half, dh, vec);
    float dl = 0.f;
#pragma unroll
    for (int j = 0; j < A::NJ; ++j) {
        const f32x4 o = load4(rows_at(out + oblock), own, j, half, dh, vec);
#pragma unroll
        for (int i = 0; i < 4; ++i) dl = fmaf(dof[j][i], o[i], dl);
    }
    dl += __shfl_xor(dl, 32, 64);
    if (wave == 0 && half == 0 && valid) delta[stat] = dl;
    const float ls = valid ? lse[stat] : INFINITY;                  // queries past the end: every probability 0
    f32x16 acc[A::NC];
#pragma unroll
    for (int cb = 0; cb < A::NC; ++cb) acc[cb] = zero16();
    const int kblocks = sh.causal ? at.block + 1 : nblocks;
    for (int kb = wave; kb < kblocks; kb += kWaves) {
        const int k0 = 32 * kb, key = k0 + l32;
        const bool masked = (sh.causal && kb == at.block) || k0 + 32 > sh.s;
        const float *rows = seq + (size_t)k0 * pitch;
        const int krow = key < sh.s ? row : kPoison;
        const f32x16 st = A::product(rows_at(rows + d), krow, qf, half, dh, vec);
        f32x16 ds = A::product(rows_at(rows + 2 * d), krow, dof, half, dh, vec);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            ds[r] = expf(st[r] * scale - ls) * (ds[r] - dl);
            if (masked && k0 + 8 * (r >> 2) + 4 * half + (r & 3) > last) ds[r] = 0.f;
        }
        A::accumulate(acc, rows_at(rows + d), pitch4, sh.s - k0, dh, l32, half, ds, masked, [&](int pos) { return k0 + pos <= last; });
    }
    A::merge_store(acc, red, wave, lane, 1.f, scale, dqkv + ((size_t)at.b * sh.s + q) * pitch + (size_t)at.h * dh, valid, dh, vec);
}

// dK and dV of 32 keys; queries are streamed
template <int DH>
__global__ __launch_bounds__(256) void attn_bwd_dkv_f32_kernel(const float *__restrict__ qkv, const float *__restrict__ lse,
                                                               const float *__restrict__ dout, float *__restrict__ dqkv,
                                                               const float *__restrict__ delta, AttnShape sh, bool vec) {
    typedef AttnF32<DH> A;
    __shared__ float red[kWaves * 16 * 64];
    const int nblocks = (sh.s + 31) / 32;
    const Place at = place_of(sh, nblocks, false);
    const int dh = sh.dh, d = sh.heads * dh;
    const size_t pitch = 3 * (size_t)d;
    const float *seq = qkv + (size_t)at.b * sh.s * pitch + (size_t)at.h * dh, *dob = dout + (size_t)at.b * sh.s * d + (size_t)at.h * dh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, half = lane >> 5;
    const int key = at.block * 32 + l32;
    const bool valid = key < sh.s;
    const int first = sh.causal ? key : 0;                          // first query that sees this lane's key
    const float scale = rsqrtf((float)dh);
    const size_t stat0 = ((size_t)at.b * sh.heads + at.h) * sh.s;
    f32x4 kf[A::NJ], vf[A::NJ];
    const int pitch4 = 12 * d, row = l32 * pitch4;                      // bytes
    const float *own = seq + (size_t)at.block * 32 * pitch;
    A::load_own(kf, rows_at(own + d), valid ? row : kPoison, half, dh, vec);
    A::load_own(vf, rows_at(own + 2 * d), valid ? row : kPoison, half, dh, vec);
    f32x16 dk[A::NC], dv[A::NC];
#pragma unroll
    for (int cb = 0; cb < A::NC; ++cb) dk[cb] = dv[cb] = zero16();
    for (int qb = (sh.causal ? at.block : 0) + wave; qb < nblocks; qb += kWaves) {
        const int q0 = 32 * qb, q = q0 + l32;
        const bool masked = (sh.causal && qb == at.block) || q0 + 32 > sh.s;
        const __amdgpu_buffer_rsrc_t qrows = rows_at(seq + (size_t)q0 * pitch), drows = rows_at(dob + (size_t)q0 * d);
        const f32x16 st = A::product(qrows, q < sh.s ? row : kPoison, kf, half, dh, vec);
        f32x16 ds = A::product(drows, q < sh.s ? l32 * 4 * d : kPoison, vf, half, dh, vec), p;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int qq = q0 + 8 * (r >> 2) + 4 * half + (r & 3);
            const int qc = min(qq, sh.s - 1);
            p[r] = expf(st[r] * scale - lse[stat0 + qc]);
            ds[r] = p[r] * (ds[r] - delta[stat0 + qc]);
            if (masked && (qq >= sh.s || qq < first)) p[r] = ds[r] = 0.f;
        }
        auto seen = [&](int pos) { return q0 + pos >= first && q0 + pos < sh.s; };
        A::accumulate(dv, drows, 4 * d, sh.s - q0, dh, l32, half, p, masked, seen);
        A::accumulate(dk, qrows, pitch4, sh.s - q0, dh, l32, half, ds, masked, seen);
    }
    float *orow = dqkv + ((size_t)at.b * sh.s + key) * pitch + (size_t)at.h * dh;
    A::merge_store(dk, red, wave, lane, 1.f, scale, orow + d, valid, dh, vec);
    A::merge_store(dv, red, wave, lane, 1.f, 1.f, orow + 2 * d, valid, dh, vec);
}

bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// Up to 128 channels a wavefront's operands and accumulators fit its registers (dK/dV: 4 x dh / 2 of them); 32 rows of [Q | K | V]
// lie inside the buffer loads' range.  Short sequences stay with one wavefront per position: they give this kernel one or two streamed
// blocks, most of its wavefronts nothing to do, and its chain of 32-position products is longer than theirs until there are so many
// heads that theirs fill the chip.  Backward of n heads in all, us here [one wavefront per position], where the two meet:
//   s    dh 32                                                 dh 128
//   32   8: 15 [9]     64: 15 [14]    512: 19 [67]             8: 43 [19]    64: 43 [35]    512: 91 [261]
//   48   8: 16 [10]    64: 16 [19]    512: 35 [94]             8: 44 [24]    64: 44 [53]    512: 166 [395]
//   64   8: 15 [16]    64: 15 [40]    512: 38 [239]            8: 42 [31]    64: 43 [144]   512: 173 [919]
// By the length and not by the number of heads in the launch: a sequence's results must not depend on how many share it.
bool attn_f32_supports(AttnShape sh) { return sh.s > 48 && sh.dh <= 128 && (double)sh.heads * sh.dh * 12 * 32 < kRange; }

#define LGA_ATTN_F32_DH(dh, CALL)           \
    do {                                    \
        if ((dh) <= 32) { CALL(32); }       \
        else if ((dh) <= 64) { CALL(64); }  \
        else { CALL(128); }                 \
    } while (0)

void launch_attn_fwd_f32(const float *qkv, float *out, float *lse, AttnShape sh, hipStream_t s) {
    const size_t blocks = (size_t)sh.n_seq * sh.heads * ((sh.s + 31) / 32);
    if (blocks == 0) return;
    const bool vec = sh.dh % 4 == 0 && al16(qkv) && al16(out);
    const double pos = (double)sh.n_seq * sh.heads * sh.s, pairs = pos * sh.s * (sh.causal ? 0.5 : 1.0);
    ProfScope scope("attn_fwd_f32_kernel", 4.0 * pairs * sh.dh, 16.0 * pos * sh.dh, s);
#define CALL(DH) hipLaunchKernelGGL(attn_fwd_f32_kernel<DH>, dim3((unsigned)blocks), dim3(256), 0, s, qkv, out, lse, sh, vec)
    LGA_ATTN_F32_DH(sh.dh, CALL);
#undef CALL
}

void launch_attn_bwd_f32(const float *qkv, const float *out, const float *lse, const float *dout, float *dqkv, float *delta,
                         AttnShape sh, hipStream_t s) {
    const size_t blocks = (size_t)sh.n_seq * sh.heads * ((sh.s + 31) / 32);
    if (blocks == 0) return;
    const bool vec = sh.dh % 4 == 0 && al16(qkv) && al16(out) && al16(dout) && al16(dqkv);
    const double pos = (double)sh.n_seq * sh.heads * sh.s, pairs = pos * sh.s * (sh.causal ? 0.5 : 1.0);
    {
        ProfScope scope("attn_bwd_dq_f32_kernel", 6.0 * pairs * sh.dh, 24.0 * pos * sh.dh, s);
#define CALL(DH) hipLaunchKernelGGL(attn_bwd_dq_f32_kernel<DH>, dim3((unsigned)blocks), dim3(256), 0, s, qkv, out, lse, dout, dqkv, delta, sh, vec)
        LGA_ATTN_F32_DH(sh.dh, CALL);
#undef CALL
    }
    {
        ProfScope scope("attn_bwd_dkv_f32_kernel", 8.0 * pairs * sh.dh, 24.0 * pos * sh.dh, s);
#define CALL(DH) hipLaunchKernelGGL(attn_bwd_dkv_f32_kernel<DH>, dim3((unsigned)blocks), dim3(256), 0, s, qkv, lse, dout, dqkv, delta, sh, vec)
        LGA_ATTN_F32_DH(sh.dh, CALL);
#undef CALL
    }
}

}  // namespace lga
