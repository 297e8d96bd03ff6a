// 16-bit MFMA GEMM for problems that do not give every compute unit a 256 x 256 tile (both operands k-contiguous, fp32
// accumulate, the same epilogues as the large-tile kernel).
//
// What bounds such a problem is latency: a workgroup's serial walk over k, one memory latency and one barrier per step, with
// few wavefronts on a compute unit to fill them.  So
//  - operands go global -> LDS without passing through registers (see the large-tile kernel for the swizzle), 64 k per step,
//    in NS stages, so that NS - 1 steps are in flight while one is multiplied;
//  - a workgroup is four wavefronts (2 x 2 over the BM x BN tile), or KG groups of four, each of which takes its own part of the
//    k range; their sums meet in LDS at the end and are added in group order (the result does not depend on scheduling);
//  - the finished tile leaves through LDS row by row, 16 bytes per lane, with the epilogue applied on the way.
// Groups and slices of k are for the weight gradients only.  With one group an element's products are added in the order of
// the large-tile kernel, so an activation does not depend on how many rows share its launch, nor on which of the two kernels
// runs: the orders and groupings of the micro-batches agree bit for bit.  (Four groups would give 160 x 1920 x 7680 another
// 28 -> 20 us; other shapes gain 0 - 10 %.)
// Measured against the register-staged 128 x 128 kernel that served these problems before (one MI355X, us): 256 x 512 x 128 with
// GELU 10.3 -> 5.0, 160 x 1920 x 7680 85 -> 28, 932 x 1280 x 5120 61 -> 35, 4096 x 768 x 3072 44 -> 30, weight gradient
// 768 x 768 x 4096 34 (256 x 256 tiles, k in 4 slices) -> 17, 512 x 512 x 4096 31 -> 11.
#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "gemm16.h"
#include "kernels.h"

namespace lga {

namespace {

template <class E> __device__ __forceinline__ f32x4 mfma_16x16x32(x8<E> a, x8<E> b, f32x4 c);
template <> __device__ __forceinline__ f32x4 mfma_16x16x32<bf16>(x8<bf16> a, x8<bf16> b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mfma_16x16x32<f16>(x8<f16> a, x8<f16> b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

template <int BM, int BN, int KG, int NS> struct SmallTile {
    static constexpr int kStageElems = (BM + BN) * BK;                 // A tile, then B tile
    static constexpr int kPitch = BN + 4;                              // of the finished tile in LDS (floats)
    static constexpr size_t kRing = (size_t)KG * NS * kStageElems * 2, kOut = (size_t)KG * BM * kPitch * 4;
    static constexpr size_t smem = kRing > kOut ? kRing : kOut;
};

// In: GemmParams<E>, or GemmGroup<E> for the weight gradients of a layer in one launch.
template <int BM, int BN, int KG, int NS, int EPI, class E, class In>
__global__ __launch_bounds__(256 * KG) void gemm_small_kernel(In in, int tiles_m, int tiles_n) {
    constexpr bool GROUP = std::is_same<In, GemmGroup<E>>::value;
    typedef SmallTile<BM, BN, KG, NS> T;
    constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 16, FN = WN / 16;
    constexpr int NL = (BM + BN) / 32;                                 // loads of a wavefront per step: 8 rows each
    constexpr int kNewer = (NS - 2) * NL;                              // loads of the steps after the one that is waited for
    static_assert(BM % 32 == 0 && BN % 32 == 0 && NS >= 2 && kNewer < 64, "whole blocks; vmcnt has six bits");
    constexpr int kWaitOlder = 0x0070 | (kNewer & 15) | (kNewer >> 4 << 14);       // s_waitcnt lgkmcnt(0) vmcnt(kNewer)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    GemmParams<E> p;
    int tile;
    if constexpr (GROUP) {
        tile = xcd_contiguous(gridDim.x);
        p = select_from_group<BM, BN>(in, tile, tiles_m, tiles_n);
    } else {
        p = in;
        tile = xcd_contiguous(tiles_m * tiles_n * ((EPI == EPI_ACCUM_F32 && p.ksplit > 1) ? p.ksplit : p.batch > 1 ? p.batch : 1));
    }
    const int ntiles = tiles_m * tiles_n;
    if (!GROUP && p.batch > 1) select_problem(p, tile, ntiles);
    if constexpr (EPI == EPI_ACCUM_F32) {
        if (p.ksplit > 1) {
            const int z = tile / ntiles, k0 = z * p.kchunk;
            tile -= z * ntiles;
            p.A += k0;
            p.B += k0;
            p.K = min(p.K - k0, p.kchunk);
            p.outf = p.partial + (size_t)z * p.M * p.N;
            p.ldc = p.N;
            p.beta = 0.f;
        }
    }
    constexpr int GROUP_M = 8;
    const int group_size = GROUP_M * tiles_n;
    const int gid = tile / group_size, first_m = gid * GROUP_M, gsz = min(tiles_m - first_m, GROUP_M);
    const int m0 = (first_m + (tile % group_size) % gsz) * BM, n0 = ((tile % group_size) / gsz) * BN;
    if (!GROUP && p.tri == 1 && n0 >= m0 + BM) return;             // whole workgroup: the tile lies above the diagonal

    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
    const int wm = wave >> 1, wn = wave & 1;

    int kbeg = 0;
    if (!GROUP && p.tri == 2) p.K = min(p.K, m0 + BM);
    if (!GROUP && p.tri == 3) kbeg = min(m0, p.K) / BK * BK;       // whole k steps before the tile's first row
    const int steps = ((p.K - kbeg + BK - 1) / BK + KG - 1) / KG;
    kbeg += group * steps * BK;

    // Load i of a wavefront fills rows [(wave NL + i) 8, + 8) of the stage's BM + BN rows; lane L's 16 bytes land at 16 L of its
    // 1 KB, i.e. physical chunk L % 8 of row L / 8, for which it fetches logical chunk (L % 8) ^ swz16(row).
    E *ring = reinterpret_cast<E *>(smem_raw) + group * NS * T::kStageElems;
    int off[NL];
    const int chunk = (lane & 7) ^ ((lane >> 4) & 3);    // swz16 of row 8 q + lane / 8 is (lane >> 4) + 4 (q odd)
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int q = wave * NL + i, r = q * 8 + (lane >> 3);
        const bool is_a = q < BM / 8;
        const int row = is_a ? r : r - BM;
        const bool in = is_a ? m0 + row < p.M : n0 + row < p.N;
        off[i] = in ? row * (is_a ? p.lda : p.ldb) * 2 + ((chunk ^ ((q & 1) << 2)) << 4) : kBufPoison;
    }
    const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A + (size_t)m0 * p.lda), rsB = make_rsrc(p.B + (size_t)n0 * p.ldb);
    typedef __attribute__((address_space(3))) void *lds_ptr;
    auto load_step = [&](int s) {
        const int k0 = kbeg + s * BK, krem = p.K - k0;
        E *stage = ring + (s % NS) * T::kStageElems;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int q = wave * NL + i;
            int vo = off[i];
            if (krem < BK) vo = ((chunk ^ ((q & 1) << 2)) * 8 < krem) ? vo : kBufPoison;      // partial or empty last step: zeros
            lds_ptr dst = (lds_ptr)(stage + q * 8 * BK);
            if (q < BM / 8) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, dst, 16, vo, krem > 0 ? k0 * 2 : 0, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, dst, 16, vo, krem > 0 ? k0 * 2 : 0, 0, 0);
        }
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < steps) load_step(s);
    const int lane_sw = lq ^ (l16 >> 1);                 // logical chunk 4 ks + lq of a row r = l16 (mod 16)
    const int off_a = (wm * WM + l16) * BK + lane_sw * 8, off_b = (BM + wn * WN + l16) * BK + lane_sw * 8;
    for (int s = 0; s < steps; ++s) {
        // this wavefront's loads of step s have landed and its LDS reads of step s - 1 have returned; after the barrier the step is
        // published and the stage of step s - 1 is free
        if (NS > 2 && s + NS - 2 < steps) __builtin_amdgcn_s_waitcnt(kWaitOlder);
        else __builtin_amdgcn_s_waitcnt(0x0070);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + NS - 1 < steps) load_step(s + NS - 1);
        const E *stage = ring + (s % NS) * T::kStageElems;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            x8<E> af[FM], bf[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) af[i] = *reinterpret_cast<const x8<E> *>(stage + (off_a ^ (ks << 5)) + i * 16 * BK);
#pragma unroll
            for (int j = 0; j < FN; ++j) bf[j] = *reinterpret_cast<const x8<E> *>(stage + (off_b ^ (ks << 5)) + j * 16 * BK);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = mfma_16x16x32<E>(bf[j], af[i], acc[i][j]);
        }
    }
    if constexpr (EPI == EPI_ACCUM_F32 && KG == 1 && BM == 128) if (gridDim.x <= 256) {
        // A whole 128 x 128 tile of fp32 results leaves from the registers, 64 bytes of 16 rows per instruction, where compute units hold
        // one workgroup: nothing would run beside the way through LDS (1024 x 4096 x 512, 256 tiles: 12.2 -> 10.9 us,
        // 2048 x 2048 x 64: 8.5 -> 7.0; but 1280 x 3840 x 256, 300 tiles: 10.6 -> 11.4).
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int m = m0 + wm * WM + i * 16 + l16, n = n0 + wn * WN + j * 16 + 4 * lq;
                const float a[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
                if (m < p.M && n < p.N) epilogue4<EPI, E>(p, m, n, a);
            }
        return;
    }
    __syncthreads();                                     // nobody reads the ring any more, no load is in flight

    float *out = reinterpret_cast<float *>(smem_raw);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
            *reinterpret_cast<f32x4 *>(out + (group * BM + wm * WM + i * 16 + l16) * T::kPitch + wn * WN + j * 16 + 4 * lq) = acc[i][j];
    __syncthreads();
    constexpr int kItems = BM * BN / 8, kThreads = 256 * KG;
    constexpr bool kReadsAux = EPI == EPI_BIAS_RESID || EPI == EPI_MUL_DGELU;
#pragma unroll
    for (int it = 0; it < (kItems + kThreads - 1) / kThreads; ++it) {
        const int item = it * kThreads + threadIdx.x, r = item / (BN / 8), c = item % (BN / 8) * 8;
        const int m = m0 + r, n = n0 + c;
        if (item >= kItems || m >= p.M || n >= p.N) continue;
        x8<E> aux8 = {};
        if constexpr (kReadsAux) aux8 = *reinterpret_cast<const x8<E> *>(p.aux + (size_t)m * p.ldc + n);
        f32x4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = b0;
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU) {
            b0 = *reinterpret_cast<const f32x4 *>(p.bias + n);
            b1 = *reinterpret_cast<const f32x4 *>(p.bias + n + 4);
        }
        f32x4 lo = *reinterpret_cast<const f32x4 *>(out + r * T::kPitch + c), hi = *reinterpret_cast<const f32x4 *>(out + r * T::kPitch + c + 4);
#pragma unroll
        for (int g = 1; g < KG; ++g) {
            lo += *reinterpret_cast<const f32x4 *>(out + (g * BM + r) * T::kPitch + c);
            hi += *reinterpret_cast<const f32x4 *>(out + (g * BM + r) * T::kPitch + c + 4);
        }
        if constexpr (EPI == EPI_ACCUM_F32) {
            f32x4 *o = reinterpret_cast<f32x4 *>(p.outf + (size_t)m * p.ldc + n);
            if (p.beta != 0.f) {
                lo += p.beta * o[0];
                hi += p.beta * o[1];
            }
            o[0] = lo;
            o[1] = hi;
        } else {
            x8<E> o8;
            if (EPI != EPI_BIAS_GELU || p.out2) epilogue8<EPI, true, E>(p, m, n, lo, hi, aux8, b0, b1, o8);
            else epilogue8<EPI, false, E>(p, m, n, lo, hi, aux8, b0, b1, o8);
        }
    }
}

template <int BM, int BN, int KG, int NS, int EPI, class E> void launch_config(const GemmParams<E> &p, hipStream_t s) {
    typedef SmallTile<BM, BN, KG, NS> T;
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    const int work = tiles_m * tiles_n * (p.ksplit > 1 ? p.ksplit : p.batch > 1 ? p.batch : 1);
    const char *et = std::is_same<E, bf16>::value ? "bf16" : "f16", *batched = p.batch > 1 ? " (batched)" : "";
    char name[96];
    snprintf(name, sizeof(name), "gemm_%s_small_kernel<%d, %d, %d, %d>%s", et, BM, BN, KG, EPI, batched);
    const double mn = (double)p.M * p.N, nb = p.batch > 1 ? p.batch : 1;
    const double out_bytes = EPI == EPI_ACCUM_F32 ? (p.beta != 0.f ? 8.0 : 4.0) : EPI == EPI_BIAS_GELU && p.out2 ? 4.0 : 2.0;
    const double aux_bytes = (EPI == EPI_BIAS_RESID || EPI == EPI_MUL_DGELU) ? 2.0 : 0.0;
    ProfScope scope(name, nb * 2.0 * mn * p.K, nb * (2.0 * ((double)p.M * p.K + (double)p.K * p.N) + mn * (out_bytes + aux_bytes)), s);
    hipLaunchKernelGGL((gemm_small_kernel<BM, BN, KG, NS, EPI, E, GemmParams<E>>), dim3((unsigned)work), dim3(256 * KG), T::smem, s, p, tiles_m, tiles_n);
}

long tiles_of(const int M, const int N, int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); }

template <int BM, int BN, int KG, int NS, int EPI, class E, template <class> class In = GemmParams> hipError_t raise_config() {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_small_kernel<BM, BN, KG, NS, EPI, E, In<E>>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)SmallTile<BM, BN, KG, NS>::smem);
}
template <int EPI, class E> hipError_t raise_epilogue() {
    hipError_t e = raise_config<64, 64, 1, 2, EPI, E>();
    auto next = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    next(raise_config<128, 128, 1, 2, EPI, E>());
    if constexpr (EPI == EPI_ACCUM_F32) {
        next(raise_config<32, 64, 4, 3, EPI, E>());
        next(raise_config<64, 64, 2, 3, EPI, E>());
        next(raise_config<64, 64, 2, 2, EPI, E>());
        next(raise_config<32, 64, 4, 3, EPI, E, GemmGroup>());
        next(raise_config<64, 64, 2, 3, EPI, E, GemmGroup>());
        next(raise_config<64, 64, 2, 2, EPI, E, GemmGroup>());
        next(raise_config<64, 64, 1, 2, EPI, E, GemmGroup>());
        next(raise_config<128, 128, 1, 2, EPI, E, GemmGroup>());
    } else {
        next(raise_config<32, 64, 1, 8, EPI, E>());
        next(raise_config<64, 64, 1, 4, EPI, E>());
        next(raise_config<128, 128, 1, 3, EPI, E>());
    }
    return e;
}
template <class E> hipError_t raise_type() {
    hipError_t e = raise_epilogue<EPI_STORE, E>();
    if (e == hipSuccess) e = raise_epilogue<EPI_BIAS, E>();
    if (e == hipSuccess) e = raise_epilogue<EPI_BIAS_RESID, E>();
    if (e == hipSuccess) e = raise_epilogue<EPI_BIAS_GELU, E>();
    if (e == hipSuccess) e = raise_epilogue<EPI_MUL_DGELU, E>();
    if (e == hipSuccess) e = raise_epilogue<EPI_ACCUM_F32, E>();
    return e;
}

}  // namespace

// A long k range over few tiles: slices over the grid, up to 256 workgroups, at least 512 k each; the second kernel costs
// 5 us and more, so not below 4096 k (128 x 512 x 4096: 10.1 in 8 slices, 10.8 in one piece; x 8192: 11.4, 18)
int gemm_small_slices(int M, int N, int K, size_t partial_floats) {
    const long t64 = tiles_of(M, N, 64, 64);
    if (K <= 4096 || t64 < 1 || t64 > 128) return 1;
    const long fit = (long)std::min<size_t>(partial_floats / ((size_t)M * N), 32);
    return (int)std::max<long>(1, std::min({256 / t64, (long)K / 512, fit}));
}

// Which tile, how many stages and k groups: by how many workgroups a tiling gives the 256 compute units, so that the tiles run in one
// round and each unit has as many loads in flight as its LDS holds.  Measured at K = 512 ... 16384 (us, best of the others in brackets):
//   32 x 64, 8 stages, one workgroup per unit    up to 256 of them: 160 x 1920 x 7680 28.5 [35.1], 80 x 4096 x 4096 16.1 [19.3]
//   64 x 64, 4 stages, two per unit              up to 512: 160 x 7680 x 1920 14.9 [15.3], 1000 x 2048 x 8192 49.9 [50.9]
//   64 x 64, 2 stages, three and more per unit   up to 768: 4096 x 768 x 3072 30.5 [31.5], 1000 x 3072 x 2048 21.4 [22.5]
//   128 x 128, 3 stages, one per unit            up to 256: 3312 x 1064 x 1064 15.4 [16.9]
//   128 x 128, 2 stages, two per unit            beyond: half the operand traffic, 1280 x 3840 x 4096 56 [71]
// and for the weight gradients with two and four groups:
//   32 x 64, 4 groups x 3 stages                 up to 256: 512 x 512 x 4096 11.1 [13.2]
//   64 x 64, 2 groups x 3 stages                 up to 256: 768 x 768 x 4096 16.7 [18.9]
//   64 x 64, 2 groups x 2 stages                 up to 512: 768 x 2304 x 4096 25.5 [26.2], 1064 x 1064 x 2048 14.0 [15.4]
//   64 x 64, 1 group, 2 stages                   up to 768: 768 x 3072 x 4096 34.4 [43.7]
template <int EPI, class E> void launch_gemm_small(const GemmParams<E> &p, hipStream_t s) {
    if (p.batch > 1) return launch_config<128, 128, 1, 2, EPI, E>(p, s);
    const long t32 = tiles_of(p.M, p.N, 32, 64), t64 = tiles_of(p.M, p.N, 64, 64);
    if constexpr (EPI == EPI_ACCUM_F32) {
        const int slices = p.partial && p.N % 4 == 0 ? gemm_small_slices(p.M, p.N, p.K, p.partial_floats) : 1;
        if (slices > 1) {
            GemmParams<E> q = p;
            q.kchunk = ((p.K + slices - 1) / slices + BK - 1) / BK * BK;
            q.ksplit = (p.K + q.kchunk - 1) / q.kchunk;
            launch_config<64, 64, 2, 2, EPI, E>(q, s);
            launch_splitk_reduce(p.partial, q.ksplit, p.outf, p.M, p.N, p.ldc, p.beta, s);
            return;
        }
        if (t32 <= 256) launch_config<32, 64, 4, 3, EPI, E>(p, s);
        else if (t64 <= 256) launch_config<64, 64, 2, 3, EPI, E>(p, s);
        else if (t64 <= 512) launch_config<64, 64, 2, 2, EPI, E>(p, s);
        else if (t64 <= 768) launch_config<64, 64, 1, 2, EPI, E>(p, s);
        else launch_config<128, 128, 1, 2, EPI, E>(p, s);
    } else {
        if (t32 <= 256) launch_config<32, 64, 1, 8, EPI, E>(p, s);
        else if (t64 <= 512) launch_config<64, 64, 1, 4, EPI, E>(p, s);
        else if (t64 <= 768) launch_config<64, 64, 1, 2, EPI, E>(p, s);
        else if (tiles_of(p.M, p.N, 128, 128) <= 256) launch_config<128, 128, 1, 3, EPI, E>(p, s);
        else launch_config<128, 128, 1, 2, EPI, E>(p, s);
    }
}
template <int BM, int BN, int KG, int NS, class E> void launch_group_config(const GemmGroup<E> &group, hipStream_t s) {
    typedef SmallTile<BM, BN, KG, NS> T;
    long work = 0;
    double flops = 0.0, bytes = 0.0;
    for (int i = 0; i < group.n; ++i) {
        const GemmParams<E> &p = group.p[i];
        const double mn = (double)p.M * p.N;
        work += tiles_of(p.M, p.N, BM, BN) * p.ksplit;
        flops += 2.0 * mn * p.K;
        bytes += 2.0 * ((double)p.M * p.K + (double)p.K * p.N) + mn * (p.beta != 0.f ? 8.0 : 4.0);
    }
    char name[96];
    snprintf(name, sizeof(name), "gemm_%s_small_kernel<%d, %d, %d, %d> (grouped)", std::is_same<E, bf16>::value ? "bf16" : "f16", BM, BN, KG, EPI_ACCUM_F32);
    ProfScope scope(name, flops, bytes, s);
    hipLaunchKernelGGL((gemm_small_kernel<BM, BN, KG, NS, EPI_ACCUM_F32, E, GemmGroup<E>>), dim3((unsigned)work), dim3(256 * KG), T::smem, s, group, 0, 0);
}

// Several weight gradients over the same k range together: the tile by the number of workgroups they give in all, slices of a long
// k range only where even together they leave compute units without one.  The four matrices of a d = 128 layer over 512 tokens: 5.8 us, in
// launches of their own 4 x 4.7; with their operands' transposes in one launch as well the stack's step went from 518 to 426 us.
template <class E> void launch_gemm_small_group(const GemmParams<E> *p, int n, hipStream_t s) {
    GemmGroup<E> group{};
    group.n = n;
    long t32 = 0, t64 = 0;
    size_t outputs = 0;
    for (int i = 0; i < n; ++i) {
        t32 += tiles_of(p[i].M, p[i].N, 32, 64);
        t64 += tiles_of(p[i].M, p[i].N, 64, 64);
        outputs += (size_t)p[i].M * p[i].N;
    }
    int slices = 1;
    if (p[0].K > 4096 && t64 <= 128 && p[0].partial)
        slices = (int)std::max<long>(1, std::min({256 / t64, (long)p[0].K / 512, (long)std::min<size_t>(p[0].partial_floats / outputs, 32)}));
    prepare_gemm_group(group, p, slices);
    if (slices > 1) launch_group_config<64, 64, 2, 2, E>(group, s);
    else if (t32 <= 256) launch_group_config<32, 64, 4, 3, E>(group, s);
    else if (t64 <= 256) launch_group_config<64, 64, 2, 3, E>(group, s);
    else if (t64 <= 512) launch_group_config<64, 64, 2, 2, E>(group, s);
    else if (t64 <= 768) launch_group_config<64, 64, 1, 2, E>(group, s);
    else launch_group_config<128, 128, 1, 2, E>(group, s);
    launch_splitk_reduce_group(group, s);
}
template void launch_gemm_small_group<bf16>(const GemmParams<bf16> *, int, hipStream_t);
template void launch_gemm_small_group<f16>(const GemmParams<f16> *, int, hipStream_t);

#define LGA_SMALL(EPI)                                                              \
    template void launch_gemm_small<EPI, bf16>(const GemmParams<bf16> &, hipStream_t); \
    template void launch_gemm_small<EPI, f16>(const GemmParams<f16> &, hipStream_t)
LGA_SMALL(EPI_STORE);
LGA_SMALL(EPI_BIAS);
LGA_SMALL(EPI_BIAS_RESID);
LGA_SMALL(EPI_BIAS_GELU);
LGA_SMALL(EPI_MUL_DGELU);
LGA_SMALL(EPI_ACCUM_F32);
#undef LGA_SMALL

hipError_t gemm_small_prepare_kernels() {
    hipError_t e = raise_type<bf16>();
    if (e == hipSuccess) e = raise_type<f16>();
    return e;
}

}  // namespace lga
