// Device code that the 16-bit attention kernels share: operand reads, tiles that go straight into LDS and are read both ways, the
// order of the workgroups.
#pragma once

#include "kernels.h"

namespace lga {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Second operand straight from global memory: 8 contiguous bf16 of one row (zero if the row is invalid or the
// columns lie beyond the head size dh, a multiple of 8 that may be smaller than the kernel's padded DH).
template <class E> __device__ __forceinline__ x8<E> frag_global(const E *row_ptr, int ks, int half, bool valid, int dh) {
    if (!valid || 16 * ks + 8 * half >= dh) return x8<E>{0, 0, 0, 0, 0, 0, 0, 0};
    return *reinterpret_cast<const x8<E> *>(row_ptr + 16 * ks + 8 * half);
}
// delta of this lane's row: sum_c dO O, of which each half of the wavefront has every other 8 columns.  The dQ kernels take it from the dO
// operands that they hold anyway, one more read of O, and leave it for the dK/dV kernels: a kernel of its own read both (2 x 1728
// positions, 54 heads of 216: 27 us, both kernels together 989 -> 980; 32768 x 768: 18, the layer backward 1887 -> 1875).
template <int NK, class E> __device__ __forceinline__ float row_delta(const x8<E> (&dof)[NK], const x8<E> (&of)[NK]) {
    float t = 0.f;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) t += (float)of[ks][e] * (float)dof[ks][e];
    const uint32_t bits = __builtin_bit_cast(uint32_t, t);
    const auto halves = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
    return __builtin_bit_cast(float, (uint32_t)halves[0]) + __builtin_bit_cast(float, (uint32_t)halves[1]);
}
// 32x32 fp32 result registers 8*kk .. 8*kk+7 -> 16-bit second operand.
template <class E> __device__ __forceinline__ x8<E> pack16(const f32x16 &v, int kk) {
    x8<E> o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (E)v[8 * kk + e];
    return o;
}

// inside the kernels, whose element type is E
#define MFMA(a, b, c) mfma_32x32x16<E>((a), (b), (c))

// ---- direct-to-LDS tile loads and transposing LDS reads --------------------------------------
// buffer_load_dwordx4 ... lds writes lane L's 16 bytes at (LDS base) + 16 L; rows beyond the sequence get
// an offset outside the buffer's range, which the hardware answers with zeros.
constexpr int kBufRange = 0x40000000;
constexpr int kBufPoison = 0x7FFFFF00;
typedef __attribute__((address_space(3))) void *lds_ptr;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int range = kBufRange) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, range, 0x00020000);
}
// All LDS reads issued so far but the newest NEWER have returned; the operands listed are tied to the wait so that no use of
// them can be scheduled above it.
template <int NEWER = 0, class V, int N> __device__ __forceinline__ void wait_tr_reads(V (&f)[N]) {
    static_assert(N <= 10 && NEWER < 16, "operand list below; lgkmcnt has four bits");
    if constexpr (N == 2) asm volatile("s_waitcnt lgkmcnt(%c2)" : "+v"(f[0]), "+v"(f[1]) : "i"(NEWER));
    else if constexpr (N == 4) asm volatile("s_waitcnt lgkmcnt(%c4)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]) : "i"(NEWER));
    else if constexpr (N == 6) asm volatile("s_waitcnt lgkmcnt(%c6)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]) : "i"(NEWER));
    else if constexpr (N == 7) asm volatile("s_waitcnt lgkmcnt(%c7)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]) : "i"(NEWER));
    else if constexpr (N == 8) asm volatile("s_waitcnt lgkmcnt(%c8)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]) : "i"(NEWER));
    else if constexpr (N == 10) asm volatile("s_waitcnt lgkmcnt(%c10)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]), "+v"(f[8]), "+v"(f[9]) : "i"(NEWER));
    else static_assert(N == 2, "unsupported operand count");
}
// Tiles that are read both ways - rows with ds_read_b128 and transposed with ds_read_b64_tr_b16 - keep the
// unpadded pitch DH and an XOR swizzle of the 16-byte chunk index that is free of bank conflicts for both:
// 16 consecutive rows put one logical chunk into 16 different bank groups, and 4 consecutive rows (from a
// multiple of 4) put an aligned group of 4 chunks into 4 different ones.
template <int DH> __device__ __forceinline__ int sw_both(int row) {
    constexpr int stagger = DH / 8 % 16;                 // chunks, of the 16 that the banks hold, that a row is shifted against the one before it
    if constexpr (stagger == 0) return ((row & 3) << 2) | ((row >> 2) & 3);                  // 128, 256
    else if constexpr (stagger == 8) return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);      // 64, 192, 320
    else return (row >> 2) & 3;              // 4 or 12 - 32, 96, 160, 224: the row pitch already staggers groups of 4 chunks
}
// DMA of a ROWS x DH tile (global row pitch gp2 bytes) into such a tile: lane L of instruction j fills chunk
// slot 64 j + L = row * (DH / 8) + physical chunk, with the logical chunk that the swizzle maps there.
template <int ROWS, int DH> struct TileDmaSw {
    static constexpr int NCH = DH / 8;
    static constexpr int NI = ROWS * NCH / 64;              // instructions per tile
    static constexpr int NJ = (NI + 3) / 4;                 // per wavefront; those beyond the tile write zeros behind it
    static constexpr int ELEMS = NJ * 4 * 512;              // LDS elements to reserve: every wavefront issues NJ instructions of 1 KB
    static_assert((ROWS * NCH) % 64 == 0, "tile is a whole number of DMA instructions");
    int row[NJ], off[NJ];
    // dh <= DH: the head size in memory; logical chunks from dh / 8 on are padding (zeros)
    __device__ __forceinline__ void init(int wave, int lane, int gp2, int dh) {
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const int slot = (i * 4 + wave) * 64 + lane, r = slot / NCH, pc = slot % NCH;
            row[i] = r < ROWS && (pc ^ sw_both<DH>(r)) < dh / 8 ? r : 0x7FFFFFFF;
            off[i] = r * gp2 + ((pc ^ sw_both<DH>(r)) << 4);
        }
    }
    // src, dst: tiles of 16-bit elements of either format
    __device__ __forceinline__ void issue(const void *src, void *dst, int nvalid, int wave) const {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(src);
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const int j = i * 4 + wave;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(static_cast<char *>(dst) + j * 1024), 16, row[i] < nvalid ? off[i] : kBufPoison,
                                                     0, 0, 0);
        }
    }
};
// Per-lane address parts (elements) of the two kinds of operand read from such a tile.  The swizzle splits
// into a part that XORs the chunk group (DH = 64, 128 only) and one that XORs within the group, which leaves
// few distinct lane values; everything else is a compile-time offset.
template <int DH> struct BothAddr {
    static constexpr int NG = DH / 8 % 16 == 0 ? 4 : DH / 8 % 16 == 8 ? 2 : 1;     // neighbouring chunk groups the swizzle permutes
    int nb[NG][2];      // natural read: [chunk group][ks & 1]
    int tb[NG][2];      // transposed read: [32-column block c (if NG > 1)][second half of the 16 positions]
    __device__ __forceinline__ void init(int lane) {
        const int lrow = lane & 31, half = lane >> 5, i = lane & 15, g = (lane >> 4) & 1;
        const int s = sw_both<DH>(lrow), s_hi = s >> 2, s_lo = s & 3;
#pragma unroll
        for (int a = 0; a < NG; ++a)
#pragma unroll
            for (int e = 0; e < 2; ++e) nb[a][e] = lrow * DH + 32 * (a ^ s_hi) + (((2 * e + half) ^ s_lo) << 3);
#pragma unroll
        for (int sec = 0; sec < 2; ++sec) {
            const int row = 8 * sec + 4 * half + (i >> 2);           // + 16 kk, which does not change the swizzle
            const int t = sw_both<DH>(row), t_hi = t >> 2, t_lo = t & 3;
            const int b = 2 * g + ((i & 3) >> 1);
#pragma unroll
            for (int c = 0; c < NG; ++c) tb[c][sec] = row * DH + 32 * (c ^ t_hi) + ((b ^ t_lo) << 3) + 4 * (i & 1);
        }
    }
    // MFMA first operand: row 32 u + lrow of the tile, k = 16 ks + 8 half + (0..7)
    template <class E> __device__ __forceinline__ x8<E> nat(const E *tile, int u, int ks) const {
        const int a = ks >> 1;
        return *reinterpret_cast<const x8<E> *>(tile + 32 * u * DH + nb[a % NG][ks & 1] + 32 * NG * (a / NG));
    }
    // MFMA first operand "row 32 c + lrow of the transposed tile, k element e <-> tile row 16 kk + 8 (e/4) + 4 half + e%4"
    template <class E> __device__ __forceinline__ x8<E> tr(const E *tile, int c, int kk) const {
        const uint32_t a0 = (uint32_t)(uintptr_t)(tile + tb[c % NG][0]);
        const uint32_t a1 = (uint32_t)(uintptr_t)(tile + tb[c % NG][1]);
        u32x2 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(a0), "i"((16 * kk * DH + 32 * NG * (c / NG)) * 2));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(a1), "i"((16 * kk * DH + 32 * NG * (c / NG)) * 2));
        const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
        return __builtin_bit_cast(x8<E>, v);
    }
};

// The same addresses as LDS byte addresses of tiles in one of two stages, moved from one stage to the other in place: one register
// each and nothing else, where the reads above keep the element offset beside the sum of it and the stage.
template <int DH, int STAGE_BYTES> struct BothStages {
    static constexpr int NG = BothAddr<DH>::NG;
    int nb[NG][2], tb[NG][2];
    __device__ __forceinline__ void init(const void *lds, int lane) {
        BothAddr<DH> ad;
        ad.init(lane);
        const int base = (int)(uintptr_t)(lds_ptr)lds;
#pragma unroll
        for (int a = 0; a < NG; ++a)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                nb[a][e] = base + 2 * ad.nb[a][e];
                tb[a][e] = base + 2 * ad.tb[a][e];
            }
    }
    // to the other stage; opaque, or the compiler goes back to a sum per tile
    __device__ __forceinline__ void move(bool up) {
        const int by = up ? STAGE_BYTES : -STAGE_BYTES;
#pragma unroll
        for (int a = 0; a < NG; ++a)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                nb[a][e] += by;
                tb[a][e] += by;
                asm volatile("" : "+v"(nb[a][e]), "+v"(tb[a][e]));
            }
    }
    // tile: byte offset of the tile in its stage
    template <class E> __device__ __forceinline__ x8<E> nat(int tile, int u, int ks) const {
        const int a = ks >> 1;
        typedef __attribute__((address_space(3))) const x8<E> *ptr;
        return *(ptr)(uintptr_t)(uint32_t)(nb[a % NG][ks & 1] + tile + (32 * u * DH + 32 * NG * (a / NG)) * 2);
    }
    template <class E> __device__ __forceinline__ x8<E> tr(int tile, int c, int kk) const {
        u32x2 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(tb[c % NG][0]), "i"(tile + (16 * kk * DH + 32 * NG * (c / NG)) * 2));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(tb[c % NG][1]), "i"(tile + (16 * kk * DH + 32 * NG * (c / NG)) * 2));
        const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
        return __builtin_bit_cast(x8<E>, v);
    }
};

// Row operands of a chain of products, read AHEAD k steps before they are multiplied and no further: left alone the compiler reads all
// of a tile's at once, and their registers push others into scratch memory.  load(ks, slot), multiply(ks, slot): slots
// 0 ... AHEAD + 1.
template <int NK, int AHEAD, class L, class M> __device__ __forceinline__ void products_ahead(L load, M multiply) {
    constexpr int SLOTS = AHEAD + 2;
#pragma unroll
    for (int ks = 0; ks < AHEAD && ks < NK; ++ks) load(ks, ks % SLOTS);
#pragma unroll
    for (int ks = 0; ks < NK; ks += 2) {
#pragma unroll
        for (int i = AHEAD; i < AHEAD + 2; ++i)
            if (ks + i < NK) load(ks + i, (ks + i) % SLOTS);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ks, ks % SLOTS);
        if (ks + 1 < NK) multiply(ks + 1, (ks + 1) % SLOTS);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Workgroup -> ((sequence, head), block rank) for a 1-D grid of n_seq * heads * nblocks workgroups, which the
// hardware hands out in index order.  With the causal mask a (sequence, head)'s blocks differ in length by up to
// the number of blocks: rank is the slow index, so every (sequence, head)'s longest block (rank 0) starts before
// anyone's second longest and the launch ends on the shortest ones.  Without the mask all blocks are equally
// long: rank is the fast index, so the blocks that stream the same keys and values run at the same time and
// share them in the caches.
__device__ __forceinline__ void block_of(const AttnShape &sh, int nblocks, int &bh, int &rank) {
    const int bhs = sh.n_seq * sh.heads;
    if (sh.causal) {
        bh = blockIdx.x % bhs;
        rank = blockIdx.x / bhs;
    } else {
        rank = blockIdx.x % nblocks;
        bh = blockIdx.x / nblocks;
    }
}

}  // namespace
}  // namespace lga
