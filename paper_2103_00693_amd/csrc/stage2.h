// Stage 2 of the two-stage scheme (the paper's classical parallel circuit,
// Section 2, Eqs. (1)-(3) and the final CNOT layer): device code shared by the
// single-instance and the batched kernels.
//
// Solution i is z_i = l ^ XOR_{bit k of g(i)} B_k with g(i) = i ^ (i >> 1).
// Writing E_j = B_j ^ B_{j-1} (B_{-1} = 0) turns this into an affine map of
// the bits of i itself:  z_i = l ^ F(i),  F(i) = XOR_{bit j of i} E_j.
// For an index split i = (T << S) | x with x < 2^S,
//     z_i = (l ^ F(x)) ^ F(T << S):
// a per-lane constant XOR a per-tile constant.  Moving from tile T to T+1
// changes the tile constant by F(((T+1) ^ T) << S) = B_{S-1} ^ B_{S+ctz(T+1)}
// (the sum telescopes): the Gray-code step lifted to whole tiles.
#pragma once

#include "hlf_device.h"
#include "hlf_internal.h"

namespace hlf {


// Status/range gate of every stage-2 kernel.  Returns false (and the caller
// writes nothing) if the record is bad or [begin, begin+count) is not inside
// [0, 2^r); the verdict is the same for every block.
__device__ __forceinline__ bool gate(int32_t *status, const int32_t *rank, uint64_t begin,
                                     uint64_t count, int &r) {
    if (*(volatile int32_t *)status != HLF_OK) return false;
    r = *rank;
    if (r > HLF_MAX_ENUM_RANK || begin > (1ull << r) || count > (1ull << r) - begin) {
        if (threadIdx.x == 0) *status = HLF_ERANGE;
        return false;
    }
    return true;
}

// Bx[j*WW + w] = word w of B_j for j < r, zero for r <= j < 64.
template <int WW>
__device__ __forceinline__ void load_basis_padded(const uint64_t *__restrict__ basis, int r,
                                                  uint64_t *Bx, int tid, int nthreads) {
    for (int idx = tid; idx < 64 * WW; idx += nthreads) {
        const int j = idx / WW;
        Bx[idx] = (j < r) ? basis[idx] : 0ull;
    }
}

template <int WW>
__device__ __forceinline__ uint64_t E_at(const uint64_t *Bx, int j, int w) {
    return Bx[j * WW + w] ^ (j ? Bx[(j - 1) * WW + w] : 0ull);
}

// Word w of F(x) for x < 2^bits.
template <int WW>
__device__ __forceinline__ uint64_t F_low(const uint64_t *Bx, uint64_t x, int bits, int w) {
    uint64_t v = 0;
    for (int j = 0; j < bits; ++j)
        if ((x >> j) & 1ull) v ^= E_at<WW>(Bx, j, w);
    return v;
}

// Word w of F(T << S).
template <int WW>
__device__ __forceinline__ uint64_t F_tile(const uint64_t *Bx, uint64_t T, int S, int w) {
    uint64_t v = 0;
    for (int j = 0; j + S < 64 && (T >> j); ++j)
        if ((T >> j) & 1ull) v ^= E_at<WW>(Bx, S + j, w);
    return v;
}

// Word w of the tile-constant step from T to T+1.
template <int WW>
__device__ __forceinline__ uint64_t tile_step(const uint64_t *Bx, uint64_t T, int S, int w) {
    const int c = S + __builtin_ctzll(T + 1);
    return Bx[(S - 1) * WW + w] ^ Bx[(c < 63 ? c : 63) * WW + w];
}

// ---------------------------------------------------------------------------
// Materialise, W = 1, 16/32/64-bit words: V values per 16-byte store.
// ---------------------------------------------------------------------------
template <typename T>
struct Vec {
    static constexpr int V = 16 / (int)sizeof(T);  // values per 16-byte store
    static constexpr int LOGV = (V == 8) ? 3 : (V == 4) ? 2 : 1;
};

// Workgroups of the one-launch solve kernels and of the multi-word circuit:
// 1024 threads; the solve's write one 16-byte store per thread per tile, so a
// tile holds 1024*V solutions.
constexpr int kTileThreads = 1024;
constexpr int kLogTileThreads = 10;
// Workgroups per CU of the one-launch solve kernel (more workgroups than
// resident slots: the dispatcher balances the tail).
constexpr int kTileBlocksPerCU = 16;
// The kernels whose workgroups factor or build tables first (the one-launch
// solve outside its one-generation sizes, the multi-word circuit) give each
// workgroup a short contiguous range of about kBlockBytes of output, and a
// launch holds many more workgroups than fit on the device, so the resident
// ones are at different points of their ranges (resident workgroups that write
// in step at a fixed stride lose 5-15% of the write bandwidth).  Longer ranges
// only for grids beyond kMaxTileBlocks.
constexpr uint64_t kBlockBytes = 128ull << 10;
constexpr uint64_t kMaxTileBlocks = 1ull << 30;

// Tiles per workgroup for such a launch over ntiles tiles of tile_bytes bytes
// each; a launch too small to give every CU two workgroups
// at that size is spread thinner.
inline uint64_t materialise_tiles_per_block(uint64_t ntiles, uint64_t tile_bytes) {
    uint64_t want = kBlockBytes / tile_bytes ? kBlockBytes / tile_bytes : 1;
    const uint64_t spread = 2ull * (uint64_t)device_cu_count();
    const uint64_t thin = (ntiles + spread - 1) / spread;
    if (thin < want) want = thin ? thin : 1;
    const uint64_t need = (ntiles + kMaxTileBlocks - 1) / kMaxTileBlocks;
    return need > want ? need : want;
}

// Bytes of one tile of the one-launch solve kernels (one 16-byte store per
// thread).
constexpr uint64_t kTileBytes = 16ull * kTileThreads;
// Grids up to this many workgroups seed their lane constants the short way.
constexpr unsigned kShortSeedGrid = 512;

// Workgroups are dealt to the 8 XCDs in turn, so dispatch index b runs on XCD
// b % 8.  xcd_block maps b (of n) to the block index it materialises such that
// each XCD's workgroups take one contiguous run of blocks, in order: XCD x
// takes the q or q + 1 blocks from x*q + min(x, n % 8) on, q = n / 8.  Stores
// from one XCD then stay in one region instead of interleaving with the other
// seven XCDs' every workgroup, which the HBM write rate favours.
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t n) {
    const uint32_t x = b & 7u, q = n >> 3, rem = n & 7u;
    return x * q + (x < rem ? x : rem) + (b >> 3);
}

template <typename T>
__host__ __device__ constexpr int tile_shift() {
    return kLogTileThreads + Vec<T>::LOGV;
}

template <typename T>
__device__ __forceinline__ void pack16(const uint64_t *v, uint32_t (&w)[4]) {
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            w[k] = (uint32_t)(v[2 * k] & 0xFFFFu) | ((uint32_t)v[2 * k + 1] << 16);
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = (uint32_t)v[k];
    } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            w[2 * k] = (uint32_t)v[k];
            w[2 * k + 1] = (uint32_t)(v[k] >> 32);
        }
    }
}

template <typename T>
__device__ __forceinline__ void spread16(uint64_t h, uint32_t (&w)[4]) {
    if constexpr (sizeof(T) == 2) {
        const uint32_t x = (uint32_t)(h & 0xFFFFu) * 0x10001u;
        w[0] = w[1] = w[2] = w[3] = x;
    } else if constexpr (sizeof(T) == 4) {
        w[0] = w[1] = w[2] = w[3] = (uint32_t)h;
    } else {
        w[0] = w[2] = (uint32_t)h;
        w[1] = w[3] = (uint32_t)(h >> 32);
    }
}

// Tiles [t0, t1) (relative to the first tile of [begin, begin+count)) of one
// instance, by a kTileThreads workgroup; out[i - begin] = z_i.  Stores are
// nontemporal where workgroups start one behind the other (a solve of eight
// instances: 137 us, 155 with plain ones) and plain where one generation of
// them writes it all (solve.hip).  Requires
// begin % V == 0 and a 16-byte aligned `out`.  Bx: LDS basis (WW = 1).
template <typename T, bool kPlain>
__device__ void enum_tiles_w1(const uint64_t *Bx, uint64_t l, uint64_t begin, uint64_t count,
                              T *__restrict__ out, uint64_t t0, uint64_t t1) {
    constexpr int V = Vec<T>::V;
    constexpr int S = tile_shift<T>();
    constexpr int LOGV = Vec<T>::LOGV;
    const int tid = threadIdx.x;
    // Lane constants l ^ F(tid*V + e).  F is linear in the bits of the index,
    // so F(tid*V + e) = F(tid << LOGV) ^ F(e): about LOGV + 10 lookups instead
    // of V * S.  The workgroups that start with the launch (all of a launch
    // that fits on the device at once) take the short form: their start-up
    // is the launch's ramp.  The later ones keep the per-index form, whose
    // longer start-up spreads their first stores (measured about 1% faster
    // than the short form everywhere).
    uint64_t lo[V];
    if (gridDim.x <= kShortSeedGrid || blockIdx.x < kShortSeedGrid) {
        uint64_t base = l;
#pragma unroll
        for (int j = 0; j < kLogTileThreads; ++j)
            if ((tid >> j) & 1) base ^= E_at<1>(Bx, LOGV + j, 0);
#pragma unroll
        for (int e = 0; e < V; ++e) lo[e] = base ^ F_low<1>(Bx, (uint64_t)e, LOGV, 0);
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) lo[e] = l ^ F_low<1>(Bx, (uint64_t)(tid * V + e), S, 0);
    }
    uint32_t lw[4];
    pack16<T>(lo, lw);

    const uint64_t end = begin + count;
    uint64_t Tt = (begin >> S) + t0;
    uint64_t hi = F_tile<1>(Bx, Tt, S, 0);
    for (uint64_t t = t0; t < t1; ++t, ++Tt) {
        const uint64_t i0 = (Tt << S) + (uint64_t)(tid * V);
        if (i0 >= begin && i0 + V <= end) {
            uint32_t hw[4];
            spread16<T>(hi, hw);
            u32x4 val;
            val.x = lw[0] ^ hw[0];
            val.y = lw[1] ^ hw[1];
            val.z = lw[2] ^ hw[2];
            val.w = lw[3] ^ hw[3];
            if constexpr (kPlain) *(u32x4 *)(out + (i0 - begin)) = val;
            else __builtin_nontemporal_store(val, (u32x4 *)(out + (i0 - begin)));
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const uint64_t i = i0 + e;
                if (i >= begin && i < end) out[i - begin] = (T)(lo[e] ^ hi);
            }
        }
        hi ^= tile_step<1>(Bx, Tt, S, 0);
    }
}

// ---------------------------------------------------------------------------
// Materialise, one 16-byte store per thread (the kernels that only write).
//
// Bound by HBM writes, and what decides their rate here is the order in which
// the addresses are written.  Plain store kernels on this card: one store per
// thread and 4 KiB per 256-thread workgroup 6.9 TB/s (512 MiB and 1 GiB), two
// stores per thread 6.6, four 6.0, 128 KiB per 1024-thread workgroup 5.7,
// resident workgroups that stride over the range at most 6.2, and nontemporal
// stores 2-4% below plain ones (15% at 128 MiB).  So a workgroup writes one
// tile of 4 KiB, and the set-up of a wave has to fit beside it: at that rate
// a SIMD starts a wave every 350 cycles, about 85 scalar and as many vector
// instructions, and holds at most eight.  Solution i is l ^ XOR of the B_j
// over the bits j of c(i), c(i) = i ^ (i >> 1) in Gray order and i in counter
// order, both linear.  A wave takes no LDS and no barrier: the rows for the
// index bits inside its run of 64 V solutions are scalar loads, applied per
// lane under the lane's bits; the others are loaded one per lane, kept where
// c of the run's first index has that bit (the mask is the select), and XORed
// across the wave by DPP.
//
// A run that begins anywhere is cut at multiples of V by index, so its
// 16-byte stores may be misaligned in memory, which costs nothing measurable
// as long as each XCD writes one contiguous run (xcd_block): dealt in turn,
// misaligned tiles straddle two XCDs' pages and drop to 4.8 TB/s.
//
// These rates hold from idle for about 1.5 ms and again from about 30 ms on;
// between, the card's power regulation holds back writes of changing data
// (the same launches writing one value dip to 6.2 TB/s only).  Calls of 8 GiB:
// 7.4 TB/s at first, 4.9 at 3 to 4 ms, 5.8 at 8 to 12, 7.1 to 7.2 from 32 on;
// with 128 KiB per workgroup, nontemporal, 5.8 to 6.2 throughout.  The longer
// form gains 7% over bursts of 3 to 20 ms from idle and loses up to 23% on
// shorter and longer ones, whatever the size of a call, so no rule takes it.
// ---------------------------------------------------------------------------
constexpr int kVecThreads = 256;
constexpr int kLogVecThreads = 8;
// A launch has at most 2^31 threads; longer ranges take more tiles each.
constexpr uint64_t kMaxVecBlocks = 1ull << 23;

// Stores at any address: the output of a call may lie at any byte.
typedef u32x4 u32x4_any __attribute__((aligned(1)));
template <typename T>
struct AnyAddress {
    typedef T type __attribute__((aligned(1)));
};

template <typename T>
struct VecTile {
    static constexpr int V = Vec<T>::V;
    static constexpr int LOGV = Vec<T>::LOGV;
    static constexpr int ND = sizeof(T) == 8 ? 2 : 1;        // dwords per constant
    static constexpr int LB = LOGV + 6;                      // index bits inside a wave's run
    static constexpr int S = LOGV + kLogVecThreads;          // log2 solutions per tile
};

// Where a range of solutions goes, worked out on the host.
struct VecRange {
    uint64_t begin, end;      // indices; end < begin for a range that wraps
    char *tile0;              // address of tile 0's first index (at or before the output)
    uint32_t ntiles;          // 0: nothing but the device gate (see vec_range)
    uint32_t full0, full1;    // tiles full0 <= t < full1 lie inside the range
};

// ntiles is 0 for a range that wraps, or that no memory holds (2^31 tiles are
// 8 TiB): the launch then runs the gate alone.
template <typename T>
inline VecRange vec_range(uint64_t begin, uint64_t count, void *out) {
    constexpr int S = VecTile<T>::S;
    constexpr uint64_t M = (1ull << S) - 1;
    VecRange g{};
    g.begin = begin;
    g.end = begin + count;
    g.tile0 = static_cast<char *>(out) - (begin & M) * sizeof(T);
    if (count == 0 || g.end < begin) return g;
    const uint64_t t = ((g.end - 1) >> S) - (begin >> S) + 1;
    if (t >> 31) return g;
    g.ntiles = (uint32_t)t;
    g.full0 = (begin & M) ? 1u : 0u;
    g.full1 = (uint32_t)((g.end - (begin & ~M)) >> S);
    return g;
}

// Tiles per workgroup for ntiles tiles: 1 up to kMaxVecBlocks of them.
inline uint32_t vec_tiles_per_block(uint64_t ntiles) {
    return ntiles ? (uint32_t)((ntiles + kMaxVecBlocks - 1) / kMaxVecBlocks) : 1u;
}

// A word as the dwords that the stores are made of (16-bit words twice).
template <typename T>
__device__ __forceinline__ void vec_dwords(uint64_t e, uint32_t (&d)[VecTile<T>::ND]) {
    if constexpr (sizeof(T) == 8) {
        d[0] = (uint32_t)e;
        d[1] = (uint32_t)(e >> 32);
    } else if constexpr (sizeof(T) == 4) {
        d[0] = (uint32_t)e;
    } else {
        d[0] = (uint32_t)(e & 0xFFFFu) * 0x10001u;
    }
}

// XOR of the wave's values, wave-uniform, by DPP row shifts and a row
// broadcast.  A pair of dwords first folds onto one register: one swap of the
// lane halves leaves the low dwords' XORs in lanes 0..31 and the high ones'
// in lanes 32..63.
__device__ __forceinline__ uint32_t dpp_half_xor(uint32_t v) {
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);  // row_shr 1, 2, 4, 8
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // lane 15 to the next row
    return v;  // lanes 31 and 63: the XORs of their halves
}

template <int ND>
__device__ __forceinline__ void wave_xor_dwords(uint32_t (&d)[ND]) {
    if constexpr (ND == 1) {
        const uint32_t v = dpp_half_xor(d[0]);
        d[0] = (uint32_t)__builtin_amdgcn_readlane((int)v, 31) ^ (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    } else {
        const auto sw = __builtin_amdgcn_permlane32_swap(d[0], d[1], false, false);
        const uint32_t v = dpp_half_xor(sw[0] ^ sw[1]);
        d[0] = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
        d[1] = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    }
}

// This thread's V solutions i0 .. i0 + V - 1 of tile t, as dwords w.
template <typename T>
__device__ __forceinline__ void vec_put(const VecRange &g, uint32_t t, uint64_t i0, const uint32_t (&w)[4]) {
    char *base = g.tile0 + ((uint64_t)t << 12);
    const uint32_t off = 16u * threadIdx.x;
    if (t >= g.full0 && t < g.full1) {  // workgroup-uniform
        const u32x4 val = {w[0], w[1], w[2], w[3]};
        *reinterpret_cast<u32x4_any *>(base + off) = val;
    } else {
        typename AnyAddress<T>::type *o = reinterpret_cast<typename AnyAddress<T>::type *>(base + off);
#pragma unroll
        for (int e = 0; e < VecTile<T>::V; ++e) {
            if (i0 + e >= g.begin && i0 + e < g.end) {
                if constexpr (sizeof(T) == 2) o[e] = (T)(w[e >> 1] >> (16 * (e & 1)));
                else if constexpr (sizeof(T) == 4) o[e] = (T)w[e];
                else o[e] = ((uint64_t)w[2 * e + 1] << 32) | w[2 * e];
            }
        }
    }
}

// Lane part of a linear map of the index: XOR of the rows low[j] over the bits
// j < LB of c(lane * V) (see above; bit LOGV + 5 of c also takes bit LOGV + 6
// of the index, which is in the run's constant).
template <typename T, bool kCounter>
__device__ __forceinline__ void vec_lane_part(const uint64_t (&low)[VecTile<T>::LB], uint32_t x,
                                              uint32_t (&lo)[VecTile<T>::ND]) {
    constexpr int LOGV = VecTile<T>::LOGV, ND = VecTile<T>::ND;
    constexpr int J0 = kCounter ? LOGV : LOGV - 1;
    const uint32_t cx = kCounter ? x : x ^ (x >> 1);
#pragma unroll
    for (int j = J0; j < VecTile<T>::LB; ++j) {
        const uint32_t m = (uint32_t)((int)(cx << (31 - j)) >> 31);
        uint32_t e[ND];
        vec_dwords<T>(low[j], e);
#pragma unroll
        for (int q = 0; q < ND; ++q)  // lo ^ (m & e)
            lo[q] = j == J0 ? m & e[q] : __builtin_amdgcn_bitop3_b32(lo[q], m, e[q], 0x78);
    }
}

// F(e) for a value's place e < V within the store.
template <typename T, bool kCounter>
__device__ __forceinline__ void vec_place(const uint64_t (&low)[VecTile<T>::LB], int e,
                                          uint32_t (&f)[VecTile<T>::ND]) {
    const int c = kCounter ? e : e ^ (e >> 1);
    uint64_t v = 0;
#pragma unroll
    for (int j = 0; j < VecTile<T>::LOGV; ++j)
        if ((c >> j) & 1) v ^= low[j];
    vec_dwords<T>(v, f);
}

// The V values of a store: lane part, run constant and places together.
template <typename T>
__device__ __forceinline__ void vec_values(const uint32_t (&lo)[VecTile<T>::ND], const uint32_t (&h)[VecTile<T>::ND],
                                           const uint32_t (&f)[VecTile<T>::V][VecTile<T>::ND], uint32_t (&w)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if constexpr (sizeof(T) == 2)
            w[k] = lo[0] ^ (h[0] ^ ((f[2 * k][0] & 0xFFFFu) | (f[2 * k + 1][0] & 0xFFFF0000u)));
        else if constexpr (sizeof(T) == 4)
            w[k] = lo[0] ^ (h[0] ^ f[k][0]);
        else
            w[k] = lo[k & 1] ^ (h[k & 1] ^ f[k >> 1][k & 1]);
    }
}

// The gate on a record, for kernels that read it with plain loads: the rank r
// of a good record and a range inside [0, 2^r).
__device__ __forceinline__ bool vec_gate(int32_t *status, int32_t st, int32_t r, const VecRange &g) {
    if (st != HLF_OK) return false;
    if (r > HLF_MAX_ENUM_RANK || g.end < g.begin || (g.end - 1) >> r) {
        if (threadIdx.x == 0) *status = HLF_ERANGE;
        return false;
    }
    return true;
}

// Tiles [t0, t1) of a range, one store per thread and tile.  The basis array
// has n rows, all loaded at once with the status and the rank: rows past r
// meet no bit (indices are below 2^r, and so is c of them).
template <typename T, bool kCounter>
__device__ __forceinline__ void vec_materialise(int32_t *status, const int32_t *__restrict__ rank,
                                                const uint64_t *__restrict__ basis,
                                                const uint64_t *__restrict__ shift, int n, const VecRange &g,
                                                uint32_t t0, uint32_t t1) {
    using X = VecTile<T>;
    constexpr int V = X::V, LOGV = X::LOGV, ND = X::ND, LB = X::LB;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t rows = (uint32_t)n;
    const uint64_t own = basis[lane < rows ? lane : rows - 1u];
    const int32_t st = *status, r = *rank;
    const uint64_t l = shift[0];
    uint64_t low[LB];
    if (n >= LB) {
#pragma unroll
        for (int j = 0; j < LB; ++j) low[j] = basis[j];
    } else {
#pragma unroll
        for (int j = 0; j < LB; ++j) low[j] = basis[j < n ? j : n - 1];
    }
    // Every load is under way before the first branch on one of them.
    asm volatile("" ::"s"(g.begin), "s"(g.end), "s"(g.tile0), "s"(g.full1), "s"(l), "s"(r), "s"(st), "s"(low[0]),
                 "s"(t0), "s"(t1));
    if (!vec_gate(status, st, r, g)) return;
    uint32_t le[ND], ls[ND], lo[ND], f[V][ND];
    vec_dwords<T>(own, le);
    vec_dwords<T>(l, ls);
    const uint32_t x = lane << LOGV;
    vec_lane_part<T, kCounter>(low, x, lo);
#pragma unroll
    for (int e = 0; e < V; ++e) vec_place<T, kCounter>(low, e, f[e]);
    const uint64_t first = g.begin & ~((1ull << X::S) - 1);
    for (uint32_t t = t0; t < t1; ++t) {
        // the wave's run begins at index iu: its constant l ^ F(iu)
        const uint64_t iu = first + ((uint64_t)t << X::S) + (wave << LB);
        const bool on = __builtin_amdgcn_inverse_ballot_w64(kCounter ? iu : iu ^ (iu >> 1));
        uint32_t h[ND];
#pragma unroll
        for (int q = 0; q < ND; ++q) h[q] = on ? le[q] : 0u;
        wave_xor_dwords<ND>(h);
#pragma unroll
        for (int q = 0; q < ND; ++q) h[q] ^= ls[q];
        uint32_t w[4];
        vec_values<T>(lo, h, f, w);
        vec_put<T>(g, t, iu + x, w);
    }
}

// ---------------------------------------------------------------------------
// Reduce.  Per-qubit counts and the XOR-fold of a range follow in closed form
// (range_count below), so only the hash visits the solutions: one wavefront
// per contiguous range of indices, tiles of 64 U of them.  A whole tile's
// solutions are the coset z(T << S) ^ span(B_0 .. B_{S-1}), whichever member
// of it represents the tile, so from tile T to T + 1 the representative
// changes by B_{S + ctz(T + 1)} alone.
//
// Bound by VALU issue.  The loop body is 17 instructions per solution word
// (the first word's first step is GF(2)-linear and is applied once per lane
// constant and once per tile): two XORs with the tile's constant in scalar
// registers, two 64-bit products of four, two shifts, four XORs, one 64-bit
// add; from the second word on, two three-input XORs, a shift and two XORs
// more.  Everything per tile is scalar, which the vector unit does not wait
// for.  A product is written so that it ends in a two-operand add, which two
// waves can issue at once where the compiler's three-operand add takes the
// unit for itself: 2.44 against 2.33 T hashes/s in a loop of one-word hashes
// alone (17 instructions at the issue peak are 2.31).
// ---------------------------------------------------------------------------
template <int WW>
struct WaveHash {
    // lane constants: 2 U WW registers
    static constexpr int LOGU = WW == 1 ? 4 : WW <= 3 ? 3 : WW <= 7 ? 2 : 0;
    static constexpr int U = 1 << LOGU;
    static constexpr int S = 6 + LOGU;
};

__device__ __forceinline__ uint64_t mul_hash(uint64_t x, uint64_t c) {
    const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32), cl = (uint32_t)c, ch = (uint32_t)(c >> 32);
    const uint64_t p = (uint64_t)lo * cl + ((uint64_t)(lo * ch) << 32);
    const uint32_t b = hi * cl, ph = (uint32_t)(p >> 32);
    uint32_t r;
    asm("v_add_u32_e32 %0, %1, %2" : "=v"(r) : "v"(ph), "v"(b));
    return ((uint64_t)r << 32) | (uint32_t)p;
}

// mix13 after its first step x ^= x >> 30.
__device__ __forceinline__ uint64_t hash_tail(uint64_t x) {
    x = mul_hash(x, 0xBF58476D1CE4E5B9ull);
    x ^= x >> 27;
    x = mul_hash(x, 0x94D049BB133111EBull);
    return x ^ (x >> 31);
}

// Lane k of a wave holds B_k, k < r (zero from r on).
template <int WW>
struct WaveRows {
    uint32_t d[2 * WW];
};

template <int WW>
__device__ __forceinline__ WaveRows<WW> wave_rows(const uint64_t *basis, int r) {
    WaveRows<WW> b;
    const int lane = lane_id();
#pragma unroll
    for (int w = 0; w < WW; ++w) {
        const uint64_t v = lane < r ? basis[(size_t)lane * WW + w] : 0ull;
        b.d[2 * w] = (uint32_t)v;
        b.d[2 * w + 1] = (uint32_t)(v >> 32);
    }
    return b;
}

template <int WW>
__device__ __forceinline__ uint64_t row_word(const WaveRows<WW> &b, int k, int w) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)b.d[2 * w], k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)b.d[2 * w + 1], k);
    return ((uint64_t)hi << 32) | lo;
}

// This lane's share of the sum of h(z_i), i in [c0, c1) (c0 < c1 <= 2^r, both
// wave-uniform).  l: the shift, wave-uniform.  next_row(k, row): word w of
// B_k to row[w], k wave-uniform.
template <int WW, typename NextRow>
__device__ __forceinline__ uint64_t wave_hash_range(const WaveRows<WW> &b, const uint64_t (&l)[WW], uint64_t c0,
                                                    uint64_t c1, NextRow next_row) {
    constexpr int U = WaveHash<WW>::U, LOGU = WaveHash<WW>::LOGU, S = WaveHash<WW>::S;
    constexpr uint64_t M = (1ull << S) - 1;
    const uint32_t lane = (uint32_t)lane_id();
    // Lane constants F(64 u + lane): the lane's part, and for u the rows at
    // the bits of c(64 u) = g(u) << 6, with bit 5 for odd u.
    uint64_t lo[U][WW];
    const uint32_t cx = lane ^ (lane >> 1);
#pragma unroll
    for (int w = 0; w < WW; ++w) {
        uint32_t v0 = 0, v1 = 0;
        uint64_t row5 = 0;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const uint64_t e = row_word<WW>(b, j, w);
            const uint32_t m = (uint32_t)((int)(cx << (31 - j)) >> 31);
            v0 ^= m & (uint32_t)e;
            v1 ^= m & (uint32_t)(e >> 32);
            row5 = e;
        }
        uint64_t rows[LOGU + 1];
#pragma unroll
        for (int j = 0; j < LOGU; ++j) rows[j] = row_word<WW>(b, 6 + j, w);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint64_t f = (u & 1) ? row5 : 0ull;
#pragma unroll
            for (int j = 0; j < LOGU; ++j)
                if (((u ^ (u >> 1)) >> j) & 1) f ^= rows[j];
            lo[u][w] = (((uint64_t)v1 << 32) | v0) ^ f;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) lo[u][0] = mix13_head(lo[u][0]);

    uint64_t T = c0 >> S;
    const uint64_t Tend = ((c1 - 1) >> S) + 1;
    const uint64_t full0 = (c0 + M) >> S, full1 = c1 >> S;
    // Tile constant l ^ gamma ^ F(T << S) without its bit S - 1.
    uint64_t hi[WW];
    const bool on = __builtin_amdgcn_inverse_ballot_w64((T ^ (T >> 1)) << S);
#pragma unroll
    for (int w = 0; w < WW; ++w) {
        uint32_t h[2] = {on ? b.d[2 * w] : 0u, on ? b.d[2 * w + 1] : 0u};
        wave_xor_dwords<2>(h);
        hi[w] = l[w] ^ kGamma ^ (((uint64_t)h[1] << 32) | h[0]);
    }
    uint64_t acc = 0;
    for (;;) {
        const bool more = T + 1 < Tend;
        uint64_t row[WW];
        if (more) next_row(S + __builtin_ctzll(T + 1), row);
        const uint64_t h0 = mix13_head(hi[0]);
        auto hash_of = [&](int u) {
            uint64_t h = hash_tail(lo[u][0] ^ h0);
#pragma unroll
            for (int w = 1; w < WW; ++w) h = hash_tail(mix13_head(h ^ lo[u][w] ^ hi[w]));
            return h;
        };
        if (U > 1 && T >= full0 && T < full1) {
#pragma unroll
            for (int u = 0; u < U; ++u) acc += hash_of(u);
        } else {
            // The first or last tile of the range, by its indices: the
            // representative leaves out bit S - 1 of g(T << S), which for odd
            // T puts index M - x of the tile in the place of x.  (With many
            // words the comparisons cost less than a second copy of the body.)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t x = (uint64_t)(64 * u) + lane, i = (T << S) + ((T & 1ull) ? M - x : x);
                const uint64_t h = hash_of(u);
                acc += (i >= c0 && i < c1) ? h : 0ull;
            }
        }
        if (!more) break;
#pragma unroll
        for (int w = 0; w < WW; ++w) hi[w] ^= row[w];
        ++T;
    }
    return acc;
}

// Bit j of every solution of [begin, end) (begin < end <= 2^r): how many have
// it set, and the parity of that for the XOR-fold.  col: bit k is B_k[j]; lj =
// l[j].  The range is cut into aligned blocks of 2^K indices, each a coset
// z(a) ^ span(B_0 .. B_{K-1}): the bit is set in half of it if some B_k, k < K,
// has it, else in all or none as in z(a).
__device__ __forceinline__ uint64_t range_count(uint64_t col, uint32_t lj, uint64_t begin, uint64_t end,
                                                uint32_t &odd) {
    uint64_t count = 0;
    odd = 0;
    for (uint64_t a = begin; a < end;) {
        const int up = a ? __builtin_ctzll(a) : 63, fit = 63 - __builtin_clzll(end - a);
        const int K = up < fit ? up : fit;
        const uint64_t size = 1ull << K;
        const uint32_t z = lj ^ ((uint32_t)__builtin_popcountll(col & (a ^ (a >> 1))) & 1u);
        const uint64_t c = (col & (size - 1)) ? size >> 1 : z ? size : 0ull;
        count += c;
        odd ^= (uint32_t)c & 1u;
        a += size;
    }
    return count;
}

}  // namespace hlf
