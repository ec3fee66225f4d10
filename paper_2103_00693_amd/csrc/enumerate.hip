// Single-instance stage-2 kernels (materialise and reduce) for gfx950; the
// tile algebra they share with the batched kernels is in stage2.h.
//
//   enum_tile_kernel<T>     W = 1, 16/32/64-bit words, any begin and address:
//                           one 16-byte store per thread (stage2.h).
//   enum_wide_tile_kernel   W > 1: the same 16-byte pieces of every tile of its
//                           workgroup per thread.
//   enum_general_kernel     W > 1 at an address that is not a multiple of 8:
//                           z_i from LDS lookup tables over the nibbles of i
//                           (method of four Russians).
//   circuit_tile_kernel<T>  the paper's circuit, W = 1; circuit_wide_kernel W > 1.
//   reduce_kernel<W>        counts and XOR-fold in closed form, the hash on
//                           wavefronts that take contiguous tile ranges.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "hlf_device.h"
#include "hlf_internal.h"
#include "stage2.h"

namespace hlf {
namespace {

__device__ __forceinline__ bool gate(const FactorIn &f, uint64_t begin, uint64_t count, int &r) {
    return hlf::gate(f.status, f.rank, begin, count, r);
}

template <typename T, bool kCounter>
__global__ __launch_bounds__(kVecThreads) void enum_tile_kernel(FactorIn f, VecRange g, uint32_t blocks,
                                                                uint32_t tiles_per_block) {
    const uint32_t t0 = xcd_block(blockIdx.x, blocks) * tiles_per_block;
    const uint32_t t1 = t0 + tiles_per_block < g.ntiles ? t0 + tiles_per_block : g.ntiles;
    vec_materialise<T, kCounter>(f.status, f.rank, f.basis, f.shift, f.n, g, t0, t1);
}

// ---------------------------------------------------------------------------
// Materialise, W > 1 words per solution: the output is one run of words, a tile
// of 2^S consecutive solutions 64 W words or a power of two times that, and a
// thread writes the same one or two 16-byte pieces of every tile of its
// workgroup: l ^ F(slot) of their words in registers, F(T << S) stepped from
// tile to tile.  An odd W lets a piece straddle two solutions.
//
// Bound by HBM writes, and like the one-word kernels (stage2.h) by their order
// and by a wave's set-up, here some 20 reads of LDS per piece, beside it.
// 268 MB of 2 words 40.6 us (6.6 TB/s), 403 MB of 6 words 70, 369 MB of 11
// words 65, 1 GiB of 16 words 179 (6.0 TB/s); with one 8-byte nontemporal
// store per word, the lanes of a power of two of words per solution and 256 KiB
// per workgroup: 59, 80, 96, 182.  Counter order takes the same set-up: tables
// of prefix sums for it, six exchanges per word, cost 33 MB of 16 words 15 us
// (9.5 now).
// ---------------------------------------------------------------------------
template <int W>
struct WideTile {
    static constexpr int S = W <= 4 ? 8 : W <= 8 ? 7 : 6;  // log2 solutions per tile
    static constexpr int kPieces = (W << S) / 2;           // at most 512
    static constexpr int kPer = (kPieces + kVecThreads - 1) / kVecThreads;
    static constexpr uint64_t kBytes = 8ull * W << S;
};

template <int W, bool kCounter>
__global__ __launch_bounds__(kVecThreads) void enum_wide_tile_kernel(FactorIn f, uint64_t begin, uint64_t count,
                                                                     uint64_t *__restrict__ out,
                                                                     uint64_t tiles_per_block) {
    using Tile = WideTile<W>;
    constexpr int S = Tile::S;
    __shared__ __align__(16) uint64_t Bx[64 * W];
    // All arguments in one wait, not the last ones behind the barrier.
    asm volatile("" ::"s"(f.shift), "s"(begin), "s"(count), "s"(out), "s"(tiles_per_block));
    int r;
    if (!gate(f, begin, count, r)) return;
    load_basis_padded<W>(f.basis, r, Bx, threadIdx.x, kVecThreads);
    __syncthreads();
    const uint64_t end = begin + count;
    const uint64_t ntiles = ((end - 1) >> S) - (begin >> S) + 1;
    const uint64_t t0 = (uint64_t)xcd_block(blockIdx.x, gridDim.x) * tiles_per_block;
    if (t0 >= ntiles) return;
    const uint64_t t1 = (t0 + tiles_per_block < ntiles) ? t0 + tiles_per_block : ntiles;
    uint64_t Tt = (begin >> S) + t0;
    // l ^ F(i) of a piece's words is l ^ the B_j over the bits j of i ^ (i >> 1),
    // or of i itself in counter order.
    int slot[Tile::kPer][2], w[Tile::kPer][2];
    uint64_t z[Tile::kPer][2];  // the words of tile Tt
    auto add = [&](int j, uint64_t mask0, uint64_t mask1, int k) {
        if constexpr (W % 2 == 0) {  // two words of one solution, side by side
            const ulonglong2 b = *reinterpret_cast<const ulonglong2 *>(&Bx[j * W + w[k][0]]);
            z[k][0] ^= b.x & mask0;
            z[k][1] ^= b.y & mask1;
        } else {
            z[k][0] ^= Bx[j * W + w[k][0]] & mask0;
            z[k][1] ^= Bx[j * W + w[k][1]] & mask1;
        }
    };
#pragma unroll
    for (int k = 0; k < Tile::kPer; ++k) {
        uint64_t gray[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = 2 * ((int)threadIdx.x + k * kVecThreads) + h;
            slot[k][h] = e / W;
            w[k][h] = e - slot[k][h] * W;
            z[k][h] = f.shift[w[k][h]];
            gray[h] = (uint64_t)(kCounter ? slot[k][h] : slot[k][h] ^ (slot[k][h] >> 1));
        }
#pragma unroll
        for (int j = 0; j < S; ++j) add(j, 0ull - ((gray[0] >> j) & 1), 0ull - ((gray[1] >> j) & 1), k);
    }
    for (uint64_t g = (Tt << S) ^ (kCounter ? 0ull : Tt << S >> 1); g; g &= g - 1) {  // Tt < 2^(62 - S)
        const int j = __builtin_ctzll(g);
#pragma unroll
        for (int k = 0; k < Tile::kPer; ++k) add(j, ~0ull, ~0ull, k);
    }
    for (uint64_t t = t0; t < t1; ++t, ++Tt) {
        const uint64_t base = Tt << S;
        uint64_t *o = out + ((int64_t)base - (int64_t)begin) * W;
        if (base >= begin && base + (1u << S) <= end) {
#pragma unroll
            for (int k = 0; k < Tile::kPer; ++k) {
                const int piece = (int)threadIdx.x + k * kVecThreads;
                if (Tile::kPieces % kVecThreads != 0 && piece >= Tile::kPieces) break;
                const u32x4 v = {(uint32_t)z[k][0], (uint32_t)(z[k][0] >> 32), (uint32_t)z[k][1],
                                 (uint32_t)(z[k][1] >> 32)};
                *reinterpret_cast<u32x4_any *>(o + 2 * piece) = v;
            }
        } else {
#pragma unroll
            for (int k = 0; k < Tile::kPer; ++k) {
                const int piece = (int)threadIdx.x + k * kVecThreads;
                if (piece >= Tile::kPieces) break;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint64_t i = base + (uint64_t)slot[k][h];
                    if (i >= begin && i < end) o[2 * piece + h] = z[k][h];
                }
            }
        }
        if (t + 1 == t1) break;
        // The step to the next tile: rows S - 1 and c in Gray order, the rows of
        // the carry, S to c, in counter order (two of them on average).
        const int c = min(S + __builtin_ctzll(Tt + 1), 63);
        if constexpr (kCounter) {
            for (int j = S; j < c; ++j) {
#pragma unroll
                for (int k = 0; k < Tile::kPer; ++k) add(j, ~0ull, ~0ull, k);
            }
        }
#pragma unroll
        for (int k = 0; k < Tile::kPer; ++k) {
            if constexpr (!kCounter) add(S - 1, ~0ull, ~0ull, k);
            add(c, ~0ull, ~0ull, k);
        }
    }
}

// ---------------------------------------------------------------------------
// W > 1 words at an address that is not a multiple of 8: z_i = l ^ XOR_m
// Tab[m][digit m of i], 16 nibble tables of 16 entries of W words (<= 32 KiB).
// ---------------------------------------------------------------------------
template <int WMAX>
struct GenTables {
    static constexpr int kDigitBits = 4;
    static constexpr int kDigits = 64 / kDigitBits;
    static constexpr int kEntries = 1 << kDigitBits;
    uint64_t tab[kDigits * kEntries * WMAX];
    uint64_t l[WMAX];
};

// Build tables from E_j = B_j ^ B_{j-1} (Gray order) or E_j = B_j (counter
// order); returns the number of digits in use.
template <int WMAX>
__device__ int build_tables(const FactorIn &f, int r, int W, bool counter, GenTables<WMAX> &g) {
    using G = GenTables<WMAX>;
    const int ndig = (r + G::kDigitBits - 1) / G::kDigitBits;
    for (int idx = threadIdx.x; idx < ndig * G::kEntries; idx += blockDim.x) {
        const int m = idx / G::kEntries, v = idx - m * G::kEntries;
        for (int w = 0; w < W; ++w) {
            uint64_t acc = 0;
            for (int q = 0; q < G::kDigitBits; ++q) {
                const int j = m * G::kDigitBits + q;
                if (((v >> q) & 1) && j < r) {
                    acc ^= f.basis[(size_t)j * W + w];
                    if (j > 0 && !counter) acc ^= f.basis[(size_t)(j - 1) * W + w];
                }
            }
            g.tab[idx * WMAX + w] = acc;
        }
    }
    if ((int)threadIdx.x < W) g.l[threadIdx.x] = f.shift[threadIdx.x];
    return ndig;
}

template <int WMAX>
__global__ __launch_bounds__(256) void enum_general_kernel(FactorIn f, uint64_t begin, uint64_t count,
                                                           uint64_t *__restrict__ out, int counter) {
    using G = GenTables<WMAX>;
    __shared__ G g;
    int r;
    if (!gate(f, begin, count, r)) return;
    const int W = f.words;
    const int ndig = build_tables<WMAX>(f, r, W, counter != 0, g);
    __syncthreads();
    // WMAX lanes per solution, lane w computes and stores word w: the
    // active lanes of a wave store one contiguous run of words.
    const int w = (int)(threadIdx.x & (WMAX - 1));
    const uint64_t stride = ((uint64_t)gridDim.x * blockDim.x) / WMAX;
    for (uint64_t j = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WMAX; j < count;
         j += stride) {
        const uint64_t i = begin + j;
        uint64_t z = (w < W) ? g.l[w] : 0ull;
        for (int m = 0; m < ndig; ++m) {
            const int d = (int)((i >> (m * G::kDigitBits)) & (G::kEntries - 1));
            z ^= g.tab[(m * G::kEntries + d) * WMAX + w];
        }
        if (w < W) *reinterpret_cast<AnyAddress<uint64_t>::type *>(out + (j * W + w)) = z;
    }
}

// ---------------------------------------------------------------------------
// The paper's circuit, evaluated literally (Section 2, Eqs. (1)-(2), Fig. 1(c))
// and fed by the binary counter of the FPGA design (Section 4).  Solution
// number i:
//   R = the bits of i scattered onto the pivot positions (R_{p_k} = bit k),
//   y = ((R & H) << 1) ^ ((R >> 1) & H)        horizontal-edge ROU layers
//     ^ ((R & Vm) << N) ^ ((R >> N) & Vm)      vertical-edge ROU layers
//     ^ (R & b)                                Toffoli layer (colours b)
//   z = y ^ l                                  final CNOT layer
// H has bit v set when the edge (v, v+1) exists, Vm when (v, v+N) exists.
// The scatter is linear in the bits of i, so R = R_lo(x) ^ R_hi(T) for
// i = (T << S) | x; the circuit itself runs for every solution.
// ---------------------------------------------------------------------------
// One 16-byte store per thread and tile, as vec_materialise (stage2.h), with
// the unit vectors of the pivots in the place of the basis rows: they give R.
// The layers then run on every solution.  16-bit words go through them in
// pairs, one in each half of a dword: no edge mask holds a bit whose shift
// would leave its half.  allowH and allowV are the vertices that have a
// right and a lower neighbour on the grid; every wave reads A's rows, takes
// the edge masks from them by ballots and checks that A has no other entry.
// Its set-up is some 40 vector instructions beside 50 per tile, so a
// workgroup takes kCircuitTiles tiles.
constexpr uint32_t kCircuitTiles = 2;

template <typename T>
__global__ __launch_bounds__(kVecThreads) void circuit_tile_kernel(
    FactorIn f, const int32_t *__restrict__ pivots, const uint64_t *__restrict__ rows, int N, uint64_t allowH,
    uint64_t allowV, VecRange g, uint32_t blocks, uint32_t tiles_per_block) {
    using X = VecTile<T>;
    constexpr int V = X::V, LOGV = X::LOGV, ND = X::ND, LB = X::LB;
    const uint32_t t0 = xcd_block(blockIdx.x, blocks) * tiles_per_block;
    const uint32_t t1 = t0 + tiles_per_block < g.ntiles ? t0 + tiles_per_block : g.ntiles;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t n = (uint32_t)f.n;
    const uint32_t own_row = lane < n ? lane : n - 1u;
    const int32_t own_pivot = pivots[own_row];
    uint64_t row = rows[own_row];
    const int32_t st = *f.status, r = *f.rank;
    const uint64_t l = f.shift[0];
    // Pivots past r are -1: their bits of the index are never set.
    int32_t p[LB];
    if (f.n >= LB) {
#pragma unroll
        for (int j = 0; j < LB; ++j) p[j] = pivots[j];
    } else {
#pragma unroll
        for (int j = 0; j < LB; ++j) p[j] = pivots[j < f.n ? j : f.n - 1];
    }
    asm volatile("" ::"s"(g.begin), "s"(g.end), "s"(g.tile0), "s"(g.full1), "s"(l), "s"(r), "s"(st), "s"(p[0]),
                 "s"(t0), "s"(t1), "s"(allowH), "s"(allowV));
    if (!vec_gate(f.status, st, r, g)) return;
    row = lane < n ? row : 0ull;
    // Row v turned right by v: bit 0 the colour, 1 and N the edges to v + 1
    // and v + N, 63 and 64 - N those to v - 1 and v - N.
    const uint64_t turned = (row >> lane) | (row << ((64u - lane) & 63u));
    const uint64_t mH = __ballot((turned >> 1) & 1ull) & allowH, mV = __ballot((turned >> N) & 1ull) & allowV,
                   mb = __ballot(turned & 1ull);
    const bool left = __builtin_amdgcn_inverse_ballot_w64(allowH << 1), right = __builtin_amdgcn_inverse_ballot_w64(allowH);
    const bool up = __builtin_amdgcn_inverse_ballot_w64(allowV << N), down = __builtin_amdgcn_inverse_ballot_w64(allowV);
    const uint64_t ok = 1ull | (right ? 2ull : 0ull) | (down ? 1ull << N : 0ull) | (left ? 1ull << 63 : 0ull) |
                        (up ? 1ull << (64 - N) : 0ull);
    if (__ballot((turned & ~ok) != 0ull)) {
        if (tid == 0) *f.status = HLF_EINVAL;
        return;
    }
    uint64_t low[LB];
#pragma unroll
    for (int j = 0; j < LB; ++j) low[j] = 1ull << (p[j] & 63);
    uint32_t le[ND], ls[ND], lo[ND], pf[V][ND], H[ND], Vm[ND], bb[ND];
    vec_dwords<T>(1ull << (own_pivot & 63), le);
    vec_dwords<T>(l, ls);
    vec_dwords<T>(mH, H);
    vec_dwords<T>(mV, Vm);
    vec_dwords<T>(mb, bb);
    const uint32_t x = lane << LOGV;
    vec_lane_part<T, true>(low, x, lo);
#pragma unroll
    for (int e = 0; e < V; ++e) vec_place<T, true>(low, e, pf[e]);
    const uint64_t first = g.begin & ~((1ull << X::S) - 1);
    for (uint32_t t = t0; t < t1; ++t) {
        const uint64_t iu = first + ((uint64_t)t << X::S) + (wave << LB);
        const bool on = __builtin_amdgcn_inverse_ballot_w64(iu);
        uint32_t h[ND];
#pragma unroll
        for (int q = 0; q < ND; ++q) h[q] = on ? le[q] : 0u;
        wave_xor_dwords<ND>(h);
        uint32_t w[4];
        vec_values<T>(lo, h, pf, w);  // R
        if constexpr (ND == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t R = w[k];
                w[k] = ((R & H[0]) << 1) ^ ((R >> 1) & H[0]) ^ ((R & Vm[0]) << N) ^ ((R >> N) & Vm[0]) ^ (R & bb[0]) ^ ls[0];
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; k += 2) {
                const uint64_t R = ((uint64_t)w[k + 1] << 32) | w[k];
                const uint64_t y = ((R & mH) << 1) ^ ((R >> 1) & mH) ^ ((R & mV) << N) ^ ((R >> N) & mV) ^ (R & mb) ^ l;
                w[k] = (uint32_t)y;
                w[k + 1] = (uint32_t)(y >> 32);
            }
        }
        vec_put<T>(g, t, iu + x, w);
    }
}

// ---------------------------------------------------------------------------
// Reduce.  The first count_blocks workgroups take the counts and the XOR-fold
// (thread j: vertex j, from column j of the basis), the others the hash, four
// waves each on contiguous ranges of tiles and one atomic add per workgroup.
// From W = 4 on the tile's next row comes by scalar loads under way during the
// tile's arithmetic; below, the wave holds the rows itself.
// ---------------------------------------------------------------------------
constexpr int kReduceThreads = 256;

template <int WW>
__global__ __launch_bounds__(kReduceThreads) void reduce_kernel(FactorIn f, uint64_t begin, uint64_t count,
                                                                uint64_t tiles_per_wave, uint32_t count_blocks,
                                                                int accumulate, uint64_t *__restrict__ counts,
                                                                uint64_t *__restrict__ hash,
                                                                uint64_t *__restrict__ xorfold) {
    constexpr int S = WaveHash<WW>::S;
    __shared__ uint64_t part[kReduceThreads / 64];
    int r;
    if (!gate(f, begin, count, r)) return;
    const uint64_t end = begin + count;
    const int lane = lane_id();
    if (blockIdx.x < count_blocks) {
        const int j = (int)blockIdx.x * kReduceThreads + (int)threadIdx.x, w = j >> 6;
        if (w >= WW) return;  // wave-uniform
        uint64_t col = 0;
        for (int k = 0; k < r; ++k) col |= ((f.basis[(size_t)k * WW + w] >> lane) & 1ull) << k;
        uint32_t odd;
        const uint64_t c = range_count(col, (uint32_t)(f.shift[w] >> lane) & 1u, begin, end, odd);
        const uint64_t fold = __ballot(odd);
        if (accumulate) {  // launches on other streams may add to the same outputs
            if (j < f.n && c) atomicAdd((unsigned long long *)&counts[j], (unsigned long long)c);
            if (xorfold && lane == 0 && fold) atomicXor((unsigned long long *)&xorfold[w], (unsigned long long)fold);
        } else {
            if (j < f.n) counts[j] = c;
            if (xorfold && lane == 0) xorfold[w] = fold;
        }
        return;
    }
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t ntiles = ((end - 1) >> S) - (begin >> S) + 1;
    const uint64_t t0 = ((uint64_t)(blockIdx.x - count_blocks) * (kReduceThreads / 64) + wave) * tiles_per_wave;
    uint64_t acc = 0;
    if (t0 < ntiles) {
        const uint64_t first_tile = begin >> S;
        const uint64_t t1 = t0 + tiles_per_wave < ntiles ? t0 + tiles_per_wave : ntiles;
        const uint64_t c0 = t0 ? (first_tile + t0) << S : begin, c1 = t1 < ntiles ? (first_tile + t1) << S : end;
        const WaveRows<WW> b = wave_rows<WW>(f.basis, r);
        uint64_t l[WW];
#pragma unroll
        for (int w = 0; w < WW; ++w) l[w] = f.shift[w];
        acc = wave_hash_range<WW>(b, l, c0, c1, [&](int k, uint64_t(&row)[WW]) {
#pragma unroll
            for (int w = 0; w < WW; ++w) {
                if constexpr (WW <= 3) row[w] = row_word<WW>(b, k, w);
                else row[w] = f.basis[(size_t)k * WW + w];
            }
        });
    }
    acc = wave_sum_u64(acc);
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t sum = 0;
#pragma unroll
        for (int v = 0; v < kReduceThreads / 64; ++v) sum += part[v];
        if (sum) atomicAdd((unsigned long long *)hash, (unsigned long long)sum);
    }
}

// Overwrite mode: the hash starts from zero, and for an empty range so do the
// others (a kernel, so the call stays capturable in a graph).
__global__ void zero_outputs_kernel(FactorIn f, uint64_t begin, uint64_t count, int n, int W,
                                    uint64_t *counts, uint64_t *hash, uint64_t *xorfold) {
    int r;
    if (!gate(f, begin, count, r)) return;
    if (threadIdx.x == 0) *hash = 0;
    if (count) return;
    for (int j = threadIdx.x; j < n; j += blockDim.x) counts[j] = 0;
    if (xorfold)
        for (int w = threadIdx.x; w < W; w += blockDim.x) xorfold[w] = 0;
}

// Even split of ntiles over at most max_units units: tiles per unit.
uint64_t tiles_per_unit_for(uint64_t ntiles, uint64_t max_units, uint64_t *units) {
    uint64_t b = ntiles < max_units ? ntiles : max_units;
    if (b == 0) b = 1;
    const uint64_t tpu = (ntiles + b - 1) / b;
    *units = (ntiles + tpu - 1) / tpu;
    return tpu;
}

// Materialise launches: materialise_tiles_per_block tiles per workgroup.
// The multi-word circuit kernel's workgroups build per-word tables before their
// first store, so they take ranges kWideRangeFactor times longer than the
// common size (passed as a smaller nominal tile size).
constexpr uint64_t kWideRangeFactor = 2;

uint64_t tiles_per_block_for(uint64_t ntiles, uint64_t tile_bytes, uint64_t *blocks) {
    const uint64_t tpb = materialise_tiles_per_block(ntiles, tile_bytes);
    *blocks = ntiles ? (ntiles + tpb - 1) / tpb : 1;
    return tpb;
}

template <typename T>
hlf_status launch_tile(const FactorIn &f, uint64_t begin, uint64_t count, T *out, int counter,
                       hipStream_t stream) {
    const VecRange g = vec_range<T>(begin, count, out);
    const uint32_t tpb = vec_tiles_per_block(g.ntiles);
    const uint32_t blocks = g.ntiles ? (g.ntiles + tpb - 1) / tpb : 1u;
    if (counter)
        hipLaunchKernelGGL((enum_tile_kernel<T, true>), dim3(blocks), dim3(kVecThreads), 0, stream, f, g, blocks, tpb);
    else
        hipLaunchKernelGGL((enum_tile_kernel<T, false>), dim3(blocks), dim3(kVecThreads), 0, stream, f, g, blocks, tpb);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

// Tiles per workgroup of the multi-word materialise kernel.  Up to kWideFill
// tiles each go to one generation of two workgroups per CU: a workgroup's
// set-up costs several tiles (21 MB of 5 words: 7.1 us in 512 workgroups of 8
// tiles, 9.5 in 2048 of 2; 8.7 with 128 KiB per 1024-thread workgroup), and a
// longer range in 32 KiB each, many more workgroups than run at once (1 GiB of
// 16 words: 178 us at 32 KiB, 182 at 64, 187 at 128; of 15 words within 3%).
constexpr uint64_t kWideBytes = 32ull << 10;
constexpr uint64_t kWideFill = 32;

template <int W>
hlf_status launch_wide_tile(const FactorIn &f, uint64_t begin, uint64_t count, uint64_t *out, int counter,
                            hipStream_t stream) {
    constexpr int S = WideTile<W>::S;
    const uint64_t end = begin + count;
    const uint64_t ntiles = (end < begin) ? 1 : ((end - 1) >> S) - (begin >> S) + 1;
    const uint64_t resident = 2ull * (uint64_t)device_cu_count();
    const uint64_t fill = (ntiles + resident - 1) / resident;
    uint64_t tpb = fill <= kWideFill ? fill : kWideBytes / WideTile<W>::kBytes;
    tpb = std::max(tpb, (ntiles + kMaxVecBlocks - 1) / kMaxVecBlocks);
    const uint64_t blocks = (ntiles + tpb - 1) / tpb;
    if (counter)
        hipLaunchKernelGGL((enum_wide_tile_kernel<W, true>), dim3((unsigned)blocks), dim3(kVecThreads), 0, stream, f,
                           begin, count, out, tpb);
    else
        hipLaunchKernelGGL((enum_wide_tile_kernel<W, false>), dim3((unsigned)blocks), dim3(kVecThreads), 0, stream, f,
                           begin, count, out, tpb);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int... Ws>
hlf_status launch_wide(int W, const FactorIn &f, uint64_t begin, uint64_t count, uint64_t *out, int counter,
                       hipStream_t stream, std::integer_sequence<int, Ws...>) {
    hlf_status st = HLF_EINVAL;
    ((W == Ws + 2 ? (st = launch_wide_tile<Ws + 2>(f, begin, count, out, counter, stream), 0) : 0), ...);
    return st;
}

template <int WMAX>
hlf_status launch_general(const FactorIn &f, uint64_t begin, uint64_t count, uint64_t *out, int counter,
                          hipStream_t stream) {
    const uint64_t per_block = 256 / WMAX;  // solutions per workgroup pass
    uint64_t blocks = (count + per_block - 1) / per_block;
    const uint64_t cap = (uint64_t)device_cu_count() * 8;
    if (blocks > cap) blocks = cap;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(enum_general_kernel<WMAX>, dim3((unsigned)blocks), dim3(256), 0,
                       stream, f, begin, count, out, counter);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int WW>
hlf_status launch_reduce_t(const FactorIn &f, uint64_t begin, uint64_t count, bool accumulate, uint64_t *counts,
                           uint64_t *hash, uint64_t *xorfold, hipStream_t stream) {
    constexpr int S = WaveHash<WW>::S;
    const uint64_t end = begin + count;
    const uint64_t ntiles = (end < begin) ? 1 : ((end - 1) >> S) - (begin >> S) + 1;
    uint64_t waves;
    // Waves per CU: more than fit, so that the last ones fill in; fewer where a
    // wave's constants are many (2^30 one-word solutions: 501 us at 16, 483 at
    // 32, 474 at 64, 478 at 96; 2^24 of 16 words: 161 at 16 and 32, 169 at 64).
    const uint64_t tpw = tiles_per_unit_for(ntiles, (uint64_t)device_cu_count() * (WW == 1 ? 64 : 32), &waves);
    const uint32_t count_blocks = (uint32_t)((f.n + kReduceThreads - 1) / kReduceThreads);
    const uint64_t blocks = count_blocks + (waves + 3) / 4;
    hipLaunchKernelGGL(reduce_kernel<WW>, dim3((unsigned)blocks), dim3(kReduceThreads), 0, stream, f, begin, count,
                       tpw, count_blocks, accumulate ? 1 : 0, counts, hash, xorfold);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int... Ws>
hlf_status launch_reduce_w(int W, const FactorIn &f, uint64_t begin, uint64_t count, bool accumulate,
                           uint64_t *counts, uint64_t *hash, uint64_t *xorfold, hipStream_t stream,
                           std::integer_sequence<int, Ws...>) {
    hlf_status st = HLF_EINVAL;
    ((W == Ws + 1 ? (st = launch_reduce_t<Ws + 1>(f, begin, count, accumulate, counts, hash, xorfold, stream), 0) : 0),
     ...);
    return st;
}

}  // namespace

hlf_status launch_enumerate(const FactorIn &f, uint64_t begin, uint64_t count, int word_bits,
                            bool counter_order, void *out, hipStream_t stream) {
    const int W = f.words;
    const int c = counter_order ? 1 : 0;
    if (W == 1 && word_bits <= 64) {
        if (word_bits == 16) return launch_tile<uint16_t>(f, begin, count, (uint16_t *)out, c, stream);
        if (word_bits == 32) return launch_tile<uint32_t>(f, begin, count, (uint32_t *)out, c, stream);
        return launch_tile<uint64_t>(f, begin, count, (uint64_t *)out, c, stream);
    }
    uint64_t *o = (uint64_t *)out;
    if (((uintptr_t)out & 7u) == 0) {
        return launch_wide(W, f, begin, count, o, c, stream, std::make_integer_sequence<int, HLF_MAX_N / 64 - 1>{});
    }
    if (W <= 2) return launch_general<2>(f, begin, count, o, c, stream);
    if (W <= 4) return launch_general<4>(f, begin, count, o, c, stream);
    if (W <= 8) return launch_general<8>(f, begin, count, o, c, stream);
    return launch_general<16>(f, begin, count, o, c, stream);
}

// ---------------------------------------------------------------------------
// The paper's circuit for grids of more than 64 vertices (W > 1 words per
// vector; the same layers as circuit_tile_kernel).  First a launch checks
// that A is a subgraph of the N x N grid (every row's bits lie on the vertex
// itself and its grid neighbours) and writes HLF_EINVAL otherwise, so the
// materialising launch behind it on the stream writes nothing (one thread per
// word of A; one workgroup for all took 9.7 us at n = 1024).  The materialising
// kernel takes one lane per word: thread (slot, w) holds word w of solutions
// base + slot + u*P, u < WMAX, P = 1024 / WMAX.  (In pieces of 16 bytes, as
// enum_wide_tile_kernel, its set-up is too long for the few solutions of a
// block: 27 MB of 13 words 22 us against 15.)  R, the counter bits scattered onto the pivots, is linear
// in the index: R = Rlo(slot + u*P) ^ Rhi(T) for a tile T of 1024 indices.
// The edge layers shift R by 1 and by N bits across words; a lane takes the
// neighbouring words of its solution from lanes w - 1 and w + 1.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void circuit_check_kernel(int32_t *status, const uint64_t *__restrict__ rows,
                                                            int n, int W, int N) {
    if (*(volatile int32_t *)status != HLF_OK) return;
    const int idx = blockIdx.x * 256 + threadIdx.x;  // one word of A each
    if (idx >= n * W) return;
    const int v = idx / W, w = idx - v * W;
    const int gr = v / N, gc = v - gr * N;
    uint64_t allowed = 0;
    auto allow = [&](int u) {
        if ((u >> 6) == w) allowed |= 1ull << (u & 63);
    };
    allow(v);
    if (gc > 0) allow(v - 1);
    if (gc < N - 1) allow(v + 1);
    if (gr > 0) allow(v - N);
    if (gr < N - 1) allow(v + N);
    if (rows[idx] & ~allowed) *status = HLF_EINVAL;
}

namespace {

// x of lane - 1 / lane + 1 within the lane's 16-lane row (0 at the row edge).
__device__ __forceinline__ uint64_t dpp_row_shr1(uint64_t x) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x111, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x111, 0xf, 0xf, true);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}
__device__ __forceinline__ uint64_t dpp_row_shl1(uint64_t x) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x101, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x101, 0xf, 0xf, true);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

template <int WMAX>
__global__ __launch_bounds__(kTileThreads) void circuit_wide_kernel(
    FactorIn f, const int32_t *__restrict__ pivots, const uint64_t *__restrict__ rows, int N,
    uint64_t begin, uint64_t count, uint64_t *__restrict__ out, uint64_t tiles_per_block) {
    constexpr int P = kTileThreads / WMAX;
    constexpr int U = WMAX;
    constexpr int S = kLogTileThreads;
    constexpr int LOGP = S - (WMAX == 2 ? 1 : WMAX == 4 ? 2 : WMAX == 8 ? 3 : 4);
    __shared__ uint64_t E[64 * WMAX];     // E[k][w] = word w of e_{p_k}, k < r
    __shared__ uint64_t M[3 * WMAX];      // H, V (edge masks), b (colours)
    int r;
    if (!gate(f, begin, count, r)) return;
    const int n = f.n, W = f.words;
    const int tid = threadIdx.x;
    for (int idx = tid; idx < 64 * WMAX; idx += blockDim.x) {
        const int k = idx / WMAX, w = idx - k * WMAX;
        uint64_t e = 0;
        if (k < r) {
            const int p = pivots[k];
            if ((p >> 6) == w) e = 1ull << (p & 63);
        }
        E[idx] = e;
    }
    // masks from three words per row: A[v][v+1], A[v][v+N], A[v][v]
    {
        const int v = tid;  // n <= 1024 = blockDim.x
        bool h = false, vv = false, bb = false;
        if (v < n) {
            const int gr = v / N, gc = v - (v / N) * N;
            const uint64_t *row = rows + (size_t)v * W;
            if (gc < N - 1) h = (row[(v + 1) >> 6] >> ((v + 1) & 63)) & 1ull;
            if (gr < N - 1) vv = (row[(v + N) >> 6] >> ((v + N) & 63)) & 1ull;
            bb = (row[v >> 6] >> (v & 63)) & 1ull;
        }
        const uint64_t H = __ballot(h), V = __ballot(vv), B = __ballot(bb);
        const int wave = tid >> 6;
        if ((tid & 63) == 0 && wave < WMAX) {
            M[wave] = H;
            M[WMAX + wave] = V;
            M[2 * WMAX + wave] = B;
        }
    }
    __syncthreads();
    const uint64_t end = begin + count;
    const uint64_t ntiles = ((end - 1) >> S) - (begin >> S) + 1;
    const uint64_t t0 = (uint64_t)xcd_block(blockIdx.x, gridDim.x) * tiles_per_block;
    if (t0 >= ntiles) return;
    const uint64_t t1 = (t0 + tiles_per_block < ntiles) ? t0 + tiles_per_block : ntiles;
    const int w = tid & (WMAX - 1);
    const int slot = tid / WMAX;
    const bool act = w < W;
    const uint64_t Hw = M[w], Vw = M[WMAX + w], Bw = M[2 * WMAX + w];
    const uint64_t Hm = w ? M[w - 1] : 0ull, Vm = w ? M[WMAX + w - 1] : 0ull;
    const uint64_t lw = act ? f.shift[w] : 0ull;
    // Rlo[u] = scatter of slot + u*P; bit j of slot is e_{p_j}, u*P adds LOGP + bits of u
    uint64_t Rlo[U];
    {
        uint64_t x = 0;
        for (int j = 0; j < LOGP; ++j)
            if ((slot >> j) & 1) x ^= E[j * WMAX + w];
        Rlo[0] = x;
    }
#pragma unroll
    for (int u = 1; u < U; ++u) Rlo[u] = Rlo[u & (u - 1)] ^ E[(LOGP + __builtin_ctz(u)) * WMAX + w];
    uint64_t Tt = (begin >> S) + t0;
    uint64_t Rhi = 0;
    for (int j = 0; j + S < 64 && (Tt >> j); ++j)
        if ((Tt >> j) & 1ull) Rhi ^= E[(S + j) * WMAX + w];
    const int Nr = 64 - N;
    for (uint64_t t = t0; t < t1; ++t, ++Tt) {
        const uint64_t base = Tt << S;
        const bool full = base >= begin && base + (1u << S) <= end;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t R = Rlo[u] ^ Rhi;
            // neighbouring words of the same solution (0 beyond the vector):
            // DPP row shifts by one lane (a solution's WMAX lanes lie in one
            // 16-lane row)
            uint64_t Rd = dpp_row_shr1(R);
            uint64_t Ru = dpp_row_shl1(R);
            if (w == 0) Rd = 0;
            if (w == WMAX - 1) Ru = 0;
            const uint64_t X1 = R & Hw, X1d = Rd & Hm, X2 = R & Vw, X2d = Rd & Vm;
            const uint64_t y = ((X1 << 1) | (X1d >> 63)) ^ (((R >> 1) | (Ru << 63)) & Hw) ^
                               ((X2 << N) | (X2d >> Nr)) ^ (((R >> N) | (Ru << Nr)) & Vw) ^ (R & Bw);
            const uint64_t z = y ^ lw;
            const uint64_t i = base + (uint64_t)slot + (uint64_t)u * P;
            if (act) {
                if (full)
                    __builtin_nontemporal_store(z, out + (i - begin) * W + w);
                else if (i >= begin && i < end)
                    out[(i - begin) * W + w] = z;
            }
        }
        // next tile: the counter's carry flips bits S .. S + ctz(T + 1)
        const int c = __builtin_ctzll(Tt + 1);
        for (int j = 0; j <= c && S + j < 64; ++j) Rhi ^= E[(S + j) * WMAX + w];
    }
}

}  // namespace

hlf_status launch_circuit(const FactorIn &f, const int32_t *pivots, const uint64_t *rows, int N,
                          uint64_t begin, uint64_t count, int word_bits, void *out,
                          hipStream_t stream) {
    const uint64_t end = begin + count;
    auto go = [&](auto tag) -> hlf_status {
        using T = decltype(tag);
        const VecRange g = vec_range<T>(begin, count, out);
        uint64_t allowH = 0, allowV = 0;
        for (int v = 0; v < f.n; ++v) {
            if (v % N < N - 1) allowH |= 1ull << v;
            if (v + N < f.n) allowV |= 1ull << v;
        }
        const uint32_t tpb = std::max(kCircuitTiles, vec_tiles_per_block(g.ntiles));
        const uint32_t blocks = g.ntiles ? (g.ntiles + tpb - 1) / tpb : 1u;
        hipLaunchKernelGGL(circuit_tile_kernel<T>, dim3(blocks), dim3(kVecThreads), 0, stream, f, pivots, rows, N,
                           allowH, allowV, g, blocks, tpb);
        return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
    };
    if (word_bits == 16) return go(uint16_t{});
    if (word_bits == 32) return go(uint32_t{});
    if (word_bits == 64 && f.words == 1) return go(uint64_t{});
    // W > 1 words per solution
    const int W = f.words;
    hipLaunchKernelGGL(circuit_check_kernel, dim3((unsigned)((f.n * W + 255) / 256)), dim3(256), 0, stream, f.status,
                       rows, f.n, W, N);
    if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    auto wide = [&](auto wm) -> hlf_status {
        constexpr int WMAX = decltype(wm)::value;
        constexpr int S = kLogTileThreads;
        const uint64_t ntiles = (end < begin) ? 1 : ((end - 1) >> S) - (begin >> S) + 1;
        uint64_t blocks;
        const uint64_t tpb = tiles_per_block_for(ntiles, (8ull * (uint64_t)W << S) / kWideRangeFactor, &blocks);
        hipLaunchKernelGGL(circuit_wide_kernel<WMAX>, dim3((unsigned)blocks), dim3(kTileThreads), 0, stream,
                           f, pivots, rows, N, begin, count, (uint64_t *)out, tpb);
        return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
    };
    if (W <= 2) return wide(std::integral_constant<int, 2>{});
    if (W <= 4) return wide(std::integral_constant<int, 4>{});
    if (W <= 8) return wide(std::integral_constant<int, 8>{});
    return wide(std::integral_constant<int, 16>{});
}

hlf_status launch_reduce(const FactorIn &f, uint64_t begin, uint64_t count, bool accumulate,
                         uint64_t *counts, uint64_t *hash, uint64_t *xorfold,
                         hipStream_t stream) {
    const int W = f.words;
    if (!accumulate) {
        hipLaunchKernelGGL(zero_outputs_kernel, dim3(1), dim3(256), 0, stream, f, begin, count,
                           f.n, W, counts, hash, xorfold);
        if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    }
    if (count == 0) return HLF_OK;
    return launch_reduce_w(W, f, begin, count, accumulate, counts, hash, xorfold, stream,
                           std::make_integer_sequence<int, HLF_MAX_WORDS>{});
}

}  // namespace hlf
