// Stage 1 of the two-stage scheme (the paper's CLA module, Section 2,
// tasks (1)-(4)) on gfx950:
//   * pack_dense_kernel (n <= 64), pack_rows_kernel + pack_check_kernel
//     (n > 64): dense 0/1 matrix -> packed uint64 rows, with the symmetry /
//     0-1 validation of the problem statement (Section 1);
//   * factor_wave_kernel: one wavefront per instance (used for n <= 64; the
//     batch path runs the same elimination for n <= 192); every lane keeps
//     its rows in VGPRs, pivots are found with a ballot and the pivot row is
//     broadcast with readlane -- no barriers in the elimination;
//   * factor_workgroup_kernel: one workgroup per instance for n <= 1024, one
//     row per thread in VGPRs, Gauss-Jordan in panels of 64 columns: one wave
//     finds a panel's pivots on one word per row, then every row applies the
//     panel with 13 lookups per word in tables of XOR combinations of the
//     panel's pivot rows (LDS).
// Both variants produce the canonical record defined in hlf.h (the RREF is
// unique, so the pivot rows chosen do not matter).
#include "factor_wave.h"
#include "hlf_device.h"
#include "hlf_internal.h"

#include <climits>

namespace hlf {
namespace {

// ---------------------------------------------------------------------------
// A0: pack + validate for n <= 64 (larger n: the two launches below).  One wave
// packs A into bit rows in LDS, one word each, and checks A = A^T.
//
// Packing: when n is a multiple of 16 and A is 16-byte aligned, each thread
// loads 16 bytes (columns 16q..16q+15 of one row) per request, all its rows in
// flight, and gathers them into 16 bits.  For a 32-bit word x holding four
// 0/1 bytes b0..b3, (x * 0x10204080) >> 28 = b0 | b1<<1 | b2<<2 | b3<<3: the
// partial product of b_k with 2^(28-7k) lands on bit 28+k, and every other
// partial product lands on a distinct bit below 28 or above 31, so there are
// no carries into bits 28..31.  Any other n falls back to byte loads (lane l
// loads column l of G rows, one ballot per row).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t gather4(uint32_t x) { return (x * 0x10204080u) >> 28; }

// Symmetry of one pair of 64x64 tiles: lane l holds x = word J of row 64I+l
// and y = word I of row 64J+l.  Column b of tile (I, J), which lane b of the
// transposed tile holds, must equal y in lane b (row 64J+b restricted to
// columns 64I..64I+63).  Returns true, wave-uniform, if some
// A[64I+l][64J+b] != A[64J+b][64I+l].  Needs all lanes active.
__device__ __forceinline__ bool tile_pair_asym(uint64_t x, uint64_t y) {
    return __ballot(wave_transpose64(x) != y) != 0;
}

// A0 for n > 64: two launches.  pack_rows_kernel packs 16 rows per
// workgroup (16-byte loads and gather4 when n is a multiple of 16 and A is
// 16-byte aligned, else byte loads and one ballot per row word) and checks
// that every byte is 0 or 1.  gather4 is only meaningful on 0/1 bytes, so a
// row holding another value may pack to arbitrary bits; the workgroup then
// marks it so that the check below must fail whatever those bits are.  When
// n is not a multiple of 64 the row gets pad bit 63 of its last word.  When
// it is, every block is 16 full rows, and the asymmetry goes inside one of
// the workgroup's own row pairs (i, i^1): if one row of the pair is bad, its
// entry towards the other becomes the complement of the other's entry back,
// if both are, the two entries become 1 and 0.  pack_check_kernel checks the
// pad bits and A = A^T on the packed rows, tile pair by tile pair; the first
// launch writes HLF_OK and the second the verdict that overrules it.
constexpr int kPackRowsPerBlock = 16;
constexpr int kPackRowsThreads = 256;

__global__ __launch_bounds__(kPackRowsThreads) void pack_rows_kernel(const uint8_t *__restrict__ A,
                                                                     int n, int W, int vec16,
                                                                     uint64_t *__restrict__ rows,
                                                                     int32_t *__restrict__ status) {
    __shared__ uint64_t lds[kPackRowsPerBlock * HLF_MAX_WORDS];
    __shared__ int badrow[kPackRowsPerBlock];
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * kPackRowsPerBlock;
    const int cpr = n >> 4;  // 16-byte chunks per row
    if (blockIdx.x == 0 && tid == 0) *status = HLF_OK;
    if (tid < kPackRowsPerBlock) badrow[tid] = 0;
    for (int idx = tid; idx < kPackRowsPerBlock * W; idx += kPackRowsThreads) lds[idx] = 0;
    __syncthreads();
    if (!vec16) {
        // (row, word) items per wave: lane l loads byte 64w + l of the row, a
        // ballot gives the packed word; eight items' loads go out together.
        const int lane = tid & 63, wave = tid >> 6;
        constexpr int kWaves = kPackRowsThreads / 64, kBatch = 8;
        const int items = kPackRowsPerBlock * W;
        for (int it0 = wave * kBatch; it0 < items; it0 += kWaves * kBatch) {
            uint32_t byte[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int it = it0 + u, lr = it / W, w = it - lr * W;
                const int i = i0 + lr, c = 64 * w + lane;
                byte[u] = (it < items && i < n && c < n) ? (uint32_t)A[(size_t)i * n + c] : 0u;
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int it = it0 + u, lr = it / W;
                const uint64_t word = __ballot(byte[u] & 1u);
                const bool badb = __ballot(byte[u] > 1u) != 0;
                if (lane == 0 && it < items) {
                    lds[it] = word;  // it = lr * W + w
                    if (badb) badrow[lr] = 1;
                }
            }
        }
    } else {
    uint16_t *l16 = reinterpret_cast<uint16_t *>(lds);
    const u32x4 *A16 = reinterpret_cast<const u32x4 *>(A);
    // at most 16 rows x 64 chunks = 4 chunks per thread, all loads first
    constexpr int kPer = kPackRowsPerBlock * (HLF_MAX_N / 16) / kPackRowsThreads;
    u32x4 v[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int idx = tid + k * kPackRowsThreads;
        const int lr = idx / cpr, c = idx - lr * cpr;
        const bool ok = lr < kPackRowsPerBlock && i0 + lr < n;
        v[k] = ok ? __builtin_nontemporal_load(&A16[(size_t)(i0 + lr) * cpr + c]) : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int idx = tid + k * kPackRowsThreads;
        const int lr = idx / cpr, c = idx - lr * cpr;
        if (lr < kPackRowsPerBlock && i0 + lr < n) {
            if (((v[k].x | v[k].y | v[k].z | v[k].w) & 0xFEFEFEFEu) != 0u) badrow[lr] = 1;
            l16[lr * 4 * W + c] = (uint16_t)(gather4(v[k].x) | (gather4(v[k].y) << 4) |
                                             (gather4(v[k].z) << 8) | (gather4(v[k].w) << 12));
        }
    }
    }
    __syncthreads();
    if ((n & 63) != 0) {  // pad bit 63 of the last word of a bad row
        if (tid < kPackRowsPerBlock && i0 + tid < n && badrow[tid]) lds[tid * W + W - 1] |= 1ull << 63;
    } else if (tid < kPackRowsPerBlock / 2) {  // row pair (a, a + 1): full blocks
        const int a = 2 * tid, b = a + 1, ia = i0 + a, ib = i0 + b;
        if (ib < n && (badrow[a] || badrow[b])) {
            uint64_t &ab = lds[a * W + (ib >> 6)];  // holds entry (ia, ib)
            uint64_t &ba = lds[b * W + (ia >> 6)];  // holds entry (ib, ia)
            const uint64_t mab = 1ull << (ib & 63), mba = 1ull << (ia & 63);
            if (badrow[a] && badrow[b]) {
                ab |= mab;
                ba &= ~mba;
            } else if (badrow[a]) {
                ab = (ba & mba) ? (ab & ~mab) : (ab | mab);
            } else {
                ba = (ab & mab) ? (ba & ~mba) : (ba | mba);
            }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < kPackRowsPerBlock * W; idx += kPackRowsThreads) {
        const int lr = idx / W, w = idx - lr * W;
        const int i = i0 + lr;
        if (i < n) rows[(size_t)i * W + w] = lds[lr * W + w];
    }
}

// One wave per tile pair (one workgroup for all of them: 11.7 us at n = 1024).
constexpr int kCheckWaves = 4;

__global__ __launch_bounds__(64 * kCheckWaves) void pack_check_kernel(const uint64_t *__restrict__ rows, int n,
                                                                      int W, int32_t *__restrict__ status) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * kCheckWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per = W / 2 + 1, I = t / per, d = t - I * per;  // tiles (I, I + d mod W)
    if (I >= W) return;
    const int J = I + d < W ? I + d : I + d - W;
    const int ri = 64 * I + lane, rj = 64 * J + lane;
    const uint64_t x = ri < n ? rows[(size_t)ri * W + J] : 0ull;
    const uint64_t y = rj < n ? rows[(size_t)rj * W + I] : 0ull;
    const uint64_t pad = ~last_word_mask(n);
    const uint64_t pads = (J == W - 1 ? x & pad : 0ull) | (I == W - 1 ? y & pad : 0ull);
    if (tile_pair_asym(x, y) || __ballot(pads != 0ull) != 0) {
        if (lane == 0) *status = HLF_ENOTSYM;
    }
}

__global__ __launch_bounds__(64) void pack_dense_kernel(const uint8_t *__restrict__ A, int n,
                                                        uint64_t *__restrict__ rows, int32_t *__restrict__ status) {
    __shared__ uint64_t lds[64];
    const int lane = threadIdx.x;
    bool bad = false;
    lds[lane] = 0;
    __syncthreads();
    if ((n & 15) == 0 && ((uintptr_t)A & 15u) == 0) {
        uint16_t *l16 = reinterpret_cast<uint16_t *>(lds);
        const int cpr = n >> 4;            // 16-byte chunks per row
        const int rpp = 64 / cpr;          // rows per pass, >= 16
        const int ri = lane / cpr, q = lane - ri * cpr;
        const u32x4 *A16 = reinterpret_cast<const u32x4 *>(A);
        constexpr int kPasses = 4;         // n <= 64 rows, at least 16 a pass
        if (ri < rpp) {
            u32x4 v[kPasses];
#pragma unroll
            for (int u = 0; u < kPasses; ++u) {
                const int i = ri + u * rpp;
                v[u] = i < n ? __builtin_nontemporal_load(&A16[(size_t)i * cpr + q]) : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int u = 0; u < kPasses; ++u) {
                const int i = ri + u * rpp;
                if (i < n) {
                    bad |= ((v[u].x | v[u].y | v[u].z | v[u].w) & 0xFEFEFEFEu) != 0u;
                    l16[i * 4 + q] = (uint16_t)(gather4(v[u].x) | (gather4(v[u].y) << 4) |
                                                (gather4(v[u].z) << 8) | (gather4(v[u].w) << 12));
                }
            }
        }
    } else {
        constexpr int G = 16;
        for (int i0 = 0; i0 < n; i0 += G) {
            uint32_t v[G];
#pragma unroll
            for (int k = 0; k < G; ++k)
                v[k] = (lane < n && i0 + k < n) ? (uint32_t)A[(size_t)(i0 + k) * n + lane] : 0u;
#pragma unroll
            for (int k = 0; k < G; ++k) {
                if (i0 + k >= n) break;
                bad |= v[k] > 1u;
                const uint64_t word = __ballot(v[k] == 1u);
                if (lane == 0) lds[i0 + k] = word;
            }
        }
    }
    __syncthreads();
    const uint64_t row = lds[lane];  // zero from row n on
    if (tile_pair_asym(row, row)) bad = true;
    if (lane < n) rows[lane] = row;
    const bool any = __ballot(bad) != 0;
    if (lane == 0) *status = any ? HLF_ENOTSYM : HLF_OK;
}

// keep_bad: out.status already holds the pack verdict for these rows; a
// verdict other than HLF_OK stays and nothing else is written.
template <int WMAX>
__global__ __launch_bounds__(64) void factor_wave_kernel(const uint64_t *__restrict__ rows, int n,
                                                         int W, FactorOut out, int keep_bad) {
    if (keep_bad && *(volatile int32_t *)out.status != HLF_OK) return;
    __shared__ WaveSmem<WMAX> sm;
    wave_load_rows<WMAX>(rows, n, W, sm);
    factor_wave_core<WMAX>(n, W, false, out, sm);
}

// ---------------------------------------------------------------------------
// A1-A4, workgroup variant: n <= 64*WMAX <= 1024, 64*W threads, thread i
// holds row i.  Gauss-Jordan in panels of 64 columns, one word of every row:
//
//   1. rows that are no pivot yet and not zero in the panel are listed in LDS;
//   2. one wave finds the panel's pivots from the list (panel_pivots below),
//      on panel words alone, 64 rows at a time, one per lane.  Elimination is
//      in place: where a pivot has been added to a row, the row's bit at the
//      pivot's column stays set, so that a row's bits at pivot columns come to
//      say which start-of-panel pivot rows it is the sum of (tau), and those
//      at the other columns are its entries there;
//   3. every row's tag t is the XOR of the tau of the pivots of the columns
//      that it has set (13 table lookups, five bits each), and its own tau if
//      it has become a pivot: t says which start-of-panel pivot rows to add;
//   4. the pivot rows lie in LDS; every word from the panel's on gets 13 tables
//      of 32 XOR combinations, and every row adds one entry of each to it.
//      (Words left of the panel are zero in rows that are no pivot yet.)
//
// The next panel's word is brought up to date first, so that its pivots are
// found by one wave while the others work on the words behind it.
//
// Which rows become pivots does not matter: the pivot columns are the leading
// ones of the row space, and the reduced echelon form is unique.
//
// Bound by the chain of one pivot after the other: a column costs some 17
// instructions of one wave, which issues one in five cycles at best.  Tables
// of 32 entries of 8 bytes spread over all 64 LDS banks: 530 cycles per word
// for 1024 rows, against 1080 with tables of 16, which use half of them.
// Measured at n = 1024 (32x32 grid, half the bonds), stage 1 with the packing:
// 158 us a pass, against 528 with panels of 8 columns, whose pivots all waves
// searched together with two barriers a column.  (Further candidates filtered
// by all waves instead of 64 at a time by the one: 173 us.)
// ---------------------------------------------------------------------------
constexpr int kTabGroups = 13;                    // groups of five bits of a word
constexpr int kTabWords = kTabGroups * 32;

template <int WMAX>
struct PanelShared {
    static constexpr int NP = 64 * WMAX;
    static constexpr int kStride = NP + 1;  // words of a column of `mat`, odd against bank conflicts
    // mat holds, in turn: A word-major (word w of row i at w*kStride + i); the
    // panel step's arrays; the reduced rows by pivot column, transposed in
    // place into the kernel vectors by free column.
    struct Panel {
        uint64_t tab[WMAX * kTabWords];   // [word][group][32]
        uint64_t start[WMAX * 64];        // [word][column]: start-of-panel pivot rows
        uint64_t ttab[kTabWords];         // the tables of tau
        uint64_t tau[64];                 // by column
        uint64_t base[64];                // the basis found so far (panel_pivots)
        uint64_t btab[kTabWords];         // its tables
        uint64_t cand_x[NP];
        uint16_t cand_row[NP];
    };
    union alignas(16) {
        uint64_t mat[WMAX * kStride];
        Panel pan;
    };
    uint64_t pivots[WMAX];     // pivot columns, by panel
    uint64_t diag[WMAX];
    int qacc[NP];
    uint16_t pivcol[NP];       // row -> its pivot column, 0xFFFF if none
    uint16_t pivlist[NP];
    int ncand[2];
    int bad, internal;
};

__device__ __forceinline__ uint32_t lane_select(uint64_t mask, uint32_t v, uint32_t other) {
    return __builtin_amdgcn_inverse_ballot_w64(mask) ? v : other;
}

// x ^ (m & p), one instruction.
__device__ __forceinline__ uint32_t xor_masked(uint32_t x, uint32_t m, uint32_t p) {
    return __builtin_amdgcn_bitop3_b32(x, m, p, 0x78);
}

// The 13 tables of the XOR combinations of vec[0..63], by one wave: lane
// 4g + q fills entries 8q .. 8q + 7 of group g (the last group has four
// vectors).
__device__ __forceinline__ void fill_tables(const uint64_t *vec, uint64_t *tab) {
    const int lane = lane_id(), g = lane >> 2, q = lane & 3;
    if (g >= kTabGroups) return;
    const uint64_t *v = vec + 5 * g;
    const uint64_t s0 = v[0], s1 = v[1], s2 = v[2], s3 = v[3], s4 = g < 12 ? v[4] : 0ull;
    uint64_t e[8];
    e[0] = ((q & 1) ? s3 : 0ull) ^ ((q & 2) ? s4 : 0ull);
    e[1] = e[0] ^ s0;
    e[2] = e[0] ^ s1;
    e[3] = e[1] ^ s1;
#pragma unroll
    for (int k = 0; k < 4; ++k) e[4 + k] = e[k] ^ s2;
    uint64_t *t = tab + 8 * lane;  // 32 g + 8 q
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = e[k];
}

// Places of the entries of v in a word's tables.
__device__ __forceinline__ void table_places(uint64_t v, uint32_t (&at)[kTabGroups]) {
#pragma unroll
    for (int g = 0; g < kTabGroups; ++g) at[g] = 32 * g + ((uint32_t)(v >> (5 * g)) & 31u);
}

// (The scheduling barrier keeps the reads together: left alone the compiler
// waits for each before the next, 750 cycles per word for one wave.)
__device__ __forceinline__ uint64_t table_sum(const uint64_t *tab, const uint32_t (&at)[kTabGroups]) {
    uint64_t e[kTabGroups];
#pragma unroll
    for (int g = 0; g < kTabGroups; ++g) e[g] = tab[at[g]];
    __builtin_amdgcn_sched_barrier(0);
    uint64_t v = e[0];
#pragma unroll
    for (int g = 1; g < kTabGroups; ++g) v ^= e[g];
    return v;
}

// 32 columns of the first 64 listed rows, one row per lane (panel word xh:xl):
// the lowest open row that has the column becomes its pivot, stays in its lane
// and is reduced with the others.
template <bool kHalf>
__device__ __forceinline__ void pivot_columns(uint32_t &xl, uint32_t &xh, uint32_t &col, uint64_t &open,
                                              uint32_t &need) {
#pragma unroll
    for (int c = 0; c < 32; ++c) {
        const uint64_t has = __ballot((kHalf ? xh : xl) & (1u << c));
        const uint64_t cand = has & open;
        if (cand != 0) {  // wave-uniform
            const int L = __builtin_ctzll(cand);
            const uint64_t me = 1ull << L;
            uint32_t m = lane_select(has & ~me, ~0u, 0u);
            asm("" : "+v"(m));  // keep the mask: one instruction per word below
            uint32_t ph = (uint32_t)__builtin_amdgcn_readlane((int)xh, L);
            uint32_t pl = (uint32_t)__builtin_amdgcn_readlane((int)xl, L);
            if (kHalf) ph &= ~(1u << c);
            else pl &= ~(1u << c);
            xh = xor_masked(xh, m, ph);
            xl = xor_masked(xl, m, pl);
            col = lane_select(me, (uint32_t)((kHalf ? 32 : 0) + c), col);
            open &= ~me;
            need &= ~(1u << c);
        }
    }
}

// Step 2, by one wave: the pivots of a panel of kb columns from nc listed
// rows.  Writes tau by column, the rows' pivot columns and returns the pivot
// mask (wave-uniform).
template <int WMAX>
__device__ uint64_t panel_pivots(PanelShared<WMAX> &sm, int nc, int kb, int panel) {
    auto &P = sm.pan;
    const int lane = lane_id();
    const uint64_t all = kb < 64 ? (1ull << kb) - 1 : ~0ull;
    uint32_t xl = 0, xh = 0, row = 0, col = ~0u;
    if (lane < nc) {
        xl = (uint32_t)P.cand_x[lane];
        xh = (uint32_t)(P.cand_x[lane] >> 32);
        row = P.cand_row[lane];
    }
    uint64_t open = __ballot((xl | xh) != 0u);
    uint32_t need_l = (uint32_t)all, need_h = (uint32_t)(all >> 32);  // columns without a pivot yet
    pivot_columns<false>(xl, xh, col, open, need_l);
    pivot_columns<true>(xl, xh, col, open, need_h);
    uint64_t need = ((uint64_t)need_h << 32) | need_l;
    // Further rows, 64 at a time: the basis found so far is added where they
    // have its columns, what is left has entries in columns of `need` only.  A
    // new pivot moves to a lane that holds none.
    for (int first = 64; first < nc && need; first += 64) {
        P.base[lane] = 0;
        wave_lds_sync();
        if (col < 64u) P.base[col] = ((uint64_t)xh << 32) | xl;
        wave_lds_sync();
        fill_tables(P.base, P.btab);
        wave_lds_sync();
        uint64_t y = 0;
        uint32_t yrow = 0;
        if (first + lane < nc) {
            const uint64_t v = P.cand_x[first + lane];
            yrow = P.cand_row[first + lane];
            uint32_t at[kTabGroups];
            table_places(v, at);
            y = (v & need) ^ table_sum(P.btab, at);
        }
        uint64_t left = __ballot((y & need) != 0ull);
        for (uint64_t cols = need; cols && left; cols &= cols - 1) {
            const int c = __builtin_ctzll(cols);
            const uint64_t has = __ballot((y >> c) & 1ull) & left;
            if (has == 0) continue;
            const int L = __builtin_ctzll(has);
            const uint64_t bit = 1ull << c, px = readlane64(y, L), add = px & ~bit;
            const uint32_t prow = (uint32_t)__builtin_amdgcn_readlane((int)yrow, L);
            left &= ~(1ull << L);
            if ((y & bit) && lane != L) y ^= add;
            const uint32_t ma = (((c < 32 ? xl : xh) >> (c & 31)) & 1u) ? ~0u : 0u;
            const uint64_t held = __ballot(col < 64u);
            const uint64_t me = ~held & (held + 1);  // the lowest lane without a pivot
            xl = lane_select(me, (uint32_t)px, xl ^ (ma & (uint32_t)add));
            xh = lane_select(me, (uint32_t)(px >> 32), xh ^ (ma & (uint32_t)(add >> 32)));
            col = lane_select(me, (uint32_t)c, col);
            row = lane_select(me, prow, row);
            need &= ~bit;
            left &= __ballot((y & need) != 0ull);
        }
    }
    const uint64_t found = all & ~need;
    P.tau[lane] = 0;
    wave_lds_sync();
    if (col < 64u) {
        P.tau[col] = (((uint64_t)xh << 32) | xl) & found;
        sm.pivcol[row] = (uint16_t)(64 * panel + (int)col);
    }
    return found;
}

template <int WMAX>
__global__ __launch_bounds__(64 * WMAX) void factor_workgroup_kernel(const uint64_t *__restrict__ rows,
                                                                     int n, int W, FactorOut out,
                                                                     int keep_bad) {
    if (keep_bad && *(volatile int32_t *)out.status != HLF_OK) return;
    using Sm = PanelShared<WMAX>;
    constexpr int ST = Sm::kStride;
    __shared__ Sm sm;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nthr = 64 * W;

    // A into LDS with consecutive loads: this thread's elements tid + k*nthr
    // are word w0 of rows i0 + 64k.
    const int i0 = tid / W, w0 = tid - i0 * W;
    {
        uint64_t v[WMAX];
#pragma unroll
        for (int k = 0; k < WMAX; ++k) v[k] = (k < W && i0 + 64 * k < n) ? rows[tid + k * nthr] : 0ull;
#pragma unroll
        for (int k = 0; k < WMAX; ++k)
            if (k < W) sm.mat[w0 * ST + i0 + 64 * k] = v[k];
    }
    sm.pivcol[tid] = 0xFFFFu;
    sm.qacc[tid] = 0;
    if (tid == 0) {
        sm.bad = 0;
        sm.internal = 0;
        sm.ncand[0] = sm.ncand[1] = 0;
    }
    __syncthreads();
    uint64_t row[WMAX];
#pragma unroll
    for (int w = 0; w < WMAX; ++w) row[w] = w < W ? sm.mat[w * ST + tid] : 0ull;

    // Pad bits, and the symmetry of the tile pairs.
    bool bad = false;
    const uint64_t lm = last_word_mask(n);
#pragma unroll
    for (int w = 0; w < WMAX; ++w) {
        if (w == W - 1 && (row[w] & ~lm)) bad = true;
        if (w == wave) {
            const uint64_t d = __ballot((row[w] >> lane) & 1ull);
            if (lane == 0) sm.diag[wave] = d;
        }
    }
    for (int d = 0; 2 * d <= W; ++d) {  // tile pairs (I, I + d mod W), wave I
        const int J = wave + d < W ? wave + d : wave + d - W;
        if (tile_pair_asym(sm.mat[J * ST + 64 * wave + lane], sm.mat[wave * ST + 64 * J + lane])) bad = true;
    }
    if (bad) sm.bad = 1;
    __syncthreads();
    if (sm.bad) {
        if (tid == 0) {
            *out.status = HLF_ENOTSYM;
            *out.rank = 0;
        }
        return;
    }

    auto &P = sm.pan;
    bool used = false;
    uint64_t x = row[0];  // the panel's word, up to date
    uint64_t t = 0;       // the last panel's tag; its words from p + 1 on are due
    for (int p = 0;; ++p) {
        // 1. the list of panel p
        const bool open = !used && x != 0ull;
        const uint64_t opens = __ballot(open);
        if (opens) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&sm.ncand[p & 1], __builtin_popcountll(opens));
            at = __builtin_amdgcn_readfirstlane(at);
            if (open) {
                at += __builtin_popcountll(opens & ((1ull << lane) - 1ull));
                P.cand_x[at] = x;
                P.cand_row[at] = (uint16_t)tid;
            }
        }
        __syncthreads();
        // 2. its pivots, beside the last panel's words behind it
        if (wave == 0) {
            __builtin_amdgcn_s_setprio(3);
            const int kb = n - 64 * p < 64 ? n - 64 * p : 64;
            const uint64_t found = panel_pivots<WMAX>(sm, __builtin_amdgcn_readfirstlane(sm.ncand[p & 1]), kb, p);
            if (lane == 0) {
                sm.pivots[p] = found;
                sm.ncand[(p + 1) & 1] = 0;
            }
            __builtin_amdgcn_s_setprio(0);
        }
        if (__ballot(t != 0ull)) {
            uint32_t at[kTabGroups];
            table_places(t, at);
#pragma unroll
            for (int w = 0; w < WMAX; ++w)
                if (w > p && w < W) row[w] ^= table_sum(P.tab + w * kTabWords, at);
        }
        t = 0;
        __syncthreads();
        const bool last = p + 1 == W;
        if (sm.pivots[p] != 0) {  // workgroup-uniform
            // 3. the tags; 4. the tables, and the panel's own and the next word
            const uint32_t pc = sm.pivcol[tid];
            const bool fresh = (int)(pc >> 6) == p;
            const int c = (int)(pc & 63u);
            if (fresh) {
                used = true;
#pragma unroll
                for (int w = 0; w < WMAX; ++w)
                    if (w >= p && w < W) P.start[w * 64 + c] = row[w];
            }
            if (wave == W - 1) fill_tables(P.tau, P.ttab);
            __syncthreads();
            uint32_t at[kTabGroups];
            if (fresh) {
                t = P.tau[c] ^ (1ull << c);
            } else if (x) {
                table_places(x, at);
                t = table_sum(P.ttab, at);
            }
            if (p + wave < W) fill_tables(&P.start[(p + wave) * 64], P.tab + (p + wave) * kTabWords);
            __syncthreads();
            if (__ballot(t != 0ull)) {
                table_places(t, at);
#pragma unroll
                for (int w = 0; w < WMAX; ++w)
                    if (w == p || (w == p + 1 && w < W)) row[w] ^= table_sum(P.tab + w * kTabWords, at);
            }
        }
        if (last) break;
#pragma unroll
        for (int w = 1; w < WMAX; ++w)
            if (w == p + 1) x = row[w];
        // the words behind the next panel's own are due, in its step 2
    }
    __syncthreads();

    // The reduced rows by pivot column, zero at the other columns, word-major.
    const uint64_t mine = sm.pivots[wave], lower = (1ull << lane) - 1ull;
    const bool is_piv = (mine >> lane) & 1ull;
    if (!is_piv) {
#pragma unroll
        for (int w = 0; w < WMAX; ++w)
            if (w < W) sm.mat[w * ST + tid] = 0ull;
    }
    if (used) {
        const int pc = sm.pivcol[tid];
#pragma unroll
        for (int w = 0; w < WMAX; ++w)
            if (w < W) sm.mat[w * ST + pc] = row[w];
    }
    // Column tid (its block is `wave`): pivots below it, and the rank.
    int below = __builtin_popcountll(mine & lower), r = 0;
    for (int v = 0; v < W; ++v) {
        const int k = __builtin_popcountll(sm.pivots[v]);
        if (v < wave) below += k;
        r += k;
    }
    if (tid < n) {
        if (is_piv) {
            out.pivots[below] = tid;
            sm.pivlist[below] = (uint16_t)tid;
        }
        if (tid >= r) out.pivots[tid] = -1;
    }
    __syncthreads();
    // B_k = row p_k of A, in consecutive words: loaded here, stored at the end.
    uint64_t bv[WMAX];
#pragma unroll
    for (int k = 0; k < WMAX; ++k) {
        const int i = i0 + 64 * k;
        bv[k] = (k < W && i < r) ? rows[(size_t)sm.pivlist[i] * W + w0] : 0ull;
    }

    // Kernel vectors: entry (c, f) of the reduced rows is entry c of k_f, so
    // transposing every 64x64 tile in place (pairs (I, J), (J, I) together)
    // leaves word I of k_f at mat[I][f]; column f of its own block also gets
    // its bit f.  Words of columns that are not free become 0.
    for (int d = 0; 2 * d <= W; ++d) {  // tile pairs (I, I + d mod W), wave I
        const int I = wave, J = wave + d < W ? wave + d : wave + d - W;
        if (2 * d == W && d && I >= d) break;  // wave J has this pair
        const uint64_t fI = (64 * I + 64 <= n ? ~0ull : lm) & ~sm.pivots[I];
        const uint64_t fJ = (64 * J + 64 <= n ? ~0ull : lm) & ~sm.pivots[J];
        uint64_t ki = 0, kj = 0;
        if (fJ) ki = wave_transpose64(sm.mat[J * ST + 64 * I + lane]);       // word I of k_{64J + lane}
        if (fI && d) kj = wave_transpose64(sm.mat[I * ST + 64 * J + lane]);  // word J of k_{64I + lane}
        if (d == 0) ki |= 1ull << lane;
        if (!((fJ >> lane) & 1ull)) ki = 0;
        if (!((fI >> lane) & 1ull)) kj = 0;
        sm.mat[I * ST + 64 * J + lane] = ki;
        if (d) sm.mat[J * ST + 64 * I + lane] = kj;
    }
    __syncthreads();
    const bool is_free = tid < n && !is_piv;
    if (out.kernel && is_free) {
        const int j = tid - below;
#pragma unroll
        for (int w = 0; w < WMAX; ++w)
            if (w < W) out.kernel[(size_t)j * W + w] = sm.mat[w * ST + tid];
    }

    // q(k_f) = k_f^T A k_f over the integers = 2 (entries of A below the
    // diagonal between members of k_f) + (its members on the diagonal).  Wave
    // v takes rows 64v + lane: their words left of the diagonal against k_f,
    // the parity over its members among them.
    {
        uint64_t a[WMAX];
        bool loaded = false;
        const uint64_t dw = sm.diag[wave];
        for (int J = 0; J < W; ++J) {
            const uint64_t own = sm.mat[wave * ST + 64 * J + lane];  // this wave's word of k_{64J + lane}
            uint64_t todo = __ballot(own != 0ull);
            if (todo && !loaded) {
                loaded = true;
#pragma unroll
                for (int w = 0; w < WMAX; ++w) {
                    a[w] = (tid < n && w <= wave) ? rows[(size_t)tid * W + w] : 0ull;
                    if (w == wave) a[w] &= lower;
                }
            }
            for (; todo; todo &= todo - 1) {
                const int f = __builtin_ctzll(todo);
                const uint64_t members = readlane64(own, f);
                // Words 0 .. wave of k_f, one per lane; most are zero for
                // sparse kernel vectors.
                const uint64_t kw = lane <= wave ? sm.mat[lane * ST + 64 * J + f] : 0ull;
                const uint32_t set = (uint32_t)__ballot(kw != 0ull);
                uint64_t acc = 0;
#pragma unroll
                for (int w = 0; w < WMAX; ++w)
                    if ((set >> w) & 1u) acc ^= a[w] & readlane64(kw, w);
                const uint64_t odd = __ballot(__builtin_popcountll(acc) & 1) & members;
                const int q = 2 * (__builtin_popcountll(odd) & 1) + __builtin_popcountll(members & dw);
                if (lane == 0 && q) atomicAdd(&sm.qacc[64 * J + f], q);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < WMAX; ++k)
        if (k < W && i0 + 64 * k < r) out.basis[tid + k * nthr] = bv[k];
    __syncthreads();
    {
        const int q = is_free ? sm.qacc[tid] : 0;
        const uint64_t sw = __ballot(q & 2);
        if (lane == 0) out.shift[wave] = sw;
        if (q & 1) sm.internal = 1;
    }
    __syncthreads();
    if (tid == 0) {
        *out.rank = r;
        *out.status = sm.internal ? HLF_EINTERNAL : HLF_OK;
    }
}

template <int WMAX>
hlf_status launch_wave_t(const uint64_t *rows, int n, int W, const FactorOut &out, int keep_bad,
                         hipStream_t stream) {
    hipLaunchKernelGGL(factor_wave_kernel<WMAX>, dim3(1), dim3(64), 0, stream, rows, n, W, out,
                       keep_bad);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int WMAX>
hlf_status launch_workgroup_t(const uint64_t *rows, int n, int W, const FactorOut &out,
                              int keep_bad, hipStream_t stream) {
    hipLaunchKernelGGL(factor_workgroup_kernel<WMAX>, dim3(1), dim3(64 * W), 0, stream, rows, n,
                       W, out, keep_bad);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

}  // namespace

hlf_status launch_pack(const uint8_t *A, int n, int W, uint64_t *rows, int32_t *status,
                       hipStream_t stream) {
    if (W >= 2) {
        const int vec16 = ((n & 15) == 0 && ((uintptr_t)A & 15u) == 0) ? 1 : 0;
        const unsigned blocks = (unsigned)((n + kPackRowsPerBlock - 1) / kPackRowsPerBlock);
        hipLaunchKernelGGL(pack_rows_kernel, dim3(blocks), dim3(kPackRowsThreads), 0, stream, A, n, W,
                           vec16, rows, status);
        if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
        hipLaunchKernelGGL(pack_check_kernel, dim3((unsigned)((W * (W / 2 + 1) + kCheckWaves - 1) / kCheckWaves)),
                           dim3(64 * kCheckWaves), 0, stream, rows, n, W, status);
        return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
    }
    hipLaunchKernelGGL(pack_dense_kernel, dim3(1), dim3(64), 0, stream, A, n, rows, status);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

hlf_status launch_factor(const uint64_t *rows, int n, int W, const FactorOut &out,
                         bool force_workgroup, bool keep_pack_status, hipStream_t stream) {
    const int kb = keep_pack_status ? 1 : 0;
    // One wave is faster up to n = 64; from two words on, the blocked
    // workgroup elimination is.
    if (!force_workgroup && W == 1) return launch_wave_t<1>(rows, n, W, out, kb, stream);
    if (W <= 1) return launch_workgroup_t<1>(rows, n, W, out, kb, stream);
    if (W <= 2) return launch_workgroup_t<2>(rows, n, W, out, kb, stream);
    if (W <= 4) return launch_workgroup_t<4>(rows, n, W, out, kb, stream);
    if (W <= 8) return launch_workgroup_t<8>(rows, n, W, out, kb, stream);
    return launch_workgroup_t<16>(rows, n, W, out, kb, stream);
}

}  // namespace hlf
