// Stage 1 (the paper's CLA module, Section 2, tasks (1)-(4)) for one
// instance with n <= 64*WMAX (WMAX in {1,2,3}) on one wavefront.
//
// Lane l holds rows l, l+64, l+128 ("slots") in VGPRs.  Gauss-Jordan over
// GF(2), column by column: a ballot per slot finds the rows with the column
// set, readlane broadcasts one, and it is XORed into every row that has the
// column -- itself included, which takes it off the list -- and kept in a
// second set of registers, the reduced pivot rows, under the lane and slot
// of its column, where later columns are eliminated the same way.  No
// barrier, no LDS.  Those registers, transposed across the wave, are the
// Ker(A) basis (task (2)); q on it (task (3)) and the canonical shift (task
// (4)) take one uniform step per free column.
//
// Bound by one wave's chain of instructions, which issue one in about five
// cycles: some 175 cycles a column at n <= 64 (425 with the candidates, the
// rank and the lists kept per lane and in LDS), 0.8 us to read A (1.6 us at
// n = 16 and 4.8 at n = 64 with one byte per lane and load).  The whole of a
// small solve is 9.0 k cycles at n = 16 (15.8 k) and 18.2 k at n = 64 (42.1 k).
//
// Only the calling wave takes part (LDS ordering by wave_lds_sync), so the
// routine can run on one wave of a larger workgroup.
#pragma once

#include <type_traits>

#include "hlf_device.h"
#include "hlf_internal.h"

namespace hlf {

template <int WMAX>
struct WaveSmem {
    uint64_t orig[64 * WMAX * WMAX];           // A, packed rows of W words
    uint32_t stream[128 * WMAX * WMAX + 2];    // A's entries, one bit each, row after row
    int piv[64 * WMAX];
    unsigned long long shiftw[WMAX];
};

// Packed rows from global memory into sm.orig.
template <int WMAX>
__device__ __forceinline__ void wave_load_rows(const uint64_t *__restrict__ rows, int n, int W,
                                               WaveSmem<WMAX> &sm) {
    for (int idx = lane_id(); idx < n * W; idx += 64) sm.orig[idx] = rows[idx];
}

// Dense row-major uint8 matrix into sm.orig: 16 consecutive entries per lane
// and load, at any address, kBatch loads in flight; each becomes 16 bits of
// the stream, and lane i then cuts rows i, i + 64, .. out of it.  The last
// load ends with the matrix and is shifted into place.  Four 0/1 bytes x
// become four bits as (x * 0x10204080) >> 28 (no carries reach bits 28..31).
// Returns true on every lane if an entry is not 0/1.
template <int WMAX>
__device__ __forceinline__ bool wave_load_dense(const uint8_t *__restrict__ A, int n, int W,
                                                WaveSmem<WMAX> &sm) {
    typedef u32x4 quad_any __attribute__((aligned(1)));
    constexpr int kBatch = WMAX == 1 ? 4 : 9;
    const int lane = lane_id();
    const int nn = n * n;
    uint16_t *s16 = reinterpret_cast<uint16_t *>(sm.stream);
    bool bad = false;
    if (nn < 16) {
        const uint32_t v = lane < nn ? (uint32_t)A[lane] : 0u;
        bad = v > 1u;
        const uint64_t bits = __ballot(v == 1u);
        if (lane == 0) sm.stream[0] = (uint32_t)bits;
    } else {
        for (int q0 = 0; 16 * q0 < nn; q0 += 64 * kBatch) {
            u32x4 v[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int at = min(16 * (q0 + 64 * k + lane), nn - 16);
                v[k] = *reinterpret_cast<const quad_any *>(A + at);
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int q = q0 + 64 * k + lane;
                bad |= ((v[k].x | v[k].y | v[k].z | v[k].w) & 0xFEFEFEFEu) != 0;
                const uint32_t bits = (v[k].x * 0x10204080u) >> 28 | (v[k].y * 0x10204080u) >> 28 << 4 |
                                      (v[k].z * 0x10204080u) >> 28 << 8 | (v[k].w * 0x10204080u) >> 28 << 12;
                if (16 * q < nn) s16[q] = (uint16_t)(bits >> max(16 * q + 16 - nn, 0));
            }
        }
    }
    wave_lds_sync();
    const uint64_t lm = last_word_mask(n);
#pragma unroll
    for (int s = 0; s < WMAX; ++s) {
        const int i = 64 * s + lane;
        if (i < n) {
#pragma unroll
            for (int w = 0; w < WMAX; ++w) {
                if (w >= W) break;
                const int bit = i * n + 64 * w, d = bit >> 5, sh = bit & 31;  // words past the stream: masked off
                const uint32_t a = sm.stream[d], b = sm.stream[d + 1], c = sm.stream[d + 2];
                const uint64_t v = (uint64_t)__builtin_amdgcn_alignbit(c, b, sh) << 32 |
                                   (uint32_t)__builtin_amdgcn_alignbit(b, a, sh);
                sm.orig[i * W + w] = w == W - 1 ? v & lm : v;
            }
        }
    }
    return __ballot(bad) != 0;
}

// The elimination for exactly W words a row.
template <int W, class Smem>
__device__ int factor_wave_words(int n, bool bad_input, const FactorOut &out, Smem &sm) {
    const int lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    wave_lds_sync();
    uint32_t x[W][2 * W];  // rows, as dwords
    bool bad = bad_input;
    {
        uint64_t row[W][W];
#pragma unroll
        for (int s = 0; s < W; ++s) {
            const int i = s * 64 + lane;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                row[s][w] = i < n ? sm.orig[i * W + w] : 0ull;
                x[s][2 * w] = (uint32_t)row[s][w];
                x[s][2 * w + 1] = (uint32_t)(row[s][w] >> 32);
            }
            if (row[s][W - 1] & ~last_word_mask(n)) bad = true;  // pad bits
        }
        // A = A^T, tile pair by tile pair
#pragma unroll
        for (int s = 0; s < W; ++s)
#pragma unroll
            for (int w = s; w < W; ++w)
                if (wave_transpose64(row[s][w]) != row[w][s]) bad = true;
    }
    if (__ballot(bad)) {
        if (lane == 0) {
            *out.rank = 0;
            *out.status = HLF_ENOTSYM;
        }
        return -1;
    }

    // Column c: a row that has it, px, is XORed into every row and every
    // pivot row that has it.  Words left of the column are zero in px.
    uint32_t p[W][2 * W];  // pivot rows: that of column 64s + l in slot s, lane l
    uint64_t pivots[W];    // columns that have one
#pragma unroll
    for (int s = 0; s < W; ++s) {
        pivots[s] = 0;
#pragma unroll
        for (int d = 0; d < 2 * W; ++d) p[s][d] = 0;
    }
#pragma unroll
    for (int h = 0; h < 2 * W; ++h) {
        const int cols = min(32, n - 32 * h);
        uint32_t found = 0;
        for (int b = 0; b < cols; ++b) {
            uint32_t m[W];
            uint64_t has[W], any = 0;
#pragma unroll
            for (int s = 0; s < W; ++s) {
                m[s] = (uint32_t)__builtin_amdgcn_sbfe((int)x[s][h], b, 1);
                has[s] = __ballot(m[s] != 0u);
                any |= has[s];
            }
            if (any == 0) continue;  // a free column
            uint32_t px[2 * W];
            auto take = [&](auto slot) {  // a branch per slot: merged, they would index x in memory
                constexpr int s = decltype(slot)::value;
                if constexpr (W > 1) asm volatile("; slot %0" ::"n"(s));
                const int at = __builtin_ctzll(has[s]);
#pragma unroll
                for (int d = h; d < 2 * W; ++d) px[d] = (uint32_t)__builtin_amdgcn_readlane((int)x[s][d], at);
            };
            if (W == 1 || has[0] != 0)
                take(std::integral_constant<int, 0>{});
            else if (W == 2 || has[1 % W] != 0)
                take(std::integral_constant<int, 1 % W>{});
            else
                take(std::integral_constant<int, 2 % W>{});
            found |= 1u << b;
#pragma unroll
            for (int s = 0; s < W; ++s)
#pragma unroll
                for (int d = h; d < 2 * W; ++d) x[s][d] = __builtin_amdgcn_bitop3_b32(x[s][d], m[s], px[d], 0x78);
            const bool mine = lane == 32 * (h & 1) + b;
#pragma unroll
            for (int s = 0; s <= h / 2; ++s) {
                const uint32_t mp = (uint32_t)__builtin_amdgcn_sbfe((int)p[s][h], b, 1);
#pragma unroll
                for (int d = h; d < 2 * W; ++d) {
                    const uint32_t v = __builtin_amdgcn_bitop3_b32(p[s][d], mp, px[d], 0x78);
                    p[s][d] = s == h / 2 && mine ? px[d] : v;
                }
            }
        }
        pivots[h >> 1] |= (uint64_t)found << (32 * (h & 1));
    }

    int r = 0;
#pragma unroll
    for (int s = 0; s < W; ++s) {
        const int c = 64 * s + lane, k = r + __builtin_popcountll(pivots[s] & below);
        if ((pivots[s] >> lane) & 1ull) {
            sm.piv[k] = c;
            out.pivots[k] = c;
#pragma unroll
            for (int w = 0; w < W; ++w) out.basis[k * W + w] = sm.orig[c * W + w];
        }
        r += __builtin_popcountll(pivots[s]);
    }
    for (int k = r + lane; k < n; k += 64) out.pivots[k] = -1;
    // Lane f of the transposed pivot rows holds column f, whose bit c is entry
    // f of column c's pivot row: k_f = e_f | column f.
    uint64_t shiftbits[W];
    bool internal = false;
#pragma unroll
    for (int t = 0; t < W; ++t) shiftbits[t] = 0;
    if (r < n) {
        uint64_t a[W][W];  // A again
#pragma unroll
        for (int s = 0; s < W; ++s)
#pragma unroll
            for (int w = 0; w < W; ++w) a[s][w] = 64 * s + lane < n ? sm.orig[(64 * s + lane) * W + w] : 0ull;
        int before = 0;  // free columns of the words before
#pragma unroll
        for (int t = 0; t < W; ++t) {
            const uint64_t cols = 64 * t + 64 <= n ? ~0ull : 64 * t < n ? (1ull << (n & 63)) - 1ull : 0ull;
            const uint64_t free = cols & ~pivots[t];
            if (free == 0) continue;
            const bool is_free = (free >> lane) & 1ull;
            uint64_t kv[W];
#pragma unroll
            for (int u = 0; u < W; ++u) {
                kv[u] = wave_transpose64((uint64_t)p[u][2 * t + 1] << 32 | p[u][2 * t]);
                if (u == t) kv[u] |= 1ull << lane;
            }
            if (out.kernel && is_free) {
                const int j = before + __builtin_popcountll(free & below);
#pragma unroll
                for (int u = 0; u < W; ++u) out.kernel[j * W + u] = kv[u];
            }
            before += __builtin_popcountll(free);
            // q(k_f) = sum over i in supp k_f of popcount(A_i & k_f): every
            // term is even (A k_f = 0 mod 2), so bit 1 of the sum is the
            // parity of the terms = 2 mod 4.
            for (uint64_t fm = free; fm; fm &= fm - 1ull) {
                const int f = __builtin_ctzll(fm);
                uint64_t k[W];
#pragma unroll
                for (int u = 0; u < W; ++u) k[u] = readlane64(kv[u], f);
                uint32_t twos = 0, ones = 0;
#pragma unroll
                for (int s = 0; s < W; ++s) {
                    uint32_t term = 0;
#pragma unroll
                    for (int u = 0; u < W; ++u) term += (uint32_t)__builtin_popcountll(a[s][u] & k[u]);
                    if (!((k[s] >> lane) & 1ull)) term = 0;
                    twos ^= term;
                    ones |= term;
                }
                if (__ballot(ones & 1u)) internal = true;
                if (__builtin_popcountll(__ballot(twos & 2u)) & 1) shiftbits[t] |= 1ull << f;
            }
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int t = 0; t < W; ++t) {
            sm.shiftw[t] = shiftbits[t];
            out.shift[t] = shiftbits[t];
        }
        *out.rank = r;
        *out.status = internal ? HLF_EINTERNAL : HLF_OK;
    }
    wave_lds_sync();
    return internal ? -1 : r;
}

// Factor the matrix in sm.orig.  `bad_input` forces HLF_ENOTSYM.  Returns the
// rank, or -1 if the record was marked invalid.
template <int WMAX>
__device__ int factor_wave_core(int n, int W, bool bad_input, const FactorOut &out,
                                WaveSmem<WMAX> &sm) {
    if constexpr (WMAX >= 3)
        if (W == 3) return factor_wave_words<3>(n, bad_input, out, sm);
    if constexpr (WMAX >= 2)
        if (W == 2) return factor_wave_words<2>(n, bad_input, out, sm);
    return factor_wave_words<1>(n, bad_input, out, sm);
}

}  // namespace hlf
