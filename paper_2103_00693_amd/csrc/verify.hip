// Verification data for a cross-entropy benchmark of a device that runs the
// circuit (Section 5): exact pair statistics of a uniform solution, and the
// membership test that gives the ideal probability 2^-r of a sampled string
// (Section 1's definition of a solution, App. A's output distribution).
#include <type_traits>
#include <utility>

#include "hlf_device.h"
#include "hlf_internal.h"

namespace hlf {
namespace {

// Row i per workgroup: quarters[i*n + j] = 0 if A_i = 0 or A_j = 0, 2 if
// A_i = A_j != 0, else 1.  z = l ^ XOR_k c_k B_k with c uniform makes
// coordinate i the functional c -> l_i ^ <c, beta_i>, beta_i = row i of A at
// the pivot columns; the pivot columns are an information set of the row
// space, so beta_i = beta_j exactly when A_i = A_j, and beta_i = 0 exactly
// when A_i = 0 (then l_i = 0: e_i is in Ker(A) with q(e_i) = A_ii = 0).
template <int WMAX>
__global__ __launch_bounds__(256) void pair_stats_kernel(FactorIn f, const uint64_t *__restrict__ rows,
                                                         uint8_t *__restrict__ quarters) {
    if (*(volatile int32_t *)f.status != HLF_OK) return;
    const int n = f.n, W = f.words;
    const int i = blockIdx.x;
    __shared__ uint64_t ri[WMAX];
    __shared__ int nz_i;
    if (threadIdx.x == 0) nz_i = 0;
    __syncthreads();
    if ((int)threadIdx.x < W) {
        const uint64_t v = rows[(size_t)i * W + threadIdx.x];
        ri[threadIdx.x] = v;
        if (v) atomicOr(&nz_i, 1);
    }
    __syncthreads();
    const bool nzi = nz_i != 0;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        uint64_t diff = 0, orj = 0;
#pragma unroll
        for (int w = 0; w < WMAX; ++w) {
            if (w < W) {
                const uint64_t x = rows[(size_t)j * W + w];
                diff |= x ^ ri[w];
                orj |= x;
            }
        }
        quarters[(size_t)i * n + j] = (!nzi || !orj) ? 0 : (diff == 0 ? 2 : 1);
    }
}

typedef int m4i __attribute__((ext_vector_type(4)));
typedef int m8i __attribute__((ext_vector_type(8)));
typedef float m16f __attribute__((ext_vector_type(16)));

// Pair statistics on the matrix cores (n > 64): quarters[i][j] needs |A_i|,
// |A_j| and the integer dot product popcount(A_i & A_j) (rows equal exactly
// when all three agree), and the dot products of all row pairs are the
// product of the packed rows with their transpose.  One wave per 32 x 32 tile
// of (i, j): v_mfma_scale_f32_32x32x64_f8f6f4 with E2M1 operands whose
// set-bit products are exactly 1 (the i rows at nibble positions 2, 1, 0, 0,
// the j rows at 0, 1, 2, 2 for bits 4t + 0..3), so the fp32 sums are the
// counts.  K chunk w is row word w; lane half h takes its 32-bit half.
// Accumulator register q of lane l holds the count of rows i = 32bi + 8(q/4)
// + 4(l/32) + q%4 and j = 32bj + l%32.
constexpr int kPairWaves = 4;

__global__ __launch_bounds__(64 * kPairWaves) void pair_stats_mfma_kernel(
    FactorIn f, const uint64_t *__restrict__ rows, uint8_t *__restrict__ quarters) {
    __shared__ uint32_t pci[kPairWaves][32];
    if (*(volatile int32_t *)f.status != HLF_OK) return;
    const int n = f.n, W = f.words;
    const int nb = (n + 31) >> 5;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, m = lane & 31;
    const int t = blockIdx.x * kPairWaves + wave;  // tile index, wave-uniform
    if (t >= nb * nb) return;                      // no barrier below
    const int bi = t / nb, bj = t - bi * nb;
    const int i = 32 * bi + m, j = 32 * bj + m;    // this lane's rows
    // words 2p + h of rows i and j, all loads at once
    uint64_t xi[HLF_MAX_N / 128], xj[HLF_MAX_N / 128];
    uint32_t pi = 0, pj = 0;
#pragma unroll
    for (int p = 0; p < HLF_MAX_N / 128; ++p) {
        const int w = 2 * p + h;
        xi[p] = (i < n && w < W) ? rows[(size_t)i * W + w] : 0ull;
        xj[p] = (j < n && w < W) ? rows[(size_t)j * W + w] : 0ull;
        pi += (uint32_t)__builtin_popcountll(xi[p]);
        pj += (uint32_t)__builtin_popcountll(xj[p]);
    }
    // whole-row popcounts: add the other half's words (lane l ^ 32)
    pi += __builtin_amdgcn_permlane32_swap(pi, pi, false, false)[h ? 0 : 1];
    pj += __builtin_amdgcn_permlane32_swap(pj, pj, false, false)[h ? 0 : 1];
    if (lane < 32) pci[wave][m] = pi;
    m16f acc;
    auto chunk = [&](int w, uint32_t yi, uint32_t yj) {
        const m8i a = {(int)((yi & 0x11111111u) << 2), (int)(yi & 0x22222222u),
                       (int)((yi & 0x44444444u) >> 2), (int)((yi & 0x88888888u) >> 3), 0, 0, 0, 0};
        const m8i b = {(int)(yj & 0x11111111u), (int)(yj & 0x22222222u),
                       (int)(yj & 0x44444444u), (int)((yj >> 1) & 0x44444444u), 0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, w == 0 ? m16f{} : acc, 4, 4, 0, 127,
                                                             0, 127);
    };
#pragma unroll
    for (int p = 0; p < HLF_MAX_N / 128; ++p) {
        if (2 * p < W) {
            const auto yi = __builtin_amdgcn_permlane32_swap((uint32_t)xi[p], (uint32_t)(xi[p] >> 32), false, false);
            const auto yj = __builtin_amdgcn_permlane32_swap((uint32_t)xj[p], (uint32_t)(xj[p] >> 32), false, false);
            chunk(2 * p, yi[0], yj[0]);
            if (2 * p + 1 < W) chunk(2 * p + 1, yi[1], yj[1]);
        }
    }
    wave_lds_sync();  // pci of this wave written above
    if (j < n) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int mi = 8 * (q >> 2) + 4 * h + (q & 3);
            const int ii = 32 * bi + mi;
            if (ii < n) {
                const uint32_t c = (uint32_t)acc[q], ni = pci[wave][mi];
                quarters[(size_t)ii * n + j] = (ni == 0u || pj == 0u) ? 0 : (ni == pj && c == ni) ? 2 : 1;
            }
        }
    }
}

// Membership for n > 192, on the matrix cores: the parities <k_j, z_s> of all
// kernel vectors are the GF(2) product of the strings (num x n) and the kernel
// basis transposed (n x (n - r)), computed as in the sampler:
// v_mfma_scale_f32_32x32x64_f8f6f4 with E2M1 operands whose set-bit products
// are exactly 1, fp32 sums that are integer counts, bit 0 their parity.
//
// A wave takes 64 strings, as two blocks of 32 that share every read of the
// kernel operand from LDS.  Lane (h, m) loads half of string m's (32 + m's)
// words, 16 bytes at a time, and the K chunks are numbered by what it then
// holds: chunk c of half h is dword string_dword<W>(c, h), nibble t of operand
// dword d its bit 4t + d.  The kernel vectors are encoded in the same order
// once per workgroup, up to 256 at a time for n = 1024 (all of them up to
// n = 512); every further group takes the strings again, leaves those that have
// failed, and is not begun by a workgroup that has none left.  The product is taken with the kernel operand first, so
// accumulator register i of lane l holds the count of kernel vector
// 8(i/4) + 4(l/32) + i%4 of its 32-chunk for string l % 32.  Two chunks share
// an accumulator: the first K chunk adds to 2^23 and the second chunk of a
// pair carries the scale 2^11, so a sum is 2^23 + c + 2^11 c' (c, c' <= n <=
// 1024) and its raw bits 0 and 11 are the two parities.
//
// Bound by the matrix cores and by what each block costs besides: n = 1024,
// n - r = 95, 2^20 strings take 43 us, of which the products are 20.5 (1.6 M
// instructions of 32 cycles), the launch and the operand about 7, reading the
// strings (134 MB, 19 us) being hidden.  With one block of 32 strings a wave,
// words loaded 8 bytes at a time, and a second launch for other n - r: 51 us;
// n - r = 221: 76 us, and 232 with that second, one-thread-per-string kernel.
// 2^20 uniform strings, which fail at once, n - r = 724: 30 us, and 69 where
// all three groups are laid out whether or not a string is left.
constexpr int kMemMfmaMinWords = 4;
// Waves per workgroup (one workgroup per CU): what the registers allow.
template <int W>
constexpr int kMemWavesOf = W <= 6 ? 12 : 8;

// The dword of a string (W words) that lane half h holds as its c-th: two
// words (16 bytes) of every four, then one word of two, then half a word.
template <int W>
__device__ __forceinline__ constexpr int string_dword(int c, int h) {
    constexpr int Q = W / 4, R = W % 4;
    if (c < 4 * Q) return 8 * (c >> 2) + 4 * h + (c & 3);
    if (R >= 2 && c < 4 * Q + 2) return 8 * Q + 2 * h + (c - 4 * Q);
    return 2 * (W - 1) + h;
}

// A string's dwords in that order.  Strings are only 8-byte aligned, which the
// 16-byte loads allow.
template <int W>
__device__ __forceinline__ void load_string(const uint64_t *z, int h, uint32_t (&y)[W]) {
    typedef uint32_t quad __attribute__((ext_vector_type(4), aligned(8)));
    constexpr int Q = W / 4, R = W % 4;
    const uint32_t *z32 = reinterpret_cast<const uint32_t *>(z);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const quad v = *reinterpret_cast<const quad *>(z32 + 8 * q + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) y[4 * q + e] = v[e];
    }
    if constexpr (R >= 2) {
        const uint64_t v = z[4 * Q + h];
        y[4 * Q] = (uint32_t)v;
        y[4 * Q + 1] = (uint32_t)(v >> 32);
    }
    if constexpr (R & 1) y[W - 1] = z32[2 * (W - 1) + h];
}

template <int W>
__global__ __launch_bounds__(64 * kMemWavesOf<W>) void membership_mfma_kernel(
    FactorIn f, const uint64_t *__restrict__ kernel, const uint64_t *__restrict__ z, uint64_t num,
    uint8_t *__restrict__ member) {
    constexpr int kMemWaves = kMemWavesOf<W>;
    constexpr int kAll = 2 * W, kFit = (128 / W) & ~1;
    constexpr int JC = kAll < kFit ? kAll : kFit;  // 32-vector chunks per group, even
    __shared__ __align__(16) uint32_t Bop[W * JC * 64 * 4];
    __shared__ uint32_t target[JC];
    __shared__ uint32_t taken;  // blocks of this workgroup that waves have claimed
    const int status = *(volatile int32_t *)f.status, nk = f.n - *(volatile int32_t *)f.rank;
    if (status != HLF_OK) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, m = lane & 31;
    m16f magic;
#pragma unroll
    for (int i = 0; i < 16; ++i) magic[i] = 8388608.0f;  // 2^23
    auto op8 = [](m4i v) { return m8i{v[0], v[1], v[2], v[3], 0, 0, 0, 0}; };
    auto encode = [](uint32_t v) {
        return m8i{(int)(v & 0x11111111u), (int)(v & 0x22222222u), (int)(v & 0x44444444u),
                   (int)((v >> 1) & 0x44444444u), 0, 0, 0, 0};
    };
    auto multiply = [](m8i b, m8i a, m16f c, auto scale) {
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b, a, c, 4, 4, 0, decltype(scale)::value, 0, 127);
    };
    uint32_t emask[4], erot0[4], erot1[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t sh = (uint32_t)(u + 4 * h);
        emask[u] = 0x01010101u << sh;
        erot0[u] = (32u - sh) & 31u;  // rotate right: bit 0 of each byte to bit sh
        erot1[u] = (35u - sh) & 31u;  // bit 3 of each byte to bit sh
    }
    const uint64_t nblk = (num + 63) >> 6;
    const uint64_t per_wg = (nblk + gridDim.x - 1) / gridDim.x;
    const uint64_t blk0 = (uint64_t)blockIdx.x * per_wg;
    const uint32_t blocks = blk0 < nblk ? (uint32_t)min(nblk - blk0, per_wg) : 0u;
    if (nk == 0) {  // every string is a solution
        const uint64_t all = (uint64_t)gridDim.x * blockDim.x;
        for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + tid; s < num; s += all) member[s] = 1;
        return;
    }
    // A block's strings are loaded while the one before it is multiplied, the
    // first block's while the operand is laid out.
    uint32_t next[2][W] = {};
    auto fetch = [&](uint32_t i) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint64_t s = min(64 * (blk0 + i) + (uint64_t)(32 * k + m), num - 1);
            load_string<W>(z + s * W, h, next[k]);
        }
    };
    int j0 = 0;          // the group's first kernel vector
    uint64_t alive = 0;  // lanes that have seen a string pass the group
    do {
        const int left = min(nk - j0, 32 * JC);
        const int jcs = (left + 31) >> 5;  // 32-vector chunks in use
        const bool first = j0 == 0;
        if (tid < JC) target[tid] = 0;
        if (tid == 0) taken = kMemWaves;
        __syncthreads();
        // Kernel operand of chunk (c, jc): lane (h, m), dword d, nibble t holds
        // bit 4t + d of dword string_dword(c, h) of k_{j0+32jc+m} at nibble
        // position 2, 1, 0, 0 for d = 0, 1, 2, 3 (0 beyond n - r).  Target bit
        // j is <k_j, l> (mod 2).  A wave takes half of a chunk's words; its
        // first strings are asked for behind its first kernel words.
        const uint32_t *l32 = reinterpret_cast<const uint32_t *>(f.shift);
        for (int t = wave; t < max(2 * jcs, kMemWaves); t += kMemWaves) {
            const int jc = t >> 1, j = 32 * jc + m;
            const uint32_t *kj = reinterpret_cast<const uint32_t *>(kernel + (size_t)(j0 + min(j, left - 1)) * W);
            constexpr int H = (W + 1) / 2;
            uint32_t y[H], l[H];
#pragma unroll
            for (int u = 0; u < H; ++u) {
                const int d = string_dword<W>(min((t & 1) * H + u, W - 1), h);
                y[u] = kj[d];
                l[u] = l32[d];
            }
            if (t == wave && (uint32_t)wave < blocks) fetch((uint32_t)wave);
            if (t >= 2 * jcs) break;
            uint32_t dot = 0;
#pragma unroll
            for (int u = 0; u < H; ++u) {
                const int c = (t & 1) * H + u;
                if (c >= W) break;
                if (j >= left) y[u] = 0;
                dot ^= y[u] & l[u];
                uint32_t *dst = &Bop[((size_t)(c * JC + jc) * 64 + lane) * 4];
                dst[0] = (y[u] & 0x11111111u) << 2;
                dst[1] = y[u] & 0x22222222u;
                dst[2] = (y[u] & 0x44444444u) >> 2;
                dst[3] = (y[u] & 0x88888888u) >> 3;
            }
            const uint64_t odd = __ballot(__builtin_popcount(dot) & 1);
            if (lane == 0) atomicXor(&target[jc], (uint32_t)odd ^ (uint32_t)(odd >> 32));
        }
        __syncthreads();
        alive = 0;
        for (uint32_t i = (uint32_t)wave, then; i < blocks; i = then) {
            const uint64_t so = 64 * (blk0 + i) + (uint64_t)lane;  // the string this lane stores
            const bool live = so < num;
            uint32_t y[2][W];
#pragma unroll
            for (int c = 0; c < W; ++c) {
                y[0][c] = next[0][c];
                y[1][c] = next[1][c];
            }
            uint32_t claim = 0;
            if (lane == 0) claim = atomicAdd(&taken, 1u);
            then = (uint32_t)__builtin_amdgcn_readfirstlane((int)claim);
            if (then < blocks) fetch(then);
            if (!first && __ballot(live && member[so] != 0) == 0) continue;
            uint32_t bad[2] = {0u, 0u};
            // An odd chunk first, then pairs, until all 64 strings have failed.
            for (int jc = 0, wide; jc < jcs; jc += wide) {
                wide = jc == 0 && (jcs & 1) ? 1 : 2;
                m16f acc[2];
                auto product = [&](auto two) {
                    constexpr bool kTwo = decltype(two)::value;
                    const uint32_t *src = &Bop[((size_t)jc * 64 + lane) * 4];
                    m4i b0 = *reinterpret_cast<const m4i *>(src), b1{};
                    if (kTwo) b1 = *reinterpret_cast<const m4i *>(src + 256);
                    m8i e[2] = {encode(y[0][0]), encode(y[1][0])};
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        // the next word's operands are read and encoded while
                        // this one's are multiplied
                        const m8i q0 = op8(b0), q1 = op8(b1), e0 = e[0], e1 = e[1];
                        if (c + 1 < W) {
                            src += JC * 256;
                            b0 = *reinterpret_cast<const m4i *>(src);
                            if (kTwo) b1 = *reinterpret_cast<const m4i *>(src + 256);
                            // here, and for every pair again: the encodings of
                            // all words together would not fit the registers
                            asm volatile("" : "+v"(y[0][c + 1]), "+v"(y[1][c + 1]));
                            e[0] = encode(y[0][c + 1]);
                            e[1] = encode(y[1][c + 1]);
                        }
                        acc[0] = multiply(q0, e0, c == 0 ? magic : acc[0], std::integral_constant<int, 127>{});
                        acc[1] = multiply(q0, e1, c == 0 ? magic : acc[1], std::integral_constant<int, 127>{});
                        if (kTwo) {
                            acc[0] = multiply(q1, e0, acc[0], std::integral_constant<int, 138>{});
                            acc[1] = multiply(q1, e1, acc[1], std::integral_constant<int, 138>{});
                        }
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
#pragma unroll
                        for (int k = 0; k < (kTwo ? 4 : 2); ++k) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);              // one product
                            __builtin_amdgcn_sched_group_barrier(0x002, kTwo ? 3 : 5, 0);  // encoding
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if (wide == 2)
                    product(std::true_type{});
                else
                    product(std::false_type{});
                // Register i = 4t + u holds the counts of vector 8t + 4h + u of
                // both chunks: byte permutes gather bytes 0 (bit 0) and 1 (bit
                // 11 = bit 3 of byte 1) of registers u, 4+u, 8+u, 12+u, a
                // rotation and a mask put each parity at bit 8t + 4h + u, and
                // one swap leaves lane (h, m) the 32 parities of chunk jc + h.
                const int vectors = h < wide ? left - 32 * (jc + h) : 0;
                const uint32_t valid = vectors >= 32 ? ~0u : vectors > 0 ? (1u << vectors) - 1u : 0u;
                const uint32_t tgt = target[min(jc + h, JC - 1)];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    uint32_t r[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) r[i] = __float_as_uint(acc[k][i]);
                    uint32_t lo = 0u, hi = 0u;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t P = __builtin_amdgcn_perm(r[4 + u], r[u], 0x05010400u);
                        const uint32_t Q = __builtin_amdgcn_perm(r[12 + u], r[8 + u], 0x05010400u);
                        const uint32_t R = __builtin_amdgcn_perm(Q, P, 0x05040100u);  // bytes 0
                        const uint32_t S = __builtin_amdgcn_perm(Q, P, 0x07060302u);  // bytes 1
                        lo |= __builtin_amdgcn_alignbit(R, R, erot0[u]) & emask[u];
                        hi |= __builtin_amdgcn_alignbit(S, S, erot1[u]) & emask[u];
                    }
                    const auto sw = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
                    bad[k] |= ((sw[0] | sw[1]) ^ tgt) & valid;
                }
                const uint64_t b0 = __ballot(bad[0] != 0), b1 = __ballot(bad[1] != 0);
                if ((uint32_t)((b0 | b0 >> 32) & (b1 | b1 >> 32)) == ~0u) break;
            }
            // lane l takes both halves' verdicts of string l
            const auto sw = __builtin_amdgcn_permlane32_swap(bad[0], bad[1], false, false);
            const uint32_t verdict = sw[0] | sw[1];
            if (live && (first || verdict)) member[so] = verdict ? 0 : 1;
            if (j0 + 32 * JC < nk) alive |= __ballot(live && verdict == 0);
        }
        j0 += 32 * JC;
        // Another group only for strings that have passed so far.  (The barrier
        // also says that this group's operand has been read.)
    } while (j0 < nk && __syncthreads_or(alive != 0));
}

// n <= 192, one thread per string: member[s] = 1 iff <k_j, z_s> = <k_j, l>
// (mod 2) for every kernel vector k_j, j < n - r.  <k_j, l> = l_{f_j} because
// k_j is 1 at its free column f_j, 0 at the other free columns, and l is 0 on
// the pivots.  The word count W is a compile-time constant, so each kernel
// vector is one wide wave-uniform (scalar) load and one wait; the targets
// <k_j, l> are staged once per workgroup as a bit mask in LDS.
template <int W>
__global__ __launch_bounds__(256) void membership_kernel(FactorIn f, const uint64_t *__restrict__ kernel,
                                                         const uint64_t *__restrict__ z,
                                                         uint64_t num, uint8_t *__restrict__ member) {
    if (*(volatile int32_t *)f.status != HLF_OK) return;
    const int n = f.n;
    const int nk = n - *f.rank;
    __shared__ uint32_t target[2 * W];
    for (int t = threadIdx.x; t < 2 * W; t += blockDim.x) target[t] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < nk; j += blockDim.x) {
        uint64_t acc = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) acc ^= kernel[(size_t)j * W + w] & f.shift[w];
        if (__builtin_popcountll(acc) & 1) atomicOr(&target[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; s < num; s += stride) {
        uint64_t zv[W];
#pragma unroll
        for (int w = 0; w < W; ++w) zv[w] = z[s * W + w];
        bool ok = true;
        for (int j = 0; j < nk; ++j) {
            const uint64_t *kj = kernel + (size_t)j * W;
            uint64_t acc = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) acc ^= kj[w] & zv[w];
            const uint32_t par = (uint32_t)__builtin_popcountll(acc) & 1u;
            if (par != ((target[j >> 5] >> (j & 31)) & 1u)) {
                ok = false;
                break;
            }
        }
        member[s] = ok ? 1 : 0;
    }
}

template <int WMAX>
hlf_status launch_pair_stats_t(const FactorIn &f, const uint64_t *rows, uint8_t *quarters,
                               hipStream_t stream) {
    hipLaunchKernelGGL(pair_stats_kernel<WMAX>, dim3((unsigned)f.n), dim3(256), 0, stream, f, rows,
                       quarters);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int W>
hlf_status launch_membership_t(const FactorIn &f, const uint64_t *kernel, const uint64_t *z,
                               uint64_t num, uint8_t *member, hipStream_t stream) {
    if constexpr (W >= kMemMfmaMinWords) {
        const uint64_t nblk = (num + 63) / 64;
        uint64_t g = (uint64_t)device_cu_count();
        const uint64_t most = (nblk + 3) / 4;
        if (g > most) g = most;
        if (g == 0) g = 1;
        hipLaunchKernelGGL(membership_mfma_kernel<W>, dim3((unsigned)g), dim3(64 * kMemWavesOf<W>), 0, stream, f,
                           kernel, z, num, member);
    } else {
        uint64_t blocks = (num + 255) / 256;
        const uint64_t cap = (uint64_t)device_cu_count() * 8;
        if (blocks > cap) blocks = cap;
        if (blocks == 0) blocks = 1;
        hipLaunchKernelGGL(membership_kernel<W>, dim3((unsigned)blocks), dim3(256), 0, stream, f, kernel, z, num,
                           member);
    }
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int... Ws>
hlf_status launch_membership_w(int W, const FactorIn &f, const uint64_t *kernel, const uint64_t *z,
                               uint64_t num, uint8_t *member, hipStream_t stream,
                               std::integer_sequence<int, Ws...>) {
    hlf_status st = HLF_EINVAL;
    ((W == Ws + 1 ? (st = launch_membership_t<Ws + 1>(f, kernel, z, num, member, stream), 0) : 0), ...);
    return st;
}

}  // namespace

hlf_status launch_pair_stats(const FactorIn &f, const uint64_t *rows, uint8_t *quarters,
                             hipStream_t stream) {
    const int W = f.words;
    if (W >= 2) {
        const int nb = (f.n + 31) / 32;
        const unsigned blocks = (unsigned)((nb * nb + kPairWaves - 1) / kPairWaves);
        hipLaunchKernelGGL(pair_stats_mfma_kernel, dim3(blocks), dim3(64 * kPairWaves), 0, stream, f,
                           rows, quarters);
        return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
    }
    return launch_pair_stats_t<1>(f, rows, quarters, stream);
}

hlf_status launch_membership(const FactorIn &f, const uint64_t *kernel, const uint64_t *z,
                             uint64_t num, uint8_t *member, hipStream_t stream) {
    return launch_membership_w(f.words, f, kernel, z, num, member, stream,
                               std::make_integer_sequence<int, HLF_MAX_N / 64>{});
}

}  // namespace hlf
