// Device-side helpers shared by the HIP kernels of libhlf (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hlf.h"

namespace hlf {

constexpr int kWave = 64;
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

// Four dwords, for 16-byte loads and stores (nontemporal builtins accept it).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Output function of SplitMix64 (Stafford's Mix13), used for the set hash and
// the sampling coefficient stream.
__device__ __forceinline__ uint64_t mix13(uint64_t x) {
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}

// The first step of mix13.  It is linear over GF(2): callers that split x into a
// per-lane and a per-tile part apply it to each part, and hash_tail does the rest.
__device__ __forceinline__ uint64_t mix13_head(uint64_t x) { return x ^ (x >> 30); }

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane) {
    uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// A value that is the same on every lane, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// 32x32 bit transposes within each half of the wave, on the VALU alone:
// lane l of a half holds row l of each matrix and gets its column l.  Step j
// exchanges, between lanes l and l ^ j, the bits whose row and column indices
// differ in bit j (the lane with bit j clear keeps the columns with bit j
// clear and takes its partner's, moved up by j; the other keeps the columns
// with bit j set and takes its partner's, moved down).  Partners: j = 16 by
// a permlane16 swap of the two rows of 16, j = 8 by a row mirror then a half
// mirror, j = 4 by a half mirror then a quad mirror, j = 2 and 1 by quad
// permutations (DPP).  Byte and halfword steps merge with one byte permute,
// the others with a masked rotate and an and-or.
template <int N>
__device__ __forceinline__ void half_transpose32_n(uint32_t (&x)[N]) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    {   // j = 16: after the swap, the first result holds the lane's own value
        // in rows 0 and 2 and its partner's in rows 1 and 3, the second the
        // other way round, so one byte permute with a per-row selector merges
        const bool up = lane & 16;
        const uint32_t sel = up ? 0x07060302u : 0x05040100u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const auto sw = __builtin_amdgcn_permlane16_swap(x[i], x[i], false, false);
            x[i] = __builtin_amdgcn_perm(sw[1], sw[0], sel);
        }
    }
    {   // j = 8
        const uint32_t sel = (lane & 8) ? 0x03070105u : 0x06020400u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int t = __builtin_amdgcn_mov_dpp((int)x[i], 0x140, 0xF, 0xF, false);   // row mirror
            const uint32_t y = (uint32_t)__builtin_amdgcn_mov_dpp(t, 0x141, 0xF, 0xF, false);  // half mirror
            x[i] = __builtin_amdgcn_perm(y, x[i], sel);
        }
    }
#pragma unroll
    for (int step = 2; step >= 0; --step) {
        const int j = 1 << step;
        const uint32_t mj = j == 4 ? 0x0F0F0F0Fu : j == 2 ? 0x33333333u : 0x55555555u;
        const uint32_t M = (lane & j) ? ~mj : mj;
        const uint32_t R = (lane & j) ? (uint32_t)j : (uint32_t)(32 - j);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            int y;
            if (j == 4) {
                const int t = __builtin_amdgcn_mov_dpp((int)x[i], 0x141, 0xF, 0xF, false);  // half mirror
                y = __builtin_amdgcn_mov_dpp(t, 0x1B, 0xF, 0xF, true);                     // quad [3,2,1,0]
            } else if (j == 2) {
                y = __builtin_amdgcn_mov_dpp((int)x[i], 0x4E, 0xF, 0xF, true);  // quad [2,3,0,1]
            } else {
                y = __builtin_amdgcn_mov_dpp((int)x[i], 0xB1, 0xF, 0xF, true);  // quad [1,0,3,2]
            }
            const uint32_t t = (uint32_t)y & M;
            x[i] = (x[i] & M) | __builtin_amdgcn_alignbit(t, t, R);
        }
    }
}

// 64x64 bit transpose across one wavefront: lane l holds row l (bit c =
// column c) and gets column l (bit r = row r).  Each half of the wave
// transposes its two 32x32 blocks; one swap of the low dwords of the upper
// half with the high dwords of the lower half exchanges the off-diagonal ones
// (33 VALU instructions; by lane shuffles through LDS it takes twelve of them
// in a chain).  Needs all lanes active.
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x) {
    uint32_t d[2] = {(uint32_t)x, (uint32_t)(x >> 32)};
    half_transpose32_n<2>(d);
    const auto sw = __builtin_amdgcn_permlane32_swap(d[0], d[1], false, false);
    return ((uint64_t)sw[1] << 32) | sw[0];
}

// Orders the LDS accesses of one wavefront around this point (waits for its
// outstanding LDS operations; no other wave is involved).  Used by code that
// runs on a single wave of a larger workgroup.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Makes what this wave has written visible to every workgroup of the device
// before anything that it stores after this (a flag, stored relaxed; its reader
// takes an acquire fence).  The wait is spelled out: the fence's own wait for
// the write-back of the L2 is dropped by the compiler where no other access of
// the wave is outstanding, since it does not count the write-back among them,
// and a flag stored right behind it was seen before the data.
__device__ __forceinline__ void release_to_device() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Mask of the valid bits of the last word of an n-bit vector (all ones when
// n is a multiple of 64).
__device__ __forceinline__ uint64_t last_word_mask(int n) {
    int rem = n & 63;
    return rem ? ((1ull << rem) - 1) : ~0ull;
}

}  // namespace hlf
