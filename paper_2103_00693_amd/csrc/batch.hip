// Batches of instances on gfx950: the whole FS2D pipeline (Sections 1-2) for
// many grid instances of mixed size with one launch per stage.
//
//   batch_factor_kernel<WMAX>   pack + validate + factor, one wavefront (a
//                               64-thread workgroup) per instance, n <= 64*WMAX.
//   batch_enum_kernel<T>        materialise for up to kMaxEnumTasks instances
//                               in one launch; each workgroup takes a short
//                               contiguous tile range of one instance.
//   batch_reduce_kernel<WMAX>   persistent: each wavefront first takes factor
//                               tasks from a device counter; an instance with
//                               r <= max_rank then claims a contiguous block of
//                               chunk indices with ONE 64-bit atomic that returns
//                               both its slot and its first chunk, writes the
//                               slot and releases it; wavefronts then take chunk
//                               indices from a second counter and find the slot
//                               by 64-way search.  A wave only waits for a slot
//                               that was already claimed (its writer is running)
//                               or for factor tasks that running waves hold, so
//                               every wait ends and the grid drains.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "factor_wave.h"
#include "hlf.h"
#include "hlf_device.h"
#include "hlf_internal.h"
#include "stage2.h"

namespace hlf {
namespace {

struct BatchDev {
    int32_t count;
    const int32_t *n;
    const int64_t *dense_off;
    const int64_t *mat_off;
    const int64_t *vec_off;
    const int64_t *piv_off;
    const int32_t *order;  // instance ids grouped by word count
    int32_t *status;
    int32_t *rank;
    int32_t *pivots;
    uint64_t *basis;
    uint64_t *shift;
    uint64_t *kernel;
    uint64_t *counts;
    uint64_t *hash;
};

__device__ __forceinline__ FactorOut record_of(const BatchDev &b, int i) {
    FactorOut out;
    out.status = &b.status[i];
    out.rank = &b.rank[i];
    out.pivots = b.pivots + b.piv_off[i];
    out.basis = b.basis + b.mat_off[i];
    out.shift = b.shift + b.vec_off[i];
    out.kernel = b.kernel ? b.kernel + b.mat_off[i] : nullptr;
    return out;
}

// ---------------------------------------------------------------------------
// Stage 1 for the instances order[first .. first + gridDim.x).
// ---------------------------------------------------------------------------
template <int WMAX>
__global__ __launch_bounds__(64) void batch_factor_kernel(BatchDev b, const uint8_t *__restrict__ A,
                                                          int first) {
    __shared__ WaveSmem<WMAX> sm;
    const int i = b.order[first + blockIdx.x];
    const int n = b.n[i];
    const int W = (n + 63) >> 6;
    const bool badv = wave_load_dense<WMAX>(A + b.dense_off[i], n, W, sm);
    factor_wave_core<WMAX>(n, W, badv, record_of(b, i), sm);
}

// A failed pack (an entry other than 0/1) overrides the factor's verdict.
__global__ void merge_pack_status_kernel(int32_t *status, const int32_t *pack_status) {
    if (threadIdx.x == 0 && *pack_status != HLF_OK) *status = *pack_status;
}

// ---------------------------------------------------------------------------
// Materialise for several instances.
// ---------------------------------------------------------------------------
constexpr int kMaxEnumTasks = 16;

struct EnumTask {
    int32_t *status;
    const int32_t *rank;
    const uint64_t *basis;
    const uint64_t *shift;
    void *out;
    uint64_t begin;
    uint64_t count;
    uint32_t block0;           // first block of this task
    uint32_t tiles_per_block;
};

// Tasks of batch_enum_kernel, read by every wave from the kernel arguments
// before its first store.
struct alignas(128) VecTask {
    const uint64_t *basis;
    const uint64_t *shift;
    int32_t inst;
    int32_t n;
    VecRange g;
    uint32_t block0;
};

struct alignas(128) EnumTasks {
    uint32_t first[kMaxEnumTasks];  // first block of tasks 1 .. (~0 past the last)
    uint32_t blocks;                // blocks of all tasks
    uint32_t tiles_per_block;
    uint32_t job_blocks;            // blocks before theirs that run the FactorJob
    int32_t *status;
    const int32_t *rank;
    VecTask t[kMaxEnumTasks];
};

// Optional stage-1 work carried by a materialise launch: the first job_blocks
// workgroups factor instances order[first .. first + num) of another batch,
// one instance per wavefront (W = 1).  The records it writes are not read by
// the same launch, so there is no dependency inside the launch.
struct FactorJob {
    BatchDev d;
    const uint8_t *A;
    int32_t first;
    int32_t num;
};

constexpr int kWavesPerVecBlock = kVecThreads / 64;

template <typename T, bool kFactor>
__global__ __launch_bounds__(kVecThreads, 8) void batch_enum_kernel(EnumTasks tasks, FactorJob job) {
    uint32_t own_first = tasks.first[threadIdx.x & (kMaxEnumTasks - 1)];
    uint32_t blocks = tasks.blocks, tpb = tasks.tiles_per_block, job_blocks = tasks.job_blocks;
    asm("" : "+v"(own_first), "+s"(blocks), "+s"(tpb), "+s"(job_blocks));  // in one wait
    uint32_t bid = blockIdx.x;
    if constexpr (kFactor) {
        __shared__ WaveSmem<1> sm[kWavesPerVecBlock];
        if (bid < job_blocks) {
            const int w = threadIdx.x >> 6;
            const int idx = (int)bid * kWavesPerVecBlock + w;
            if (idx < job.num) {
                const int i = job.d.order[job.first + idx];
                const int n = job.d.n[i];
                const bool badv = wave_load_dense<1>(job.A + job.d.dense_off[i], n, 1, sm[w]);
                factor_wave_core<1>(n, 1, badv, record_of(job.d, i), sm[w]);
            }
            return;
        }
        bid -= job_blocks;
    }
    bid = xcd_block(bid, blocks);
    // The task of this block: the first blocks of the others, one per lane,
    // counted where they are at or before it.  (Fifteen scalar compares cost
    // 30 scalar issues a wave, and the launch a third of its rate.)
    const uint64_t le = __ballot(own_first <= bid);
    const uint32_t k = (uint32_t)__builtin_popcount((uint32_t)le & ((1u << kMaxEnumTasks) - 1u));
    VecTask t = tasks.t[k];
    asm("" : "+s"(t.inst), "+s"(t.n), "+s"(t.g.begin), "+s"(t.g.end), "+s"(t.g.ntiles), "+s"(t.g.full0),
        "+s"(t.g.full1), "+s"(t.block0));
    const uint32_t t0 = (bid - t.block0) * tpb;
    const uint32_t t1 = t0 + tpb < t.g.ntiles ? t0 + tpb : t.g.ntiles;
    vec_materialise<T, false>(tasks.status + t.inst, tasks.rank + t.inst, t.basis, t.shift, t.n, t.g, t0, t1);
}

// ---------------------------------------------------------------------------
// Stage 1 + stage 2 materialise in one launch (instances with n <= 64).
// The first workgroup of an instance to start claims its factorisation with a
// CAS on flags[inst] (0 idle, 1 claimed, 2 done) and runs it on its first wave;
// the instance's other workgroups wait for 2 -- a claim is only ever held by a
// running workgroup, so every wait ends.  The last workgroup to finish resets
// the flags of the launch, so each launch starts from idle flags.  Every
// workgroup reaches the final counter (no early return).
// ---------------------------------------------------------------------------
struct SolveTasks {
    EnumTask t[kMaxEnumTasks];
    int32_t inst[kMaxEnumTasks];
    int32_t num;
};

template <typename T>
__global__ __launch_bounds__(kTileThreads) void batch_solve_kernel(BatchDev b,
                                                                   const uint8_t *__restrict__ A,
                                                                   SolveTasks tasks, int32_t *flags,
                                                                   unsigned int *blocks_done) {
    constexpr int S = tile_shift<T>();
    __shared__ WaveSmem<1> sm;
    __shared__ uint64_t Bx[64];
    __shared__ int role;
    __shared__ int ok;
    __shared__ int rank_s;
    const int tid = threadIdx.x;
    int k = 0;
    for (int j = 1; j < tasks.num; ++j)
        if (tasks.t[j].block0 <= blockIdx.x) k = j;
    const EnumTask &t = tasks.t[k];
    const int i = tasks.inst[k];

    // Agent-scope acquire/release fences invalidate / write back the XCD's L2,
    // so the claim and the wait use relaxed atomics and each workgroup takes
    // exactly one acquire (thread 0) after it has seen the flag at 2.
    if (tid == 0) {
        int mine = 0;
        if (__hip_atomic_load(&flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
            int expected = 0;
            mine = __hip_atomic_compare_exchange_strong(&flags[i], &expected, 1, __ATOMIC_RELAXED,
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                       ? 1 : 0;
        }
        role = mine;
    }
    __syncthreads();
    if (role) {
        if (tid < 64) {
            const int n = b.n[i];
            const bool badv = wave_load_dense<1>(A + b.dense_off[i], n, 1, sm);
            factor_wave_core<1>(n, 1, badv, record_of(b, i), sm);
            release_to_device();
            if (tid == 0) __hip_atomic_store(&flags[i], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else if (tid == 0) {
        while (__hip_atomic_load(&flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 2)
            __builtin_amdgcn_s_sleep(8);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (tid == 0) {
        int r = 0;
        ok = gate(t.status, t.rank, t.begin, t.count, r) ? 1 : 0;
        rank_s = r;
    }
    __syncthreads();
    if (ok) {
        load_basis_padded<1>(t.basis, rank_s, Bx, tid, blockDim.x);
        __syncthreads();
        const uint64_t end = t.begin + t.count;
        const uint64_t ntiles = ((end - 1) >> S) - (t.begin >> S) + 1;
        const uint64_t t0 = (uint64_t)(blockIdx.x - t.block0) * t.tiles_per_block;
        if (t0 < ntiles) {
            const uint64_t t1 = (t0 + t.tiles_per_block < ntiles) ? t0 + t.tiles_per_block : ntiles;
            enum_tiles_w1<T, false>(Bx, t.shift[0], t.begin, t.count, (T *)t.out, t0, t1);
        }
    }
    __syncthreads();
    // Thread 0's flag accesses have all returned before its increment is
    // issued, so the last workgroup can reset the flags; the end of the kernel
    // makes the reset visible to the next launch.
    if (tid == 0) {
        const unsigned int prev =
            __hip_atomic_fetch_add(blocks_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == gridDim.x - 1) {
            for (int j = 0; j < tasks.num; ++j)
                __hip_atomic_store(&flags[tasks.inst[j]], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(blocks_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---------------------------------------------------------------------------
// Persistent factor + reduce.
// ---------------------------------------------------------------------------
constexpr int kClaimShift = 40;  // claim word: (slots << 40) | chunks
constexpr unsigned long long kChunkMask = (1ull << kClaimShift) - 1;

// The drawn counters and the polled words lie on cache lines of their own.
struct QueueHead {
    unsigned long long claim;  // published slots and chunks
    unsigned int fskip;        // factor tasks finished without a claim
    char pad0[128 - 12];
    unsigned int fnext;        // next factor task
    char pad1[64 - 4];
    unsigned long long cnext;  // next chunk index past the first gridDim.x
};

// One word per slot, zero until published: (first chunk + 1) << kInstBits |
// instance.  First chunks are below 2^40, instances below 2^20.
constexpr int kInstBits = 20;
struct ChunkSlot {
    unsigned long long entry;
};

__global__ void batch_queue_reset_kernel(QueueHead *q, ChunkSlot *slots, int count) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) {
        q->fnext = 0;
        q->fskip = 0;
        q->cnext = 0;
        q->claim = 0;
    }
    if (t < count) slots[t].entry = 0;
}

// Offsets of the batch layout (prefix sums over the instance sizes) for the
// allocation-free reduce, and the queue reset: one workgroup of 1024 threads,
// count <= 1024 * kLayoutPer.  An n outside [1, max_n] counts as 0 (no space;
// its factor task reports HLF_EINVAL).  n_eff receives the sizes the other
// kernels use.  Every sum fits 32 bits (16384 * 192^2 < 2^30).  54 sizes took
// 8.7 us and the reset another launch of 4.6, with 16 sizes a thread, one
// after the other, and ten rounds of a scan over LDS.
constexpr int kLayoutPer = 16;

__global__ __launch_bounds__(1024) void noalloc_layout_kernel(const int32_t *__restrict__ n_in,
                                                              int count, int max_n, int32_t *n_eff,
                                                              int64_t *dense_off, int64_t *mat_off,
                                                              int64_t *vec_off, int64_t *piv_off,
                                                              QueueHead *q, ChunkSlot *slots) {
    __shared__ uint32_t part[16][4];
    const int t = threadIdx.x, lane = lane_id(), wave = t >> 6;
    const int per = (count + 1023) >> 10;
    const int i0 = t * per, i1 = min(count, i0 + per);
    for (int i = t; i < count; i += 1024) slots[i].entry = 0;
    if (t == 0) {
        q->fnext = 0;
        q->fskip = 0;
        q->cnext = 0;
        q->claim = 0;
    }
    auto sizes = [&](int i, uint32_t (&v)[4]) {
        const int n = n_in[i];
        const uint32_t ne = (n >= 1 && n <= max_n) ? (uint32_t)n : 0u, W = (ne + 63) >> 6;
        v[0] = ne * ne;
        v[1] = ne * W;
        v[2] = W;
        v[3] = ne;
    };
    uint32_t loc[4] = {0, 0, 0, 0};
    for (int i = i0; i < i1; ++i) {
        uint32_t v[4];
        sizes(i, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) loc[k] += v[k];
    }
    uint32_t run[4];  // inclusive over the wave, then exclusive over all
#pragma unroll
    for (int k = 0; k < 4; ++k) run[k] = loc[k];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t up = (uint32_t)__shfl_up((int)run[k], d);
            if (lane >= d) run[k] += up;
        }
    }
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < 4; ++k) part[wave][k] = run[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        run[k] -= loc[k];
        for (int v = 0; v < wave; ++v) run[k] += part[v][k];
    }
    for (int i = i0; i < i1; ++i) {
        uint32_t v[4];
        sizes(i, v);
        n_eff[i] = (int32_t)v[3];
        dense_off[i] = run[0];
        mat_off[i] = run[1];
        vec_off[i] = run[2];
        piv_off[i] = run[3];
#pragma unroll
        for (int k = 0; k < 4; ++k) run[k] += v[k];
    }
}

template <typename V>
__device__ __forceinline__ V relaxed_load(const V *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Entry of the last of nslots claimed slots whose first chunk is <= c (first
// chunks increase with the slot, slot 0's is 0).  64 slots are read at a time,
// one per lane, evenly over what is left: two rounds for 4096 slots.  A claimed
// slot that is still zero is about to be written by a running wave.
__device__ __forceinline__ unsigned long long find_slot(const ChunkSlot *slots, int nslots, unsigned long long c) {
    const int lane = lane_id();
    int lo = 0, len = nslots;
    for (;;) {
        const int step = (len + 63) >> 6;
        const bool in = lane * step < len;
        unsigned long long e = 0;
        for (;;) {
            if (in && e == 0) e = relaxed_load(&slots[lo + lane * step].entry);
            if (__ballot(in && e == 0) == 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
        const unsigned long long below = __ballot(in && (e >> kInstBits) - 1 <= c);  // lane 0 always
        const int k = 63 - __builtin_clzll(below);
        if (step == 1) return readlane64(e, k);
        lo += k * step;
        len = min(step, len - k * step);
    }
}

template <int WW>
__device__ void reduce_chunk(const BatchDev &b, int inst, int r, unsigned long long c0, unsigned long long c1) {
    const WaveRows<WW> rows = wave_rows<WW>(b.basis + b.mat_off[inst], r);
    uint64_t l[WW];
    const uint64_t *sh = b.shift + b.vec_off[inst];
#pragma unroll
    for (int w = 0; w < WW; ++w) l[w] = uniform64(sh[w]);
    const uint64_t acc = wave_sum_u64(wave_hash_range<WW>(rows, l, uniform64(c0), uniform64(c1),
                                                          [&](int k, uint64_t(&row)[WW]) {
#pragma unroll
                                                              for (int w = 0; w < WW; ++w) row[w] = row_word<WW>(rows, k, w);
                                                          }));
    if (lane_id() == 0 && acc) atomicAdd((unsigned long long *)&b.hash[inst], (unsigned long long)acc);
}

template <int WMAX>
__global__ __launch_bounds__(64) void batch_reduce_kernel(BatchDev b, const uint8_t *__restrict__ A,
                                                          int max_rank, int chunk_log2, int drawn,
                                                          QueueHead *q, ChunkSlot *slots) {
    __shared__ WaveSmem<WMAX> sm;
    const int lane = lane_id();

    // Phase 1: factor tasks.  Drawn, the first one too: a wave that is not
    // running yet must not hold one that running waves wait for.  Draws come
    // one in 12 ns and hold up all other accesses meanwhile (2048 waves: 24 us
    // before the first task was done), so waves beyond the number of tasks let
    // the others draw first, and nobody draws once all are taken.
    for (bool first = true;; first = false) {
        if (!first || blockIdx.x >= (unsigned int)b.count) {
            if (first)
                for (int k = 0; k <= b.count >> 5; ++k) __builtin_amdgcn_s_sleep(16);
            if ((unsigned int)__builtin_amdgcn_readfirstlane((int)relaxed_load(&q->fnext)) >= (unsigned int)b.count)
                break;
        }
        unsigned int f = 0;
        if (lane == 0) f = atomicAdd(&q->fnext, 1u);
        f = (unsigned int)__builtin_amdgcn_readfirstlane((int)f);
        if (f >= (unsigned int)b.count) break;
        const int n = b.n[f];
        const int W = (n + 63) >> 6;
        const FactorOut out = record_of(b, (int)f);
        int r = -1;
        if (n >= 1 && W <= WMAX) {
            const bool badv = wave_load_dense<WMAX>(A + b.dense_off[f], n, W, sm);
            r = factor_wave_core<WMAX>(n, W, badv, out, sm);
        } else if (lane == 0) {
            *out.rank = 0;
            *out.status = HLF_EINVAL;
        }
        // Counts over all 2^r solutions: half of them where row j of A (and so
        // bit j of some B_k) is not zero; elsewhere none, since then A e_j = 0
        // and q(e_j) = A_jj = 0 give l_j = 0.
        uint64_t *cnt = b.counts + b.piv_off[f];
        const uint64_t half = r >= 1 && r <= max_rank ? 1ull << (r - 1) : 0ull;
        for (int j = lane; j < n; j += 64) {
            uint64_t any = 0;
            if (half)
                for (int w = 0; w < W; ++w) any |= sm.orig[j * W + w];
            cnt[j] = any ? half : 0ull;
        }
        if (lane == 0) b.hash[f] = 0;
        if (r >= 0 && r <= max_rank) {  // wave-uniform
            // The release makes the record and the zeroed hash visible to
            // whoever reads the entry.
            release_to_device();
            if (lane == 0) {
                const unsigned long long nch = r > chunk_log2 ? 1ull << (r - chunk_log2) : 1ull;
                const unsigned long long old = atomicAdd(&q->claim, (1ull << kClaimShift) | nch);
                __hip_atomic_store(&slots[old >> kClaimShift].entry,
                                   (((old & kChunkMask) + 1) << kInstBits) | (unsigned long long)f, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        } else if (lane == 0) {
            __hip_atomic_fetch_add(&q->fskip, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();  // LDS is reused by the next factor task
    }

    // Phase 2: chunk tasks, the first one by the wave's index, the others drawn
    // or, where they are short (see kShortPieceLog2), in turn.
    unsigned long long c = blockIdx.x;
    for (;;) {
        unsigned long long e = 0;
        for (int naps = 0;; ++naps) {
            const unsigned long long cl = uniform64(relaxed_load(&q->claim));
            if (c < (cl & kChunkMask)) {
                e = find_slot(slots, (int)(cl >> kClaimShift), c);
                break;
            }
            // Every task claims a slot or is counted in fskip: where the slots
            // of this claim word and the others make up the batch, the word is
            // the last one and no chunk is left.  (A count of all tasks would
            // have to be released after each claim, which writes back the L2:
            // 2048 instances with nothing to reduce 203 us against 148.)
            const unsigned int skipped = (unsigned int)__builtin_amdgcn_readfirstlane((int)relaxed_load(&q->fskip));
            if ((unsigned int)(cl >> kClaimShift) + skipped >= (unsigned int)b.count) break;
            // Thousands of waves polling at full rate hold up the atomics that
            // they wait for: back off, with the grid, to 7 us at 2048 waves.
            const int units = naps < 4 ? 1 : 1 + (int)(gridDim.x >> 7);
            for (int k = 0; k < units; ++k) __builtin_amdgcn_s_sleep(16);
        }
        if (e == 0) break;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the record behind the entry
        const int inst = (int)(e & ((1u << kInstBits) - 1));
        const unsigned long long local = c - ((e >> kInstBits) - 1);
        const int n = b.n[inst];
        const int W = (n + 63) >> 6;
        const int r = __builtin_amdgcn_readfirstlane(b.rank[inst]);
        const unsigned long long total = 1ull << r;
        const unsigned long long c0 = local << chunk_log2;
        unsigned long long c1 = c0 + (1ull << chunk_log2);
        if (c1 > total) c1 = total;
        if (W == 1) reduce_chunk<1>(b, inst, r, c0, c1);
        if constexpr (WMAX >= 2)
            if (W == 2) reduce_chunk<2>(b, inst, r, c0, c1);
        if constexpr (WMAX >= 3)
            if (W == 3) reduce_chunk<3>(b, inst, r, c0, c1);
        if (drawn) {
            unsigned long long next = 0;
            if (lane == 0) next = atomicAdd(&q->cnext, 1ull);
            c = gridDim.x + uniform64(next);
        } else {
            c += gridDim.x;
        }
    }
}

}  // namespace
}  // namespace hlf

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
struct hlf_batch_s {
    int device = 0;
    int32_t count = 0;
    int32_t max_n = 0;
    std::vector<int32_t> n;
    std::vector<int64_t> dense_off, mat_off, vec_off, piv_off;
    int64_t dense_bytes = 0, mat_words = 0, vec_words = 0, piv_entries = 0;
    // instances ordered by word count: W = 1, 2, 3, then larger
    std::vector<int32_t> order;
    int bucket_start[5] = {0, 0, 0, 0, 0};
    // device arrays
    int32_t *d_n = nullptr;
    int64_t *d_dense_off = nullptr, *d_mat_off = nullptr, *d_vec_off = nullptr, *d_piv_off = nullptr;
    int32_t *d_order = nullptr;
    int32_t *status = nullptr, *rank = nullptr, *pivots = nullptr;
    uint64_t *basis = nullptr, *shift = nullptr, *kernel = nullptr, *counts = nullptr, *hash = nullptr;
    uint64_t *rows = nullptr;  // packed rows of instances with n > 192
    int32_t *pack_status = nullptr;
    int32_t *solve_flags = nullptr;        // per instance, idle between launches
    unsigned int *solve_done = nullptr;    // workgroups finished in a solve launch
    hlf::QueueHead *queue = nullptr;
    hlf::ChunkSlot *slots = nullptr;
    hlf_batch_params tuned = {20, 8};
    bool has_tuned = false;
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    std::vector<void *> allocations;
};

namespace {

template <typename T>
hlf_status dev_alloc(hlf_batch_s *b, T **p, size_t elems) {
    void *q = nullptr;
    const size_t bytes = std::max<size_t>(elems, 1) * sizeof(T);
    if (hipMalloc(&q, bytes) != hipSuccess) return HLF_ENOMEM;
    b->allocations.push_back(q);
    *p = (T *)q;
    return HLF_OK;
}

hlf::BatchDev view_of(const hlf_batch_s *b) {
    hlf::BatchDev d;
    d.count = b->count;
    d.n = b->d_n;
    d.dense_off = b->d_dense_off;
    d.mat_off = b->d_mat_off;
    d.vec_off = b->d_vec_off;
    d.piv_off = b->d_piv_off;
    d.order = b->d_order;
    d.status = b->status;
    d.rank = b->rank;
    d.pivots = b->pivots;
    d.basis = b->basis;
    d.shift = b->shift;
    d.kernel = b->kernel;
    d.counts = b->counts;
    d.hash = b->hash;
    return d;
}

bool params_ok(const hlf_batch_params &p) {
    return p.chunk_log2 >= 10 && p.chunk_log2 <= 30 && p.waves_per_cu >= 1 && p.waves_per_cu <= 16;
}

// The claim word keeps the running chunk total in its low kClaimShift bits:
// every instance with r <= max_rank claims max(1, 2^(r - chunk_log2)) chunks,
// so the total over the batch must stay below 2^kClaimShift (else it would
// carry into the slot field).
bool claims_fit_count(int count, int max_rank, int chunk_log2) {
    const int e = max_rank > chunk_log2 ? max_rank - chunk_log2 : 0;
    if (e >= hlf::kClaimShift) return false;
    const unsigned long long per = 1ull << e;
    return (unsigned long long)count < ((1ull << hlf::kClaimShift) / per);
}

// The pieces that a chunk is drawn in: 2^17 solutions, as far as the queue
// counts that many.  A wave takes 0.6 ms for 2^20 solutions beside another on
// its SIMD, and the last ones run while the rest of the card is idle (4096
// grids at chunk_log2 20, 8 waves per CU: 6.51 ms in whole chunks, 6.19 in
// pieces of 2^17, 6.27 of 2^16, 6.49 of 2^15, where the draws begin to queue).
constexpr int kPieceLog2 = 17;

// Batches that cannot hold that many solutions for every wave take shorter
// pieces, an eighth of what a wave could get at most, down to 2^12: an
// instance of rank 16 is then the work of 16 waves instead of one, 2 us
// instead of 37.  Draws come one in 9 ns at best, so waves take short pieces
// in turn, without.
constexpr int kShortPieceLog2 = 12;

int piece_log2(int count, int max_rank, int chunk_log2, int grid, int *drawn) {
    int most = max_rank;  // log2 of the solutions per wave, at most
    for (int c = count; c > grid; c >>= 1) ++most;
    for (int c = count; c < grid; c <<= 1) --most;
    const int want = std::min(kPieceLog2, std::max(kShortPieceLog2, most - 3));
    *drawn = want == kPieceLog2;  // also where the caller's chunks are shorter
    int p = chunk_log2;
    while (p > want && claims_fit_count(count, max_rank, p - 1)) --p;
    return p;
}

bool claims_fit(const hlf_batch_s *b, int max_rank, int chunk_log2) {
    return claims_fit_count(b->count, max_rank, chunk_log2);
}

// What a reduce launches for given parameters.
struct ReducePlan {
    int piece, drawn, grid;
    bool operator==(const ReducePlan &o) const { return piece == o.piece && drawn == o.drawn && grid == o.grid; }
};

template <int WMAX>
ReducePlan reduce_plan(int count, int max_rank, const hlf_batch_params &p) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, hlf::batch_reduce_kernel<WMAX>, 64, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    ReducePlan plan;
    plan.grid = hlf::device_cu_count() * std::min(p.waves_per_cu, per_cu);
    plan.piece = piece_log2(count, max_rank, p.chunk_log2, plan.grid, &plan.drawn);
    // no more waves than factor tasks or pieces there can be
    const int e = std::max(max_rank - plan.piece, 0);
    if (e < 20 && (int64_t)count << e < plan.grid) plan.grid = count << e;
    return plan;
}

// The persistent factor/reduce kernel over the instances of a device view,
// with the given queue and slot arrays, which have been reset.
template <int WMAX>
hlf_status launch_reduce_view(const hlf::BatchDev &d, const uint8_t *A, int max_rank,
                              const hlf_batch_params &p, hlf::QueueHead *queue,
                              hlf::ChunkSlot *slots, hipStream_t stream) {
    const ReducePlan plan = reduce_plan<WMAX>(d.count, max_rank, p);
    hipLaunchKernelGGL(hlf::batch_reduce_kernel<WMAX>, dim3(plan.grid), dim3(64), 0, stream, d, A, max_rank,
                       plan.piece, plan.drawn, queue, slots);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

template <int WMAX>
hlf_status launch_batch_reduce_t(hlf_batch_s *b, const uint8_t *A, int max_rank,
                                 const hlf_batch_params &p, hipStream_t stream) {
    hipLaunchKernelGGL(hlf::batch_queue_reset_kernel, dim3((b->count + 255) / 256), dim3(256), 0, stream,
                       b->queue, b->slots, b->count);
    if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    return launch_reduce_view<WMAX>(view_of(b), A, max_rank, p, b->queue, b->slots, stream);
}

hlf_status batch_reduce_impl(hlf_batch_s *b, const uint8_t *A, int max_rank,
                             const hlf_batch_params &p, hipStream_t stream) {
    if (b->max_n <= 64) return launch_batch_reduce_t<1>(b, A, max_rank, p, stream);
    return launch_batch_reduce_t<3>(b, A, max_rank, p, stream);
}

std::mutex g_tune_mu;
std::map<std::tuple<int, int, int64_t, int>, std::pair<hlf_batch_params, float>> g_tune_cache;

}  // namespace

extern "C" {

hlf_status hlf_batch_create(int32_t count, const int32_t *n_host, hlf_batch *out) {
    if (!out || !n_host || count < 1 || count > (1 << 20)) return HLF_EINVAL;
    *out = nullptr;
    for (int i = 0; i < count; ++i)
        if (n_host[i] < 1 || n_host[i] > HLF_MAX_N) return HLF_EINVAL;
    hlf_batch_s *b = new hlf_batch_s();
    if (hipGetDevice(&b->device) != hipSuccess) {
        delete b;
        return HLF_EDEVICE;
    }
    b->count = count;
    b->n.assign(n_host, n_host + count);
    b->dense_off.resize(count);
    b->mat_off.resize(count);
    b->vec_off.resize(count);
    b->piv_off.resize(count);
    std::vector<std::vector<int32_t>> buckets(4);
    for (int i = 0; i < count; ++i) {
        const int64_t n = b->n[i], W = (n + 63) / 64;
        b->dense_off[i] = b->dense_bytes;
        b->mat_off[i] = b->mat_words;
        b->vec_off[i] = b->vec_words;
        b->piv_off[i] = b->piv_entries;
        b->dense_bytes += n * n;
        b->mat_words += n * W;
        b->vec_words += W;
        b->piv_entries += n;
        b->max_n = std::max<int32_t>(b->max_n, (int32_t)n);
        buckets[W <= 3 ? W - 1 : 3].push_back(i);
    }
    for (int k = 0; k < 4; ++k) {
        b->bucket_start[k] = (int)b->order.size();
        b->order.insert(b->order.end(), buckets[k].begin(), buckets[k].end());
    }
    b->bucket_start[4] = (int)b->order.size();
    int64_t big_words = 0;
    for (int i : buckets[3]) big_words = std::max<int64_t>(big_words, (int64_t)b->n[i] * ((b->n[i] + 63) / 64));

    hlf_status st = HLF_OK;
    auto chk = [&](hlf_status s) { if (st == HLF_OK) st = s; };
    chk(dev_alloc(b, &b->d_n, count));
    chk(dev_alloc(b, &b->d_dense_off, count));
    chk(dev_alloc(b, &b->d_mat_off, count));
    chk(dev_alloc(b, &b->d_vec_off, count));
    chk(dev_alloc(b, &b->d_piv_off, count));
    chk(dev_alloc(b, &b->d_order, count));
    chk(dev_alloc(b, &b->status, count));
    chk(dev_alloc(b, &b->rank, count));
    chk(dev_alloc(b, &b->pivots, b->piv_entries));
    chk(dev_alloc(b, &b->basis, b->mat_words));
    chk(dev_alloc(b, &b->shift, b->vec_words));
    chk(dev_alloc(b, &b->kernel, b->mat_words));
    chk(dev_alloc(b, &b->counts, b->piv_entries));
    chk(dev_alloc(b, &b->hash, count));
    chk(dev_alloc(b, &b->rows, big_words));
    chk(dev_alloc(b, &b->pack_status, 1));
    chk(dev_alloc(b, &b->solve_flags, count));
    chk(dev_alloc(b, &b->solve_done, 1));
    chk(dev_alloc(b, &b->queue, 1));
    chk(dev_alloc(b, &b->slots, count));
    if (st == HLF_OK) {
        auto up = [&](void *dst, const void *src, size_t bytes) {
            if (hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice) != hipSuccess) st = HLF_EDEVICE;
        };
        up(b->d_n, b->n.data(), count * sizeof(int32_t));
        up(b->d_dense_off, b->dense_off.data(), count * sizeof(int64_t));
        up(b->d_mat_off, b->mat_off.data(), count * sizeof(int64_t));
        up(b->d_vec_off, b->vec_off.data(), count * sizeof(int64_t));
        up(b->d_piv_off, b->piv_off.data(), count * sizeof(int64_t));
        up(b->d_order, b->order.data(), count * sizeof(int32_t));
        std::vector<int32_t> init(count, HLF_EINVAL);  // not factored yet
        up(b->status, init.data(), count * sizeof(int32_t));
        std::vector<int32_t> zero(count, 0);
        up(b->solve_flags, zero.data(), count * sizeof(int32_t));
        const unsigned int zero_u = 0;
        up(b->solve_done, &zero_u, sizeof(zero_u));
    }
    if (st != HLF_OK) {
        hlf_batch_destroy(b);
        return st;
    }
    *out = b;
    return HLF_OK;
}

hlf_status hlf_batch_destroy(hlf_batch b) {
    if (!b) return HLF_OK;
    // Best-effort teardown: the handle is gone whatever these return.
    (void)hipDeviceSynchronize();
    if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    for (void *p : b->allocations) (void)hipFree(p);
    delete b;
    return HLF_OK;
}

hlf_status hlf_batch_get_layout(hlf_batch b, hlf_batch_layout *L) {
    if (!b || !L) return HLF_EINVAL;
    L->count = b->count;
    L->max_n = b->max_n;
    L->dense_bytes = b->dense_bytes;
    L->mat_words = b->mat_words;
    L->vec_words = b->vec_words;
    L->piv_entries = b->piv_entries;
    L->dense_off = b->dense_off.data();
    L->mat_off = b->mat_off.data();
    L->vec_off = b->vec_off.data();
    L->piv_off = b->piv_off.data();
    L->status = b->status;
    L->rank = b->rank;
    L->pivots = b->pivots;
    L->basis = b->basis;
    L->shift = b->shift;
    L->kernel = b->kernel;
    L->counts = b->counts;
    L->hash = b->hash;
    return HLF_OK;
}

hlf_status hlf_batch_factor_dense(hlf_batch b, const uint8_t *A_dev, hipStream_t stream) {
    if (!b || !A_dev) return HLF_EINVAL;
    const hlf::BatchDev d = view_of(b);
    for (int k = 0; k < 3; ++k) {
        const int first = b->bucket_start[k];
        const int num = b->bucket_start[k + 1] - first;
        if (num == 0) continue;
        if (k == 0) hipLaunchKernelGGL(hlf::batch_factor_kernel<1>, dim3(num), dim3(64), 0, stream, d, A_dev, first);
        if (k == 1) hipLaunchKernelGGL(hlf::batch_factor_kernel<2>, dim3(num), dim3(64), 0, stream, d, A_dev, first);
        if (k == 2) hipLaunchKernelGGL(hlf::batch_factor_kernel<3>, dim3(num), dim3(64), 0, stream, d, A_dev, first);
        if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    }
    for (int idx = b->bucket_start[3]; idx < b->bucket_start[4]; ++idx) {
        const int i = b->order[idx];
        const int n = b->n[i], W = (n + 63) / 64;
        hlf::FactorOut out;
        out.status = b->status + i;
        out.rank = b->rank + i;
        out.pivots = b->pivots + b->piv_off[i];
        out.basis = b->basis + b->mat_off[i];
        out.shift = b->shift + b->vec_off[i];
        out.kernel = b->kernel + b->mat_off[i];
        hlf_status s = hlf::launch_pack(A_dev + b->dense_off[i], n, W, b->rows, b->pack_status, stream);
        if (s != HLF_OK) return s;
        s = hlf::launch_factor(b->rows, n, W, out, false, false, stream);
        if (s != HLF_OK) return s;
        hipLaunchKernelGGL(hlf::merge_pack_status_kernel, dim3(1), dim3(64), 0, stream, out.status,
                           b->pack_status);
        if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    }
    return HLF_OK;
}

}  // extern "C"

namespace {

template <typename T>
void launch_enum_group(const hlf::EnumTasks &tasks, const hlf::FactorJob *job, hipStream_t stream) {
    if (job) {
        hipLaunchKernelGGL((hlf::batch_enum_kernel<T, true>), dim3(tasks.job_blocks + tasks.blocks),
                           dim3(hlf::kVecThreads), 0, stream, tasks, *job);
    } else {
        hipLaunchKernelGGL((hlf::batch_enum_kernel<T, false>), dim3(tasks.blocks),
                           dim3(hlf::kVecThreads), 0, stream, tasks, hlf::FactorJob{});
    }
}

hlf_status batch_enumerate_impl(hlf_batch b, int32_t num, const int32_t *inst,
                                const uint64_t *begin, const uint64_t *count, void *const *out,
                                int32_t word_bits, const hlf::FactorJob *job, hipStream_t stream) {
    if (!b || num < 0 || (num > 0 && (!inst || !begin || !count || !out))) return HLF_EINVAL;
    if (word_bits != 16 && word_bits != 32 && word_bits != 64) return HLF_EINVAL;
    for (int k = 0; k < num; ++k) {
        if (inst[k] < 0 || inst[k] >= b->count) return HLF_EINVAL;
        if (b->n[inst[k]] > word_bits) return HLF_EINVAL;
        if (count[k] > 0 && !out[k]) return HLF_EINVAL;
    }
    auto range_of = [&](int k) {
        return word_bits == 16   ? hlf::vec_range<uint16_t>(begin[k], count[k], out[k])
               : word_bits == 32 ? hlf::vec_range<uint32_t>(begin[k], count[k], out[k])
                                 : hlf::vec_range<uint64_t>(begin[k], count[k], out[k]);
    };
    std::vector<int> todo;
    for (int k = 0; k < num; ++k)
        if (count[k] > 0) todo.push_back(k);
    bool job_done = job == nullptr;
    for (size_t g = 0; g < todo.size() || !job_done; g += hlf::kMaxEnumTasks) {
        const size_t m = g < todo.size() ? std::min<size_t>(hlf::kMaxEnumTasks, todo.size() - g) : 0;
        uint64_t total = 0;
        for (size_t j = 0; j < m; ++j) total += range_of(todo[g + j]).ntiles;
        hlf::EnumTasks tasks;
        std::memset(&tasks, 0, sizeof(tasks));
        const uint32_t tpb = hlf::vec_tiles_per_block(total);
        tasks.tiles_per_block = tpb;
        uint64_t block = 0;
        std::fill(tasks.first, tasks.first + hlf::kMaxEnumTasks, ~0u);
        for (size_t j = 0; j < m; ++j) {
            const int k = todo[g + j];
            const int i = inst[k];
            hlf::VecTask &t = tasks.t[j];
            t.inst = i;
            t.n = b->n[i];
            t.basis = b->basis + b->mat_off[i];
            t.shift = b->shift + b->vec_off[i];
            t.g = range_of(k);
            t.block0 = (uint32_t)block;
            if (j > 0) tasks.first[j - 1] = (uint32_t)block;
            // a range without tiles (vec_range) still takes a workgroup for the gate
            block += t.g.ntiles ? (t.g.ntiles + (uint64_t)tpb - 1) / tpb : 1u;
        }
        tasks.blocks = (uint32_t)block;
        tasks.status = b->status;
        tasks.rank = b->rank;
        const hlf::FactorJob *jb = job_done ? nullptr : job;
        job_done = true;
        if (jb) tasks.job_blocks = (uint32_t)((jb->num + hlf::kWavesPerVecBlock - 1) / hlf::kWavesPerVecBlock);
        if (word_bits == 16) launch_enum_group<uint16_t>(tasks, jb, stream);
        else if (word_bits == 32) launch_enum_group<uint32_t>(tasks, jb, stream);
        else launch_enum_group<uint64_t>(tasks, jb, stream);
        if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    }
    return HLF_OK;
}

}  // namespace

extern "C" {

hlf_status hlf_batch_enumerate(hlf_batch b, int32_t num, const int32_t *inst,
                               const uint64_t *begin, const uint64_t *count, void *const *out,
                               int32_t word_bits, hipStream_t stream) {
    return batch_enumerate_impl(b, num, inst, begin, count, out, word_bits, nullptr, stream);
}

hlf_status hlf_batch_enumerate_overlap(hlf_batch b, int32_t num, const int32_t *inst,
                                       const uint64_t *begin, const uint64_t *count,
                                       void *const *out, int32_t word_bits, hlf_batch next,
                                       const uint8_t *A_next_dev, hipStream_t stream) {
    if (!next || !A_next_dev || next == b || next->max_n > 64) return HLF_EINVAL;
    hlf::FactorJob job;
    job.d = view_of(next);
    job.A = A_next_dev;
    job.first = 0;
    job.num = next->count;
    return batch_enumerate_impl(b, num, inst, begin, count, out, word_bits, &job, stream);
}

hlf_status hlf_batch_solve(hlf_batch b, const uint8_t *A_dev, int32_t num, const int32_t *inst,
                           const uint64_t *begin, const uint64_t *count, void *const *out,
                           int32_t word_bits, hipStream_t stream) {
    if (!b || !A_dev || num < 1 || num > hlf::kMaxEnumTasks || !inst || !begin || !count || !out)
        return HLF_EINVAL;
    if (word_bits != 16 && word_bits != 32 && word_bits != 64) return HLF_EINVAL;
    const int V = 16 / (word_bits / 8);
    const int S = word_bits == 16 ? hlf::tile_shift<uint16_t>()
                  : word_bits == 32 ? hlf::tile_shift<uint32_t>() : hlf::tile_shift<uint64_t>();
    std::vector<uint64_t> tiles(num);
    uint64_t total = 0;
    for (int k = 0; k < num; ++k) {
        const int i = inst[k];
        if (i < 0 || i >= b->count || b->n[i] > word_bits) return HLF_EINVAL;
        if (count[k] == 0 || !out[k] || begin[k] % V != 0 || ((uintptr_t)out[k] & 15u) != 0 ||
            begin[k] + count[k] < begin[k])
            return HLF_EINVAL;
        const uint64_t end = begin[k] + count[k];
        tiles[k] = ((end - 1) >> S) - (begin[k] >> S) + 1;
        total += tiles[k];
    }
    const uint64_t target_blocks = (uint64_t)hlf::device_cu_count() * hlf::kTileBlocksPerCU;
    const uint64_t tpb = std::max<uint64_t>(1, (total + target_blocks - 1) / target_blocks);
    hlf::SolveTasks tasks;
    std::memset(&tasks, 0, sizeof(tasks));
    tasks.num = num;
    uint64_t block = 0;
    for (int k = 0; k < num; ++k) {
        const int i = inst[k];
        hlf::EnumTask &t = tasks.t[k];
        t.status = b->status + i;
        t.rank = b->rank + i;
        t.basis = b->basis + b->mat_off[i];
        t.shift = b->shift + b->vec_off[i];
        t.out = out[k];
        t.begin = begin[k];
        t.count = count[k];
        t.block0 = (uint32_t)block;
        t.tiles_per_block = (uint32_t)tpb;
        tasks.inst[k] = i;
        block += (tiles[k] + tpb - 1) / tpb;
    }
    if (block > 0xFFFFFFFFull) return HLF_EINVAL;
    const hlf::BatchDev d = view_of(b);
    if (word_bits == 16)
        hipLaunchKernelGGL(hlf::batch_solve_kernel<uint16_t>, dim3((unsigned)block), dim3(hlf::kTileThreads), 0, stream, d, A_dev, tasks, b->solve_flags, b->solve_done);
    else if (word_bits == 32)
        hipLaunchKernelGGL(hlf::batch_solve_kernel<uint32_t>, dim3((unsigned)block), dim3(hlf::kTileThreads), 0, stream, d, A_dev, tasks, b->solve_flags, b->solve_done);
    else
        hipLaunchKernelGGL(hlf::batch_solve_kernel<uint64_t>, dim3((unsigned)block), dim3(hlf::kTileThreads), 0, stream, d, A_dev, tasks, b->solve_flags, b->solve_done);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

hlf_status hlf_batch_reduce(hlf_batch b, const uint8_t *A_dev, int32_t max_rank,
                            const hlf_batch_params *params, hipStream_t stream) {
    if (!b || !A_dev || max_rank < 0 || max_rank > HLF_MAX_ENUM_RANK) return HLF_EINVAL;
    if (b->max_n > 192) return HLF_EINVAL;
    const hlf_batch_params p = params ? *params : b->tuned;
    if (!params_ok(p) || !claims_fit(b, max_rank, p.chunk_log2)) return HLF_EINVAL;
    return batch_reduce_impl(b, A_dev, max_rank, p, stream);
}

hlf_status hlf_batch_tune(hlf_batch b, const uint8_t *A_dev, int32_t max_rank,
                          hlf_batch_params *best, float *best_ms, hipStream_t stream) {
    if (!b || !A_dev || max_rank < 0 || max_rank > HLF_MAX_ENUM_RANK) return HLF_EINVAL;
    if (b->max_n > 192) return HLF_EINVAL;
    const auto key = std::make_tuple(b->count, b->max_n, b->piv_entries, (int)max_rank);
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune_cache.find(key);
        if (it != g_tune_cache.end()) {
            b->tuned = it->second.first;
            b->has_tuned = true;
            if (best) *best = it->second.first;
            if (best_ms) *best_ms = it->second.second;
            return HLF_OK;
        }
    }
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return HLF_EDEVICE;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return HLF_EDEVICE;
    }
    // Several chunk sizes come to one launch (piece_log2): the largest of them
    // stands for it, which leaves the most room for a later call's max_rank.
    const int chunks[] = {22, 20, 18, 16, 14};
    const int waves[] = {2, 4, 8, 12};
    std::vector<ReducePlan> timed;
    hlf_batch_params bestp = b->tuned;
    float bestt = 1e30f;
    hlf_status st = HLF_OK;
    bool any = false;
    for (int c : chunks) {
        if (!claims_fit(b, max_rank, c)) continue;
        any = true;
        for (int w : waves) {
            const hlf_batch_params p = {c, w};
            const ReducePlan plan = b->max_n <= 64 ? reduce_plan<1>(b->count, max_rank, p) : reduce_plan<3>(b->count, max_rank, p);
            if (std::find(timed.begin(), timed.end(), plan) != timed.end()) continue;
            timed.push_back(plan);
            st = batch_reduce_impl(b, A_dev, max_rank, p, stream);  // warm
            if (st != HLF_OK) break;
            float tsum = 0;
            for (int rep = 0; rep < 2 && st == HLF_OK; ++rep) {
                if (hipEventRecord(e0, stream) != hipSuccess) st = HLF_EDEVICE;
                if (st == HLF_OK) st = batch_reduce_impl(b, A_dev, max_rank, p, stream);
                if (st == HLF_OK && hipEventRecord(e1, stream) != hipSuccess) st = HLF_EDEVICE;
                if (st == HLF_OK && hipEventSynchronize(e1) != hipSuccess) st = HLF_EDEVICE;
                float ms = 0;
                if (st == HLF_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) st = HLF_EDEVICE;
                tsum += ms;
            }
            if (st != HLF_OK) break;
            if (tsum / 2 < bestt) {
                bestt = tsum / 2;
                bestp = p;
            }
        }
        if (st != HLF_OK) break;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != HLF_OK) return st;
    if (!any) return HLF_EINVAL;
    b->tuned = bestp;
    b->has_tuned = true;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune_cache[key] = {bestp, bestt};
    }
    if (best) *best = bestp;
    if (best_ms) *best_ms = bestt;
    return HLF_OK;
}

hlf_status hlf_batch_graph_capture(hlf_batch b, const uint8_t *A_dev, int32_t max_rank,
                                   const hlf_batch_params *params) {
    if (!b || !A_dev || max_rank < 0 || max_rank > HLF_MAX_ENUM_RANK) return HLF_EINVAL;
    if (b->max_n > 192) return HLF_EINVAL;
    const hlf_batch_params p = params ? *params : b->tuned;
    if (!params_ok(p) || !claims_fit(b, max_rank, p.chunk_log2)) return HLF_EINVAL;
    hipStream_t s;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return HLF_EDEVICE;
    hlf_status st = HLF_OK;
    hipGraph_t g = nullptr;
    if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) != hipSuccess) st = HLF_EDEVICE;
    if (st == HLF_OK) {
        st = batch_reduce_impl(b, A_dev, max_rank, p, s);
        if (hipStreamEndCapture(s, &g) != hipSuccess) st = HLF_EDEVICE;
    }
    hipGraphExec_t exec = nullptr;
    if (st == HLF_OK && hipGraphInstantiate(&exec, g, nullptr, nullptr, 0) != hipSuccess)
        st = HLF_EDEVICE;
    (void)hipStreamDestroy(s);
    if (st != HLF_OK) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->graph = g;
    b->graph_exec = exec;
    return HLF_OK;
}

hlf_status hlf_batch_graph_launch(hlf_batch b, hipStream_t stream) {
    if (!b || !b->graph_exec) return HLF_EINVAL;
    return hipGraphLaunch(b->graph_exec, stream) == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Allocation-free batched reduce.  Its scratch -- the work queue, the chunk
// slots, the layout offsets and the checked sizes -- is one file-scope device
// array; each device holds its own copy, located once per device with
// hipGetSymbolAddress and used through that address only.
// ---------------------------------------------------------------------------
namespace {
constexpr int kNoAllocMaxCount = 16384;
constexpr size_t kNoAllocQueueBytes = 256;
constexpr size_t kNoAllocSlotBytes = sizeof(hlf::ChunkSlot) * kNoAllocMaxCount;
constexpr size_t kNoAllocOffBytes = sizeof(int64_t) * kNoAllocMaxCount;
constexpr size_t kNoAllocScratchBytes =
    kNoAllocQueueBytes + kNoAllocSlotBytes + 4 * kNoAllocOffBytes + sizeof(int32_t) * kNoAllocMaxCount;
static_assert(sizeof(hlf::QueueHead) <= kNoAllocQueueBytes, "queue head fits its space");
static_assert(kNoAllocMaxCount <= 1024 * hlf::kLayoutPer, "one layout workgroup covers every instance");
}  // namespace

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {};

// Device address of this device's scratch array (looked up once per device).
hlf_status scratch_address(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return HLF_EDEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr)
            return HLF_EDEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return HLF_OK;
}
}  // namespace

extern "C" {

hlf_status hlf_batch_reduce_noalloc(int32_t count, int32_t max_n, const int32_t *n_dev,
                                    const uint8_t *A_dev, int32_t max_rank,
                                    const hlf_batch_params *params, int32_t *status_dev,
                                    int32_t *rank_dev, int32_t *pivots_dev, uint64_t *basis_dev,
                                    uint64_t *shift_dev, uint64_t *kernel_dev,
                                    uint64_t *counts_dev, uint64_t *hash_dev, hipStream_t stream) {
    if (count < 1 || count > kNoAllocMaxCount || max_n < 1 || max_n > 192) return HLF_EINVAL;
    if (!n_dev || !A_dev || !status_dev || !rank_dev || !pivots_dev || !basis_dev || !shift_dev ||
        !counts_dev || !hash_dev)
        return HLF_EINVAL;
    if (max_rank < 0 || max_rank > HLF_MAX_ENUM_RANK) return HLF_EINVAL;
    const hlf_batch_params p = params ? *params : hlf_batch_params{20, 8};
    if (!params_ok(p) || !claims_fit_count(count, max_rank, p.chunk_log2)) return HLF_EINVAL;
    void *base = nullptr;
    const hlf_status st = scratch_address(&base);
    if (st != HLF_OK) return st;
    unsigned char *sb = static_cast<unsigned char *>(base);
    auto *queue = reinterpret_cast<hlf::QueueHead *>(sb);
    auto *slots = reinterpret_cast<hlf::ChunkSlot *>(sb + kNoAllocQueueBytes);
    auto *offs = reinterpret_cast<int64_t *>(sb + kNoAllocQueueBytes + kNoAllocSlotBytes);
    auto *n_eff = reinterpret_cast<int32_t *>(offs + 4 * kNoAllocMaxCount);
    hlf::BatchDev d;
    d.count = count;
    d.n = n_eff;
    d.dense_off = offs;
    d.mat_off = offs + kNoAllocMaxCount;
    d.vec_off = offs + 2 * kNoAllocMaxCount;
    d.piv_off = offs + 3 * kNoAllocMaxCount;
    d.order = nullptr;
    d.status = status_dev;
    d.rank = rank_dev;
    d.pivots = pivots_dev;
    d.basis = basis_dev;
    d.shift = shift_dev;
    d.kernel = kernel_dev;
    d.counts = counts_dev;
    d.hash = hash_dev;
    hipLaunchKernelGGL(hlf::noalloc_layout_kernel, dim3(1), dim3(1024), 0, stream, n_dev, count,
                       max_n, n_eff, offs, offs + kNoAllocMaxCount, offs + 2 * kNoAllocMaxCount,
                       offs + 3 * kNoAllocMaxCount, queue, slots);
    if (hipGetLastError() != hipSuccess) return HLF_EDEVICE;
    if (max_n <= 64) return launch_reduce_view<1>(d, A_dev, max_rank, p, queue, slots, stream);
    return launch_reduce_view<3>(d, A_dev, max_rank, p, queue, slots, stream);
}

}  // extern "C"
