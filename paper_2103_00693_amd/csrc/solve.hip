// Stage 1 and stage 2 of one small instance in ONE launch (n <= 64): every
// workgroup packs and validates A and factors it on its first wave (the
// paper's Section 2 tasks (1)-(4): a few microseconds of one wave at this
// size), then materialises its own tiles of [begin, begin + count) (Eq. (3)
// and the final CNOT layer, as in stage2.h).  Workgroup 0 writes the caller's
// record; every other workgroup writes a private copy in LDS, so the record
// has a single writer and a range error cannot race with another
// workgroup's verdict.  The redundant factorisations run side by side and no
// workgroup waits for another: this is the latency path for small instances.
#include "factor_wave.h"
#include "hlf_device.h"
#include "hlf_internal.h"
#include "stage2.h"

namespace hlf {
namespace {

template <typename T, bool kAtOnce>
__global__ __launch_bounds__(kTileThreads) void solve_dense_kernel(const uint8_t *__restrict__ A,
                                                                   int n, FactorOut rec,
                                                                   uint64_t begin, uint64_t count,
                                                                   T *__restrict__ out,
                                                                   uint64_t tiles_per_block) {
    constexpr int S = tile_shift<T>();
    __shared__ WaveSmem<1> sm;
    __shared__ uint64_t Bx[64];
    __shared__ int32_t own_status, own_rank, own_piv[64];
    __shared__ uint64_t own_basis[64], own_shift[1];
    __shared__ int go;
    if (threadIdx.x < 64) {
        FactorOut o = rec;
        if (blockIdx.x != 0) {  // generic pointers into this workgroup's LDS
            o.status = &own_status;
            o.rank = &own_rank;
            o.pivots = own_piv;
            o.basis = own_basis;
            o.shift = own_shift;
            o.kernel = nullptr;
        }
        const bool badv = wave_load_dense<1>(A, n, 1, sm);
        const int r = factor_wave_core<1>(n, 1, badv, o, sm);  // -1: invalid matrix
        const bool ok = r >= 0 && r <= HLF_MAX_ENUM_RANK && begin <= (1ull << r) &&
                        count <= (1ull << r) - begin;
        // After this lane's own status write in factor_wave_core.
        if (r >= 0 && !ok && blockIdx.x == 0 && threadIdx.x == 0) *rec.status = HLF_ERANGE;
        if (ok) Bx[threadIdx.x] = ((int)threadIdx.x < r) ? sm.orig[sm.piv[threadIdx.x]] : 0ull;
        if (threadIdx.x == 0) go = (ok && count > 0) ? 1 : 0;
    }
    __syncthreads();
    if (!go) return;
    const uint64_t end = begin + count;
    const uint64_t ntiles = ((end - 1) >> S) - (begin >> S) + 1;
    const uint64_t t0 = (uint64_t)(kAtOnce ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x) * tiles_per_block;
    if (t0 >= ntiles) return;
    const uint64_t t1 = (t0 + tiles_per_block < ntiles) ? t0 + tiles_per_block : ntiles;
    enum_tiles_w1<T, kAtOnce>(Bx, sm.shiftw[0], begin, count, out, t0, t1);
}

template <typename T>
hlf_status launch_solve_dense_t(const uint8_t *A, int n, const FactorOut &rec, uint64_t begin,
                                uint64_t count, T *out, hipStream_t stream) {
    constexpr int S = tile_shift<T>();
    const uint64_t end = begin + count;
    uint64_t ntiles = 1;  // count = 0 or a wrapping range: one workgroup (stage 1 only)
    if (count > 0 && end > begin) ntiles = ((end - 1) >> S) - (begin >> S) + 1;
    // As many workgroups as run at once (two per CU), since each one factors
    // first, where that gives them 128 to 512 KiB each; their stores are then
    // plain and by XCD.  2^24 32-bit words 15.9 us, 64-bit 25.3, 2^25 44, and
    // 16.7, 30, 55 in blocks of at most 128 KiB, nontemporal and in launch
    // order, which is as good or better below and above: 2^22 64-bit words
    // 12.3 us against 13.0, 2^26 102 against 106.
    const uint64_t resident = 2ull * (uint64_t)device_cu_count();
    const uint64_t fill = (ntiles + resident - 1) / resident;
    const bool at_once = fill * kTileBytes >= kBlockBytes && fill * kTileBytes <= 4 * kBlockBytes;
    const uint64_t tpb = at_once ? fill : materialise_tiles_per_block(ntiles, kTileBytes);
    const uint64_t blocks = (ntiles + tpb - 1) / tpb;
    if (at_once)
        hipLaunchKernelGGL((solve_dense_kernel<T, true>), dim3((unsigned)blocks), dim3(kTileThreads), 0, stream, A, n,
                           rec, begin, count, out, tpb);
    else
        hipLaunchKernelGGL((solve_dense_kernel<T, false>), dim3((unsigned)blocks), dim3(kTileThreads), 0, stream, A, n,
                           rec, begin, count, out, tpb);
    return hipGetLastError() == hipSuccess ? HLF_OK : HLF_EDEVICE;
}

}  // namespace

hlf_status launch_solve_dense(const uint8_t *A, int n, const FactorOut &rec, uint64_t begin,
                              uint64_t count, int word_bits, void *out, hipStream_t stream) {
    if (word_bits == 16)
        return launch_solve_dense_t<uint16_t>(A, n, rec, begin, count, (uint16_t *)out, stream);
    if (word_bits == 32)
        return launch_solve_dense_t<uint32_t>(A, n, rec, begin, count, (uint32_t *)out, stream);
    return launch_solve_dense_t<uint64_t>(A, n, rec, begin, count, (uint64_t *)out, stream);
}

}  // namespace hlf
