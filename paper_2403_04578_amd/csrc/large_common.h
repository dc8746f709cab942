// Helpers shared by the per-sweep paths for large networks (fpi_large.hip, fpi_large64.hip).
#pragma once

#include <algorithm>

#include "tpf_internal.h"

namespace tpf {
namespace {

// ZIP shares of Eq. (2) per PQ bus: all NULL for constant-power loads; aZ NULL when no
// bus has a constant-impedance share.
struct ZipShares {
    const double *aP, *aI, *aZ;
};

// Tells the host that queues the sweeps that none is left to do (a store to pinned host
// memory, visible to the host without any wait on the device).
__device__ __forceinline__ void post_done(int *done_flag, int seq) {
    if (done_flag) __hip_atomic_store(done_flag, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Places of the staying columns of a chunk in the next list: a rank from the
// block's ballots and one atomic per chunk (a counter shared by every column of the sweep
// would serialise a million atomics).  Returns the slot, or -1 when `stay` is false.
__device__ __forceinline__ int chunk_slot(bool stay, int *counter, int *wsum, int *base) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long m = __ballot(stay);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(m);
    __syncthreads();
    if (tid == 0) {
        const int tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        *base = tot ? atomicAdd(counter, tot) : 0;
    }
    __syncthreads();
    int off = *base;
    for (int w = 0; w < wave; ++w) off += wsum[w];
    return stay ? off + rank : -1;
}

}  // namespace

// Whether a sweep of solve `seq` already found every column retired: the sweeps queued
// after it would all exit at once, so the host queues no more.  A read of pinned host
// memory; it never waits for the device.
[[maybe_unused]] static bool all_retired(const DeviceNet &dn, int seq) {
    return dn.done_host && __atomic_load_n(dn.done_host, __ATOMIC_ACQUIRE) == seq;
}

// Columns per finish chunk: about 16,384 buses' worth, a power of two in [4, 256] (one
// atomic per chunk keeps a million-column sweep from serialising on the list counter,
// and small chunks keep a few wide columns spread over many wavefronts).
[[maybe_unused]] static int finish_chunk(int n) {
    int c = 4;
    while (c < 256 && 2 * c * n <= 16384) c *= 2;
    return c;
}

// Fixed grids of the queued sweeps: enough blocks to fill the chip, few enough that a
// sweep with nothing left to do costs little.
constexpr int64_t kGemmGrid = 1024, kFinishGrid = 1024;

// Grid of a persistent GEMM: at most kGemmGrid blocks and no more than are resident at
// once (CUs x blocks per CU).  Its blocks share the tiles evenly, so blocks beyond the
// resident ones would start only after others had finished all of theirs and run the
// kernel's second half at a fraction of the occupancy (the 16-bit GEMM, three blocks per
// CU for its 43 KB of LDS, took twice as long with 1,024 blocks).
[[maybe_unused]] static int64_t gemm_grid(const void *kernel, int threads, int64_t tiles) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return std::max<int64_t>(1, std::min<int64_t>({kGemmGrid, (int64_t)num_cus() * per_cu, tiles}));
}

}  // namespace tpf
