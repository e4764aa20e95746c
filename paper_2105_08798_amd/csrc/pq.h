// Work queues of the persistent product kernels (PqLists).
#pragma once
#include <algorithm>
#include <map>
#include <mutex>

#include "common.h"

// Next job for thread 0's caller: with one list per XCD the caller takes jobs from the list
// of its own XCD, then, as lists run out, from the others in turn; past the end of all of
// them: 0x7fffffff.  `cur` counts the lists the caller has exhausted.
__device__ inline int pq_take(const PqLists& q, int& cur) {
    const int home = q.nl > 1 ? (int)(blockIdx.x % q.nl) : 0;
    while (cur < q.nl) {
        const int l = (home + cur) % q.nl;
        const int s = atomicAdd(&q.ctr[l], 1);
        if (s < q.start[l + 1] - q.start[l]) return q.start[l] + s;
        ++cur;
    }
    return 0x7fffffff;
}
// The last of `leavers` callers to leave sets the counters back to zero for the next launch
// (so the launch can be replayed from a graph).
__device__ inline void pq_leave(const PqLists& q, int leavers) {
    __threadfence();
    if (atomicAdd(&q.ctr[8], 1) == leavers - 1) {
        for (int l = 0; l < q.nl; ++l) atomicExch(&q.ctr[l], 0);
        atomicExch(&q.ctr[8], 0);
    }
}

// Per wave: every wave of the launch takes its own jobs (no barrier).
__device__ inline int pq_next_wave(const PqLists& q, int& cur) {
    int j = 0;
    if ((threadIdx.x & 63) == 0) j = pq_take(q, cur);
    return __builtin_amdgcn_readfirstlane(j);
}
__device__ inline void pq_done_wave(const PqLists& q) {
    if ((threadIdx.x & 63) == 0) pq_leave(q, (int)gridDim.x * (int)(blockDim.x >> 6));
}

// Per work group: thread 0 takes the job for all of them.
__device__ inline int pq_next(const PqLists& q, int* slot, int& cur) {
    if (threadIdx.x == 0) *slot = pq_take(q, cur);
    __syncthreads();
    const int j = __builtin_amdgcn_readfirstlane(*slot);   // uniform: the job fields go to SGPRs
    __syncthreads();                     // every thread has read the slot; LDS of the last job free
    return j;
}
__device__ inline void pq_done(const PqLists& q) {
    if (threadIdx.x == 0) pq_leave(q, (int)gridDim.x);
}

// Compute units of the current device (one device type per process).
static inline int device_cus() {
    static const int n = [] {
        int dev = 0, cus = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        return std::max(1, cus);
    }();
    return n;
}

// Work groups of a persistent launch: the kernel's occupancy per CU times the CUs
// (queried once per kernel and cached; the library runs on one device type per process).
template <typename K>
static int pq_groups_of(K kernel, int threads) {
    static std::mutex mu;
    static std::map<const void*, int> cache;
    std::lock_guard<std::mutex> lock(mu);
    const void* key = (const void*)kernel;
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0);
    const int g = std::max(1, per_cu) * device_cus();
    cache[key] = g;
    return g;
}
