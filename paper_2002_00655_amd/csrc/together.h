// Decisions to leave that a workgroup takes as a whole.  The handle's error flag may be set by other workgroups of the
// same launch at any moment, so wavefronts that look at it one by one can see different values; where the rest of a
// kernel needs every thread (shares of a check, a barrier, tables filled together), one answer must hold for all.
#pragma once
#include <stdint.h>

#include "dpaps.h"

// Whether a call of few keys is to do nothing: a key is out of range, or the flag is set.  Every workgroup of the call's
// one kernel looks at all of the keys before it does anything else, so that a bad call changes nothing, and no thread
// leaves before all have looked.  Sets the error; the same in all threads.
// AHEAD: keys of a thread whose reads are on their way together.  keep(p, k): called for every key as it is read.
constexpr int64_t FEW_KEYS = 2048;
template <int AHEAD, class Keep>
__device__ __forceinline__ bool few_keys_off(const int64_t *keys, int64_t n, int64_t K, int32_t *err, Keep keep) {
    const bool was_off = *(volatile const int32_t *)err != 0;
    bool off = was_off;
#pragma unroll AHEAD
    for (int64_t p = threadIdx.x; p < n; p += blockDim.x) {
        const int64_t k = keys[p];
        keep(p, k);
        off |= k < 0 || k >= K;
    }
    const bool any = __syncthreads_or(off ? 1 : 0) != 0;
    if (any && threadIdx.x == 0 && !was_off) atomicExch(err, PS_EKEY);     // (an error that stands already is kept)
    return any;
}
template <int AHEAD = 1>
__device__ __forceinline__ bool few_keys_off(const int64_t *keys, int64_t n, int64_t K, int32_t *err) {
    return few_keys_off<AHEAD>(keys, n, K, err, [](int64_t, int64_t) {});
}

// The flag as work before this launch left it: asked for here, looked at when the kernel's first reads, which need no check, are on their
// way - a trip to memory less for every kernel of a call.  In the kernels that check the keys beside other work - the first count of
// a sort, a step's keys - the launch may set the flag itself, so that wavefronts see it differently and part of a workgroup leaves.  There that is
// harmless: what the others count or write lies in range, and every kernel behind them sees the flag and uses none of it.
__device__ __forceinline__ int32_t flag_ahead(const int32_t *err) { return *(volatile const int32_t *)err; }

// One thread's look at the flag, for the whole workgroup: what stands in `word` (in LDS) after the next barrier holds for all.
__device__ __forceinline__ void look_for_all(const int32_t *err, int *word) {
    if (threadIdx.x == 0) *word = *(volatile const int32_t *)err;
}
