// Byte offsets into the factors of a block's rows or columns, a buffer each.  An access at an offset past a buffer's end reads
// zero and writes nothing, and the hardware takes the offset as an unsigned number of 32 bits: that is how lanes without an
// entry or a component are switched off without branching.
#pragma once
#include <stdint.h>

// Past the end of every buffer that is taken: the host refuses a block whose factors span as many bytes or more.
#define DPAPS_PAST_END 0x7FFFF000
static inline bool dpaps_span_ok(int64_t rows, int64_t L) { return rows * L * 4 < (int64_t)DPAPS_PAST_END; }

// where row `row` of the block starts, if there is one; where component k of a row lies in it, if the rank has one
__device__ __forceinline__ int row_start(bool there, int row, int L) { return there ? row * L * 4 : DPAPS_PAST_END; }
__device__ __forceinline__ int component_at(int k, int L) { return k < L ? k * 4 : DPAPS_PAST_END; }

// The sum of two of them, either of which may be DPAPS_PAST_END: two of those, with an access of 16 bytes behind, still fit.
__device__ __forceinline__ int past_end_sum(int a, int b) { return (int)((uint32_t)a + (uint32_t)b); }
static_assert(2 * (uint64_t)DPAPS_PAST_END + 16 <= (uint64_t)1 << 32, "no sum of two offsets comes round to the buffer's start");
