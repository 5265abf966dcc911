// The factors of a block that are fetched ahead of its second part.
#pragma once
#include <stdint.h>

// Touches a word of every 128 bytes of the factors of `nrows` rows and `ncols` columns (their numbers in rows, cols;
// column c's factor is the store's m + c), `by` threads side by side, this one the `first`: load(i) reads float i of the store.
// The loads are ordinary ones, which leave their lines in the die's cache.  AGENT_H: the columns come from and go to
// workgroups on other dies within the launch and are read and written past that cache; they are left alone.
template <bool AGENT_H, class Load>
__device__ __forceinline__ void touch_factors(int first, int by, int nrows, int ncols, const int32_t *rows, const int32_t *cols, int64_t m, int L, Load load) {
    const int lines = (L * 4 + 127) / 128, count = AGENT_H ? nrows : nrows + ncols;
    for (int t = first; t < count; t += by) {
        const int64_t k = t < nrows ? rows[t] : m + cols[t - nrows];
        for (int i = 0; i < lines; ++i) load(k * L + 32 * i);
    }
}
