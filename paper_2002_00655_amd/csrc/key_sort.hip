// Stable sort of (key, position) pairs by key, for the cumulative push (Sec. 2.1: a push
// adds an update term to the stored value; Sec. 3.7: the operations on one key are applied
// one after the other).  A push with repeated keys must apply a key's terms in argument
// order, so the pairs are brought into the order (key, position) first.
//
// What is known here and a general sort cannot assume: keys are below num_keys (19 bits for
// half a million keys, 24 for eleven million), and positions are 0 .. n-1 in input order,
// so a stable sort by the key's digits alone yields (key, position) order and the positions
// need not be read in the first pass.  Least-significant-digit passes; each pass is
//   1. k_sort_count    one workgroup per tile of the input: how many pairs of the tile fall
//                      into each bucket (LDS counters), written bucket-major;
//   2. k_sort_rowsum   one workgroup per bucket: the bucket's total;
//   3. k_sort_scan     one workgroup per bucket: where the bucket starts (pairs in lower
//                      buckets) and, from there, where each tile's share of it starts;
//   4. k_sort_scatter  one workgroup per tile: a wavefront takes 64 consecutive pairs at a
//                      time; lanes with the same digit find each other with one ballot per
//                      bit of the digit, the first of them advances the wavefront's own
//                      counter of that bucket in LDS, the others take their place behind it
//                      in lane order; the wavefronts' counters are then turned into
//                      offsets in wavefront order, so that pairs of one bucket keep their
//                      input order - the pass is stable - and every pair is stored.
// Up to MID_MAX pairs the tiles are few and larger, and every workgroup of the scatter works out its offsets from all
// tiles' counters itself: two launches per pass instead of four; so they are from BIG_MIN up to BIG_MAX pairs, in larger
// tiles that are put in order in LDS before they are stored.  Up to FEW_MAX pairs one workgroup sorts them in LDS.
// A caller that has not checked its keys asks for it: the first kernel then sets the handle's error, which ends the rest.
// Integer work only: the result is the same bit for bit whatever the scheduling.
#include "common.h"
#include "together.h"

#include <algorithm>

namespace {

constexpr int SORT_THREADS = 256;          // 4 wavefronts per tile
constexpr int SORT_WAVES = SORT_THREADS / 64;
constexpr int SORT_MAX_BITS = 10;          // bits of a digit at most: 1024 buckets

__device__ __forceinline__ uint32_t digit_of(uint64_t key, int shift, uint32_t mask) { return (uint32_t)(key >> shift) & mask; }

// FIRST: the input is the caller's key array (int64, checked to be in range or the handle is frozen) and the
// positions are the indices; otherwise the pairs come from the previous pass.
template <int ITEMS, bool FIRST>
__global__ __launch_bounds__(SORT_THREADS) void k_sort_count(const int64_t *keys_in, const uint64_t *pk_in, int64_t n, int shift, int bits,
                                                             int64_t num_tiles, uint32_t *hist, int64_t check_below, int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ uint32_t cnt[1 << SORT_MAX_BITS];
    const int R = 1 << bits;
    const uint32_t mask = (uint32_t)R - 1u;
    const int64_t base = (int64_t)blockIdx.x * (SORT_THREADS * ITEMS);
    uint64_t key[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t q = base + (int64_t)r * SORT_THREADS + threadIdx.x;
        key[r] = q < n ? (FIRST ? (uint64_t)keys_in[q] : pk_in[q]) : 0;
    }
    if (stop) return;
    for (int i = threadIdx.x; i < R; i += SORT_THREADS) cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (base + (int64_t)r * SORT_THREADS + threadIdx.x < n) {
            if (FIRST && check_below > 0 && key[r] >= (uint64_t)check_below) atomicExch(err, PS_EKEY);
            atomicAdd(&cnt[digit_of(key[r], shift, mask)], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < R; i += SORT_THREADS) hist[(int64_t)i * num_tiles + blockIdx.x] = cnt[i];
}

__global__ __launch_bounds__(256) void k_sort_rowsum(const uint32_t *hist, int64_t num_tiles, uint32_t *row_total, const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ uint32_t s[256];
    const uint32_t *row = hist + (int64_t)blockIdx.x * num_tiles;
    uint32_t acc = 0;
    for (int64_t t = threadIdx.x; t < num_tiles; t += 256) acc += row[t];
    if (stop) return;
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) row_total[blockIdx.x] = s[0];
}

// hist[b][t] <- pairs in buckets below b + pairs of bucket b in tiles before t
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t *hist, int64_t num_tiles, const uint32_t *row_total, const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ uint32_t s[256];
    __shared__ uint32_t carry;
    const int b = blockIdx.x;
    uint32_t acc = 0;
    for (int i = threadIdx.x; i < b; i += 256) acc += row_total[i];
    if (stop) return;
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) carry = s[0];
    __syncthreads();
    uint32_t *row = hist + (int64_t)b * num_tiles;
    for (int64_t t0 = 0; t0 < num_tiles; t0 += 256) {
        const int64_t t = t0 + threadIdx.x;
        const uint32_t v = t < num_tiles ? row[t] : 0u;
        // inclusive scan of the 256 values in LDS (Hillis-Steele, two buffers in one array by barriers)
        s[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const uint32_t add = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0u;
            __syncthreads();
            s[threadIdx.x] += add;
            __syncthreads();
        }
        const uint32_t incl = s[threadIdx.x], c = carry;
        if (t < num_tiles) row[t] = c + incl - v;
        __syncthreads();
        if (threadIdx.x == 255) carry = c + incl;
        __syncthreads();
    }
}

template <int ITEMS, bool FIRST>
__global__ __launch_bounds__(SORT_THREADS) void k_sort_scatter(const int64_t *keys_in, const uint64_t *pk_in, const uint32_t *pp_in, int64_t n,
                                                               int shift, int bits, int64_t num_tiles, const uint32_t *hist, uint64_t *pk_out,
                                                               uint32_t *pp_out, const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ uint32_t wh[SORT_WAVES][1 << SORT_MAX_BITS];
    const int R = 1 << bits;
    const uint32_t mask = (uint32_t)R - 1u;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // wavefront w takes the pairs [base + w * 64 * ITEMS, + 64 * ITEMS), 64 consecutive ones per round
    const int64_t base = (int64_t)blockIdx.x * (SORT_THREADS * ITEMS) + (int64_t)wave * 64 * ITEMS;
    uint64_t key[ITEMS];
    uint32_t pos[ITEMS], rank[ITEMS];
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t q = base + r * 64 + lane;
        key[r] = 0; pos[r] = 0;
        if (q < n) {
            key[r] = FIRST ? (uint64_t)keys_in[q] : pk_in[q];
            pos[r] = FIRST ? (uint32_t)q : pp_in[q];
        }
    }
    // where the tile's pairs of this thread's buckets go
    constexpr int OWN = (1 << SORT_MAX_BITS) / SORT_THREADS;
    uint32_t starts[OWN];
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        const int b = threadIdx.x + i * SORT_THREADS;
        starts[i] = b < R ? hist[(int64_t)b * num_tiles + blockIdx.x] : 0u;
    }
    if (stop) return;
    for (int i = threadIdx.x; i < SORT_WAVES * (1 << SORT_MAX_BITS); i += SORT_THREADS) (&wh[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = base + r * 64 + lane < n;
        const uint32_t d = digit_of(key[r], shift, mask);
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = ((d >> b) & 1u) != 0u;
            const uint64_t v = __ballot(valid && bit);
            same &= bit ? v : ~v;
        }
        // `same`: the valid lanes with this lane's digit (meaningful in valid lanes only)
        uint32_t before = 0;
        const int leader = valid ? __ffsll((long long)same) - 1 : lane;
        if (valid && lane == leader) {
            before = wh[wave][d];
            wh[wave][d] = before + (uint32_t)__popcll(same);
        }
        before = (uint32_t)__shfl((int)before, leader);
        rank[r] = before + (uint32_t)__popcll(same & below);
    }
    __syncthreads();
    // a wavefront's counters become the offsets of its first pair of each bucket
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        const int b = threadIdx.x + i * SORT_THREADS;
        if (b >= R) break;
        uint32_t run = starts[i];
#pragma unroll
        for (int w = 0; w < SORT_WAVES; ++w) {
            const uint32_t c = wh[w][b];
            wh[w][b] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t q = base + r * 64 + lane;
        if (q < n) {
            const uint32_t dst = wh[wave][digit_of(key[r], shift, mask)] + rank[r];
            pk_out[dst] = key[r];
            pp_out[dst] = pos[r];
        }
    }
}

// ---- up to MID_MAX pairs: counters tile by tile, every workgroup of the scatter sums them itself -------------------
// MID_ITEMS pairs per thread: 4, or 2 up to MID_SHORT pairs, where tiles are what there are too few of.
// TILES_AHEAD: tiles whose counters a thread asks for together - always so many (an unrolled loop's remainder goes one trip to memory
// after the other: a scatter of 20,001 pairs 7.3 us, this way 6.7).
constexpr int TILES_AHEAD = 16;
constexpr int MID_THREADS = 512, MID_WAVES = MID_THREADS / 64, MID_MAX_TILES = 64;
constexpr int64_t MID_MAX = (int64_t)MID_THREADS * 4 * MID_MAX_TILES, MID_SHORT = MID_MAX / 4;
static_assert(2 * MID_THREADS >= 1 << SORT_MAX_BITS, "two buckets per thread");

template <int MID_ITEMS, bool FIRST>
__global__ __launch_bounds__(MID_THREADS) void k_sort_mid_count(const int64_t *keys_in, const uint64_t *pk_in, int64_t n, int shift, int bits,
                                                                uint32_t *hist, int64_t check_below, int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ uint32_t cnt[1 << SORT_MAX_BITS];
    const int R = 1 << bits, tid = threadIdx.x;
    const uint32_t mask = (uint32_t)R - 1u;
    const int64_t base = (int64_t)blockIdx.x * (MID_THREADS * MID_ITEMS);
    uint64_t key[MID_ITEMS];
#pragma unroll
    for (int r = 0; r < MID_ITEMS; ++r) {
        const int64_t q = base + r * MID_THREADS + tid;
        key[r] = q < n ? (FIRST ? (uint64_t)keys_in[q] : pk_in[q]) : 0;
    }
    if (stop) return;
    for (int i = tid; i < R; i += MID_THREADS) cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MID_ITEMS; ++r) {
        if (base + r * MID_THREADS + tid < n) {
            if (FIRST && check_below > 0 && key[r] >= (uint64_t)check_below) atomicExch(err, PS_EKEY);
            atomicAdd(&cnt[digit_of(key[r], shift, mask)], 1u);
        }
    }
    __syncthreads();
    for (int i = tid; i < R; i += MID_THREADS) hist[(int64_t)blockIdx.x * R + i] = cnt[i];
}

template <int MID_ITEMS, bool FIRST>
__global__ __launch_bounds__(MID_THREADS) void k_sort_mid_scatter(const int64_t *keys_in, const uint64_t *pk_in, const uint32_t *pp_in, int64_t n,
                                                                  int shift, int bits, const uint32_t *hist, uint64_t *pk_out, uint32_t *pp_out,
                                                                  const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ __attribute__((aligned(8))) uint32_t wh[MID_WAVES][1 << SORT_MAX_BITS];
    __shared__ uint32_t wave_sum[MID_WAVES];
    const int R = 1 << bits, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tile = blockIdx.x, tiles = gridDim.x;
    const uint32_t mask = (uint32_t)R - 1u;
    const int64_t base = (int64_t)tile * (MID_THREADS * MID_ITEMS) + (int64_t)wave * 64 * MID_ITEMS;
    uint64_t key[MID_ITEMS];
    uint32_t pos[MID_ITEMS], rank[MID_ITEMS];
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < MID_ITEMS; ++r) {
        const int64_t q = base + r * 64 + lane;
        const bool valid = q < n;
        key[r] = valid ? (FIRST ? (uint64_t)keys_in[q] : pk_in[q]) : 0;
        pos[r] = valid ? (FIRST ? (uint32_t)q : pp_in[q]) : 0u;
    }
    // this thread's two buckets: pairs in all tiles, and in the tiles before this one
    uint2 total = make_uint2(0u, 0u), before_tile = total;
    if (2 * tid < R) {
        for (int t0 = 0; t0 < tiles; t0 += TILES_AHEAD) {
            uint2 v[TILES_AHEAD];
#pragma unroll
            for (int i = 0; i < TILES_AHEAD; ++i) v[i] = *reinterpret_cast<const uint2 *>(&hist[(int64_t)(t0 + i < tiles ? t0 + i : t0) * R + 2 * tid]);
#pragma unroll
            for (int i = 0; i < TILES_AHEAD; ++i) {
                total.x += t0 + i < tiles ? v[i].x : 0u; total.y += t0 + i < tiles ? v[i].y : 0u;
                before_tile.x += t0 + i < tile ? v[i].x : 0u; before_tile.y += t0 + i < tile ? v[i].y : 0u;
            }
        }
    }
    if (stop) return;
    // (of the buckets only what the digit has)
    for (int w = 0; w < MID_WAVES; ++w)
        if (2 * tid < R) *reinterpret_cast<uint2 *>(&wh[w][2 * tid]) = make_uint2(0u, 0u);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MID_ITEMS; ++r) {
        const bool valid = base + r * 64 + lane < n;
        const uint32_t d = digit_of(key[r], shift, mask);
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = ((d >> b) & 1u) != 0u;
            const uint64_t v = __ballot(valid && bit);
            same &= bit ? v : ~v;
        }
        uint32_t before = 0;
        const int leader = valid ? __ffsll((long long)same) - 1 : lane;
        if (valid && lane == leader) {
            before = wh[wave][d];
            wh[wave][d] = before + (uint32_t)__popcll(same);
        }
        before = (uint32_t)__shfl((int)before, leader);
        rank[r] = before + (uint32_t)__popcll(same & below);
    }
    // the pairs in lower buckets: a scan over the buckets' totals
    const uint32_t both = total.x + total.y;
    uint32_t incl = both;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t lower = incl - both;
    for (int w = 0; w < wave; ++w) lower += wave_sum[w];
    // a wavefront's counters become the offsets of its first pair of each bucket
    if (2 * tid < R) {
        uint32_t run0 = lower + before_tile.x, run1 = lower + total.x + before_tile.y;
#pragma unroll
        for (int w = 0; w < MID_WAVES; ++w) {
            uint2 *at = reinterpret_cast<uint2 *>(&wh[w][2 * tid]);
            const uint2 c = *at;
            *at = make_uint2(run0, run1);
            run0 += c.x; run1 += c.y;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MID_ITEMS; ++r) {
        if (base + r * 64 + lane < n) {
            const uint32_t dst = wh[wave][digit_of(key[r], shift, mask)] + rank[r];
            pk_out[dst] = key[r];
            pp_out[dst] = pos[r];
        }
    }
}

// ---- from BIG_MIN up to BIG_MAX pairs: two launches per digit with tiles of 8,192 pairs, which a workgroup brings into the order of
// their buckets in LDS first, so that the stores of a bucket's pairs (8 of a tile at 1,024 buckets) leave side by side.
// Every workgroup sums all tiles' counters itself: 0.5 MB of them at a million pairs.  1,000,003 pairs of 19 bits: 63 us
// in four launches; 78 in eight, as below BIG_MIN, where smaller tiles give up to one workgroup per compute unit: pushes of rows of 4 with
// keys of 19 bits, 131,073 pairs 68 us and 73 with large tiles, 180,000 72.6 and 75.9, 262,144 79.5 and 80.3 (keys of 22 bits 87.8 and 91.6); 280,000
// 91.6 and 88.0, 400,000 102 and 96.5.
constexpr int BIG_THREADS = 1024, BIG_WAVES = BIG_THREADS / 64, BIG_ITEMS = 8, BIG_TILE = BIG_THREADS * BIG_ITEMS;
constexpr int64_t BIG_MIN = ((int64_t)1 << 18) + 1, BIG_MAX = (int64_t)1 << 21;
static_assert(BIG_THREADS >= 1 << SORT_MAX_BITS && BIG_TILE < 1 << 16, "a bucket per thread, places in a tile of 16 bits");
struct BigLds {
    uint64_t key[BIG_TILE];
    uint32_t pos[BIG_TILE];
    uint16_t place[BIG_WAVES][1 << SORT_MAX_BITS];     // a wavefront's pairs of a bucket, then where the first of them lies in the tile
    int32_t out[1 << SORT_MAX_BITS];                   // from a pair's place in the tile to its place in the output
    uint32_t sums[2][BIG_WAVES];
};

template <bool FIRST>
__global__ __launch_bounds__(BIG_THREADS) void k_sort_big_count(const int64_t *keys_in, const uint64_t *pk_in, int64_t n, int shift, int bits, uint32_t *hist,
                                                                int64_t check_below, int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ uint32_t cnt[1 << SORT_MAX_BITS];
    const int R = 1 << bits, tid = threadIdx.x;
    const uint32_t mask = (uint32_t)R - 1u;
    const int64_t base = (int64_t)blockIdx.x * BIG_TILE;
    uint64_t key[BIG_ITEMS];
#pragma unroll
    for (int r = 0; r < BIG_ITEMS; ++r) {
        const int64_t q = base + r * BIG_THREADS + tid;
        key[r] = q < n ? (FIRST ? (uint64_t)keys_in[q] : pk_in[q]) : 0;
    }
    if (stop) return;
    if (tid < R) cnt[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < BIG_ITEMS; ++r) {
        const bool valid = base + r * BIG_THREADS + tid < n;
        if (FIRST && check_below > 0 && valid && key[r] >= (uint64_t)check_below) atomicExch(err, PS_EKEY);
        // (a wavefront whose pairs are all of one bucket - few keys, keys in order - counts them at once: additions to one word
        // come one by one)
        const uint32_t d = digit_of(key[r], shift, mask), d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const uint64_t there = __ballot(valid);
        if (__ballot(valid && d != d0) == 0) {
            if ((tid & 63) == 0 && there != 0) atomicAdd(&cnt[d0], (uint32_t)__popcll(there));
        } else if (valid) atomicAdd(&cnt[d], 1u);
    }
    __syncthreads();
    if (tid < R) hist[(int64_t)blockIdx.x * R + tid] = cnt[tid];
}

template <bool FIRST>
__global__ __launch_bounds__(BIG_THREADS) void k_sort_big_scatter(const int64_t *keys_in, const uint64_t *pk_in, const uint32_t *pp_in, int64_t n, int shift,
                                                                  int bits, const uint32_t *hist, uint64_t *pk_out, uint32_t *pp_out, const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    extern __shared__ __attribute__((aligned(16))) unsigned char big_mem[];
    BigLds &l = *reinterpret_cast<BigLds *>(big_mem);
    const int R = 1 << bits, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tile = blockIdx.x, tiles = gridDim.x;
    const uint32_t mask = (uint32_t)R - 1u;
    // wavefront w takes the tile's pairs [w * 64 * BIG_ITEMS, + 64 * BIG_ITEMS), 64 consecutive ones per round
    const int64_t base = (int64_t)tile * BIG_TILE;
    const int size = (int)(n - base < BIG_TILE ? n - base : BIG_TILE), first = wave * 64 * BIG_ITEMS;
    uint64_t key[BIG_ITEMS];
    uint32_t pos[BIG_ITEMS], rank[BIG_ITEMS];
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < BIG_ITEMS; ++r) {
        const int q = first + r * 64 + lane;
        key[r] = q < size ? (FIRST ? (uint64_t)keys_in[base + q] : pk_in[base + q]) : 0;
        pos[r] = q < size ? (FIRST ? (uint32_t)(base + q) : pp_in[base + q]) : 0u;
    }
    // this thread's bucket: pairs in all tiles, and in the tiles before this one
    uint32_t total = 0, before_tile = 0;
    if (tid < R) {
        for (int t0 = 0; t0 < tiles; t0 += TILES_AHEAD) {
            uint32_t v[TILES_AHEAD];
#pragma unroll
            for (int i = 0; i < TILES_AHEAD; ++i) v[i] = hist[(int64_t)(t0 + i < tiles ? t0 + i : t0) * R + tid];
#pragma unroll
            for (int i = 0; i < TILES_AHEAD; ++i) {
                total += t0 + i < tiles ? v[i] : 0u;
                before_tile += t0 + i < tile ? v[i] : 0u;
            }
        }
    }
    if (stop) return;
    for (int b = lane; b < R; b += 64) l.place[wave][b] = 0;
    __asm__ volatile("" ::: "memory");                 // (a wavefront's own counters: LDS serves its accesses in order)
#pragma unroll
    for (int r = 0; r < BIG_ITEMS; ++r) {
        const bool valid = first + r * 64 + lane < size;
        const uint32_t d = digit_of(key[r], shift, mask);
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = ((d >> b) & 1u) != 0u;
            const uint64_t v = __ballot(valid && bit);
            same &= bit ? v : ~v;
        }
        uint32_t before = 0;
        const int leader = valid ? __ffsll((long long)same) - 1 : lane;
        if (valid && lane == leader) {
            before = l.place[wave][d];
            l.place[wave][d] = (uint16_t)(before + (uint32_t)__popcll(same));
        }
        before = (uint32_t)__shfl((int)before, leader);
        rank[r] = before + (uint32_t)__popcll(same & below);
    }
    __syncthreads();
    // the bucket's pairs in the tile, wavefront by wavefront
    uint32_t in_tile = 0;
    if (tid < R)
#pragma unroll
        for (int w = 0; w < BIG_WAVES; ++w) {
            const uint32_t c = l.place[w][tid];
            l.place[w][tid] = (uint16_t)in_tile;
            in_tile += c;
        }
    // the pairs in lower buckets, of all tiles and of this one: scans over the buckets
    uint32_t all = total, own = in_tile;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t a = (uint32_t)__shfl_up((int)all, off), o = (uint32_t)__shfl_up((int)own, off);
        if (lane >= off) { all += a; own += o; }
    }
    if (lane == 63) { l.sums[0][wave] = all; l.sums[1][wave] = own; }
    __syncthreads();
    uint32_t lower = all - total, start = own - in_tile;
    for (int w = 0; w < wave; ++w) { lower += l.sums[0][w]; start += l.sums[1][w]; }
    if (tid < R) {
        l.out[tid] = (int32_t)(lower + before_tile - start);
#pragma unroll
        for (int w = 0; w < BIG_WAVES; ++w) l.place[w][tid] = (uint16_t)(l.place[w][tid] + start);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < BIG_ITEMS; ++r)
        if (first + r * 64 + lane < size) {
            const uint32_t at = l.place[wave][digit_of(key[r], shift, mask)] + rank[r];
            l.key[at] = key[r];
            l.pos[at] = pos[r];
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < BIG_ITEMS; ++r) {
        const int i = r * BIG_THREADS + tid;
        if (i < size) {
            const uint64_t k = l.key[i];
            const uint32_t dst = (uint32_t)(l.out[digit_of(k, shift, mask)] + i);
            pk_out[dst] = k;
            pp_out[dst] = l.pos[i];
        }
    }
}

// ---- up to FEW_MAX pairs: one workgroup, a bitonic network over key << FEW_BITS | position in LDS -----------------
// A thread takes one comparison of every step.  Up to a distance of 64 a wavefront's comparisons stay within its 128
// numbers, and LDS serves a wavefront's accesses in order: only longer distances need a barrier.
constexpr int FEW_BITS = 11, FEW_MAX = 1 << FEW_BITS, FEW_THREADS = FEW_MAX / 2;
__global__ __launch_bounds__(FEW_THREADS) void k_sort_few(const int64_t *keys, int n, uint64_t *skeys, uint32_t *spos, int64_t check_below, int32_t *err) {
    if (*(volatile const int32_t *)err) return;
    __shared__ uint64_t x[FEW_MAX];
    const int tid = threadIdx.x;
    int N = 128;
    while (N < n) N <<= 1;
    bool bad = false;
    for (int i = tid; i < N; i += FEW_THREADS) {
        const uint64_t k = i < n ? (uint64_t)keys[i] : 0;
        bad |= i < n && check_below > 0 && k >= (uint64_t)check_below;
        x[i] = i < n ? (k << FEW_BITS) | (uint64_t)i : ~0ull;
    }
    if (__syncthreads_or(bad ? 1 : 0)) {
        if (tid == 0) atomicExch(err, PS_EKEY);
        return;
    }
    for (int k = 2; k <= N; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (2 * tid < N) {
                const int i = ((tid & -j) << 1) | (tid & (j - 1));      // (j: a power of two)
                const uint64_t a = x[i], b = x[i + j];
                const bool up = (i & k) == 0;
                if ((a > b) == up) { x[i] = b; x[i + j] = a; }
            }
            __asm__ volatile("" ::: "memory");
            // the next step reads what other wavefronts wrote: this one, or the next, reaches past 64
            if (j > 64 || (j == 1 && k >= 128)) __syncthreads();
        }
    }
    __syncthreads();
    for (int i = tid; i < n; i += FEW_THREADS) {
        skeys[i] = x[i] >> FEW_BITS;
        spos[i] = (uint32_t)x[i] & (FEW_MAX - 1);
    }
}

inline size_t up256(size_t x) { return (x + 255) / 256 * 256; }

struct SortPlan {
    int items;            // a tile holds 256 * items pairs (beyond BIG_MAX; up to there no tile is smaller than that)
    int passes;
    int bits[8];
    int64_t num_tiles;
    size_t off_pk, off_pp, off_hist, off_tot, bytes;   // the second pair of buffers, the counts, the bucket totals
};

SortPlan sort_plan(int64_t n, int key_bits) {
    SortPlan p{};
    p.items = n <= BIG_MAX ? 4 : 16;
    // short inputs are bound by the number of launches: wide digits, few passes; long ones by memory
    // traffic, where narrower digits keep a tile's pairs of one bucket next to each other in the output
    const int max_bits = n <= BIG_MAX ? SORT_MAX_BITS : 8;
    p.passes = (key_bits + max_bits - 1) / max_bits;
    if (p.passes < 1) p.passes = 1;
    for (int i = 0, left = key_bits; i < p.passes; ++i) {
        p.bits[i] = (left + (p.passes - i) - 1) / (p.passes - i);
        if (p.bits[i] < 1) p.bits[i] = 1;
        left -= p.bits[i];
    }
    p.num_tiles = (n + (int64_t)SORT_THREADS * p.items - 1) / ((int64_t)SORT_THREADS * p.items);
    if (p.num_tiles < 1) p.num_tiles = 1;
    p.off_pk = 0;
    p.off_pp = up256((size_t)n * 8);
    p.off_hist = p.off_pp + up256((size_t)n * 4);
    p.off_tot = p.off_hist + up256((size_t)(1 << SORT_MAX_BITS) * (size_t)p.num_tiles * 4);
    p.bytes = p.off_tot + up256((size_t)(1 << SORT_MAX_BITS) * 4);
    return p;
}

// MID: up to MID_MAX pairs; ITEMS 0: BIG_MIN to BIG_MAX
template <int ITEMS, bool MID>
int sort_run(dpaps_ps *ps, const SortPlan &p, const int64_t *keys, int64_t n, int64_t check_below, uint64_t *skeys, uint32_t *spos, void *scratch,
             hipStream_t st) {
    uint64_t *alt_k = (uint64_t *)((char *)scratch + p.off_pk);
    uint32_t *alt_p = (uint32_t *)((char *)scratch + p.off_pp);
    uint32_t *hist = (uint32_t *)((char *)scratch + p.off_hist);
    uint32_t *tot = (uint32_t *)((char *)scratch + p.off_tot);
    // the last pass must write (skeys, spos): with an even number of passes the first one writes there too
    uint64_t *out_k = (p.passes & 1) ? skeys : alt_k, *in_k = nullptr;
    uint32_t *out_p = (p.passes & 1) ? spos : alt_p, *in_p = nullptr;
    const unsigned tiles = (unsigned)p.num_tiles;
    int shift = 0;
    for (int i = 0; i < p.passes; ++i) {
        const int bits = p.bits[i], R = 1 << bits;
        if constexpr (MID) {
            constexpr int TILE = MID_THREADS * ITEMS;
            const unsigned mid = (unsigned)((n + TILE - 1) / TILE);
            if (i == 0) k_sort_mid_count<ITEMS, true><<<mid, MID_THREADS, 0, st>>>(keys, nullptr, n, shift, bits, hist, check_below, ps->err);
            else k_sort_mid_count<ITEMS, false><<<mid, MID_THREADS, 0, st>>>(nullptr, in_k, n, shift, bits, hist, 0, ps->err);
            PS_HIP(ps, hipGetLastError());
            if (i == 0) k_sort_mid_scatter<ITEMS, true><<<mid, MID_THREADS, 0, st>>>(keys, nullptr, nullptr, n, shift, bits, hist, out_k, out_p, ps->err);
            else k_sort_mid_scatter<ITEMS, false><<<mid, MID_THREADS, 0, st>>>(nullptr, in_k, in_p, n, shift, bits, hist, out_k, out_p, ps->err);
            PS_HIP(ps, hipGetLastError());
        } else if constexpr (ITEMS == 0) {
            static LdsAllowed first, other;
            int rc = dpaps_allow_lds(ps, first, reinterpret_cast<const void *>(&k_sort_big_scatter<true>), sizeof(BigLds));
            if (!rc) rc = dpaps_allow_lds(ps, other, reinterpret_cast<const void *>(&k_sort_big_scatter<false>), sizeof(BigLds));
            if (rc) return rc;
            const unsigned big = (unsigned)((n + BIG_TILE - 1) / BIG_TILE);
            if (i == 0) k_sort_big_count<true><<<big, BIG_THREADS, 0, st>>>(keys, nullptr, n, shift, bits, hist, check_below, ps->err);
            else k_sort_big_count<false><<<big, BIG_THREADS, 0, st>>>(nullptr, in_k, n, shift, bits, hist, 0, ps->err);
            PS_HIP(ps, hipGetLastError());
            if (i == 0) k_sort_big_scatter<true><<<big, BIG_THREADS, sizeof(BigLds), st>>>(keys, nullptr, nullptr, n, shift, bits, hist, out_k, out_p, ps->err);
            else k_sort_big_scatter<false><<<big, BIG_THREADS, sizeof(BigLds), st>>>(nullptr, in_k, in_p, n, shift, bits, hist, out_k, out_p, ps->err);
            PS_HIP(ps, hipGetLastError());
        } else {
            if (i == 0) k_sort_count<ITEMS, true><<<tiles, SORT_THREADS, 0, st>>>(keys, nullptr, n, shift, bits, p.num_tiles, hist, check_below, ps->err);
            else k_sort_count<ITEMS, false><<<tiles, SORT_THREADS, 0, st>>>(nullptr, in_k, n, shift, bits, p.num_tiles, hist, 0, ps->err);
            PS_HIP(ps, hipGetLastError());
            k_sort_rowsum<<<R, 256, 0, st>>>(hist, p.num_tiles, tot, ps->err);
            PS_HIP(ps, hipGetLastError());
            k_sort_scan<<<R, 256, 0, st>>>(hist, p.num_tiles, tot, ps->err);
            PS_HIP(ps, hipGetLastError());
            if (i == 0) k_sort_scatter<ITEMS, true><<<tiles, SORT_THREADS, 0, st>>>(keys, nullptr, nullptr, n, shift, bits, p.num_tiles, hist, out_k, out_p, ps->err);
            else k_sort_scatter<ITEMS, false><<<tiles, SORT_THREADS, 0, st>>>(nullptr, in_k, in_p, n, shift, bits, p.num_tiles, hist, out_k, out_p, ps->err);
            PS_HIP(ps, hipGetLastError());
        }
        in_k = out_k; in_p = out_p;
        out_k = in_k == skeys ? alt_k : skeys;
        out_p = in_p == spos ? alt_p : spos;
        shift += bits;
    }
    return PS_OK;
}

}  // namespace

// bits needed for keys below num_keys
int dpaps_key_bits(int64_t num_keys) {
    int b = 1;
    while (b < 63 && ((int64_t)1 << b) < num_keys) ++b;
    return b;
}

// scratch (bytes) that dpaps_sort_pairs needs for n pairs, besides its two output arrays
// (no less for more pairs)
size_t dpaps_sort_scratch_bytes(int64_t n, int key_bits) {
    const size_t bytes = sort_plan(n, key_bits).bytes;
    return n <= BIG_MAX ? bytes : std::max(bytes, sort_plan(BIG_MAX, key_bits).bytes);
}

// skeys[q], spos[q] (n each) <- the pairs (keys[p], p) ordered by key, equal keys by p.  Keys must be in
// [0, 2^key_bits) - or `check` is asked for: a key outside [0, num_keys) then sets the handle's error, and the kernels do
// nothing once it is set.  Allocates nothing; asynchronous on st.
int dpaps_sort_pairs(dpaps_ps *ps, const int64_t *keys, int64_t n, int key_bits, bool check, uint64_t *skeys, uint32_t *spos, void *scratch, hipStream_t st) {
    if (n <= 0) return PS_OK;
    const int64_t check_below = check ? ps->K : 0;
    if (n <= FEW_MAX && key_bits + FEW_BITS < 64) {
        k_sort_few<<<1, FEW_THREADS, 0, st>>>(keys, (int)n, skeys, spos, check_below, ps->err);
        PS_HIP(ps, hipGetLastError());
        return PS_OK;
    }
    const SortPlan p = sort_plan(n, key_bits);
    if (n <= MID_SHORT) return sort_run<2, true>(ps, p, keys, n, check_below, skeys, spos, scratch, st);
    if (n <= MID_MAX) return sort_run<4, true>(ps, p, keys, n, check_below, skeys, spos, scratch, st);
    if (n < BIG_MIN) return sort_run<4, false>(ps, p, keys, n, check_below, skeys, spos, scratch, st);
    if (n <= BIG_MAX) return sort_run<0, false>(ps, p, keys, n, check_below, skeys, spos, scratch, st);
    return sort_run<16, false>(ps, p, keys, n, check_below, skeys, spos, scratch, st);
}
