// Parameter server primitives on one GPU: dense store, owner map, pull / push /
// localize and the integer routing statistics (Table "Primitives", Sec. 3.1-3.3,
// Sec. 3.5, Sec. 3.7 of the paper).
#include "common.h"
#include "route.h"
#include "together.h"

#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------
int dpaps_fail_hip(dpaps_ps *ps, hipError_t e, const char *what) {
    if (ps) {
        ps->last_error = std::string(what) + ": " + hipGetErrorString(e);
    }
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? PS_ENOMEM : PS_EHIP;
}

static size_t ws_with_room(size_t bytes) { return bytes + bytes / 4 + 4096; }
int dpaps_ws_reserve(dpaps_ps *ps, size_t bytes) {
    if (bytes <= ps->ws_bytes) return PS_OK;
    if (ps->ws) {
        PS_HIP(ps, hipDeviceSynchronize());
        PS_HIP(ps, hipFree(ps->ws));
        ps->ws = nullptr;
        ps->ws_bytes = 0;
    }
    const size_t want = ws_with_room(bytes);
    PS_HIP(ps, hipMalloc(&ps->ws, want));
    ps->ws_bytes = want;
    return PS_OK;
}

int dpaps_allow_lds(dpaps_ps *ps, LdsAllowed &allowed, const void *kernel, size_t bytes) {
    static std::mutex mutex;                           // (so that it never shrinks under a launch of another handle)
    const bool kept = ps->device >= 0 && ps->device < DPAPS_DEVICES;
    if (kept && bytes <= allowed.on[ps->device].load(std::memory_order_acquire)) return PS_OK;
    std::lock_guard<std::mutex> lock(mutex);
    if (kept && bytes <= allowed.on[ps->device].load(std::memory_order_relaxed)) return PS_OK;
    PS_HIP(ps, hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    if (kept) allowed.on[ps->device].store(bytes, std::memory_order_release);
    return PS_OK;
}

static inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
__global__ void k_init_owner(int32_t *owner, int64_t K, int64_t per_home) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < K) owner[k] = (int32_t)(k / per_home);
}

__global__ void k_check_keys(const int64_t *keys, int64_t n, int64_t K, int32_t *err) {
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) {
        int64_t k = keys[p];
        if (k < 0 || k >= K) atomicExch(err, PS_EKEY);
    }
}

__global__ __launch_bounds__(256) void k_route_access(RouteArgs a, const int32_t *err) {
    __shared__ RouteLds l;
    route_access_block(a, l, blockIdx.x, flag_ahead(err));
}

// The replies of a pull or push have arrived: the requester's node knows the owner of every remote key it asked
// for (Sec. 3.3: the caches change without messages of their own).  Several mentions of a key write the same.
__global__ void k_cache_replies(const int64_t *keys, int64_t n, int32_t worker, const int32_t *owner, int16_t *loc_row, const int32_t *err) {
    if (*(volatile const int32_t *)err) return;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t k = keys[p];
    const int32_t o = owner[k];
    if (o != worker) loc_row[k] = (int16_t)o;
}

// localize: the home node updates the location at once (Sec. 3.2, step 1); the
// exchange makes exactly one of several mentions of a key the one that moves it.
// few: a call of few keys, checked here
__global__ __launch_bounds__(256) void k_localize(const int64_t *keys, int64_t n, int32_t worker, int32_t *owner, int64_t per_home, int32_t W,
                                                   uint32_t *named, uint32_t *stamp_pair, uint32_t call_id, u64 *stats,
                                                   int16_t *loc, int64_t K, bool few, int32_t *err) {
    const int32_t stop = few ? 0 : flag_ahead(err);
    if (few && few_keys_off<8>(keys, n, K, err)) return;
    __shared__ RouteLds l;
    route_lds_init(l, W);
    const double inv_per_home = 1.0 / (double)per_home;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    uint32_t n_keys = 0, n_moved = 0;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += step * ROUTE_AHEAD) {
        int64_t k[ROUTE_AHEAD];
        int32_t old[ROUTE_AHEAD];
        bool active[ROUTE_AHEAD];
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u) {
            const int64_t p = base + u * step + threadIdx.x;
            active[u] = p < n;
            k[u] = active[u] ? keys[p] : 0;
        }
        if (stop) return;
        // (a key that is seen to be the worker's already is left alone: a stale read only costs an exchange, and
        // a key mentioned a million times in one call does not turn into a million exchanges on one word)
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u) old[u] = active[u] ? __hip_atomic_load(&owner[k[u]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : worker;
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u)
            if (old[u] != worker) old[u] = atomicExch(&owner[k[u]], worker);
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u) {
            if (base + u * step >= n) break;
            const bool moved = active[u] && old[u] != worker;
            if (moved && loc) loc[(int64_t)old[u] * K + k[u]] = (int16_t)worker;     // the old owner hands the value over: it knows where to
            n_keys += lanes_with(active[u]);
            n_moved += lanes_with(moved);
            route_key(moved, worker, home_node(k[u], per_home, inv_per_home), old[u], W, stamp_pair, call_id, l);
        }
    }
    if ((threadIdx.x & 63) == 0) { atomicAdd(&l.count[0], n_keys); atomicAdd(&l.count[1], n_moved); }
    route_settle(l, W, named, blockIdx.x, gridDim.x);
    route_lds_flush(l, stats, PS_STAT_LOCALIZE_KEYS, PS_STAT_RELOCATED, PS_STAT_MSG_LOC_REQ, PS_STAT_MSG_LOC_INSTRUCT, PS_STAT_MSG_LOC_TRANSFER);
}

__global__ __launch_bounds__(256) void k_owner(const int64_t *keys, int64_t n, const int32_t *owner, int32_t *out, int64_t K, bool few, int32_t *err) {
    const int32_t stop = few ? 0 : flag_ahead(err);
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t k = p < n ? keys[p] : 0;
    if (few ? few_keys_off<8>(keys, n, K, err) : stop != 0) return;
    if (p < n) out[p] = owner[k];
}

// Pieces of a row: built-in vectors (arrays of float4 structures end up in LDS and scratch memory).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// pull: the rows in pieces of 16, 8 or 4 bytes (what value_len and the result's alignment allow), P pieces a row, a
// workgroup 256 * AHEAD consecutive pieces of the result, a thread every 256th of them: its keys, then its pieces, are
// asked for together.  The first route.blocks workgroups count the statistics beside that; a call of few keys checks
// them here (a larger one in a launch before).
// Bound by the memory's random reads.  1,000,003 Zipf keys of 100 values on 256 nodes with the check (5 us) and the statistics: 130 us, 104
// where the last-level cache still holds the store's 200 MB; 3,000 keys 10, 100 keys 7 in one launch; with the statistics in a launch of their own and one
// piece per thread 172, 20 and 10.  4 pieces ahead of 16 bytes instead of one: 133 us instead of 151; 8 of 4 bytes (rows
// of 51): 80 instead of 157, 4: 90.
// STREAM: results that no cache holds are written past them: 300,000 rows of 400: 90 us instead of 143, a million of 100:
// 117 instead of 133.  A result of 120 MB gains nothing (27.2 and 27.6), and its reader may find it in the last-level cache of
// 256 MB: hence half of that.
constexpr int64_t PULL_STREAM_BYTES = (int64_t)128 << 20;
template <class Piece, int AHEAD, bool STREAM>
__global__ __launch_bounds__(256) void k_pull(RouteArgs route, const int64_t *keys, int64_t n, uint32_t P, double inv_P, const Piece *val, Piece *out,
                                              int64_t K, int32_t *err) {
    // (of a larger call the flag was set, or not, by the launch before)
    const bool few = n <= FEW_KEYS;
    const int32_t stop = few ? 0 : flag_ahead(err);
    __shared__ RouteLds l;
    if ((int)blockIdx.x < route.blocks) {
        if (few && few_keys_off(keys, n, K, err)) return;
        route_access_block(route, l, blockIdx.x, stop);
        return;
    }
    const int64_t block = blockIdx.x - route.blocks;
    // the workgroup's first piece: row p0, piece c0 of it (quotients by way of 1 / P, rounded: the first in double and
    // put right, the others, of numbers up to P - 1 + 256 AHEAD - 1 - 3069 at most, with 8 pieces of 4 bytes ahead and rows of
    // 1023 -, exact with the half added: the quotient then lies 1 / (2 P) or more from a whole number, and is off by 2e-7 of itself)
    const int64_t first = block * (256 * AHEAD), total = n * P;
    const int64_t p0 = quotient(first, P, inv_P);
    const uint32_t c0 = (uint32_t)(first - p0 * P);
    const float inv_Pf = (float)inv_P;
    int64_t key[AHEAD];
    uint32_t c[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
        const uint32_t t = c0 + u * 256u + threadIdx.x, row = (uint32_t)(((float)t + 0.5f) * inv_Pf);
        c[u] = t - row * P;
        key[u] = first + u * 256 + threadIdx.x < total ? keys[p0 + row] : 0;
    }
    if (few ? few_keys_off(keys, n, K, err) : stop != 0) return;
    Piece x[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) x[u] = val[key[u] * P + c[u]];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
        if (first + u * 256 + threadIdx.x < total) {
            if constexpr (STREAM) __builtin_nontemporal_store(x[u], &out[first + u * 256 + threadIdx.x]);
            else out[first + u * 256 + threadIdx.x] = x[u];
        }
}

// push, after the (key, position) pairs have been sorted by key with a stable
// sort: one wavefront per sorted position; the wavefront at the head of a run
// of equal keys adds that key's update terms one after the other, in
// increasing position - the order a sequential server would apply them in.
// (One wavefront per key however often it is mentioned: the checking mode.)
__global__ void k_push_apply(const uint64_t *skeys, const uint32_t *spos, int64_t n, int32_t L, const float *deltas,
                             float *val, const int32_t *err) {
    if (*(volatile const int32_t *)err) return;
    const int lane = threadIdx.x & 63;
    int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (q >= n) return;
    uint64_t k = skeys[q];
    if (q > 0 && skeys[q - 1] == k) return;
    int64_t end = q + 1;
    while (end < n && skeys[end] == k) ++end;
    for (int32_t c = lane; c < L; c += 64) {
        float v = val[(int64_t)k * L + c];
        for (int64_t t = q; t < end; ++t) v = v + deltas[(int64_t)spos[t] * L + c];
        val[(int64_t)k * L + c] = v;
    }
}

// push, the default: the sorted positions are cut into ranges of PUSH_RANGE, one wavefront each, so that a key
// mentioned thousands of times is summed by many wavefronts.  Inside a range the terms of a key are added
// one after the other in argument order, starting from the stored value; a key whose terms fill one range
// only (any key mentioned once, most keys mentioned a few times) therefore gets the sequential server's
// bits.  Where a key's terms continue from the previous range they are summed from zero into part[2 r];
// where they start here and continue into the next range the running value goes to part[2 r + 1]; the
// second kernel adds a key's partial sums in range order.  The result depends on the arguments only.
constexpr int PUSH_RANGE = 64;
constexpr int PUSH_FEW_WAVES = 8;     // wavefronts per compute unit up to which four share a range

__device__ __forceinline__ uint64_t readlane_u64(uint64_t x, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// x, which is the same in all lanes, as a scalar
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

constexpr uint64_t NOKEY = ~0ull;                                      // no key looks like this

// Of one range of cnt sorted positions, lane t holding position t's key (mk), the key before it (before) and where its
// term lies (mp), the keys whose terms start in [p0, p1), without the positions in `skips` (keys that are mentioned once
// and have been updated by the step itself); prevk, nextk: the keys of the positions before and after the range.
// A row is P pieces, this lane's is c.
template <class Piece>
__device__ __forceinline__ void push_range(int cnt, int p0, int p1, u64 skips, uint64_t mk, uint64_t before, int mp, uint64_t prevk, uint64_t nextk,
                                           int64_t r, int c, int32_t P, const Piece *deltas, Piece *val, Piece *part) {
    constexpr int UN = sizeof(Piece) == 16 ? 8 : 16;
    const int lane = threadIdx.x & 63;
    const u64 heads = __ballot(lane < cnt && (lane == 0 || before != mk));   // positions where a key's terms start
    const bool first_open = readlane_u64(mk, 0) == prevk;              // the first key's terms continue from the range before
    const bool in = c < P;
    // from the first key that starts in [p0, p1) to the last one's end
    const u64 from = heads & (~0ull << p0), after = p1 < 64 ? heads & (~0ull << p1) : 0;
    const int start = from ? __ffsll((long long)from) - 1 : 64, end = after ? __ffsll((long long)after) - 1 : cnt;
    if (start >= p1 || start >= cnt) return;
    u64 left = (end < 64 ? (1ull << end) - 1ull : ~0ull) & (~0ull << start) & ~skips;
    // UN positions at a time: all their loads first (update terms, and the stored value where a key's terms
    // start), then the additions in order
    Piece v = {};
    uint64_t key = NOKEY;                                              // key of the terms being summed
    bool key_open = false;                                             // ... which continue from the range before
    while (left != 0) {
        Piece d[UN], b[UN];
        int at[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            at[i] = left != 0 ? __ffsll((long long)left) - 1 : -1;
            left &= left - 1ull;
            const int u = at[i] >= 0 ? at[i] : 0;
            const bool is_head = at[i] >= 0 && ((heads >> u) & 1) != 0 && !(u == 0 && first_open);
            d[i] = Piece{};
            b[i] = Piece{};
            if (in && at[i] >= 0) d[i] = deltas[(int64_t)__builtin_amdgcn_readlane(mp, u) * P + c];
            if (is_head && in) b[i] = val[(int64_t)readlane_u64(mk, u) * P + c];
        }
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int u = at[i];
            if (u >= 0) {
                if ((heads >> u) & 1) {
                    if (key != NOKEY && in) {                          // the previous key's terms end here
                        if (key_open) part[(2 * r) * P + c] = v;
                        else val[(int64_t)key * P + c] = v;
                    }
                    key = readlane_u64(mk, u);
                    key_open = u == 0 && first_open;
                    v = b[i];
                }
                v = v + d[i];
            }
        }
    }
    if (in && key != NOKEY) {
        if (key_open) part[(2 * r) * P + c] = v;
        else if (end == cnt && key == nextk) part[(2 * r + 1) * P + c] = v;
        else val[(int64_t)key * P + c] = v;
    }
}

// The ranges of a call; the first route.blocks workgroups (of the first 64 components) count its statistics instead.
// SPLIT wavefronts share a range, each the keys whose terms start in its part: where there are few ranges that is what
// makes wavefronts enough (20,001 keys of 50 values: 12 us instead of 19); with many it only repeats the reading of the keys.
template <class Piece, int SPLIT>
__global__ __launch_bounds__(256) void k_push_ranges(RouteArgs route, PushDone done, const uint64_t *skeys, const uint32_t *spos, int64_t n, int32_t P,
                                                      const Piece *deltas, Piece *val, Piece *part, const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    __shared__ RouteLds l;
    if ((int)blockIdx.x < route.blocks) {
        if (blockIdx.y == 0) route_access_block(route, l, blockIdx.x, stop);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)(blockIdx.x - (unsigned)route.blocks) * blockDim.x + threadIdx.x) >> 6, r = wave / SPLIT;
    const int p0 = (int)(wave % SPLIT) * (PUSH_RANGE / SPLIT);
    const int64_t q0 = r * PUSH_RANGE;
    if (q0 + p0 >= n) return;
    const int cnt = (int)(n - q0 < PUSH_RANGE ? n - q0 : PUSH_RANGE);
    const uint64_t mk = lane < cnt ? skeys[q0 + lane] : NOKEY;         // lane t: sorted position q0 + t
    const int mp = lane < cnt ? (int)spos[q0 + lane] : 0;
    const uint64_t prevk = q0 > 0 ? skeys[q0 - 1] : NOKEY;
    const uint64_t nextk = q0 + cnt < n ? skeys[q0 + cnt] : NOKEY;
    const uint64_t before = lane > 0 && lane < cnt ? skeys[q0 + lane - 1] : NOKEY;
    if (stop) return;
    u64 skips = 0;
    if (done.shared) skips = __ballot(lane < cnt && done.in_place((uint32_t)mp));
    push_range(cnt, p0, p0 + PUSH_RANGE / SPLIT, skips, mk, before, mp, prevk, nextk, r, blockIdx.y * 64 + lane, P, deltas, val, part);
}

// A push of at most 64 keys in one launch: one range.  Every wavefront (64 components each) checks the keys, brings them
// into the order (key, position) in its registers - a key's place is the number of keys before it - and adds; the
// last workgroup counts the statistics.
__global__ __launch_bounds__(64) void k_push_tiny(RouteArgs route, const int64_t *keys, int n, int32_t L, const float *deltas, float *val, int64_t K,
                                                  int32_t *err) {
    const int lane = threadIdx.x;
    const uint64_t k = lane < n ? (uint64_t)keys[lane] : NOKEY;
    if (few_keys_off(keys, n, K, err)) return;
    __shared__ RouteLds l;
    if (route.blocks && blockIdx.x == gridDim.x - 1) { route_access_block(route, l, 0); return; }
    int place = 0;
    for (int i = 0; i < n; ++i) {
        const uint64_t ki = readlane_u64(k, i);
        place += ki < k || (ki == k && i < lane) ? 1 : 0;
    }
    if (lane >= n) place = lane;
    // lane t <- the key and position whose place is t
    const int mp = __builtin_amdgcn_ds_permute(place << 2, lane);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_permute(place << 2, (int)(uint32_t)k), hi = (uint32_t)__builtin_amdgcn_ds_permute(place << 2, (int)(uint32_t)(k >> 32));
    const uint64_t mk = ((uint64_t)hi << 32) | lo;
    const uint64_t up = __shfl_up(mk, 1);
    push_range(n, 0, PUSH_RANGE, 0, mk, lane > 0 && lane < n ? up : NOKEY, mp, NOKEY, NOKEY, 0, blockIdx.x * 64 + lane, L, deltas, val, (float *)nullptr);
}

// A push of up to FEW_KEYS keys in one launch, without a sort: the sums are those of k_push_ranges and k_push_join, bit for
// bit, and what they need of a key's place in the order is counted.  Every workgroup checks all keys and has them in LDS.  A
// wavefront takes a position: it compares the position's key with all keys, and if no position before it has the same, the number
// of smaller keys is where the key's terms start among the sorted ones - so where its ranges of 64 begin - and the positions
// with the same key are its terms, in order.  A key of more than FEW_OWN ranges is worked on by the whole workgroup, a
// range per wavefront, its sums in LDS.  The first route.blocks workgroups count the statistics.
// Bound by a launch and two trips to memory behind each other (keys, rows), above 1,024 keys by the comparisons.  A push of 333 keys of
// 100 values on 256 nodes: 7.6 us, sorted and added in three launches 16.8; 2,048 keys 13.3 and 27.3, all of them one key 28.2 and 33.1,
// of 20 keys 17.2 and 32.0 (78 with a workgroup's positions side by side).  On 8 nodes, rows of 1, 16, 64, 256 and 400: 65 to 1,024 keys take
// 0.32 to 0.63 of what sort and sums take, 2,048 keys 0.4 to 0.9; longer rows: see push_without_sort.
constexpr int FEW_THREADS = 1024, FEW_WAVES = FEW_THREADS / 64, FEW_OWN = 2, FEW_RANGES = (int)FEW_KEYS / PUSH_RANGE + 1;
template <class Piece>
__global__ __launch_bounds__(FEW_THREADS) void k_push_few(RouteArgs route, const int64_t *keys, int n, int32_t P, const Piece *deltas, Piece *val,
                                                          int64_t K, int32_t *err) {
    constexpr size_t SUMS = (size_t)FEW_KEYS * 8, FEW_LDS = SUMS + (size_t)FEW_RANGES * 64 * sizeof(Piece);
    __shared__ __attribute__((aligned(16))) unsigned char mem[FEW_LDS > sizeof(RouteLds) ? FEW_LDS : sizeof(RouteLds)];
    __shared__ uint32_t many;                                          // which wavefronts' keys the whole workgroup works on,
    __shared__ u64 many_mask[FEW_WAVES][FEW_KEYS / 64], many_key[FEW_WAVES];   // and what they found of them
    __shared__ int many_start[FEW_WAVES], many_count[FEW_WAVES];
    const bool counts = (int)blockIdx.x < route.blocks;
    uint64_t *lk = reinterpret_cast<uint64_t *>(mem);
    Piece *sums = reinterpret_cast<Piece *>(mem + SUMS);
    if (threadIdx.x == 0) many = 0;
    if (few_keys_off<2>(keys, n, K, err, [&](int64_t p, int64_t k) { lk[p] = (uint64_t)k; })) return;
    if (counts) {
        __syncthreads();                                               // (the keys in LDS are not needed here)
        if (blockIdx.y == 0) route_access_block(route, *reinterpret_cast<RouteLds *>(mem), blockIdx.x);
        return;
    }
    constexpr int UN = sizeof(Piece) == 16 ? 16 : 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), chunks = (n + 63) / 64;
    // (the positions dealt out to the workgroups in turn, shifted from turn to turn: frequent keys are first named by the first
    // positions, or at equal distances, and a workgroup takes its own one after the other)
    const int groups = (int)(gridDim.x - (unsigned)route.blocks), mine = wave * groups + ((int)(blockIdx.x - (unsigned)route.blocks) + 5 * wave) % groups;
    const int c = blockIdx.y * 64 + lane;
    const bool in = c < P;
    u64 mask = 0;                                                      // lane i: which of the positions 64 i .. have the key
    int start = 0, count = 0;                                          // its terms among the sorted ones: the first, how many
    uint64_t key = 0;
    // position p's key; false if a position before p has it, or there is no position p
    auto look = [&](int p) {
        mask = 0; start = 0; count = 0;
        if (p >= n) return false;
        key = uniform_u64(lk[p]);
        for (int i = 0; i < chunks; ++i) {
            const bool there = 64 * i + lane < n;
            const uint64_t k = there ? lk[64 * i + lane] : NOKEY;
            const u64 same = __ballot(there && k == key);
            if (64 * i <= p && (64 * i + 63 < p ? same : same & ((1ull << (p & 63)) - 1ull)) != 0) return false;
            start += __popcll(__ballot(there && k < key));
            count += __popcll(same);
            mask = lane == i ? same : mask;
        }
        return true;
    };
    // the sum of the key's terms [lo, hi), one after the other, onto the stored value (STORED) or zero
    auto sum = [&](int lo, int hi, auto stored) {
        Piece v = {};
        if constexpr (decltype(stored)::value)
            if (in) v = val[(int64_t)key * P + c];
        int at = 0, seen = 0;                                          // the positions from 64 at on, `seen` terms are before those
        u64 m = readlane_u64(mask, 0);
        while (seen + __popcll(m) <= lo) { seen += __popcll(m); m = readlane_u64(mask, ++at); }
        for (; seen < lo; ++seen) m &= m - 1ull;
        while (lo < hi) {
            Piece d[UN];
            int got = 0;
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                d[u] = Piece{};
                if (lo + u < hi) {
                    while (m == 0) m = readlane_u64(mask, ++at);
                    const int p = 64 * at + __ffsll((long long)m) - 1;
                    m &= m - 1ull;
                    if (in) d[u] = deltas[(int64_t)p * P + c];
                    ++got;
                }
            }
#pragma unroll
            for (int u = 0; u < UN; ++u)
                if (u < got) v = v + d[u];
            lo += got;
        }
        return v;
    };
    constexpr std::integral_constant<bool, true> onto_stored{};
    constexpr std::integral_constant<bool, false> onto_zero{};
    // range r of the key's terms ends before term
    auto end_of = [&](int r) { const int e = (start / PUSH_RANGE + r + 1) * PUSH_RANGE - start; return e < count ? e : count; };
    if (look(mine)) {
        const int ranges = (start + count - 1) / PUSH_RANGE - start / PUSH_RANGE + 1;
        if (ranges <= FEW_OWN) {
            Piece v = sum(0, end_of(0), onto_stored);
            for (int r = 1; r < ranges; ++r) v = v + sum(end_of(r - 1), end_of(r), onto_zero);
            if (in) val[(int64_t)key * P + c] = v;
        } else {
            if (lane < (int)FEW_KEYS / 64) many_mask[wave][lane] = mask;
            if (lane == 0) { many_key[wave] = key; many_start[wave] = start; many_count[wave] = count; atomicOr(&many, 1u << wave); }
        }
    }
    __syncthreads();
    uint32_t left = (uint32_t)__builtin_amdgcn_readfirstlane((int)many);
    while (left != 0) {
        const int w = __ffs((int)left) - 1;
        left &= left - 1u;
        mask = lane < (int)FEW_KEYS / 64 ? many_mask[w][lane] : 0;
        key = uniform_u64(many_key[w]);
        start = __builtin_amdgcn_readfirstlane(many_start[w]);
        count = __builtin_amdgcn_readfirstlane(many_count[w]);
        const int ranges = (start + count - 1) / PUSH_RANGE - start / PUSH_RANGE + 1;
        for (int r = wave; r < ranges; r += FEW_WAVES) sums[r * 64 + lane] = r == 0 ? sum(0, end_of(0), onto_stored) : sum(end_of(r - 1), end_of(r), onto_zero);
        __syncthreads();
        if (wave == 0 && in) {
            Piece v = sums[lane];
            for (int r = 1; r < ranges; ++r) v = v + sums[r * 64 + lane];
            val[(int64_t)key * P + c] = v;
        }
        __syncthreads();                                               // the sums' place is used again
    }
}

// Second kernel: the wavefront of the range in which a key's terms start and do not end adds the partial sums
// of the following ranges, in order, and stores the value.  blockIdx.y: which 64 components.
// Bound by the chain of one wavefront on the most frequent key: a million Zipf keys, over a thousand ranges of one:
// 19 us; 25 with that key's ranges found 64 at a time one after the other and 16 rows asked for together, 23 with 64 rows
// but every address in vector registers.
constexpr int JOIN_AHEAD = 64;
__global__ __launch_bounds__(256) void k_push_join(const uint64_t *skeys, int64_t n, int32_t L, const float *part, float *val,
                                                    const int32_t *err) {
    const int32_t stop = flag_ahead(err);
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);   // the same in all lanes: addresses in scalars
    const int64_t q1 = (r + 1) * PUSH_RANGE;
    if (q1 >= n) return;                                               // nothing follows this range
    const uint64_t key = skeys[q1 - 1], next = skeys[q1];
    if (stop != 0 || next != key) return;                              // its last key ends here
    if (r > 0 && skeys[q1 - PUSH_RANGE] == key && skeys[q1 - PUSH_RANGE - 1] == key) return;   // it started earlier
    // m: how many of the following ranges begin with this key.  The keys are sorted, so those ranges follow one another:
    // 64 at a time are looked at, and where all of them do, 64 spread over what is left, until the first that does not.
    const int64_t nranges = (n + PUSH_RANGE - 1) / PUSH_RANGE;
    int64_t lo = r + 1, hi = nranges, by = 1;                          // ranges below lo begin with the key, hi and above do not
    while (lo < hi) {
        const int64_t at = lo + lane * by;
        const u64 b = __ballot(at < hi && skeys[(at < hi ? at : lo) * PUSH_RANGE] == key);
        const int run = b == ~0ull ? 64 : __ffsll((long long)~b) - 1;
        if (run < 64 && lo + run * by < hi) hi = lo + run * by;
        if (run > 0) lo += (run - 1) * by + 1;
        by = (hi - lo + 63) / 64;
    }
    const int64_t m = lo - (r + 1);
    const int c = blockIdx.y * 64 + lane;
    if (c >= L) return;
    float v = part[(2 * r + 1) * L + c];
    int64_t j = 1;
    for (; j + JOIN_AHEAD <= m + 1; j += JOIN_AHEAD) {
        float d[JOIN_AHEAD];
#pragma unroll
        for (int i = 0; i < JOIN_AHEAD; ++i) d[i] = part[(2 * (r + j + i)) * L + c];
#pragma unroll
        for (int i = 0; i < JOIN_AHEAD; ++i) v = v + d[i];
    }
    for (; j + 8 <= m + 1; j += 8) {
        float d[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) d[i] = part[(2 * (r + j + i)) * L + c];
#pragma unroll
        for (int i = 0; i < 8; ++i) v = v + d[i];
    }
    for (; j <= m; ++j) v = v + part[(2 * (r + j)) * L + c];
    val[(int64_t)key * L + c] = v;
}

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
static inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }
// Workgroups for the statistics of n keys.  A single one has nobody to compare its destinations with, but goes through its
// keys' trips to memory alone: on 8 nodes, localize of 2,048 keys takes 28 us with one and 22.5 with eight.
static inline int route_grid(int64_t n) {
    if (n <= 512) return 1;
    const int64_t need = (n + 255) / 256;
    return (int)(need < ROUTE_BLOCKS ? need : ROUTE_BLOCKS);
}

static int static_scratch_init(dpaps_ps *ps);

extern "C" int ps_create(int64_t num_keys, int32_t value_len, int32_t num_workers, ps_handle *out) {
    if (!out) return PS_EINVAL;
    *out = nullptr;
    if (num_keys <= 0 || value_len <= 0 || value_len > 1024 || num_workers <= 0 || num_workers > 2048) return PS_EINVAL;
    dpaps_ps *ps = new (std::nothrow) dpaps_ps();
    if (!ps) return PS_ENOMEM;
    ps->K = num_keys; ps->L = value_len; ps->W = num_workers;
    ps->per_home = (num_keys + num_workers - 1) / num_workers;
    hipError_t e;
#define CR(call) do { e = (call); if (e != hipSuccess) { int rc_ = dpaps_fail_hip(ps, e, #call); ps_destroy(ps); return rc_; } } while (0)
    CR(hipGetDevice(&ps->device));
    {
        const int rc_ = static_scratch_init(ps);
        if (rc_) { ps_destroy(ps); return rc_; }
    }
    int v = 0;
    CR(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, ps->device));
    ps->lds_bytes = v;
    CR(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, ps->device));
    ps->num_cu = v;
    // slack after the last row: a read of as many components as the longest factor has (256) that starts in it stays inside the allocation
    size_t vbytes = ((size_t)num_keys * value_len + 256) * sizeof(float);
    CR(hipMalloc(&ps->val, vbytes));
    CR(hipMemset(ps->val, 0, vbytes));
    CR(hipMalloc(&ps->owner, (size_t)num_keys * sizeof(int32_t)));
    static_assert(PS_STAT_COUNT <= PS_STAT_STRIDE, "a slot holds all counters");
    CR(hipMalloc(&ps->stats, PS_STAT_SLOTS * PS_STAT_STRIDE * sizeof(u64)));
    CR(hipMemset(ps->stats, 0, PS_STAT_SLOTS * PS_STAT_STRIDE * sizeof(u64)));
    CR(hipMalloc(&ps->err, sizeof(int32_t)));
    CR(hipMemset(ps->err, 0, sizeof(int32_t)));
    CR(hipMalloc(&ps->d_sse, sizeof(double)));
    size_t W = (size_t)num_workers;
    const size_t route_words = NAMED_WORDS + (W * W > PAIR_BITS ? W * W : 0);
    CR(hipMalloc(&ps->named, route_words * sizeof(uint32_t)));
    CR(hipMemset(ps->named, 0, route_words * sizeof(uint32_t)));
    ps->stamp_pair = ps->named + NAMED_WORDS;
    k_init_owner<<<grid_for(num_keys, 256), 256>>>(ps->owner, num_keys, ps->per_home);
    CR(hipGetLastError());
    CR(hipDeviceSynchronize());
#undef CR
    *out = ps;
    return PS_OK;
}

void dpaps_mf_free(dpaps_ps *ps);   // mf_prepare.hip

extern "C" int ps_destroy(ps_handle ps) {
    if (!ps) return PS_EINVAL;
    (void)hipDeviceSynchronize();
    dpaps_mf_free(ps);
    if (ps->val) (void)hipFree(ps->val);
    if (ps->owner) (void)hipFree(ps->owner);
    if (ps->stats) (void)hipFree(ps->stats);
    if (ps->err) (void)hipFree(ps->err);
    if (ps->d_sse) (void)hipFree(ps->d_sse);
    if (ps->named) (void)hipFree(ps->named);
    if (ps->ws) (void)hipFree(ps->ws);
    if (ps->kge_ws) (void)hipFree(ps->kge_ws);
    if (ps->kge_seen) (void)hipFree(ps->kge_seen);
    if (ps->kge_shared) (void)hipFree(ps->kge_shared);
    if (ps->handoff_ws) (void)hipFree(ps->handoff_ws);
    if (ps->loc) (void)hipFree(ps->loc);
    if (ps->side_stream) (void)hipStreamDestroy(ps->side_stream);
    if (ps->ev_fork) (void)hipEventDestroy(ps->ev_fork);
    if (ps->ev_join) (void)hipEventDestroy(ps->ev_join);
    if (ps->ev_sorted) (void)hipEventDestroy(ps->ev_sorted);
    for (hipEvent_t e : ps->ev_added)
        if (e) (void)hipEventDestroy(e);
    if (ps->ev_keys) (void)hipEventDestroy(ps->ev_keys);
    if (ps->d_tasks) (void)hipFree(ps->d_tasks);
    for (hipEvent_t e : ps->ev_pool) (void)hipEventDestroy(e);
    delete ps;
    return PS_OK;
}

static int launch_check(dpaps_ps *ps, const int64_t *keys, int64_t n, hipStream_t st) {
    if (n > 0) {
        k_check_keys<<<grid_for(n, 256), 256, 0, st>>>(keys, n, ps->K, ps->err);
        PS_HIP(ps, hipGetLastError());
    }
    return PS_OK;
}

// the library's second stream (default priority) and the events that tie it to the caller's
int dpaps_side_stream(dpaps_ps *ps) {
    if (!ps->side_stream) {
        PS_HIP(ps, hipStreamCreateWithFlags(&ps->side_stream, hipStreamNonBlocking));
        PS_HIP(ps, hipEventCreateWithFlags(&ps->ev_fork, hipEventDisableTiming));
        PS_HIP(ps, hipEventCreateWithFlags(&ps->ev_join, hipEventDisableTiming));
        PS_HIP(ps, hipEventCreateWithFlags(&ps->ev_sorted, hipEventDisableTiming));
        for (hipEvent_t &e : ps->ev_added) PS_HIP(ps, hipEventCreateWithFlags(&e, hipEventDisableTiming));
        PS_HIP(ps, hipEventCreateWithFlags(&ps->ev_keys, hipEventDisableTiming));
    }
    return PS_OK;
}

__global__ void k_fill_u32(uint32_t *p, size_t n, uint32_t v) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// p[0 .. words) <- 0 (a kernel, not a memset node: callers may be capturing)
int dpaps_zero_words(uint32_t *p, size_t words, hipStream_t st) {
    k_fill_u32<<<grid_for((int64_t)words, 256), 256, 0, st>>>(p, words, 0u);
    return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
}

static uint32_t next_call_id(dpaps_ps *ps, hipStream_t st) {
    if (++ps->call_id == 0) {   // wrapped: forget all stamps
        const size_t W = (size_t)ps->W, words = W * W > PAIR_BITS ? W * W : 0;
        if (words) (void)dpaps_zero_words(ps->stamp_pair, words, st);
        ps->call_id = 1;
    }
    return ps->call_id;
}

// the statistics of one access, to be counted by the first `blocks` workgroups of a launch
static RouteArgs route_args(dpaps_ps *ps, int32_t worker, const int64_t *keys, int64_t n, int st_local, int st_remote, int st_local2, int st_remote2,
                            hipStream_t st) {
    RouteArgs a{};
    if (worker < 0 || n == 0) return a;
    a.keys = keys; a.n = n; a.worker = worker; a.W = ps->W; a.owner = ps->owner; a.per_home = ps->per_home;
    a.named = ps->named; a.stamp_pair = ps->stamp_pair; a.call_id = next_call_id(ps, st);
    a.stats = ps->stats; a.stat_local = st_local; a.stat_remote = st_remote; a.stat_local2 = st_local2; a.stat_remote2 = st_remote2;
    a.loc_row = ps->loc ? ps->loc + (int64_t)worker * ps->K : nullptr;
    a.blocks = route_grid(n);
    return a;
}
static int cache_replies(dpaps_ps *ps, int32_t worker, const int64_t *keys, int64_t n, hipStream_t st) {
    if (worker < 0 || n == 0 || !ps->loc) return PS_OK;
    k_cache_replies<<<grid_for(n, 256), 256, 0, st>>>(keys, n, worker, ps->owner, ps->loc + (int64_t)worker * ps->K, ps->err);
    PS_HIP(ps, hipGetLastError());
    return PS_OK;
}

// the statistics in a launch of their own
static int route_access(dpaps_ps *ps, int32_t worker, const int64_t *keys, int64_t n, int st_local, int st_remote,
                        hipStream_t st, int st_local2 = -1, int st_remote2 = -1) {
    if (worker < 0 || n == 0) return PS_OK;
    if (ps->loc && st_local2 >= 0) {      // with location caches the second access is routed after the first one's replies
        const int rc = route_access(ps, worker, keys, n, st_local, st_remote, st);
        return rc ? rc : route_access(ps, worker, keys, n, st_local2, st_remote2, st);
    }
    const RouteArgs a = route_args(ps, worker, keys, n, st_local, st_remote, st_local2, st_remote2, st);
    k_route_access<<<a.blocks, 256, 0, st>>>(a, ps->err);
    PS_HIP(ps, hipGetLastError());
    return cache_replies(ps, worker, keys, n, st);
}

extern "C" int ps_pull(ps_handle ps, int32_t worker, const int64_t *keys, int64_t n, float *out, void *stream) {
    if (!ps || n < 0 || (n > 0 && (!keys || !out))) return PS_EINVAL;
    if (worker < -1 || worker >= ps->W) return PS_EWORKER;
    if (n == 0) return PS_OK;
    hipStream_t st = (hipStream_t)stream;
    int rc = n <= FEW_KEYS ? PS_OK : launch_check(ps, keys, n, st);
    if (rc) return rc;
    const RouteArgs a = route_args(ps, worker, keys, n, PS_STAT_PULL_LOCAL, PS_STAT_PULL_REMOTE, -1, -1, st);
#define PULL(PIECE, BYTES)                                                                                                                   \
    do {                                                                                                                                     \
        const uint32_t P = (uint32_t)((int64_t)ps->L * 4 / BYTES);                                                                           \
        const PIECE *val = reinterpret_cast<const PIECE *>(ps->val);                                                                         \
        PIECE *to = reinterpret_cast<PIECE *>(out);                                                                                          \
        constexpr int AHEAD = BYTES == 4 ? 8 : 4;                                                                                            \
        const unsigned grid = (unsigned)a.blocks + grid_for(n * P, 256 * AHEAD);                                                             \
        if (n * ps->L * 4 > PULL_STREAM_BYTES) k_pull<PIECE, AHEAD, true><<<grid, 256, 0, st>>>(a, keys, n, P, 1.0 / P, val, to, ps->K, ps->err); \
        else k_pull<PIECE, AHEAD, false><<<grid, 256, 0, st>>>(a, keys, n, P, 1.0 / P, val, to, ps->K, ps->err);                             \
    } while (0)
    if (ps->L % 4 == 0 && ((uintptr_t)out & 15) == 0) PULL(f32x4, 16);
    else if (ps->L % 2 == 0 && ((uintptr_t)out & 7) == 0) PULL(f32x2, 8);
    else PULL(float, 4);
#undef PULL
    PS_HIP(ps, hipGetLastError());
    return cache_replies(ps, worker, keys, n, st);
}

// The adding itself, for keys that have been checked (the kernels do nothing once the error flag is set), in two
// halves: the sort, which needs the keys only (a step that computes its update rows meanwhile runs it beside that
// work), and the sums, which need the rows.  The sorted pairs stay in the scratch between the two.
// Scratch of a push of n pairs: sorted keys, sorted positions, two partial-sum rows per range, the sort's own.
struct PushLayout { size_t off_pos, off_part, off_sort, bytes; };
static PushLayout push_layout(const dpaps_ps *ps, int64_t n) {
    const int64_t nranges = (n + PUSH_RANGE - 1) / PUSH_RANGE;
    const size_t part_bytes = ps->opt_push_sequential ? 0 : align_up((size_t)nranges * 2 * ps->L * sizeof(float));
    PushLayout l;
    l.off_pos = align_up((size_t)n * 8);
    l.off_part = l.off_pos + align_up((size_t)n * 4);
    l.off_sort = l.off_part + part_bytes;
    l.bytes = l.off_sort + dpaps_sort_scratch_bytes(n, dpaps_key_bits(ps->K));
    return l;
}

// the sort into `base` (scratch of at least push_layout(n).bytes, not allocated here)
static int push_sort_into(dpaps_ps *ps, void *base, const int64_t *keys, int64_t n, bool check, hipStream_t st) {
    const PushLayout l = push_layout(ps, n);
    uint64_t *skeys = (uint64_t *)base;
    uint32_t *spos = (uint32_t *)((char *)base + l.off_pos);
    const int rc = dpaps_sort_pairs(ps, keys, n, dpaps_key_bits(ps->K), check, skeys, spos, (char *)base + l.off_sort, st);
    if (rc) return rc;
    ps->push_base = base; ps->push_sorted_n = n; ps->push_off_pos = l.off_pos; ps->push_off_part = l.off_part;
    return PS_OK;
}

int dpaps_push_sort(dpaps_ps *ps, const int64_t *keys, int64_t n, hipStream_t st) {
    const int rc = dpaps_ws_reserve(ps, push_layout(ps, n).bytes);
    return rc ? rc : push_sort_into(ps, ps->ws, keys, n, false, st);
}
// The same for steps that sort ahead of the sums of the step before: scratch for two steps of up to n keys each, and the sort
// into one of the two halves.  (No number of keys needs more than a larger one.)
// Where there is no memory for two (*two false) the steps share one.  The scratch that is there is given up only for a larger one that
// has been allocated, and a size that was refused is not asked for again: otherwise every call of that size would wait for the device.
static size_t push_half(const dpaps_ps *ps, int64_t most) { return align_up(push_layout(ps, most).bytes); }
int dpaps_push_reserve_steps(dpaps_ps *ps, int64_t most, bool *two) {
    const size_t one = push_half(ps, most), both = 2 * one;
    *two = true;
    if (both <= ps->ws_bytes) return PS_OK;
    if (both < ps->ws_two_refused) {
        void *larger = nullptr;
        const hipError_t e = hipMalloc(&larger, ws_with_room(both));
        if (e == hipSuccess) {
            if (ps->ws) {
                const hipError_t through = hipDeviceSynchronize();
                if (through != hipSuccess) { (void)hipFree(larger); PS_HIP(ps, through); }
                (void)hipFree(ps->ws);
            }
            ps->ws = larger; ps->ws_bytes = ws_with_room(both);
            return PS_OK;
        }
        if (e != hipErrorOutOfMemory) PS_HIP(ps, e);
        (void)hipGetLastError();
        ps->ws_two_refused = both;
    }
    *two = false;
    return dpaps_ws_reserve(ps, one);
}
int dpaps_push_sort_half(dpaps_ps *ps, int half, int64_t most, const int64_t *keys, int64_t n, hipStream_t st) {
    return push_sort_into(ps, (char *)ps->ws + (half ? push_half(ps, most) : 0), keys, n, false, st);
}

static int push_tiny(dpaps_ps *ps, const RouteArgs &stats, const int64_t *keys, int64_t n, const float *deltas, hipStream_t st) {
    k_push_tiny<<<(unsigned)((ps->L + 63) / 64 + (stats.blocks ? 1 : 0)), 64, 0, st>>>(stats, keys, (int)n, ps->L, deltas, ps->val, ps->K, ps->err);
    PS_HIP(ps, hipGetLastError());
    return PS_OK;
}

// How many components a lane of a push's sums holds: as few as let one wavefront take a row (up to four).
// A row that several wavefronts take is read in overlapping lines, long after one another.  A million keys, rows of 100:
// the push 240 us with 2, 281 with 1; rows of 400, 20,000 keys: 47 with 4, 58 with 1.  Rows of 64 with 2: 198 instead of
// 176 (half the lanes idle).  4 components with 16 rows at once instead of 8: 50.
static int push_width(int32_t L, const float *deltas) {
    if (L > 128 && L % 4 == 0 && ((uintptr_t)deltas & 15) == 0) return 4;
    if (L > 64 && L % 2 == 0 && ((uintptr_t)deltas & 7) == 0) return 2;
    return 1;
}
static int push_few(dpaps_ps *ps, RouteArgs stats, const int64_t *keys, int64_t n, const float *deltas, hipStream_t st) {
    if (stats.blocks) stats.blocks = 1;                // (its threads take all keys in one go)
    const int width = push_width(ps->L, deltas);
    const int32_t P = ps->L / width;
    const dim3 grid((unsigned)stats.blocks + grid_for(n, FEW_WAVES), (unsigned)((P + 63) / 64));
#define FEW(PIECE)                                                                                                                       \
    k_push_few<PIECE><<<grid, FEW_THREADS, 0, st>>>(stats, keys, (int)n, P, reinterpret_cast<const PIECE *>(deltas), reinterpret_cast<PIECE *>(ps->val), ps->K, ps->err)
    if (width == 4) FEW(f32x4); else if (width == 2) FEW(f32x2); else FEW(float);
#undef FEW
    PS_HIP(ps, hipGetLastError());
    return PS_OK;
}
// Whether a push of n checked or unchecked keys goes without sorted pairs, in one launch.  What k_push_few takes grows with its workgroups - one
// for 16 keys and 64 pieces of a row - and in each with the keys it compares; the sort and the sums take 17 to 21 us up to 1,024
// keys and 27 above, nearly whatever the row.  Up to so many workgroups it is the faster or as fast: 1,024 keys of 1,022 values
// (512 workgroups) 20.5 us both ways, 850 of 1,023 (864) 23.1 and sorted 21.3, 700 (704) 16.9 and 21.6; 2,048 of 768 (384) 25.4 and 26.1, of
// 510 (512) 29.9 and 28.0, of 255 (512; one value per piece, so few registers that two workgroups share a compute unit) 22.7 and 27.3, of
// 1,023 (2,048) 68 and 28.
static bool push_without_sort(const dpaps_ps *ps, int64_t n, const float *deltas) {
    if (ps->opt_push_sequential || n > FEW_KEYS) return false;
    if (n <= PUSH_RANGE) return true;
    const int width = push_width(ps->L, deltas);
    const int64_t groups = ceil_div64(n, FEW_WAVES) * ceil_div64(ps->L / width, 64);
    return groups <= (n <= 1024 ? 768 : width == 1 ? 512 : 448);
}
// A push whose sums need no sorted pairs: one launch.
static int push_at_once(dpaps_ps *ps, const RouteArgs &stats, const int64_t *keys, int64_t n, const float *deltas, hipStream_t st) {
    return n <= PUSH_RANGE ? push_tiny(ps, stats, keys, n, deltas, st) : push_few(ps, stats, keys, n, deltas, st);
}
// stats: an access to be counted along with the sums; done: what has been added already
static int push_add(dpaps_ps *ps, int64_t n, const float *deltas, const RouteArgs &stats, const PushDone &done, hipStream_t st) {
    if (n != ps->push_sorted_n || !ps->push_base) { ps->last_error = "push: the sums do not follow their sort"; return PS_EINVAL; }
    const int64_t nranges = (n + PUSH_RANGE - 1) / PUSH_RANGE;
    const uint64_t *skeys = (const uint64_t *)ps->push_base;
    const uint32_t *spos = (const uint32_t *)((char *)ps->push_base + ps->push_off_pos);
    float *part = (float *)((char *)ps->push_base + ps->push_off_part);
    if (ps->opt_push_sequential) {
        if (stats.blocks) {
            k_route_access<<<stats.blocks, 256, 0, st>>>(stats, ps->err);
            PS_HIP(ps, hipGetLastError());
        }
        k_push_apply<<<grid_for(n * 64, 256), 256, 0, st>>>(skeys, spos, n, ps->L, deltas, ps->val, ps->err);
        PS_HIP(ps, hipGetLastError());
        return PS_OK;
    }
    const int width = push_width(ps->L, deltas);
    const unsigned slices = (unsigned)((ps->L / width + 63) / 64);
    const bool split = nranges * slices <= PUSH_FEW_WAVES * (int64_t)ps->num_cu;
    const dim3 grid((unsigned)stats.blocks + grid_for(nranges * (split ? 4 : 1) * 64, 256), slices);
#define RANGES(PIECE, SPLIT)                                                                                                                  \
    k_push_ranges<PIECE, SPLIT><<<grid, 256, 0, st>>>(stats, done, skeys, spos, n, ps->L / width, reinterpret_cast<const PIECE *>(deltas),      \
                                                      reinterpret_cast<PIECE *>(ps->val), reinterpret_cast<PIECE *>(part), ps->err)
    if (width == 4) { if (split) RANGES(f32x4, 4); else RANGES(f32x4, 1); }
    else if (width == 2) { if (split) RANGES(f32x2, 4); else RANGES(f32x2, 1); }
    else { if (split) RANGES(float, 4); else RANGES(float, 1); }
#undef RANGES
    PS_HIP(ps, hipGetLastError());
    if (nranges > 1) {
        k_push_join<<<dim3(grid_for(nranges * 64, 256), (unsigned)((ps->L + 63) / 64)), 256, 0, st>>>(skeys, n, ps->L, part, ps->val, ps->err);
        PS_HIP(ps, hipGetLastError());
    }
    return PS_OK;
}

int dpaps_push_add(dpaps_ps *ps, int64_t n, const float *deltas, const PushDone &done, hipStream_t st) { return push_add(ps, n, deltas, RouteArgs{}, done, st); }

// The sums of a step that has pulled the keys it pushes, with the statistics of both accesses.
int dpaps_push_add_step(dpaps_ps *ps, int32_t worker, const int64_t *keys, int64_t n, const float *deltas, const PushDone &done, hipStream_t st) {
    if (ps->loc) {                          // (counted one after the other, see route_access)
        const int rc = dpaps_route_pull_push(ps, worker, keys, n, st);
        return rc ? rc : dpaps_push_add(ps, n, deltas, done, st);
    }
    return push_add(ps, n, deltas, route_args(ps, worker, keys, n, PS_STAT_PULL_LOCAL, PS_STAT_PULL_REMOTE, PS_STAT_PUSH_LOCAL, PS_STAT_PUSH_REMOTE, st),
                    done, st);
}

RouteArgs dpaps_step_route(dpaps_ps *ps, int32_t worker, int64_t n, hipStream_t st) {
    RouteArgs a = route_args(ps, worker, nullptr, n, PS_STAT_PULL_LOCAL, PS_STAT_PULL_REMOTE, PS_STAT_PUSH_LOCAL, PS_STAT_PUSH_REMOTE, st);
    if (a.blocks) a.blocks = 1;
    return a;
}

// The same for a step of at most dpaps_few_keys() keys: one launch, unless its rows are too long for that, its terms are to be added
// strictly in order or its accesses are counted one after the other.
int64_t dpaps_few_keys() { return FEW_KEYS; }
int dpaps_push_few_step(dpaps_ps *ps, int32_t worker, const int64_t *keys, int64_t n, const float *deltas, hipStream_t st) {
    if (ps->loc || !push_without_sort(ps, n, deltas)) {
        const int rc = dpaps_push_sort(ps, keys, n, st);
        return rc ? rc : dpaps_push_add_step(ps, worker, keys, n, deltas, PushDone{}, st);
    }
    const RouteArgs a = route_args(ps, worker, keys, n, PS_STAT_PULL_LOCAL, PS_STAT_PULL_REMOTE, PS_STAT_PUSH_LOCAL, PS_STAT_PUSH_REMOTE, st);
    return push_at_once(ps, a, keys, n, deltas, st);
}

// One push call with its scratch in `base` (NULL: the handle's own, which grows): the keys checked by the sort's first
// kernel, the sums with the statistics beside them.
static int push_call(dpaps_ps *ps, void *base, int32_t worker, const int64_t *keys, int64_t n, const float *deltas, hipStream_t st) {
    const bool at_once = push_without_sort(ps, n, deltas);
    int rc;
    if (!at_once) {
        if (!base) {
            rc = dpaps_ws_reserve(ps, push_layout(ps, n).bytes);
            if (rc) return rc;
            base = ps->ws;
        }
        rc = push_sort_into(ps, base, keys, n, true, st);
        if (rc) return rc;
    }
    const RouteArgs a = route_args(ps, worker, keys, n, PS_STAT_PUSH_LOCAL, PS_STAT_PUSH_REMOTE, -1, -1, st);
    rc = at_once ? push_at_once(ps, a, keys, n, deltas, st) : push_add(ps, n, deltas, a, PushDone{}, st);
    return rc ? rc : cache_replies(ps, worker, keys, n, st);
}

extern "C" int ps_push(ps_handle ps, int32_t worker, const int64_t *keys, int64_t n, const float *deltas, void *stream) {
    if (!ps || n < 0 || (n > 0 && (!keys || !deltas))) return PS_EINVAL;
    if (worker < -1 || worker >= ps->W) return PS_EWORKER;
    if (n >= ((int64_t)1 << 31)) return PS_ELIMIT;
    if (n == 0) return PS_OK;
    hipStream_t st = (hipStream_t)stream;
    return push_call(ps, nullptr, worker, keys, n, deltas, st);
}

// ---- a push that allocates nothing -------------------------------------------------------------------------
// For callers that cannot allocate (code under graph capture, serving loops, harnesses that forbid it): the
// scratch of the push - sorted pairs, the sort's buffers and counters, partial sums - lives in a fixed array in
// device memory, one copy per device that the library runs on, held until the process ends.  Its address on a
// device is looked up once, by ps_create with that device current, and kept per device; host code uses that
// address only, never the array's name.
constexpr size_t PUSH_STATIC_BYTES = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[PUSH_STATIC_BYTES];
static void *g_scratch_ptr[DPAPS_DEVICES];
static std::mutex g_scratch_mutex;

static int static_scratch_init(dpaps_ps *ps) {
    if (ps->device < 0 || ps->device >= DPAPS_DEVICES) return PS_OK;     // ps_push_noalloc will refuse
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[ps->device]) {
        void *p = nullptr;
        PS_HIP(ps, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch_ptr[ps->device] = p;
    }
    return PS_OK;
}

extern "C" int ps_push_noalloc(ps_handle ps, int32_t worker, const int64_t *keys, int64_t n, const float *deltas, void *stream) {
    if (!ps || n < 0 || (n > 0 && (!keys || !deltas))) return PS_EINVAL;
    if (worker < -1 || worker >= ps->W) return PS_EWORKER;
    if (n == 0) return PS_OK;
    void *base = ps->device >= 0 && ps->device < DPAPS_DEVICES ? g_scratch_ptr[ps->device] : nullptr;
    if (!base) { ps->last_error = "ps_push_noalloc: no fixed scratch on this device"; return PS_EINVAL; }
    if (n > PS_PUSH_NOALLOC_MAX_KEYS || (n + PUSH_RANGE - 1) / PUSH_RANGE * ps->L > PS_PUSH_NOALLOC_MAX_PARTIAL ||
        push_layout(ps, n).bytes > PUSH_STATIC_BYTES) {
        ps->last_error = "ps_push_noalloc: at most 262144 keys and ceil(n / 64) * value_len <= 2^20 per call; use ps_push";
        return PS_ELIMIT;
    }
    hipStream_t st = (hipStream_t)stream;
    return push_call(ps, base, worker, keys, n, deltas, st);
}

// Keys up to which localize and owner, whose launches are a workgroup per 256 keys, check them in that launch: 2,049 keys
// on 8 nodes, localize 22.2 us instead of 24.3 with a launch for the check, 5,000 keys 22.8 instead of 24.2, 8,192 keys 22.8 and, with the
// launch, 8,193 keys 23.9 (host time of a call).
constexpr int64_t CHECKED_KEYS = 8192;

// the owner updates and statistics of a localize call; few: of keys that have not been checked (at most CHECKED_KEYS)
static int localize_call(dpaps_ps *ps, const int64_t *keys, int64_t n, int32_t worker, bool few, hipStream_t st) {
    if (n == 0) return PS_OK;
    uint32_t id = next_call_id(ps, st);
    k_localize<<<route_grid(n), 256, 0, st>>>(keys, n, worker, ps->owner, ps->per_home, ps->W, ps->named, ps->stamp_pair, id, ps->stats, ps->loc, ps->K, few, ps->err);
    PS_HIP(ps, hipGetLastError());
    return PS_OK;
}
int dpaps_localize_checked(dpaps_ps *ps, const int64_t *keys, int64_t n, int32_t worker, hipStream_t st) {
    return localize_call(ps, keys, n, worker, false, st);
}
int dpaps_route_pull_push(dpaps_ps *ps, int32_t worker, const int64_t *keys, int64_t n, hipStream_t st) {
    return route_access(ps, worker, keys, n, PS_STAT_PULL_LOCAL, PS_STAT_PULL_REMOTE, st, PS_STAT_PUSH_LOCAL, PS_STAT_PUSH_REMOTE);
}

extern "C" int ps_localize(ps_handle ps, const int64_t *keys, int64_t n, int32_t worker, void *stream) {
    if (!ps || n < 0 || (n > 0 && !keys)) return PS_EINVAL;
    if (worker < 0 || worker >= ps->W) return PS_EWORKER;
    if (n == 0) return PS_OK;
    hipStream_t st = (hipStream_t)stream;
    const bool few = n <= CHECKED_KEYS;
    const int rc = few ? PS_OK : launch_check(ps, keys, n, st);
    return rc ? rc : localize_call(ps, keys, n, worker, few, st);
}

extern "C" int ps_owner(ps_handle ps, const int64_t *keys, int64_t n, int32_t *owner_out, void *stream) {
    if (!ps || n < 0 || (n > 0 && (!keys || !owner_out))) return PS_EINVAL;
    if (n == 0) return PS_OK;
    hipStream_t st = (hipStream_t)stream;
    const bool few = n <= CHECKED_KEYS;
    const int rc = few ? PS_OK : launch_check(ps, keys, n, st);
    if (rc) return rc;
    k_owner<<<grid_for(n, 256), 256, 0, st>>>(keys, n, ps->owner, owner_out, ps->K, few, ps->err);
    PS_HIP(ps, hipGetLastError());
    return PS_OK;
}

// Synchronize, fetch and clear the sticky device error.
int dpaps_take_error(dpaps_ps *ps, hipStream_t st) {
    int32_t e = 0;
    PS_HIP(ps, hipMemcpyAsync(&e, ps->err, sizeof(e), hipMemcpyDeviceToHost, st));
    PS_HIP(ps, hipStreamSynchronize(st));
    if (e != 0) {
        PS_HIP(ps, hipMemsetAsync(ps->err, 0, sizeof(int32_t), st));
        PS_HIP(ps, hipStreamSynchronize(st));
        switch (e) {
        case PS_EKEY: ps->last_error = "a key or index was out of range in an earlier call"; break;
        case PS_EREMOTE: ps->last_error = "an SGD task touched a parameter that is not allocated to its worker"; break;
        case PS_ESTALL: ps->last_error = "a kernel gave up a wait that did not end (inconsistent layout tables, or more workgroups than the device runs at once)"; break;
        case PS_ELAYOUT: ps->last_error = "the ratings are not laid out block by block as mf_load_ratings requires"; break;
        case PS_ELIMIT: ps->last_error = "the ratings exceed a limit of the layout (rows with several entries per block, or entries per row or column in a block)"; break;
        default: ps->last_error = "a kernel of an earlier call reported an error"; break;
        }
    }
    return e;
}

extern "C" int ps_status(ps_handle ps, void *stream) {
    if (!ps) return PS_EINVAL;
    return dpaps_take_error(ps, (hipStream_t)stream);
}

extern "C" int ps_stats(ps_handle ps, int64_t *host_out, void *stream) {
    if (!ps || !host_out) return PS_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    u64 h[PS_STAT_SLOTS * PS_STAT_STRIDE];
    PS_HIP(ps, hipMemcpyAsync(h, ps->stats, sizeof(h), hipMemcpyDeviceToHost, st));
    int rc = dpaps_take_error(ps, st);      // synchronizes
    for (int c = 0; c < PS_STAT_COUNT; ++c) {
        u64 sum = 0;
        for (int sl = 0; sl < PS_STAT_SLOTS; ++sl) sum += h[sl * PS_STAT_STRIDE + c];
        host_out[c] = (int64_t)sum;
    }
    return rc;
}

extern "C" int ps_set_option(ps_handle ps, int32_t option, int64_t value) {
    if (!ps) return PS_EINVAL;
    switch (option) {
    case PS_OPT_MF_EXACT: ps->opt_exact = value != 0; return PS_OK;
    case PS_OPT_MF_CACHE_ROWS: if (value < -1) return PS_EINVAL; ps->opt_cache_rows = value; return PS_OK;
    case PS_OPT_MF_WAVES: if (value < 0 || value > 16) return PS_EINVAL; ps->opt_waves = (int)value; return PS_OK;
    case PS_OPT_MF_PROFILE: ps->opt_profile = value != 0; return PS_OK;
    case PS_OPT_MF_GROUPED: ps->opt_grouped = value != 0; return PS_OK;
    case PS_OPT_PUSH_SEQUENTIAL: ps->opt_push_sequential = value != 0; return PS_OK;
    case PS_OPT_MF_CLASSIC: if (value < 0 || value > 2) return PS_EINVAL; ps->opt_classic = (int)value; return PS_OK;
    case PS_OPT_LOCATION_CACHES: {
        // one entry of two bytes per node and key (-1: none); switching on or off empties them
        PS_HIP(ps, hipDeviceSynchronize());
        if (ps->loc) { PS_HIP(ps, hipFree(ps->loc)); ps->loc = nullptr; }
        if (value != 0) {
            const size_t bytes = (size_t)ps->W * (size_t)ps->K * sizeof(int16_t);
            if (bytes > ((size_t)16 << 30)) { ps->last_error = "location caches: nodes x keys x 2 bytes exceeds 16 GiB"; return PS_ELIMIT; }
            PS_HIP(ps, hipMalloc(&ps->loc, bytes));
            PS_HIP(ps, hipMemset(ps->loc, 0xFF, bytes));
            PS_HIP(ps, hipDeviceSynchronize());
        }
        return PS_OK;
    }
    case PS_OPT_KGE_EXACT: ps->opt_kge_exact = value != 0; return PS_OK;
    case PS_OPT_MF_TEAM_MAX: if (value < 0 || value > 14) return PS_EINVAL; ps->opt_team_max = (int)value; return PS_OK;
    case PS_OPT_MF_HEAVY_LEN:
        if (value < 1 || value > (1 << 30)) return PS_EINVAL;
        ps->opt_heavy_len = (int)value; return PS_OK;
    default: return PS_EINVAL;
    }
}

extern "C" const char *ps_last_error(ps_handle ps) { return ps ? ps->last_error.c_str() : "null handle"; }
