// The integer routing statistics of the parameter server's calls (Sec. 3.3, Sec. 3.5, Sec. 3.7 of the paper), counted on
// the device along with a call's other work.
#pragma once

#include "common.h"

// ---- routing statistics ----------------------------------------------------
// A call's kernels run a bounded number of workgroups that walk over the keys.  Each workgroup counts in LDS
// and adds its counts to the statistics once, at its end.  The message counts need the number of different
// destinations in the call.  A workgroup collects the destinations of its keys in LDS, a bit each, and when it has seen all
// its keys it puts the words that are not zero into the call's bits in memory; what the atomic returns tells which of its
// destinations nobody had named before.  The workgroup that is the last to do so clears the call's bits again.  (A call's
// only workgroup counts its own bits.)  With a stamp per destination, looked at or exchanged at its first mention
// between the keys, a chain of trips past the die's caches was what the statistics cost: a million Zipf keys on 256
// nodes 96 us; now 22, and 5 for 20,000 keys on 8 nodes.  More keys per workgroup (128 or 256 workgroups): 35 and 24 us.
constexpr int ROUTE_BLOCKS = 512;                      // at most
constexpr int NODE_WORDS = 2048 / 32;                  // one bit per node (at most 2048 workers)
constexpr int PAIR_BITS = 1 << 16;                     // one bit per (from, to) pair where W x W fits (W <= 256) ...
constexpr int SEEN_PAIR = 1024;                        // ... else direct-mapped: entry holds idx + 1 of a settled pair

struct RouteLds {
    uint32_t count[8];
    uint32_t bits_h[NODE_WORDS], bits_o[NODE_WORDS];   // nodes this workgroup's keys name as request / reply destinations
    uint32_t bits_pair[PAIR_BITS / 32];
    uint32_t seen_pair[SEEN_PAIR];
};

__device__ __forceinline__ void route_lds_init(RouteLds &l, int32_t W) {
    // (of the pairs only what W nodes can name)
    const bool bits = (int64_t)W * W <= PAIR_BITS;
    const int np = bits ? (W * W + 31) / 32 : 0, ns = bits ? 0 : SEEN_PAIR;
    if (threadIdx.x < 8) l.count[threadIdx.x] = 0;
    for (int i = threadIdx.x; i < NODE_WORDS; i += blockDim.x) { l.bits_h[i] = 0; l.bits_o[i] = 0; }
    for (int i = threadIdx.x; i < np; i += blockDim.x) l.bits_pair[i] = 0;
    for (int i = threadIdx.x; i < ns; i += blockDim.x) l.seen_pair[i] = 0;
    __syncthreads();
}

// the lanes of a wavefront with the flag set, the same number in all lanes
__device__ __forceinline__ uint32_t lanes_with(bool flag) { return (uint32_t)__popcll(__ballot(flag)); }

// Marks stamps[idx] with this call's id and tells whether this was the first mark of the call: true for exactly one
// thread of the whole call per idx.  A destination the workgroup has settled before is skipped, and so is the exchange
// where the stamp is seen to carry the id already (a stale read only costs an exchange).  All lanes ask at once, also where
// several name one idx: one after the other, a lane for each, was a wavefront's 64 trips (300 keys on 2048 nodes: a pull
// 66 to 93 us, now 27).
__device__ __forceinline__ bool stamp_first(bool want, uint32_t *stamps, int32_t idx, uint32_t call_id, uint32_t *seen, int seen_mask) {
    if (!want || *(volatile uint32_t *)&seen[idx & seen_mask] == (uint32_t)idx + 1u) return false;
    bool first = false;
    if (__hip_atomic_load(&stamps[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != call_id) first = atomicExch(&stamps[idx], call_id) != call_id;
    *(volatile uint32_t *)&seen[idx & seen_mask] = (uint32_t)idx + 1u;
    return first;
}

// Where every idx has a bit of its own in LDS: the bit set.  It is looked at first: after a workgroup's first few keys
// nearly every bit is set, and lanes that read one word are served together while atomics on it come one by one.
__device__ __forceinline__ void name_bit(bool want, int32_t idx, uint32_t *bits) {
    if (want) {
        const uint32_t m = 1u << (idx & 31);
        if ((*(volatile uint32_t *)&bits[idx >> 5] & m) == 0u) atomicOr(&bits[idx >> 5], m);
    }
}
__device__ __forceinline__ uint32_t name_pair(bool want, uint32_t *stamp_pair, int32_t from, int32_t to, int32_t W, uint32_t call_id, RouteLds &l) {
    if (W * W <= PAIR_BITS) { name_bit(want, from * W + to, l.bits_pair); return 0u; }
    return stamp_first(want, stamp_pair, from * W + to, call_id, l.seen_pair, SEEN_PAIR - 1) ? 1u : 0u;
}
// home node of key k: k / per_home without the 64-bit division (double has 53 bits, keys and per_home fewer; the
// quotient estimate is off by at most one)
__device__ __forceinline__ int64_t quotient(int64_t k, int64_t d, double inv_d) {
    int64_t h = (int64_t)((double)k * inv_d);
    if (h * d > k) --h;
    else if ((h + 1) * d <= k) ++h;
    return h;
}
__device__ __forceinline__ int32_t home_node(int64_t k, int64_t per_home, double inv_per_home) { return (int32_t)quotient(k, per_home, inv_per_home); }

// One key that must travel for requester `worker`: home h, current owner o.
// Within one call the messages to one destination are grouped (Sec. 3.7); the
// stamps record which destinations this call has already been charged for.
// count[2..4]: request, forward, reply (or their localize counterparts).
__device__ __forceinline__ void route_key(bool travels, int32_t worker, int32_t h, int32_t o, int32_t W, uint32_t *stamp_pair, uint32_t call_id,
                                          RouteLds &l) {
    name_bit(travels && h != worker, h, l.bits_h);
    const uint32_t fwd = name_pair(travels && h != o, stamp_pair, h, o, W, call_id, l);
    name_bit(travels && o != worker, o, l.bits_o);
    if (fwd) atomicAdd(&l.count[3], 1u);
}
// all keys seen: the destinations that were named are charged.  named: the call's bits (as in RouteLds, zero between
// calls) and, behind them, the number of workgroups that are through: counted by THROUGH_GROUPS words of their own
// cache lines, whose last workgroups are counted by one more.  (Atomics on one word come one by one: with 512 workgroups on
// it, localize of 131,072 keys that are all the worker's already, which settles nothing, took 10.3 us, now 6.5.)
constexpr int SETTLE_AHEAD = 9, THROUGH_GROUPS = 16, THROUGH_STRIDE = 32, THROUGH_ONE = 32;   // up to THROUGH_ONE workgroups: the one word
constexpr int NAMED_O = NODE_WORDS, NAMED_PAIR = 2 * NODE_WORDS, NAMED_THROUGH = NAMED_PAIR + PAIR_BITS / 32,
              NAMED_WORDS = NAMED_THROUGH + (1 + THROUGH_GROUPS) * THROUGH_STRIDE;
static_assert(offsetof(RouteLds, bits_o) == offsetof(RouteLds, bits_h) + 4 * NAMED_O && offsetof(RouteLds, bits_pair) == offsetof(RouteLds, bits_h) + 4 * NAMED_PAIR,
              "a workgroup's words lie as the call's do");
__device__ __forceinline__ void route_settle(RouteLds &l, int32_t W, uint32_t *named, int block, int blocks) {
    __shared__ bool last;
    __syncthreads();
    const int nw = (W + 31) / 32, np = W * W <= PAIR_BITS ? (W * W + 31) / 32 : 0, tid = threadIdx.x, T = blockDim.x;
    // the workgroup's words as they lie, of nodes asked, nodes that reply and pairs; SETTLE_AHEAD of a thread at once (each
    // answer is a trip to memory: 256 nodes' words in one)
    const uint32_t *bits = l.bits_h;
    const int words = NAMED_PAIR + np;
    uint32_t req = 0, fwd = 0, back = 0;
    for (int base = tid; base < words; base += T * SETTLE_AHEAD) {
        uint32_t m[SETTLE_AHEAD], was[SETTLE_AHEAD];
#pragma unroll
        for (int u = 0; u < SETTLE_AHEAD; ++u) m[u] = base + u * T < words ? bits[base + u * T] : 0u;
#pragma unroll
        for (int u = 0; u < SETTLE_AHEAD; ++u) was[u] = blocks > 1 && m[u] != 0u ? atomicOr(&named[base + u * T], m[u]) : 0u;
#pragma unroll
        for (int u = 0; u < SETTLE_AHEAD; ++u) {
            const int i = base + u * T;
            (i < NAMED_O ? req : (i < NAMED_PAIR ? back : fwd)) += (uint32_t)__popc(m[u] & ~was[u]);
        }
    }
    if (req) atomicAdd(&l.count[2], req);
    if (fwd) atomicAdd(&l.count[3], fwd);
    if (back) atomicAdd(&l.count[4], back);
    if (blocks == 1) return;
    // (every atomic's answer has arrived, so it has been carried out; a fence would write back the die's whole cache)
    __syncthreads();
    auto clear = [&](uint32_t *word) { __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (tid == 0) {
        const int groups = blocks > THROUGH_ONE ? THROUGH_GROUPS : blocks, g = block % groups, size = (blocks - g + groups - 1) / groups;
        uint32_t *word = &named[NAMED_THROUGH + (1 + g) * THROUGH_STRIDE];
        bool through = size == 1;
        if (!through && atomicAdd(word, 1u) == (uint32_t)size - 1u) { clear(word); through = true; }
        last = through && atomicAdd(&named[NAMED_THROUGH], 1u) == (uint32_t)groups - 1u;
    }
    __syncthreads();
    if (last) {
        for (int i = tid; i < nw; i += T) { clear(&named[i]); clear(&named[NAMED_O + i]); }
        for (int i = tid; i < np; i += T) clear(&named[NAMED_PAIR + i]);
        if (tid == 0) clear(&named[NAMED_THROUGH]);
    }
}

// adds count[i] to the statistic which[i] (i < 7; -1: none), one workgroup's share
__device__ __forceinline__ void route_lds_flush(RouteLds &l, u64 *stats, int w0, int w1, int w2, int w3, int w4, int w5 = -1, int w6 = -1) {
    __syncthreads();
    const int which[7] = {w0, w1, w2, w3, w4, w5, w6};
    if (threadIdx.x < 7 && which[threadIdx.x] >= 0 && l.count[threadIdx.x] != 0)
        atomicAdd(&stat_slot(stats)[which[threadIdx.x]], (u64)l.count[threadIdx.x]);
}

// One key that `worker` reads or writes remotely: home h, owner o, c = what the worker's node's location cache says
// (Sec. 3.3 "Location caching"; -1: no entry, or no caches).  No entry: request to the home node, which forwards
// to the owner, which replies.  Correct entry: request straight to the owner.  Stale entry: request to the node
// named, which forwards to the home node, which forwards to the owner (double-forward).  Grouped per call like
// route_key: one request per node asked, one forward per (from, to), one reply per owner.
// count[2..4]: request, forward, reply; count[5], count[6]: accesses with a correct / a stale entry.
__device__ __forceinline__ void route_access_key(bool remote, int32_t worker, int32_t h, int32_t o, int32_t c, int32_t W, uint32_t *stamp_pair,
                                                 uint32_t call_id, RouteLds &l) {
    const bool hit = remote && c == o, stale = remote && c >= 0 && c != o;
    const int32_t asked = hit ? o : (stale ? c : h);
    name_bit(remote && asked != worker, asked, l.bits_h);
    uint32_t fwd = name_pair(remote && !hit && h != o, stamp_pair, h, o, W, call_id, l);
    if (__ballot(stale) != 0) fwd += name_pair(stale && c != h, stamp_pair, c, h, W, call_id, l);
    name_bit(remote, o, l.bits_o);
    if (fwd) atomicAdd(&l.count[3], fwd);
    if (hit) atomicAdd(&l.count[5], 1u);
    if (stale) atomicAdd(&l.count[6], 1u);
}

// Locality statistics and message counts of one pull or push call: block `block` of `blocks`, every thread ROUTE_AHEAD
// keys at a time, so that as many owners are on their way.  A call's statistics need nothing of its other work and
// nothing of theirs is needed by it, so they ride in the launch of another of the call's kernels, as its first blocks.
struct RouteArgs {
    const int64_t *keys; int64_t n;
    int32_t worker, W;
    const int32_t *owner; int64_t per_home;
    uint32_t *named, *stamp_pair; uint32_t call_id;     // stamp_pair, call_id: where the pairs do not fit in bits
    u64 *stats; int stat_local, stat_remote, stat_local2, stat_remote2;
    const int16_t *loc_row;
    int blocks;                  // 0: nothing to count
};
constexpr int ROUTE_AHEAD = 4;

// stop: the handle's error flag, the same in all threads; looked at when the first keys are on their way.
__device__ __forceinline__ void route_access_block(const RouteArgs &a, RouteLds &l, int block, int32_t stop = 0) {
    route_lds_init(l, a.W);
    const double inv_per_home = 1.0 / (double)a.per_home;
    const int64_t step = (int64_t)a.blocks * blockDim.x;
    uint32_t n_local = 0, n_remote = 0;
    for (int64_t base = (int64_t)block * blockDim.x; base < a.n; base += step * ROUTE_AHEAD) {     // whole workgroups walk together
        int64_t k[ROUTE_AHEAD];
        int32_t o[ROUTE_AHEAD];
        bool active[ROUTE_AHEAD];
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u) {
            const int64_t p = base + u * step + threadIdx.x;
            active[u] = p < a.n;
            k[u] = active[u] ? a.keys[p] : 0;
        }
        if (stop) return;
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u) o[u] = active[u] ? a.owner[k[u]] : 0;
#pragma unroll
        for (int u = 0; u < ROUTE_AHEAD; ++u) {
            if (base + u * step >= a.n) break;                                                      // (the same in the whole workgroup)
            const bool local = active[u] && o[u] == a.worker, remote = active[u] && o[u] != a.worker;
            n_local += lanes_with(local);
            n_remote += lanes_with(remote);
            const int32_t c = remote && a.loc_row ? (int32_t)a.loc_row[k[u]] : -1;       // this node's location cache, if there are caches
            route_access_key(remote, a.worker, home_node(k[u], a.per_home, inv_per_home), o[u], c, a.W, a.stamp_pair, a.call_id, l);
        }
    }
    if ((threadIdx.x & 63) == 0) { atomicAdd(&l.count[0], n_local); atomicAdd(&l.count[1], n_remote); }
    route_settle(l, a.W, a.named, block, a.blocks);
    route_lds_flush(l, a.stats, a.stat_local, a.stat_remote, PS_STAT_MSG_ACC_REQ, PS_STAT_MSG_ACC_FWD, PS_STAT_MSG_ACC_REPLY, PS_STAT_CACHE_HIT,
                    PS_STAT_CACHE_STALE);
    // a second access to the same keys by the same worker right after (a pull and a push of one step) has the
    // same locality and sends the same messages once more
    // (only without location caches: with them the first access's replies change how the second is routed)
    if (a.stat_local2 >= 0) route_lds_flush(l, a.stats, a.stat_local2, a.stat_remote2, PS_STAT_MSG_ACC_REQ, PS_STAT_MSG_ACC_FWD, PS_STAT_MSG_ACC_REPLY);
}

// ps_store.hip: the statistics of a step that pulls and pushes the same n keys, counted by one workgroup (which puts the keys in)
RouteArgs dpaps_step_route(dpaps_ps *ps, int32_t worker, int64_t n, hipStream_t st);
