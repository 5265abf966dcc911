// One mini-batch step of knowledge-graph-embedding training through the parameter
// server (Sec. 4.1 "Knowledge graph embeddings" and Appendix A of the paper: SGD with
// AdaGrad and negative sampling, the AdaGrad metadata stored in the parameter server;
// model ComplEx, cited there, whose score Re sum_k e_s[k] w_r[k] conj(e_o[k]) is the
// standard one).  The step is what a worker does for a batch of data points: pull the
// parameters of the positive triples and of their negatives, compute the updates, push
// them.  Pull and push are accounted exactly like ps_pull and ps_push for every key
// occurrence (key check, locality statistics, message counts).  The pulled values are read
// from the store by the kernel that uses them instead of being copied out first, and the
// update terms that one data point has for the same key slot are added up before the push,
// which then runs as in ps_push (deterministic order of the cumulative updates).
//
// Key space: entity e is key e, relation r is key num_entities + r.  A value has 4 D
// numbers: [0, D) real parts, [D, 2 D) imaginary parts, [2 D, 4 D) the AdaGrad
// accumulators of those 2 D numbers.
#include "common.h"
#include "kge_slots.h"
#include "mf_device.h"
#include "route.h"
#include "together.h"

#include <algorithm>
#include <type_traits>

static inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// The keys of the batch; check_below > 0: checked, before anything indexes the store with them.  seen (may be NULL): which
// slots share their key with another slot of the batch is worked out as well (kge_mark_slot); the call does without where
// that could be many, see in_place_step.
// ent (may be NULL): the keys of the subjects, objects and negatives of another `ent_batch` triples, from triple
// ent_first on, which the caller localizes next.
__device__ __forceinline__ int64_t entity_key(const KgeBatch &t, int64_t b, int32_t j) { return slot_key(t, b, j == 0 ? 0 : j + 1); }
__global__ void k_kge_keys(KgeBatch t, int64_t *keys, int64_t check_below, u64 *seen, uint32_t *shared, uint32_t id, KgeBatch ent, int64_t *ent_keys,
                           int32_t *err) {
    const int32_t stop = flag_ahead(err);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t rows = 3 + t.ns + t.no;
    if (i < t.batch * rows) {
        const int64_t b = i / rows, k = slot_key(t, b, (int32_t)(i - b * rows));
        if (stop) return;
        const bool bad = check_below > 0 && (k < 0 || k >= check_below);
        if (bad) atomicExch(err, PS_EKEY);
        keys[i] = k;
        if (seen && !bad) kge_mark_slot(t.num_entities, (uint32_t)i, (int32_t)(i - b * rows), k, seen, shared, id);
    }
    const int32_t ents = 2 + ent.ns + ent.no;
    if (stop == 0 && i < ent.batch * ents) {
        const int64_t b = i / ents;
        ent_keys[i] = entity_key(ent, b, (int32_t)(i - b * ents));
    }
}

// AdaGrad with the gradient g of a key slot and the accumulator G as pulled:
//   dtheta = -lr g / sqrt(G + g^2 + eps),  dG = g^2
// EXACT: root in double and a correctly rounded division, operation by operation what a sequential fp32 program
// does; otherwise the hardware's reciprocal square root, good to one unit in the last place (G + g^2 + eps >= eps > 0).
struct Upd { float dt, dg; };
template <bool EXACT>
__device__ __forceinline__ Upd adagrad(float g, float G, float lr, float eps) {
    if constexpr (EXACT) return {-lr * g / (float)sqrt((double)(G + g * g + eps)), g * g};
    else return {(-lr * g) * __builtin_amdgcn_rsqf(G + g * g + eps), g * g};
}

// dloss/dscore of one scored triple: -label sigmoid(-label score), written so that nothing overflows; EXACT: the
// exponential in double and rounded to float, as a sequential fp32 program has it
template <bool EXACT>
__device__ __forceinline__ float dloss(float label, float sc) {
    const float z = -label * sc;
    const float na = z >= 0.0f ? -z : z;                             // -|z|
    float ex;
    if constexpr (EXACT) ex = (float)exp((double)na);
    else ex = __builtin_amdgcn_exp2f(na * 1.44269504088896340736f);   // the hardware's 2^x, good to one unit in the last place
    const float sig = z >= 0.0f ? 1.0f / (1.0f + ex) : ex / (1.0f + ex);
    return -label * sig;
}
// the losses of a data point's scored triples, added in their order (lane t: triple t, t < per; the positive one is triple 0);
// the same in all lanes
__device__ __forceinline__ double loss_of(float score, int per) {
    const float label = (threadIdx.x & 63) == 0 ? 1.0f : -1.0f;
    const float z = -label * score;
    const double en = exp((double)(z >= 0.0f ? -z : z));
    const double ls = z >= 0.0f ? (double)z + log1p(en) : log1p(en);
    double sum = 0.0;
    for (int i = 0; i < per; ++i) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, ls);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, i);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), i);
        sum += __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    }
    return sum;
}

// One wavefront per data point - a positive triple and its negatives (Appendix A: the negatives are derived from
// the data point) -, lane l the components l, l + 64, ...  The values come from the store as it holds them (the
// pull).  The data point's loss is the sum over its scored triples; the gradient of a key slot - subject,
// relation, object, each negative - is the sum of the terms of the triples the slot occurs in, added in the order of
// the triples (positive, subject negatives, object negatives), and every slot takes one AdaGrad step on it: the
// data point pushes one row per slot.  The positive triple first, then every negative in one go: its row, its
// score, the derivative of its loss (the same in all lanes), its terms for the two slots it shares with the
// positive triple, its own AdaGrad step.  Score t is also kept in lane t, and the losses of all scored triples
// are evaluated together at the end.
//   loss = log(1 + exp(-label score)),  g = dloss/dscore * dscore/dtheta
// EXACT: every score is summed in index order (the lanes' terms one after the other), for bit-for-bit comparisons
// with a sequential program; otherwise per lane and then across the lanes.
// rows: (3 + ns + no) per data point in upd.  keys_out (few data points; else NULL): the wavefront writes its data
// point's keys there and checks them first, so that the step needs no launch for that.  1 + ns + no <= 64.
// done: a negative whose key no other slot of the batch names gets its new row stored right away, value + update term,
// which is the one addition the push would make - nobody else reads or writes that row in this step -, and the push
// leaves it out.  8,192 data points with 5 + 5 negatives from 500,000 entities: the push's sums take 33 us (41 with a
// component per lane), 93 with every row.
template <int NC, bool EXACT>
__global__ __launch_bounds__(256) void k_kge_group(KgeBatch t, int32_t D, float lr, float eps, float *store, float *__restrict__ upd,
                                                    int64_t *keys_out, int64_t num_keys, PushDone done, double *loss, bool add_loss, int32_t *err) {
    const int32_t stop = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int lane = threadIdx.x & 63;
    // the data point is the same for all lanes of a wavefront: said so, its keys and row addresses stay in scalar registers
    const int64_t b = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (b >= t.batch) return;
    const int32_t ns = t.ns, no = t.no;
    const int64_t ks = t.subj[b], kr = t.num_entities + t.rel[b], ko = t.obj[b];
    if (stop != 0) return;                                           // (looked at when the first keys have been asked for)
    constexpr int CH = NC <= 2 ? 5 : 1;                              // negatives whose rows are in flight together
    const int L = 4 * D, rows = 3 + ns + no;
    if (keys_out) {
        bool bad = false;
        for (int j = lane; j < rows; j += 64) {
            const int64_t k = slot_key(t, b, j);
            bad |= k < 0 || k >= num_keys;
            keys_out[b * rows + j] = k;
        }
        if (__ballot(bad) != 0) {
            if (lane == 0) atomicExch(err, PS_EKEY);
            return;
        }
    }
    const uint32_t Du = (uint32_t)D;                                 // row addresses and field offsets are scalars, k the only lane offset
    const float *vs = store + ks * L, *vr = store + kr * L, *vo = store + ko * L;
    float *u0 = upd + b * rows * L;
    // the sum of the lanes' terms: term[c] belongs to component lane + 64 c
    auto total = [&](const float (&term)[NC]) {
        if constexpr (EXACT) {
            float acc = 0.0f;
            for (int k = 0; k < D; ++k) {
                float t = 0.0f;
#pragma unroll
                for (int c = 0; c < NC; ++c) t = (k >> 6) == c ? rl_f(term[c], k & 63) : t;
                acc = acc + t;
            }
            return acc;
        } else {
            float part = 0.0f;
#pragma unroll
            for (int c = 0; c < NC; ++c) part += term[c];
            return wave_sum(part);
        }
    };
    float sr[NC], si[NC], rr[NC], ri[NC], orl[NC], oi[NC];
    float score = 0.0f;                                              // lane t: score of scored triple t
    {
        float term[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t k = (uint32_t)lane + 64u * c;
            const bool in = k < Du;
            sr[c] = in ? vs[k] : 0.0f; si[c] = in ? (vs + Du)[k] : 0.0f;
            rr[c] = in ? vr[k] : 0.0f; ri[c] = in ? (vr + Du)[k] : 0.0f;
            orl[c] = in ? vo[k] : 0.0f; oi[c] = in ? (vo + Du)[k] : 0.0f;
            // Re((sr + i si)(rr + i ri)(or - i oi))
            term[c] = sr[c] * rr[c] * orl[c] + si[c] * rr[c] * oi[c] + sr[c] * ri[c] * oi[c] - si[c] * ri[c] * orl[c];
        }
        const float sc = total(term);
        score = lane == 0 ? sc : score;
    }
    // the gradients of the subject's, the relation's and the object's slot, started by the positive triple
    float gs[NC][2], gr[NC][2], go[NC][2];
    {
        const float dl = dloss<EXACT>(1.0f, rl_f(score, 0));
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            gs[c][0] = 0.0f + dl * (rr[c] * orl[c] + ri[c] * oi[c]); gs[c][1] = 0.0f + dl * (rr[c] * oi[c] - ri[c] * orl[c]);
            gr[c][0] = 0.0f + dl * (sr[c] * orl[c] + si[c] * oi[c]); gr[c][1] = 0.0f + dl * (sr[c] * oi[c] - si[c] * orl[c]);
            go[c][0] = 0.0f + dl * (sr[c] * rr[c] - si[c] * ri[c]);  go[c][1] = 0.0f + dl * (si[c] * rr[c] + sr[c] * ri[c]);
        }
    }
    // The negatives, CH at a time: their rows (values and accumulators) are asked for together, so that a wavefront
    // waits for memory once per CH negatives, then per negative in order its score, the derivative of its loss,
    // its terms for the two slots it shares with the positive triple, and its own step.
    // OBJ false: subject replaced by n, the triple (n, r, o); true: object replaced by n, the triple (s, r, n); label -1
    auto negatives = [&](auto obj_tag, const int32_t *list, int n_list, int slot0) {
        constexpr bool OBJ = decltype(obj_tag)::value;
        for (int j0 = 0; j0 < n_list; j0 += CH) {
            float nr[CH][NC], ni[CH][NC], Gn[CH][NC][2], sc[CH];
            int64_t kq[CH];
            uint32_t flag[CH];                                       // the slot shares its key
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                const bool valid = j0 + q < n_list;
                const int64_t kn = valid ? (int64_t)list[b * n_list + j0 + q] : ks;
                kq[q] = kn;
                flag[q] = done.shared && valid ? done.shared[b * rows + slot0 + j0 + q] : done.id;
                const float *vn = store + kn * L;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const uint32_t k = (uint32_t)lane + 64u * c;
                    const bool in = valid && k < Du;
                    nr[q][c] = in ? vn[k] : 0.0f; ni[q][c] = in ? (vn + Du)[k] : 0.0f;
                    Gn[q][c][0] = in ? (vn + 2 * Du)[k] : 0.0f; Gn[q][c][1] = in ? (vn + 3 * Du)[k] : 0.0f;
                }
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                float term[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    term[c] = OBJ ? sr[c] * rr[c] * nr[q][c] + si[c] * rr[c] * ni[q][c] + sr[c] * ri[c] * ni[q][c] - si[c] * ri[c] * nr[q][c]
                                  : nr[q][c] * rr[c] * orl[c] + ni[q][c] * rr[c] * oi[c] + nr[q][c] * ri[c] * oi[c] - ni[q][c] * ri[c] * orl[c];
                sc[q] = total(term);
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                if (j0 + q >= n_list) break;
                const bool alone = flag[q] != done.id;                 // (the same in all lanes)
                float *un = alone ? store + kq[q] * L : u0 + (int64_t)(slot0 + j0 + q) * L;
                score = lane == slot0 - 2 + j0 + q ? sc[q] : score;
                const float dl = dloss<EXACT>(-1.0f, sc[q]);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const uint32_t k = (uint32_t)lane + 64u * c;
                    if (k >= Du) continue;
                    float g0, g1;                                      // the negative's own slot
                    if constexpr (OBJ) {
                        gs[c][0] = gs[c][0] + dl * (rr[c] * nr[q][c] + ri[c] * ni[q][c]); gs[c][1] = gs[c][1] + dl * (rr[c] * ni[q][c] - ri[c] * nr[q][c]);
                        gr[c][0] = gr[c][0] + dl * (sr[c] * nr[q][c] + si[c] * ni[q][c]); gr[c][1] = gr[c][1] + dl * (sr[c] * ni[q][c] - si[c] * nr[q][c]);
                        g0 = 0.0f + dl * (sr[c] * rr[c] - si[c] * ri[c]); g1 = 0.0f + dl * (si[c] * rr[c] + sr[c] * ri[c]);
                    } else {
                        g0 = 0.0f + dl * (rr[c] * orl[c] + ri[c] * oi[c]); g1 = 0.0f + dl * (rr[c] * oi[c] - ri[c] * orl[c]);
                        gr[c][0] = gr[c][0] + dl * (nr[q][c] * orl[c] + ni[q][c] * oi[c]); gr[c][1] = gr[c][1] + dl * (nr[q][c] * oi[c] - ni[q][c] * orl[c]);
                        go[c][0] = go[c][0] + dl * (nr[q][c] * rr[c] - ni[q][c] * ri[c]);  go[c][1] = go[c][1] + dl * (ni[q][c] * rr[c] + nr[q][c] * ri[c]);
                    }
                    const Upd u_0 = adagrad<EXACT>(g0, Gn[q][c][0], lr, eps), u_1 = adagrad<EXACT>(g1, Gn[q][c][1], lr, eps);
                    un[k] = alone ? nr[q][c] + u_0.dt : u_0.dt; (un + 2 * Du)[k] = alone ? Gn[q][c][0] + u_0.dg : u_0.dg;
                    (un + Du)[k] = alone ? ni[q][c] + u_1.dt : u_1.dt; (un + 3 * Du)[k] = alone ? Gn[q][c][1] + u_1.dg : u_1.dg;
                }
            }
        }
    };
    negatives(std::false_type{}, t.neg_subj, ns, 3);
    negatives(std::true_type{}, t.neg_obj, no, 3 + ns);
    // the losses of all scored triples at once, if anybody asks for them
    if (loss) {
        const double sum = loss_of(score, 1 + ns + no);
        if (lane == 0) loss[b] = add_loss ? loss[b] + sum : sum;
    }
    // subject, relation, object: one AdaGrad step each on the summed gradient, with the accumulators as pulled
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t k = (uint32_t)lane + 64u * c;
        if (k >= Du) continue;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t ft = p * Du, fg = (2 + p) * Du;              // the field of the values and that of their accumulators
            const Upd us = adagrad<EXACT>(gs[c][p], (vs + fg)[k], lr, eps);
            const Upd ur = adagrad<EXACT>(gr[c][p], (vr + fg)[k], lr, eps);
            const Upd uo = adagrad<EXACT>(go[c][p], (vo + fg)[k], lr, eps);
            (u0 + ft)[k] = us.dt; (u0 + fg)[k] = us.dg;
            (u0 + L + ft)[k] = ur.dt; (u0 + L + fg)[k] = ur.dg;
            (u0 + 2 * L + ft)[k] = uo.dt; (u0 + 2 * L + fg)[k] = uo.dg;
        }
    }
}

// A step of so few data points that their slots fit side by side in one workgroup's LDS: all of it in one launch - the keys
// checked, every slot's row read once, a wavefront per scored triple for the scores and one per slot for gradient, AdaGrad step and
// sum, each slot's terms in the order of the other path.  A second workgroup counts the statistics.
// Bound by a launch and two trips to memory, keys and rows, one compute unit's way to them.  A data point with 5 + 5 negatives, dim 100, and its
// rows read back: 13.4 us, 22.5 with the update rows and the push in launches of their own (11 + 6 us).  A step by itself, this way and
// that: 13 slots of dim 16, 100 and 256 6.9 us and 14.7, 7.9 and 19.9, 11.8 and 26.6; 52 to 64 slots of dim 16 and 50 9.3 to 13.9 and 22.8 to 28.0; what
// no longer fits in LDS (52 slots of dim 100: 28.8) is not measured this way.  One workgroup is the faster one wherever it fits.
// LDS: the keys, the rows as pulled, the update rows, and the derivatives of the scored triples' losses.
constexpr int KGE_FEW_SLOTS = 64, KGE_FEW_THREADS = 1024, KGE_FEW_LDS = 128 << 10;
static size_t kge_few_lds(int64_t slots, int32_t L) { return (size_t)slots * 2 * L * 4 > sizeof(RouteLds) ? (size_t)slots * 2 * L * 4 : sizeof(RouteLds); }
__global__ __launch_bounds__(KGE_FEW_THREADS) void k_kge_few(RouteArgs route, KgeBatch t, int32_t D, float lr, float eps, float *store, int64_t K, double *loss,
                                                             int32_t *err) {
    extern __shared__ __attribute__((aligned(16))) float mem[];
    __shared__ int64_t key[KGE_FEW_SLOTS];
    __shared__ float score[KGE_FEW_SLOTS], dl[KGE_FEW_SLOTS];
    const int ns = t.ns, no = t.no, rows = 3 + ns + no, per = 1 + ns + no, slots = (int)t.batch * rows, L = 4 * D;
    if ((int)threadIdx.x < slots) key[threadIdx.x] = slot_key(t, (int)threadIdx.x / rows, (int)threadIdx.x % rows);
    __syncthreads();
    if (few_keys_off(key, slots, K, err)) return;
    if (blockIdx.x > 0) {
        route.keys = key;
        route_access_block(route, *reinterpret_cast<RouteLds *>(mem), 0);
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), waves = blockDim.x >> 6;
    float *const val = mem, *const upd = mem + (size_t)slots * L;
    for (int j = wave; j < slots; j += waves) {
        const float *from = store + key[j] * L;
        for (int k = lane; k < L; k += 64) val[j * L + k] = from[k];
    }
    __syncthreads();
    // the score of triple i of data point b (0: the positive one, then the subject and the object negatives) - its subject's, relation's and
    // object's slots - and the derivative of its loss
    for (int i = wave; i < (int)t.batch * per; i += waves) {
        const int b = i / per, q = i - b * per;
        const float *base = val + b * rows * L, *n = base + (q + 2) * L;
        const float *s = q >= 1 && q <= ns ? n : base, *r = base + L, *o = q > ns ? n : base + 2 * L;
        float part = 0.0f;
        for (int k = lane; k < D; k += 64)
            part += s[k] * r[k] * o[k] + s[D + k] * r[k] * o[D + k] + s[k] * r[D + k] * o[D + k] - s[D + k] * r[D + k] * o[k];
        const float sc = wave_sum(part), d = dloss<false>(q == 0 ? 1.0f : -1.0f, sc);
        if (lane == 0) { score[i] = sc; dl[i] = d; }
    }
    __syncthreads();
    // every slot's gradient, the terms of the triples it occurs in in their order, and its AdaGrad step with the accumulators as pulled
    for (int j = wave; j < slots; j += waves) {
        const int b = j / rows, jj = j - b * rows;
        const float *base = val + b * rows * L, *s = base, *r = base + L, *o = base + 2 * L, *own = base + jj * L, *d = dl + b * per;
        for (int k = lane; k < D; k += 64) {
            const float sr = s[k], si = s[D + k], rr = r[k], ri = r[D + k], orl = o[k], oi = o[D + k];
            float g0, g1;
            if (jj == 0) {
                g0 = 0.0f + d[0] * (rr * orl + ri * oi); g1 = 0.0f + d[0] * (rr * oi - ri * orl);
                for (int q = 0; q < no; ++q) {
                    const float *n = base + (3 + ns + q) * L;
                    const float nr = n[k], ni = n[D + k], dq = d[1 + ns + q];
                    g0 = g0 + dq * (rr * nr + ri * ni); g1 = g1 + dq * (rr * ni - ri * nr);
                }
            } else if (jj == 1) {
                g0 = 0.0f + d[0] * (sr * orl + si * oi); g1 = 0.0f + d[0] * (sr * oi - si * orl);
                for (int q = 0; q < ns; ++q) {
                    const float *n = base + (3 + q) * L;
                    const float nr = n[k], ni = n[D + k], dq = d[1 + q];
                    g0 = g0 + dq * (nr * orl + ni * oi); g1 = g1 + dq * (nr * oi - ni * orl);
                }
                for (int q = 0; q < no; ++q) {
                    const float *n = base + (3 + ns + q) * L;
                    const float nr = n[k], ni = n[D + k], dq = d[1 + ns + q];
                    g0 = g0 + dq * (sr * nr + si * ni); g1 = g1 + dq * (sr * ni - si * nr);
                }
            } else if (jj == 2) {
                g0 = 0.0f + d[0] * (sr * rr - si * ri); g1 = 0.0f + d[0] * (si * rr + sr * ri);
                for (int q = 0; q < ns; ++q) {
                    const float *n = base + (3 + q) * L;
                    const float nr = n[k], ni = n[D + k], dq = d[1 + q];
                    g0 = g0 + dq * (nr * rr - ni * ri); g1 = g1 + dq * (ni * rr + nr * ri);
                }
            } else {
                const float dq = d[jj - 2];
                if (jj < 3 + ns) { g0 = 0.0f + dq * (rr * orl + ri * oi); g1 = 0.0f + dq * (rr * oi - ri * orl); }
                else { g0 = 0.0f + dq * (sr * rr - si * ri); g1 = 0.0f + dq * (si * rr + sr * ri); }
            }
            const Upd u0 = adagrad<false>(g0, own[2 * D + k], lr, eps), u1 = adagrad<false>(g1, own[3 * D + k], lr, eps);
            float *u = upd + j * L + k;
            u[0] = u0.dt; u[D] = u1.dt; u[2 * D] = u0.dg; u[3 * D] = u1.dg;
        }
    }
    __syncthreads();
    // the push: the first slot that names a key adds the terms of all that do, in their order, onto the value
    for (int j = wave; j < slots; j += waves) {
        const int64_t kj = key[j];
        const u64 same = __ballot(lane < slots && key[lane < slots ? lane : 0] == kj);
        if ((same & ((1ull << j) - 1ull)) != 0) continue;
        float *to = store + kj * L;
        for (int k = lane; k < L; k += 64) {
            float v = val[j * L + k];
            for (u64 left = same; left != 0; left &= left - 1ull) v = v + upd[(__ffsll((long long)left) - 1) * L + k];
            to[k] = v;
        }
    }
    if (loss)
        for (int b = wave; b < (int)t.batch; b += waves) {
            const double sum = loss_of(lane < per ? score[b * per + lane] : 0.0f, per);
            if (lane == 0) loss[b] = sum;
        }
}

__global__ __launch_bounds__(256) void k_kge_loss_sum(const double *loss, int64_t n, double *out) {
    __shared__ double s[256];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) acc += loss[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

// *p <- `words` words of device memory, zero once st has passed this point; NULL if that cannot be had.  True: the memory was refused.
template <class T>
static bool zeroed(T **p, size_t words, hipStream_t st) {
    *p = nullptr;
    if (hipMalloc((void **)p, words * sizeof(uint32_t)) != hipSuccess) { (void)hipGetLastError(); *p = nullptr; return true; }
    if (dpaps_zero_words((uint32_t *)*p, words, st)) { (void)hipFree(*p); *p = nullptr; }
    return false;
}

// Whether a step updates the rows of keys that are named once in place (see k_kge_group), and its flags then.  It pays
// where most negatives are alone: drawn from more entities than twice the batch's negatives, three quarters and more
// are.  Not where the terms are to be added strictly one after the other, nor for rows so short that the
// bookkeeping (8 bytes a key) would weigh.  Steps take turns with two sets of flags: the flags of one may be in use while the
// next one's are written.  most: the data points of the call's largest batch.  st: the stream of the keys' kernel, which
// the work of earlier calls precedes: marks and flags are made and cleared there.  Where there is no memory for them the
// step does without, and what was refused once is not asked for again.
static bool in_place_step(dpaps_ps *ps, const KgeBatch &t, int64_t most, hipStream_t st, PushDone &done) {
    done = PushDone{};
    const int64_t negatives = t.batch * (t.ns + t.no), slots = most * (3 + t.ns + t.no);
    if (negatives == 0 || 2 * negatives > t.num_entities || ps->L < 32 || ps->opt_push_sequential) return false;
    const size_t mark_words = 2 * (size_t)ps->K;
    if (!ps->kge_seen && !ps->kge_seen_refused) ps->kge_seen_refused = zeroed(&ps->kge_seen, mark_words, st);
    if (!ps->kge_seen) return false;
    if ((size_t)slots > ps->kge_shared_slots) {
        if ((size_t)slots >= ps->kge_shared_refused) return false;
        if (hipStreamSynchronize(st) != hipSuccess) return false;
        if (ps->kge_shared) (void)hipFree(ps->kge_shared);
        ps->kge_shared = nullptr; ps->kge_shared_slots = 0;
        if (zeroed(&ps->kge_shared, 2 * (size_t)slots, st)) ps->kge_shared_refused = (size_t)slots;
        if (!ps->kge_shared) return false;
        ps->kge_shared_slots = (size_t)slots;
    }
    if (++ps->kge_id == 0) {                 // wrapped: forget everything
        if (hipDeviceSynchronize() != hipSuccess || dpaps_zero_words((uint32_t *)ps->kge_seen, mark_words, st) ||
            dpaps_zero_words(ps->kge_shared, 2 * ps->kge_shared_slots, st)) {
            --ps->kge_id;
            return false;
        }
        ps->kge_id = 1;
    }
    done.shared = ps->kge_shared + (ps->kge_id & 1u ? ps->kge_shared_slots : 0);
    done.id = ps->kge_id;
    done.slots = (uint32_t)(3 + t.ns + t.no);
    return true;
}

static int launch_group(dpaps_ps *ps, const KgeBatch &t, int32_t dim, float lr, float eps, float *upd, int64_t *keys_out, const PushDone &done, double *loss,
                        bool add_loss, hipStream_t st) {
    const unsigned blocks = grid_for(t.batch * 64, 256);
#define KGE_GROUP(NC)                                                                                                                       \
    do {                                                                                                                                    \
        if (ps->opt_kge_exact) k_kge_group<NC, true><<<blocks, 256, 0, st>>>(t, dim, lr, eps, ps->val, upd, keys_out, ps->K, done, loss, add_loss, ps->err); \
        else k_kge_group<NC, false><<<blocks, 256, 0, st>>>(t, dim, lr, eps, ps->val, upd, keys_out, ps->K, done, loss, add_loss, ps->err);                  \
    } while (0)
    switch ((dim + 63) / 64) {
    case 1: KGE_GROUP(1); break;
    case 2: KGE_GROUP(2); break;
    case 3: KGE_GROUP(3); break;
    default: KGE_GROUP(4); break;
    }
#undef KGE_GROUP
    PS_HIP(ps, hipGetLastError());
    return PS_OK;
}

extern "C" int kge_sgd_step(ps_handle ps, int32_t worker, int64_t num_entities, int32_t dim, int64_t batch, const int32_t *subj,
                            const int32_t *rel, const int32_t *obj, int32_t n_neg_subj, const int32_t *neg_subj,
                            int32_t n_neg_obj, const int32_t *neg_obj, float lr, float eps, double *loss_host_out, void *stream) {
    if (!ps || batch < 0 || dim <= 0 || n_neg_subj < 0 || n_neg_obj < 0 || num_entities <= 0) return PS_EINVAL;
    if (4 * (int64_t)dim != ps->L || num_entities > ps->K) return PS_EINVAL;
    if (dim > 256 || 1 + (int64_t)n_neg_subj + n_neg_obj > 64) return PS_ELIMIT;
    if (worker < -1 || worker >= ps->W) return PS_EWORKER;
    if (batch > 0 && (!subj || !rel || !obj || (n_neg_subj > 0 && !neg_subj) || (n_neg_obj > 0 && !neg_obj))) return PS_EINVAL;
    if (loss_host_out) *loss_host_out = 0.0;
    if (batch == 0) return PS_OK;
    const int64_t rows = batch * (3 + n_neg_subj + n_neg_obj);        // keys pulled and pushed: the slots of the data points
    if (rows >= ((int64_t)1 << 31)) return PS_ELIMIT;
    hipStream_t st = (hipStream_t)stream;
    // scratch of the step: the keys of all slots, the update rows (one per slot), the losses
    const size_t off_upd = (size_t)((rows * 8 + 255) / 256 * 256);
    const size_t off_loss = off_upd + (size_t)((rows * ps->L * 4 + 255) / 256 * 256);
    const size_t bytes = off_loss + (size_t)(batch + 1) * 8;
    if (bytes > ps->kge_ws_bytes) {
        PS_HIP(ps, hipStreamSynchronize(st));
        if (ps->kge_ws) PS_HIP(ps, hipFree(ps->kge_ws));
        ps->kge_ws = nullptr; ps->kge_ws_bytes = 0;
        hipError_t e = hipMalloc(&ps->kge_ws, bytes);
        if (e != hipSuccess) { (void)hipGetLastError(); ps->last_error = "out of device memory for the step's scratch"; return PS_ENOMEM; }
        ps->kge_ws_bytes = bytes;
    }
    int64_t *ukeys = (int64_t *)ps->kge_ws;
    float *upd = (float *)((char *)ps->kge_ws + off_upd);
    double *loss = (double *)((char *)ps->kge_ws + off_loss);
    const KgeBatch t{subj, rel, obj, neg_subj, neg_obj, n_neg_subj, n_neg_obj, num_entities, batch};
    int rc;
    double *const wanted = loss_host_out ? loss : nullptr;            // the losses, if the caller asks for them
    if (rows <= KGE_FEW_SLOTS && kge_few_lds(rows, ps->L) <= KGE_FEW_LDS && !ps->opt_kge_exact && !ps->opt_push_sequential && !ps->loc) {
        static LdsAllowed allowed;
        rc = dpaps_allow_lds(ps, allowed, reinterpret_cast<const void *>(&k_kge_few), KGE_FEW_LDS);
        if (rc) return rc;
        const RouteArgs a = dpaps_step_route(ps, worker, rows, st);
        k_kge_few<<<1 + a.blocks, KGE_FEW_THREADS, kge_few_lds(rows, ps->L), st>>>(a, t, dim, lr, eps, ps->val, ps->K, wanted, ps->err);
        PS_HIP(ps, hipGetLastError());
    } else if (rows <= dpaps_few_keys()) {
        // Few slots: what costs is launches, and the two streams' waiting for each other.  The update rows' kernel checks
        // and writes the keys, then the sums follow on the one stream.
        rc = launch_group(ps, t, dim, lr, eps, upd, ukeys, PushDone{}, wanted, false, st);
        if (rc) return rc;
        rc = dpaps_push_few_step(ps, worker, ukeys, rows, upd, st);
        if (rc) return rc;
    } else {
        PushDone done;
        const bool in_place = in_place_step(ps, t, batch, st, done);
        k_kge_keys<<<grid_for(rows, 256), 256, 0, st>>>(t, ukeys, ps->K, in_place ? ps->kge_seen : nullptr, const_cast<uint32_t *>(done.shared), done.id,
                                                        KgeBatch{}, nullptr, ps->err);
        PS_HIP(ps, hipGetLastError());
        // The sort of the push needs the keys only: it runs on the library's second stream beside the kernel that computes
        // the update rows, and the sums wait for it.  The statistics of the pull and of the push (every slot is
        // pulled, and pushed below) are counted along with the sums.
        rc = dpaps_side_stream(ps);
        if (rc) return rc;
        hipStream_t bs = ps->side_stream;
        PS_HIP(ps, hipEventRecord(ps->ev_fork, st));
        PS_HIP(ps, hipStreamWaitEvent(bs, ps->ev_fork, 0));
        rc = dpaps_push_sort(ps, ukeys, rows, bs);
        if (rc) return rc;
        PS_HIP(ps, hipEventRecord(ps->ev_sorted, bs));
        rc = launch_group(ps, t, dim, lr, eps, upd, nullptr, done, wanted, false, st);
        if (rc) return rc;
        PS_HIP(ps, hipStreamWaitEvent(st, ps->ev_sorted, 0));
        rc = dpaps_push_add_step(ps, worker, ukeys, rows, upd, done, st);
        if (rc) return rc;
    }
    if (loss_host_out) {
        k_kge_loss_sum<<<1, 256, 0, st>>>(loss, batch, loss + batch);
        PS_HIP(ps, hipGetLastError());
        PS_HIP(ps, hipMemcpyAsync(loss_host_out, loss + batch, sizeof(double), hipMemcpyDeviceToHost, st));
        PS_HIP(ps, hipStreamSynchronize(st));
    }
    return PS_OK;
}

// ---------------------------------------------------------------------------
// One epoch over workers, with the parameters allocated where they are used (Appendix A of the paper)
// ---------------------------------------------------------------------------
// every index of the epoch's triples inside its range (the kernels that follow index the store with them)
__global__ void k_kge_validate(int64_t num_entities, int64_t num_relations, int64_t n, const int32_t *subj, const int32_t *rel,
                               const int32_t *obj, int32_t ns, const int32_t *neg_subj, int32_t no, const int32_t *neg_obj, int32_t *err) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    bool bad = subj[t] < 0 || subj[t] >= num_entities || obj[t] < 0 || obj[t] >= num_entities || rel[t] < 0 || rel[t] >= num_relations;
    for (int32_t j = 0; j < ns; ++j) bad |= neg_subj[t * ns + j] < 0 || neg_subj[t * ns + j] >= num_entities;
    for (int32_t j = 0; j < no; ++j) bad |= neg_obj[t * no + j] < 0 || neg_obj[t * no + j] >= num_entities;
    if (bad) atomicExch(err, PS_EKEY);
}

// the entity keys the triples [t0, t1) will access: per triple its subject, its object, its negatives
__global__ void k_kge_entity_keys(int64_t t0, int64_t t1, const int32_t *subj, const int32_t *obj, int32_t ns, const int32_t *neg_subj,
                                  int32_t no, const int32_t *neg_obj, int64_t *keys) {
    const int64_t t = t0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= t1) return;
    int64_t *k = keys + (t - t0) * (2 + ns + no);
    k[0] = subj[t]; k[1] = obj[t];
    for (int32_t j = 0; j < ns; ++j) k[2 + j] = neg_subj[t * ns + j];
    for (int32_t j = 0; j < no; ++j) k[2 + ns + j] = neg_obj[t * no + j];
}

__global__ void k_kge_relation_keys(int64_t num_entities, int64_t t0, int64_t t1, const int32_t *rel, int64_t *keys) {
    const int64_t t = t0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < t1) keys[t - t0] = num_entities + rel[t];
}

extern "C" int kge_sgd_epoch(ps_handle ps, int64_t num_entities, int32_t dim, int64_t num_triples, const int32_t *subj, const int32_t *rel,
                             const int32_t *obj, int32_t n_neg_subj, const int32_t *neg_subj, int32_t n_neg_obj, const int32_t *neg_obj,
                             const int64_t *part_ptr_host, int32_t num_parts, int64_t batch, int32_t lookahead, float lr, float eps,
                             double *loss_host_out, void *stream) {
    if (!ps || num_triples < 0 || dim <= 0 || n_neg_subj < 0 || n_neg_obj < 0 || num_entities <= 0 || batch <= 0 || !part_ptr_host) return PS_EINVAL;
    if (4 * (int64_t)dim != ps->L || num_entities > ps->K) return PS_EINVAL;
    if (dim > 256 || 1 + (int64_t)n_neg_subj + n_neg_obj > 64) return PS_ELIMIT;
    if (num_parts <= 0 || num_parts > ps->W) return PS_EWORKER;
    if (part_ptr_host[0] != 0 || part_ptr_host[num_parts] != num_triples) return PS_EINVAL;
    int64_t longest = 0;
    for (int32_t w = 0; w < num_parts; ++w) {
        if (part_ptr_host[w + 1] < part_ptr_host[w]) return PS_EINVAL;
        longest = std::max(longest, part_ptr_host[w + 1] - part_ptr_host[w]);
    }
    if (num_triples > 0 && (!subj || !rel || !obj || (n_neg_subj > 0 && !neg_subj) || (n_neg_obj > 0 && !neg_obj))) return PS_EINVAL;
    if (loss_host_out) *loss_host_out = 0.0;
    if (num_triples == 0) return PS_OK;
    const int32_t ns = n_neg_subj, no = n_neg_obj, per = 1 + ns + no, ent = 2 + ns + no;
    const int64_t bmax = std::min(batch, longest);
    if (bmax * (per + 2) >= ((int64_t)1 << 31) || longest * ent >= ((int64_t)1 << 31)) return PS_ELIMIT;
    hipStream_t vs = (hipStream_t)stream;                  // the work on the values
    {
        const int rc = dpaps_side_stream(ps);
        if (rc) return rc;
    }
    hipStream_t bs = ps->side_stream;                      // localize calls and statistics: owner map and counters only
    // scratch: localize keys (second stream), the slots' keys, update rows and the losses (first)
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    const int64_t rows_max = bmax * (3 + ns + no);
    const size_t off_loc = 0;
    const size_t off_ukeys = off_loc + up((size_t)std::max(longest, bmax * ent) * 8);
    const size_t off_upd = off_ukeys + up((size_t)rows_max * 8);
    const size_t off_loss = off_upd + up((size_t)rows_max * ps->L * 4);
    const size_t bytes = off_loss + (size_t)(bmax + 2) * 8;
    if (bytes > ps->kge_ws_bytes) {
        PS_HIP(ps, hipStreamSynchronize(vs));
        if (ps->kge_ws) PS_HIP(ps, hipFree(ps->kge_ws));
        ps->kge_ws = nullptr; ps->kge_ws_bytes = 0;
        hipError_t e = hipMalloc(&ps->kge_ws, bytes);
        if (e != hipSuccess) { (void)hipGetLastError(); ps->last_error = "out of device memory for the epoch's scratch"; return PS_ENOMEM; }
        ps->kge_ws_bytes = bytes;
    }
    int64_t *lkeys = (int64_t *)((char *)ps->kge_ws + off_loc);
    int64_t *ukeys = (int64_t *)((char *)ps->kge_ws + off_ukeys);
    float *upd = (float *)((char *)ps->kge_ws + off_upd);
    double *loss = (double *)((char *)ps->kge_ws + off_loss);

    // every index is checked once; both streams start after that
    k_kge_validate<<<grid_for(num_triples, 256), 256, 0, vs>>>(num_entities, ps->K - num_entities, num_triples, subj, rel, obj, ns, neg_subj,
                                                             no, neg_obj, ps->err);
    PS_HIP(ps, hipGetLastError());
    PS_HIP(ps, hipEventRecord(ps->ev_fork, vs));
    PS_HIP(ps, hipStreamWaitEvent(bs, ps->ev_fork, 0));
    // (without memory for two sets of sorted pairs the steps share one)
    bool two = false;
    int rc = dpaps_push_reserve_steps(ps, rows_max, &two);
    if (rc) return rc;
    if (loss_host_out && dpaps_zero_words((uint32_t *)loss, 2 * (size_t)bmax, vs)) { ps->last_error = "knowledge-graph epoch: clearing the losses"; return PS_EHIP; }
    auto localize_entities = [&](int64_t t0, int64_t t1, int32_t w) {
        if (t1 <= t0) return (int)PS_OK;
        k_kge_entity_keys<<<grid_for(t1 - t0, 256), 256, 0, bs>>>(t0, t1, subj, obj, ns, neg_subj, no, neg_obj, lkeys);
        PS_HIP(ps, hipGetLastError());
        return dpaps_localize_checked(ps, lkeys, (t1 - t0) * ent, w, bs);
    };
    if (lookahead) {
        for (int32_t w = 0; w < num_parts && !rc; ++w) {              // relations go where their triples are
            const int64_t t0 = part_ptr_host[w], t1 = part_ptr_host[w + 1];
            if (t1 <= t0) continue;
            k_kge_relation_keys<<<grid_for(t1 - t0, 256), 256, 0, bs>>>(num_entities, t0, t1, rel, lkeys);
            PS_HIP(ps, hipGetLastError());
            rc = dpaps_localize_checked(ps, lkeys, t1 - t0, w, bs);
        }
        for (int32_t w = 0; w < num_parts && !rc; ++w)                // the first batch's entities
            rc = localize_entities(part_ptr_host[w], std::min(part_ptr_host[w] + batch, part_ptr_host[w + 1]), w);
    }
    int64_t steps_done = 0;
    for (int64_t r = 0; r * batch < longest && !rc; ++r) {
        for (int32_t w = 0; w < num_parts && !rc; ++w) {
            const int64_t t0 = part_ptr_host[w] + r * batch, end = part_ptr_host[w + 1];
            if (t0 >= end) continue;
            const int64_t t1 = std::min(t0 + batch, end), nb = t1 - t0;
            // second stream: the next batch's entities come to this worker, then this batch's accesses are counted
            const KgeBatch t{subj + t0, rel + t0, obj + t0, neg_subj + t0 * ns, neg_obj + t0 * no, ns, no, num_entities, nb};
            const int64_t n1 = lookahead && t1 < end ? std::min(t1 + batch, end) - t1 : 0;
            const KgeBatch next{subj + t1, rel + t1, obj + t1, neg_subj + t1 * ns, neg_obj + t1 * no, ns, no, num_entities, n1};
            // (sorted pairs and flags: two steps take turns with them, so the step before the last has to be through; with one
            // set of pairs, a step's sort waited for the sums of the one before it, and these for the sort: 2,970 us for 32 steps of
            // 1,024 data points over four workers with a launch for the losses after each, and 2,300 this way)
            const int half = two ? (int)(steps_done & 1) : 0;
            if (steps_done > (two ? 1 : 0)) PS_HIP(ps, hipStreamWaitEvent(bs, ps->ev_added[half], 0));
            PushDone done;
            const bool in_place = in_place_step(ps, t, bmax, bs, done);
            k_kge_keys<<<grid_for(std::max(nb * (3 + ns + no), n1 * ent), 256), 256, 0, bs>>>(t, ukeys, 0, in_place ? ps->kge_seen : nullptr,
                                                                                              const_cast<uint32_t *>(done.shared), done.id, next, lkeys, ps->err);
            PS_HIP(ps, hipGetLastError());
            if (in_place) PS_HIP(ps, hipEventRecord(ps->ev_keys, bs));
            if (n1 > 0) rc = dpaps_localize_checked(ps, lkeys, n1 * ent, w, bs);
            if (rc) break;
            rc = dpaps_route_pull_push(ps, w, ukeys, nb * (3 + ns + no), bs);
            if (rc) break;
            // ... and the push's sort, which needs the keys only
            rc = dpaps_push_sort_half(ps, half, rows_max, ukeys, nb * (3 + ns + no), bs);
            if (rc) break;
            PS_HIP(ps, hipEventRecord(ps->ev_sorted, bs));
            // first stream: the values
            if (in_place) PS_HIP(ps, hipStreamWaitEvent(vs, ps->ev_keys, 0));
            // (its losses onto those of the data points at the same places of the batches before; added up once, at the end: after every
            // step that was a launch of one workgroup on the stream that the steps wait for)
            rc = launch_group(ps, t, dim, lr, eps, upd, nullptr, done, loss_host_out ? loss : nullptr, true, vs);
            if (rc) break;
            PS_HIP(ps, hipStreamWaitEvent(vs, ps->ev_sorted, 0));
            rc = dpaps_push_add(ps, nb * (3 + ns + no), upd, done, vs);
            if (rc) break;
            PS_HIP(ps, hipEventRecord(ps->ev_added[half], vs));
            ++steps_done;
        }
    }
    // the second stream joins the first
    PS_HIP(ps, hipEventRecord(ps->ev_join, bs));
    PS_HIP(ps, hipStreamWaitEvent(vs, ps->ev_join, 0));
    if (rc) return rc;
    if (loss_host_out) {
        k_kge_loss_sum<<<1, 256, 0, vs>>>(loss, bmax, loss + bmax);
        PS_HIP(ps, hipGetLastError());
        PS_HIP(ps, hipMemcpyAsync(loss_host_out, loss + bmax, sizeof(double), hipMemcpyDeviceToHost, vs));
        PS_HIP(ps, hipStreamSynchronize(vs));
    }
    return PS_OK;
}
