// The key slots of a knowledge-graph batch, and which of them share their key.
#pragma once
#include <stdint.h>

// Slot j of data point b - subject, relation, object, subject negatives, object negatives - in pull and push order
struct KgeBatch {
    const int32_t *subj, *rel, *obj, *neg_subj, *neg_obj;
    int32_t ns, no;
    int64_t num_entities, batch;
};
__device__ __forceinline__ int64_t slot_key(const KgeBatch &t, int64_t b, int32_t j) {
    if (j == 0) return t.subj[b];
    if (j == 1) return t.num_entities + t.rel[b];
    if (j == 2) return t.obj[b];
    if (j < 3 + t.ns) return t.neg_subj[b * t.ns + (j - 3)];
    return t.neg_obj[b * t.no + (j - 3 - t.ns)];
}

// Slot i of the batch, the j-th of its data point, names key k: it leaves its number at the key, and where it finds one of
// this step (the id in front), both are flagged: shared[slot] = id.  A negative whose flag is not set in the end is the
// only slot of the batch with its key.
// A key named a thousand times is a thousand exchanges on one word, so the relations, of which there are few, are left
// out: no entity has their keys.  But only the key as a whole is checked to be in range: an entity number past the
// entities may be a relation's key, and is flagged; a relation number below zero is an entity's key, and takes part.
__device__ __forceinline__ void kge_mark_slot(int64_t num_entities, uint32_t i, int32_t j, int64_t k, unsigned long long *seen, uint32_t *shared,
                                              uint32_t id) {
    if (j == 1 && k >= num_entities) return;
    const unsigned long long old = atomicExch(&seen[k], ((unsigned long long)id << 32) | i);
    if ((uint32_t)(old >> 32) == id) { shared[i] = id; shared[(uint32_t)old] = id; }
    if (k >= num_entities) shared[i] = id;
}
