// Work items of a count launch on the device: claiming runs of them from the
// launch's cursors, and decoding a run.
#pragma once

#include "kernels.h"

namespace citron {

constexpr int kMaxClaim = 16;           // items claimed at once, at most
// decoded items of a claimed run, one int32 per field and item
enum ItemField { kItQuery, kItKind, kItRowsOff, kItTag, kItArc0, kItDegree, kItRow, kItPart, kItFields };

// First item of run j, and the items of the run that starts at g.
__device__ __forceinline__ int64_t run_begin(const ItemSpace& P, int64_t j)
{
    return j < P.singles ? j : P.singles + (j - P.singles) * P.chunk;
}
__device__ __forceinline__ int run_length(const ItemSpace& P, int g)
{
    return g < P.singles ? 1 : min(P.chunk, P.total - g);
}

// Runs for `claimers` waves or workgroups: about eight claims each, after two
// single ones.  Items are in descending cost order, so a run's cost about the
// same; a first run of 16 of a deep count's costliest items held one wave for
// 21 ms of a launch whose waves were busy 4.6 ms on average (Chung-Lu 2^14,
// k = 9).
inline void set_runs(ItemSpace& P, int64_t claimers, int max_chunk)
{
    P.singles = (int32_t)(2 * claimers < P.total ? 2 * claimers : P.total);
    const int64_t c = (P.total - P.singles) / (claimers * 8);
    P.chunk = (int32_t)(c < 1 ? 1 : (c > max_chunk ? max_chunk : c));
}

// The claimer's next run of items.  Runs of consecutive items are dealt to
// kClaimShards cursors in turn (run j to cursor j mod kClaimShards), so
// that the items still start in order of cost.  A claimer's (a
// wave's, or a block's) first run is fixed by its number and costs no atomic; later ones come from the cursor of its
// home shard, and once that is dry from any that is not, found by one load of
// all cursors.  Returns the run's first item, or -1 when none is left.
//
// One cursor for all waves served 85 M claims a second: G(50001, 37) at
// k = 4, one light vertex per item, took 590 us of claims alone, and every
// launch of 4,096 waves about 50 us for their last, empty-handed claims.
__device__ __forceinline__ int claim_run(const ItemSpace& P, int wave, int waves, int& shard, bool& fresh)
{
    const int lane = threadIdx.x & (kWave - 1);
    int c;
    if (fresh) {
        fresh = false;
        c = wave / kClaimShards;
    } else {
        int v = 0;
        if (lane == 0) v = atomicAdd(P.cursors + shard * kClaimStride, 1);
        c = __builtin_amdgcn_readfirstlane(v) + (waves - shard + kClaimShards - 1) / kClaimShards;
    }
    for (;;) {
        const int64_t g = run_begin(P, (int64_t)c * kClaimShards + shard);
        if (g < P.total) return (int)g;
        bool has = false;
        if (lane < kClaimShards) {
            const int64_t next = (int64_t)__hip_atomic_load(P.cursors + lane * kClaimStride, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT) +
                                 (waves - lane + kClaimShards - 1) / kClaimShards;
            has = run_begin(P, next * kClaimShards + lane) < P.total;
        }
        const unsigned left = (unsigned)__ballot(has);
        if (left == 0u) return -1;
        // the next shard with work after the present one, cyclically
        const unsigned after = left & ~((2u << shard) - 1u);
        shard = __builtin_ctz(after ? after : left);
        int v = 0;
        if (lane == 0) v = atomicAdd(P.cursors + shard * kClaimStride, 1);
        c = __builtin_amdgcn_readfirstlane(v) + (waves - shard + kClaimShards - 1) / kClaimShards;
    }
}
static_assert(kClaimShards <= 31, "shard masks are 32-bit words");

// Lane j < n decodes item g0 + j of the space into LDS fields:
// its query, then one part of a heavy arc or (a part of) a light vertex.  The
// chain of dependent loads (query, bucket, arc or vertex, DAG offsets, row
// offset: about 14 on a graph with a few hundred buckets) is paid once per
// run instead of once per item.
template <int kSpace>
__device__ __forceinline__ void decode_run(const ItemSpace& P, int g0, int n, int32_t* item)
{
    const int j = threadIdx.x & (kWave - 1);
    if (j >= n) return;
    const int g = g0 + j;
    int qi;
    {
        int lo = 0, hi = P.n_queries - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (P.queries[mid].space_begin[kSpace] <= g) lo = mid;
            else hi = mid - 1;
        }
        qi = lo;
    }
    const QueryDesc& q = P.queries[qi];
    const bool sorted = kSpace != kRestSpace;      // the dense kernel reads the sorted rows
    const int i = q.item_lo + (g - q.space_begin[kSpace] + q.space_off[kSpace]) * q.item_stride;
    int u, r = -1, part, nparts, tag, kind = kItemHeavyArc;
    if (q.arc_list) {
        // list mode: one part of one listed arc; counts go to its list slot
        tag = q.arc_items[2 * i];
        const int pw = q.arc_items[2 * i + 1];
        const int e = q.arc_list[tag];
        u = q.dag_src[e];
        kind = q.dag_ptr[u + 1] - q.dag_ptr[u] > kLightMaxDeg ? kItemHeavyArc : kItemLightVertex;
        r = e - q.dag_ptr[u];
        part = pw & 0xffff;
        nparts = pw >> 16;
    } else {
        // bucket holding item i, then the arc or vertex and the part (part-major)
        int lo = 0, hi = q.n_buckets - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (q.buckets[4 * mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        const int key = q.buckets[4 * lo + 3] >> kItemKindBits;
        kind = q.buckets[4 * lo + 3] & ((1 << kItemKindBits) - 1);
        const int cnt = q.buckets[4 * lo + 2];
        const int local = i - q.buckets[4 * lo];
        part = local / cnt;
        const int which = q.buckets[4 * lo + 1] + (local - part * cnt);
        if (kind == kItemHeavyArc || kind == kItemDenseArc) {
            const int e = q.rows.harcs[which];
            u = q.dag_src[e];
            r = sorted ? q.rows.hpos[e] : e - q.dag_ptr[u];
            nparts = kind == kItemDenseArc ? dense_parts(key, q.k, q.split_pct) : arc_parts(key, q.k, q.split_pct);
            tag = e;
        } else if (kind == kItemHeavyVertex || kind == kItemDenseVertex) {
            u = q.order[which];
            nparts = 1;
            tag = -1;
        } else {
            u = q.order[q.light_first + which];
            nparts = kind == kItemLightRoot ? 1 : light_arcs(key + 1, q.k, q.split_pct);
            if (kind == kItemDeepVertex) nparts *= kLightSubs;
            tag = -1;
        }
    }
    const int a0 = q.dag_ptr[u];
    item[kItQuery * kMaxClaim + j] = qi;
    item[kItKind * kMaxClaim + j] = kind;
    item[kItRowsOff * kMaxClaim + j] = sorted ? q.rows.hoff[u] : q.rows.rows_off[u];
    item[kItTag * kMaxClaim + j] = tag;
    item[kItArc0 * kMaxClaim + j] = a0;
    item[kItDegree * kMaxClaim + j] = q.dag_ptr[u + 1] - a0;
    item[kItRow * kMaxClaim + j] = r;
    item[kItPart * kMaxClaim + j] = part | (nparts << 16);
}

}  // namespace citron
