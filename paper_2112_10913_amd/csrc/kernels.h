// Launch wrappers of the HIP kernels of libcitron (host-callable).
#pragma once

#include "internal.h"
#include "peel.h"

namespace citron {

// ---- ordering phase (kernels_order.hip)
size_t scan_workspace_ints(int64_t n);
hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int32_t* ws, hipStream_t s);
// *err, *max_outdeg, *kept: zeroed before the call.  Leaves the error bits and,
// when there are none, the out-degrees under the degree ordering, the largest
// of them and their sum, which is nnz / 2 iff the graph is symmetric.
hipError_t launch_validate(int32_t n, int64_t nnz, const int32_t* row_ptr, const int32_t* col, int32_t* err,
                           int32_t* outdeg, int32_t* max_outdeg, unsigned long long* kept, hipStream_t s);
// key: nullptr for the degree ordering, else the per-vertex order key (ties by
// id).  count: outdeg is counted here (*max_outdeg, zeroed before, too); else
// it is launch_validate's, which is the degree ordering's
hipError_t launch_orient(int32_t n, const int32_t* row_ptr, const int32_t* col, int32_t* outdeg,
                         int32_t* dag_ptr, int32_t* dag_col, int32_t* dag_src, int32_t* max_outdeg,
                         int32_t* scan_ws, hipStream_t s, const int32_t* key, bool count);

// ---- core ordering by level-synchronous peeling (kernels_core.hip)
hipError_t launch_peel_init(int32_t n, const PeelParams& P, hipStream_t s);
// launches first .. first + steps - 1 (0 follows launch_peel_init); those after
// the last phase return at once.  Copy (first + steps) & 1 of the control
// block then names the next phase.
hipError_t launch_peel_steps(const PeelParams& P, int64_t first, int32_t steps, hipStream_t s);

// ---- deterministic schedule order (kernels_sched.hip)
struct SortBuffers {
    unsigned long long* keys_a;   // n keys
    unsigned long long* keys_b;   // n keys
    void* temp;                   // sched_sort_temp_bytes
    size_t temp_bytes;
};
size_t sched_sort_temp_bytes(int64_t n, int32_t nb);   // n keys of nb buckets
// order[0 .. bounds[D-1]) = vertices with out-degree >= 2 by out-degree
// descending, ties by id; bounds[i] (i < D) = vertices of out-degree > D - i
hipError_t sched_plan_order(int32_t n, const int32_t* dag_ptr, int32_t D, int32_t* bounds, int32_t* order,
                            const SortBuffers& sb, hipStream_t s);
// harcs[0 .. bounds[kHeavyGroups D]) = arcs of vertices with out-degree > 64 by
// group, each by |C_uv| descending, ties by arc index; bucket (g, c) is
// g D + D - 1 - c, and bounds[b] = arcs in the buckets before b.  density[u]
// is the class of a heavy vertex u (launch_density); null: all of class 0.
hipError_t sched_heavy_arcs(int64_t m, const int32_t* dag_ptr, const int32_t* dag_src, const int32_t* arc_c,
                            const uint8_t* density, int32_t D, int32_t* bounds, int32_t* harcs, const SortBuffers& sb,
                            hipStream_t s);
// out[0 .. n) = the light vertices order[0 .. n) (out-degrees 64 .. kDeepDeg),
// those of a deep subgraph first, each group by out-degree descending, ties by
// place in `order`; bucket (g, d) is g kDeepBuckets + 64 - d
constexpr int kDeepBuckets = kLightMaxDeg - kDeepDeg + 1;
hipError_t sched_deep_order(int32_t n, const int32_t* order, const int32_t* dag_ptr, const int32_t* rows_off,
                            const unsigned long long* rows, int32_t* bounds, int32_t* out, const SortBuffers& sb,
                            hipStream_t s);

// ---- vertex schedule (kernels_sched.hip)
struct PlanBuffers {
    int32_t* hist_scan;    // max_outdeg + 3
    int32_t* order;        // n
    int32_t* light_deg;    // n
    int32_t* light_pre;    // n + 1
    int32_t* batch_start;  // n + 1
    PlanHeader* header;    // device
};
hipError_t launch_plan(int32_t n, const int32_t* dag_ptr, int32_t max_outdeg, int32_t light_rows,
                       int32_t split_min_deg, int32_t split_factor, const PlanBuffers& pb,
                       int32_t* scan_ws, const SortBuffers& sb, hipStream_t s);
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long* p, unsigned long long v, int64_t n, hipStream_t s);

// ---- subgraph rows (kernels_rows.hip)
// Sums of a build, kept in kBuildSlots copies a line apart (the workgroups'
// atomics on one word are serialised at about 12 ns) and added by the host.
constexpr int kBuildSlots = 16;
struct alignas(128) BuildSums {
    unsigned long long tri;      // triangles (the k = 3 count)
    unsigned long long verts, rows, entries, bytes;
    int32_t tri_ovf;
};
struct BuildParams {
    const int32_t* dag_ptr;
    const int32_t* dag_col;
    const int32_t* order;
    const int32_t* light_pre;
    const int32_t* batch_start;
    PlanHeader plan;
    int32_t max_deg;
    const int32_t* rows_off;
    unsigned long long* rows;
    int32_t* arc_c;
    BuildSums* sums;             // kBuildSlots
};
// len[u] = row words of u, or of the heavy u only
hipError_t launch_rows_len(int32_t n, const int32_t* dag_ptr, bool heavy_only, int32_t* len, hipStream_t s);
// rows of the heavy vertices (order[0 .. n_heavy)) in sorted positions
struct SortedRowsParams {
    int32_t n_heavy;
    const int32_t* order;
    const int32_t* dag_ptr;
    const int32_t* dag_col;
    const int32_t* row_ptr;
    const int32_t* key;          // order key, or nullptr for the degree ordering
    const int32_t* rows_off;
    const unsigned long long* rows;
    const int32_t* hoff;
    unsigned long long* hrows;
    uint16_t* hpos;
    uint16_t* hinv;
};
hipError_t launch_sorted_rows(const SortedRowsParams& P, hipStream_t s);
// density[u] = class (density_class) of every heavy vertex u; the sorted rows are built
hipError_t launch_density(const SortedRowsParams& P, const int32_t* arc_c, uint8_t* density, hipStream_t s);
hipError_t launch_build_rows(const BuildParams& P, int32_t blocks, hipStream_t s);
hipError_t launch_arc_c_to_u64(int64_t m, const int32_t* arc_c, unsigned long long* out, hipStream_t s);

// ---- counting phase (kernels_count.hip)
struct CountLaunch {
    const QueryDesc* queries;   // device table
    int32_t n_queries;
    int32_t space_items[kSpaces] = {};   // items of each space (place_query)
    int32_t* item_ctr;          // device: kLaunchInts cursors, zeroed by the launch sequence
    unsigned long long* scratch;   // stacks of k > 12, scratch_words per block
    int64_t scratch_words;
    int32_t max_k;
    int32_t blocks;
    int32_t wg_waves;
    int32_t lds_bytes;          // dynamic LDS per block
    int32_t flush_rows;
    int32_t arc_lds_max = 256;  // heavy nodes with 64 < c <= this are copied to LDS
    bool stats;                 // instrumented launch
    bool per_arc;               // some query writes per-arc counts
    int32_t* progress = nullptr;   // host-mapped word for the items claimed (nullable)
};
// device-memory stack words per block of a count launch
int64_t count_scratch_words(int32_t max_deg, int32_t max_k, int32_t wg_waves);
// the part of them that grows with k (all stacks of k > 12)
int64_t count_deep_scratch_words(int32_t max_k, int32_t wg_waves);
// dynamic LDS of a count launch: arc_max is its arc_lds_max tuning value
int32_t count_lds_bytes(int32_t arc_max, int32_t max_k, int32_t wg_waves, bool per_arc);
hipError_t launch_count(const CountLaunch& cl, hipStream_t s);
// its dense spaces (kernels_dense.hip)
hipError_t launch_dense(const CountLaunch& cl, hipStream_t s);
inline int64_t launch_items(const CountLaunch& cl)
{
    int64_t n = 0;
    for (int s = 0; s < kSpaces; ++s) n += cl.space_items[s];
    return n;
}
hipError_t launch_check_arcs(const int32_t* arcs, int32_t n, int64_t m, int32_t* err, hipStream_t s);
hipError_t launch_list_parts(const int32_t* arcs, int32_t n, const int32_t* dag_src, const int32_t* dag_ptr,
                             const int32_t* arc_c, int32_t k, int32_t pct, int32_t* parts, hipStream_t s);
hipError_t launch_list_items(int32_t n, const int32_t* parts, const int32_t* offs, int32_t* items, hipStream_t s);
hipError_t launch_gather_arc_c(const int32_t* arcs, int32_t n, const int32_t* arc_c, unsigned long long* out,
                               hipStream_t s);

// Items that the waves or workgroups of one kernel claim in runs (items.h).
struct ItemSpace {
    const QueryDesc* queries;
    int32_t n_queries;
    int32_t total;
    int32_t* cursors;       // kClaimInts words, zeroed before the launch
    int32_t singles;        // the first, costliest items are claimed one at a time,
    int32_t chunk;          // the others in runs of this many consecutive items
};

// ---- k-clique listing (kernels_list.hip)
constexpr int kListMaxK = 16;                    // largest k listing supports
struct ListParams {
    const int32_t* arcs;         // listed arcs (DAG arc indices)
    int32_t n_arcs;
    int32_t k;
    const int32_t* dag_ptr;
    const int32_t* dag_col;
    const int32_t* dag_src;
    const int32_t* rows_off;
    const unsigned long long* rows;
    const long long* offsets;    // n_arcs + 1: first output clique of each arc
    int32_t* out;                // cliques, k ids each
    int32_t* cursors;            // kClaimInts words, zeroed before the launch
    ItemSpace items;             // runs of arcs (set by launch_list_arcs)
    bool wide;                   // 16-byte stores (set by launch_list_arcs)
    int32_t stride;              // claim j lists arc j * stride mod n_arcs (set by launch_list_arcs)
    int32_t* err;                // zeroed before the launch; 1 = slot overrun, 2 = count mismatch
};
hipError_t launch_list_arcs(const ListParams& P, int32_t blocks, hipStream_t s);
size_t scan64_workspace(int64_t n);
hipError_t scan_exclusive64(const unsigned long long* in, long long* out, int64_t n, long long* ws, hipStream_t s);

}  // namespace citron
