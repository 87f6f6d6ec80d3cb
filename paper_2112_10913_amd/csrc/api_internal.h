// Host-side state of libcitron shared by api.cpp, batch.cpp and server.cpp.
#pragma once

#include <mutex>
#include <string>
#include <vector>

#include "../../include/citron.h"
#include "kernels.h"

namespace citron {

// Small device-side words of one graph (zeroed by fill kernels, never by
// hipMemsetAsync, so that the sequences stay valid inside captured graphs).
struct SmallDev {
    int32_t err;
    int32_t max_outdeg;
    unsigned long long kept;     // sum of the out-degrees (validation)
    PeelCtl peel[2];
    PeelCounters peel_cnt;
    BuildSums build[kBuildSlots];
    int32_t list_cursors[kClaimInts];
};
static_assert(sizeof(SmallDev) % 8 == 0, "cleared in 8-byte words");

// What one count launch reads and updates: uploaded as one copy before the
// launch (partial sums, flag and cursors in their starting state); the sums
// and the flag come back as one copy.
// What is only read, what waves add to and what they claim from lie in lines
// of their own.
struct CountCtl {
    alignas(256) unsigned long long acc[kAccWords];
    int32_t overflow;
    alignas(256) QueryDesc query;
    alignas(256) int32_t cursors[kLaunchInts];
};

// Pinned host mirror for the copies back.
struct SmallHost {
    CountCtl ctl;
    int32_t err;                 // err, max_outdeg, kept: copied together
    int32_t max_outdeg;
    unsigned long long kept;
    int32_t ends[2];
    PlanHeader plan;
    uint64_t stats[kNumStats];
    int32_t rows_total;
    int32_t hist[2 * kMaxDeg + 2];   // bucket bounds of a schedule order
    PeelCtl peel[2];
    BuildSums build[kBuildSlots];
};

}  // namespace citron

struct citron_graph {
    int device = 0;
    hipStream_t stream = nullptr;
    int32_t n = 0;
    int64_t nnz = 0;
    int64_t m = 0;
    int state = 0;                 // 0 LOADED, 1 ORDERED
    int order_kind = 0;            // 0 degree ordering, 1 core ordering (peeling)
    int32_t peel_rounds = 0;       // rounds of the peeling (core ordering)
    int32_t max_outdeg = 0;
    int64_t device_bytes = 0;
    std::mutex mu;

    int32_t* d_row_ptr = nullptr;
    int32_t* d_col = nullptr;
    int32_t* d_outdeg = nullptr;
    bool outdeg_replaced = false;          // d_outdeg no longer holds the load's counts
    int32_t* d_dag_ptr = nullptr;
    int32_t* d_dag_col = nullptr;
    int32_t* d_dag_src = nullptr;
    int32_t* d_scan_ws = nullptr;
    int32_t* d_key = nullptr;              // core ordering: round of each vertex
    size_t scan_ws_ints = 0;
    citron::SmallDev* d_small = nullptr;
    citron::SmallHost* h_small = nullptr;

    citron_tuning tuning;
    citron::PlanBuffers pb = {};
    citron::PlanHeader plan = {};
    citron_tuning plan_tuning = {};
    bool plan_valid = false;
    citron::CountCtl* d_ctl = nullptr;
    unsigned long long* d_scratch = nullptr;
    int64_t scratch_bytes = 0;
    unsigned long long* d_stats = nullptr;

    uint64_t seed_base = 0;
    bool seed_pending = false;

    // subgraph rows, built at the first count (they do not depend on k)
    bool rows_valid = false;
    int32_t* d_rows_off = nullptr;          // n + 1
    unsigned long long* d_rows = nullptr;
    int32_t* d_arc_c = nullptr;             // m
    bool hrows_valid = false;
    int32_t* d_hoff = nullptr;              // n + 1: the heavy vertices' rows in sorted positions
    unsigned long long* d_hrows = nullptr;
    uint16_t* d_hpos = nullptr;             // m
    uint16_t* d_hinv = nullptr;             // m
    // heavy arcs by group and |C_uv|: of counts of k < kDensityK, which take all
    // vertices for one class, and of deeper ones
    struct HeavyArcs {
        int32_t* d_arcs = nullptr;          // m
        std::vector<int32_t> h_scan;        // bucket bounds (empty: not built)
    } harcs[2];
    std::vector<int32_t> h_vscan;           // vertices by out-degree, scanned
    int32_t* d_deep_order = nullptr;        // n: plan order of deep counts (sched_deep_order)
    std::vector<int32_t> h_deep;            // its bucket bounds (empty: not built)
    uint64_t tri = 0;
    bool tri_ovf = false;
    // per k, and one more (schedule_slot): the merged bucket table of the
    // count's work items
    int32_t* d_buckets[CITRON_KMAX + 2] = {};
    // tables superseded by a split change: kept until the graph is freed,
    // since a captured batch or an admitted server request may still read one
    std::vector<int32_t*> retired_buckets;
    int32_t bucket_split[CITRON_KMAX + 2] = {};   // split_pct each table was built with
    int64_t bucket_bytes[CITRON_KMAX + 2] = {};   // device bytes of each table
    int32_t n_buckets[CITRON_KMAX + 2] = {};
    int32_t n_work[CITRON_KMAX + 2] = {};
    int32_t sched_end[CITRON_KMAX + 2][citron::kDenseClasses] = {};   // ends of the dense spaces
    // per k: the vertex-rooted schedule (whole vertices, no split)
    int32_t* d_vbuckets[CITRON_KMAX + 1] = {};
    int64_t vbucket_bytes[CITRON_KMAX + 1] = {};
    int32_t n_vbuckets[CITRON_KMAX + 1] = {};
    int32_t n_vwork[CITRON_KMAX + 1] = {};
    uint64_t build_stats[citron::kNumStats] = {};
};

namespace citron {

// Device blocks on the current device and pinned host blocks, reused between
// graphs (pool.cpp).  A block goes back only after the work that used it.
hipError_t pool_malloc(void** p, size_t bytes);
void pool_free(void* p);
// Gives all idle blocks back.
void pool_release();
// hipMalloc, with the pool's idle blocks given back first if it fails.
hipError_t device_malloc(void** p, size_t bytes);
hipError_t pool_host_malloc(void** p, size_t bytes);
void pool_host_free(void* p, size_t bytes);

extern thread_local std::string g_last_error;
citron_status fail(citron_status st, const std::string& msg);
citron_status hip_fail(hipError_t e, const char* what);
citron_tuning default_tuning();
citron_status resolve_tuning(const citron_tuning* in, citron_tuning* out);
int32_t arc_max_for(const citron_tuning& t, int32_t max_k);
int device_cus(int dev);
citron_status ensure_plan(citron_graph* g, const citron_tuning& t);
citron_status ensure_rows(citron_graph* g);
citron_status ensure_heavy_arcs(citron_graph* g, bool deep);
// The schedule of a k-clique count: that of k, except that per-arc counts of
// k = 5 keep to arcs.  The dense kernel adds a vertex's products up over all
// its arcs, and separating them again, an accumulator pass per arc, cost more
// than it gained (R-MAT 14: 1.61 ms, 0.78 ms by arcs of the count kernel).
constexpr int32_t kPerArcSlot = CITRON_KMAX + 1;
inline int32_t schedule_slot(int32_t k, bool per_arc) { return per_arc && k == 5 ? kPerArcSlot : k; }
citron_status ensure_buckets(citron_graph* g, int32_t k, int32_t slot);
citron_status ensure_vbuckets(citron_graph* g, int32_t k);
citron_status check_count_args(const citron_graph* g, int32_t k, bool* trivial, uint64_t* value);
QueryDesc make_query(const citron_graph* g, int32_t k, int32_t slot, unsigned long long* acc, int32_t* ovf,
                     unsigned long long* per_arc, unsigned long long* stats);
void batch_forget_graph(const citron_graph* g);

}  // namespace citron
