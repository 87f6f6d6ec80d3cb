// Internal declarations shared by the HIP kernels and the host side of
// libcitron.  Not part of the public ABI (include/citron.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace citron {

constexpr int kWave = 64;            // gfx950 wavefront width
constexpr int kLightMaxDeg = 64;     // out-degree that fits one 64-bit row word
constexpr int kMaxWords = 64;        // row words per subgraph (out-degree <= 4096)
constexpr int kMaxDeg = kMaxWords * 64;
constexpr int kKMax = 32;
constexpr int kArcLdsMax = 256;      // largest candidate set an LDS subgraph copy holds

// Shared words of a count launch.  Atomics on one word are serialised by the
// device at about 12 ns each, so what every wave of a launch touches is
// spread out: work items are claimed from kClaimShards cursors (128 bytes
// apart), and a query's sum is kept in kAccSlots partial sums (64 bytes
// apart), which the host adds up with the same carry check.
constexpr int kClaimShards = 16;
constexpr int kClaimStride = 32;                        // int32 words
constexpr int kClaimInts = kClaimShards * kClaimStride;
constexpr int kAccSlots = 8;
constexpr int kAccStride = 8;                           // uint64 words
constexpr int kAccWords = kAccSlots * kAccStride;

// Sum of a query's partial sums (mod 2^64); *carry is set when one carries.
inline unsigned long long sum_acc_slots(const unsigned long long* acc, bool* carry)
{
    unsigned long long s = 0;
    for (int i = 0; i < kAccSlots; ++i) {
        const unsigned long long v = acc[i * kAccStride];
        if (s + v < s) *carry = true;
        s += v;
    }
    return s;
}

// Count-kernel statistics slots (citron_work_stats).
enum StatSlot {
    kStatVertices = 0,     // subgraphs built
    kStatRows = 1,         // rows built (arcs)
    kStatEntries = 2,      // out-list entries read by the build
    kStatWordOps = 3,      // last-level AND+popcount row-word operations
    kStatPushes = 4,       // recursion nodes pushed (both engines)
    kStatBytes = 5,        // DAG bytes read by the build
    kStatHeavySteps = 6,   // wave-uniform search steps on multi-word masks
    kStatCompactions = 7,  // nodes compacted to one word per row
    kStatCompactRows = 8,  // rows written by compaction
    kStatLightIters = 9,   // light-engine loop iterations (per wave)
    kStatLightActive = 10, // sum over those iterations of lanes with a unit
    kStatLightUnits = 11,  // units started by the light engine
    kStatFlushes = 12,     // task-buffer flushes
    kStatHeavyLeafCand = 13, // last-level candidates handled on multi-word masks
    kStatLightPops = 14,   // light-engine pops
    kStatWaveBusy = 15,    // sum over waves of (last item done - first item taken), wall-clock ticks
    kStatWaveFirst = 16,   // earliest start of a wave (wall-clock ticks, atomic min)
    kStatWaveLast = 17,    // latest end of a wave (atomic max)
    kStatWaves = 18,       // waves that ran
    kStatArcLds = 19,      // heavy arcs searched from an LDS copy of their subgraph
    kStatNeed3Lanes = 20,  // children handled whole by one lane (two levels left)
    kStatDonations = 21,   // light-engine work donations taken by idle lanes
    kStatWaveBusyMax = 22, // longest busy time of one wave (atomic max)
    kStatItemMax = 23,     // longest item: (ticks << 32) | item index (atomic max)
    kStatResidentNow = 24, // waves resident right now (live counter)
    kStatResidentMax = 25, // most waves resident at once (atomic max)
    kStatCycTotal = 26,    // shader-clock cycles of the waves, start to end
    kStatCycLight = 27,    // ... of which in the light engine
    kStatCycCopy = 28,     // ... of which copying or compacting subgraphs
    kStatCycNeed3 = 29,    // ... of which in lane-per-child two-level searches
    kStatNeed3Nodes = 30,  // nodes finished by lane-per-child two-level searches
    kStatNeed3MinOps = 31, // their row-word operations had rows been ceil(c / 64) words wide
    kNumStats = 32
};

// Schedule of one graph for the count kernel: vertices sorted by out-degree
// (descending), the heavy prefix processed one vertex per workgroup (the
// first n_split of them shared by split_factor workgroups), the light rest
// grouped into batches of about light_rows rows.
struct PlanHeader {
    int32_t n_heavy;      // vertices with out-degree > kLightMaxDeg
    int32_t n_split;      // heavy vertices shared by several workgroups
    int32_t split_factor;
    int32_t n_light;      // vertices with 2 <= out-degree <= kLightMaxDeg
    int32_t n_batches;
    int32_t n_items;      // n_split * split_factor + (n_heavy - n_split) + n_batches
    int32_t light_rows;
    int32_t max_rows;     // largest number of rows of one light batch
};

// Subgraph rows of one graph, built once (they do not depend on k): for
// every vertex u with out-list v_0 < ... < v_{d-1}, row i is the bitmap over
// positions 0..d-1 of N->(u) of N->(v_i) cap N->(u), W(u) = ceil(d/64) words.
struct RowsDev {
    const int32_t* rows_off;        // n + 1: first word of u's rows (< 2^31 words)
    const unsigned long long* rows; // all rows
    const int32_t* arc_c;           // m: popcount of arc e's row = |C_uv|
    const int32_t* harcs;           // arcs of heavy vertices by group (heavy_group), then |C_uv| descending
    // Rows of the heavy vertices again, in the order of the DAG: positions
    // sorted by the ordering (key, id), so that a vertex's neighbours come
    // after it and every matrix of rows is strictly upper triangular.  The
    // dense kernel works on these; the count kernel, whose lanes take a row
    // each, keeps to the id order, which spreads the long rows (with sorted
    // rows its k = 4 launch on a 2^20-vertex power-law graph took twice as
    // long).
    const int32_t* hoff;            // n: first word of u's rows in hrows (heavy u)
    const unsigned long long* hrows;
    const uint16_t* hpos;           // m: sorted position of arc e among its source's (heavy sources)
    const uint16_t* hinv;           // m: the way back, per sorted position
};

// Item spaces of a launch: dense arcs by row words, kDenseClasses of them
// down to 1, then everything else.
constexpr int kDenseClasses = 6;
constexpr int kSpaces = kDenseClasses + 1;
constexpr int kRestSpace = kDenseClasses;
constexpr int kLaunchInts = kSpaces * kClaimInts;
__host__ __device__ inline int dense_space(int c) { return kDenseClasses - (c + 63) / 64; }

// One query of the count kernel (a (graph, k) pair).
struct QueryDesc {
    const int32_t* dag_ptr;
    const int32_t* dag_src;      // source vertex of every arc
    const int32_t* order;        // vertices by out-degree descending (k >= kDeepK: light ones of a deep subgraph first)
    RowsDev rows;
    unsigned long long* acc;     // kAccSlots partial sums, kAccStride words apart
    int32_t* overflow;           // set to 1 when an addition carried
    unsigned long long* per_arc; // optional per-arc counts (nullptr: off)
    unsigned long long* stats;   // optional work counters (nullptr: off)
    // Work items, in buckets of equal cost key, largest key first: heavy-arc
    // buckets (key |C_uv|) and light-vertex buckets (key out-degree - 1),
    // merged.  Bucket b: buckets[4b] = first item, [4b+1] = first arc (index
    // into harcs) or first light vertex (index into the light part of order),
    // [4b+2] = arcs or vertices in the bucket, [4b+3] = key << 3 | kind
    // (BucketKind).  An arc or vertex is split into parts (arc_parts,
    // light_arcs); items of a bucket are part-major.  buckets[4 n_buckets]
    // = item count.  The vertex-rooted schedule has only the two vertex
    // kinds, each item one whole vertex (heavy ones indexed in order itself).
    const int32_t* buckets;
    int32_t n_buckets;
    int32_t light_first;         // index in order of the first light vertex
    int32_t k;
    int32_t n_work;              // items of the query (all buckets)
    int32_t n_items;             // items of this query in the launch
    int32_t item_lo;             // schedule item of the query's j-th launch item: item_lo + j * item_stride
    int32_t item_stride;
    // The kernels of a launch each take a space of items: the dense kernel's
    // instances by row words, largest first, then the count kernel.  In the
    // schedule the spaces follow one another (sched_end); place_query sets
    // where the query's launch items of space s start among all of s's items
    // (space_begin), and how many launch items come before them (space_off).
    int32_t sched_end[kDenseClasses];
    int32_t space_begin[kSpaces];
    int32_t space_off[kSpaces];
    int32_t split_pct;           // split scale the buckets were built with (arc_parts, light_arcs)
    // list mode (arc_list != nullptr): item j is (slot, part) = (arc_items[2j],
    // arc_items[2j+1] & 0xffff) of arc arc_list[slot], split into
    // arc_items[2j+1] >> 16 parts; its counts go to per-arc slot `slot`
    const int32_t* arc_list;
    const int32_t* arc_items;
};

// Kinds of work item (low bits of a bucket's key word).
constexpr int kItemKindBits = 3;
enum BucketKind {
    kItemHeavyArc = 0,     // one part of an arc of a heavy vertex (edge-rooted)
    kItemLightVertex = 1,  // (a part of) a light vertex, its arcs the units (edge-rooted)
    kItemHeavyVertex = 2,  // a whole heavy vertex, searched from its own root (vertex-rooted)
    kItemLightRoot = 3,    // a whole light vertex, one unit rooted at the vertex (vertex-rooted)
    kItemDenseArc = 4,     // one part of a heavy vertex's arc for the dense kernel (edge-rooted)
    kItemDenseVertex = 5,  // one part of a heavy vertex for the dense kernel: its arcs in turn
    kItemDeepVertex = 6    // (a part of) a light vertex with its arcs' branches dealt to kLightSubs sub-parts (edge-rooted)
};

// Parts a heavy arc with |C_uv| = c is split into for a k-clique count; each
// part takes every P-th first-level branch of the arc (speed only).  pct
// scales the default (percent); arcs are split only for k >= 6, where the
// root of an arc has at least four levels left.
__host__ __device__ inline int scale_parts(int base, int pct)
{
    if (base <= 1) return 1;
    const int p = base * pct / 100;
    return p < 1 ? 1 : (p > 64 ? 64 : p);
}

__host__ __device__ inline int arc_parts(int c, int k, int pct)
{
    if (k <= 5) return 1;
    if (k == 6) return scale_parts(c < 64 ? 1 : (c / 32 < 8 ? c / 32 : 8), pct);
    return scale_parts(c < 16 ? 1 : (c / 8 < 32 ? c / 8 : 32), pct);
}

// Arcs of heavy vertices the dense kernel takes in a k-clique count: sizes
// whose tiles fit LDS, at k >= 6, where an arc's subgraph, once laid out,
// serves many triangle counts, and at k = 5 for the vertices above kDenseMax,
// which dense_vertex leaves (R-MAT 20, k = 5: their arcs took 84 of 102 ms in
// the count kernel; 28 ms in all here, build included, from 17 or 65
// candidates on alike).  From 33, 17 and 9 candidates on: 100.9, 96 and 94.8
// ms for R-MAT 20, k = 6; 23.2, 21.7 and 21.7 for R-MAT 16, k = 7; 4.29, 4.0
// and 4.0 for a served mix of 48 counts.
//
// A mask costs the dense kernel the same however few candidates it has left,
// while the count kernel packs them, so the deeper the count the denser a
// subgraph has to be.  Random graphs of edge probability p, dense kernel and
// count kernel, about 50 candidates an arc: k = 6, p = 0.2 0.30 and 0.27 ms,
// 0.4 0.31 and 0.41; k = 7, 0.3 0.79 and 0.64, 0.4 1.0 and 1.0, 0.5 1.6 and
// 2.2; k = 8, 0.5 8.1 and 3.3, 0.7 12.8 and 12.3, 0.8 13.7 and 16.5; k = 9, 0.7
// 71 and 36, 0.8 72 and 65, 0.9 144 and 202; k = 10, 0.8 449 and 252.  About
// 200 candidates: k = 8, 0.6 546 and 546, 0.7 557 and 1255; k = 9 (an eighth),
// 0.7 1089 and 961, 0.8 1165 and 2971.  In power-law graphs the subgraphs get
// denser with every level, so what counts is the density one level down, of
// the neighbours of a candidate: 0.86 to 0.99 on R-MAT, where an arc's own
// is 0.6 to 0.95 and the dense kernel wins at every one of them (R-MAT 20, k = 8:
// 240 and 2606 ms for a share).
constexpr int kDenseMin = 17;
constexpr int kDenseMax = 64 * kDenseClasses;
__host__ __device__ inline bool dense_size(int c) { return c >= kDenseMin && c <= kDenseMax; }
// class of subgraphs where `edges` of `pairs` pairs of a candidate's neighbours
// are adjacent (pairs < 2^25)
constexpr int kDensities = 5;
constexpr int kDensityK = 7;         // counts that look at it
__host__ __device__ inline int density_class(unsigned edges, unsigned pairs)
{
    const unsigned e = 100 * edges;
    return (e >= 40 * pairs) + (e >= 66 * pairs) + (e >= 80 * pairs) + (e >= 88 * pairs);
}
__host__ __device__ inline bool dense_arc(int c, int k, int density)
{
    return k >= 5 && dense_size(c) && density >= (k < kDensityK ? 0 : k <= 10 ? k - kDensityK + 1 : kDensities - 1);
}
// Group of a heavy vertex's arc in harcs: arcs of vertices above kDenseMax
// first, and, where the dense kernel may take them, by their vertex's class.
constexpr int kHeavyGroups = 2 * kDensities;
__host__ __device__ inline int heavy_group(int d, int c, int density)
{
    return (d > kDenseMax ? 0 : kDensities) + (dense_size(c) ? density : 0);
}

// Heavy vertices the dense kernel takes whole in counts of k = 4 and 5, where
// an arc's subgraph would serve one triangle count at most: the vertex's own
// subgraph serves one per arc (k = 5), or all its 4-cliques are its triangles
// (k = 4), and its sorted rows need no packing.
__host__ __device__ inline bool dense_vertex(int d, int k)
{
    return (k == 4 || k == 5) && d > kLightMaxDeg && d <= kDenseMax;
}

// Parts of a dense arc (every P-th first-level branch).  One to four waves
// share an arc, so counts of k >= 8 are cut finely for the launch's tail
// (R-MAT 14, k = 8: c / 64 parts 52.1 ms, c / 24 43.6, c / 12 41.7, c / 4 40.6;
// Chung-Lu 2^14, k = 9: c / 8 7.3 ms, c / 4 6.5 ms); at k = 7 the
// parts' repeated layout costs more than it saves (R-MAT 16: c / 64 21.6 ms,
// c / 24 22.2 ms).
__host__ __device__ inline int dense_parts(int c, int k, int pct)
{
    if (k <= 6) return 1;
    if (k == 7) return scale_parts(c / 64, pct);
    return scale_parts(c / 4 < 64 ? c / 4 : 64, pct);
}

// Parts a light vertex (out-degree d <= 64, its subgraph one word per row)
// is split into: light_arcs of them take every light_arcs-th arc of the
// vertex, and for deep counts each of these is split again into kLightSubs
// (a power of two) that take the first-level branches of the same arcs at
// positions of one residue (speed only).  One wave searching two arcs of a
// planted 40-clique at k = 9 ran 24 of a launch's 28 ms while 88 % of the
// wave time was idle (Chung-Lu 2^14; with 4 sub-parts and short runs 15.2 ms,
// with 16 of them 12.3 ms, with complete nodes counted as binomials 6.4 ms).
// At k = 6 the tail of small launches decides: 24 graphs of up to 2^13
// vertices at k = 3..6 in one launch take 1.67 ms with d / 8 parts from
// d = 32, 1.59 with d / 4, 1.17 with 3 parts for 24 to 31 as well, 1.27 with
// d / 4 there too; a full chip (R-MAT 20) does not notice.
__host__ __device__ inline int light_arcs(int d, int k, int pct)
{
    if (k <= 5) return 1;
    if (k == 6) return scale_parts(d >= 32 ? d / 4 : (d >= 24 ? 3 : 1), pct);
    return scale_parts(d >= 12 ? d / 2 : 1, pct);
}
// Only vertices of a deep subgraph are split that far: one that closes at
// least as many triangles as a complete graph of kDeepDeg vertices.  Where
// every vertex of out-degree 24 and more was, a power-law graph without
// planted cliques (Chung-Lu 2^17, k = 9) took 4.1 ms for its millions of empty
// items; 0.95 ms now.
constexpr int kDeepK = 9;
constexpr int kDeepDeg = 24;
constexpr int kDeepTriangles = kDeepDeg * (kDeepDeg - 1) * (kDeepDeg - 2) / 6;
constexpr int kLightSubs = 16;

// Place a query's launch items (n_items, item_lo, item_stride set) in the
// item spaces, after those placed before.  Without `dense` the count kernel
// takes them all.
inline void place_query(QueryDesc& q, bool dense, int32_t* space_items)
{
    int64_t before = 0;
    for (int s = 0; s < kSpaces; ++s) {
        int64_t upto = q.n_items;
        if (s < kRestSpace) {
            // launch items j with item_lo + j * item_stride < sched_end[s]
            const int64_t end = dense && !q.arc_list ? q.sched_end[s] : 0;
            upto = end > q.item_lo ? (end - q.item_lo + q.item_stride - 1) / q.item_stride : 0;
            if (upto > q.n_items) upto = q.n_items;
        }
        q.space_off[s] = (int32_t)before;
        q.space_begin[s] = space_items[s];
        space_items[s] += (int32_t)(upto - before);
        before = upto;
    }
}

}  // namespace citron
