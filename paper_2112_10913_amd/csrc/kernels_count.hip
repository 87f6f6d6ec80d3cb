// Counting phase of the degree-ordered k-clique counter (Lonkar & Beamer,
// Section III Algorithm 2, Section V-B heuristics), as one persistent HIP
// kernel for gfx950.
//
// Input: the subgraph rows built once per graph (kernels_rows.hip): for an
// arc u -> v_i, row i of u is the candidate mask C_uv over the positions of
// N->(u).  The k-cliques whose two lowest vertices (in the degree ordering)
// are u and v_i are the (k-2)-cliques of the subgraph induced on C_uv; they
// are counted by depth-first recursion over masks M' = M AND row_x, with the
// last level summing popcounts only (degrees-only heuristic) and masks too
// small for the rest of the clique pruned (size heuristic).
//
// Scheduling.  Every wave works on its own and claims runs of items from a
// few global cursors, in order of cost: the arcs of heavy vertices
// (out-degree > 64) by |C_uv| and the light vertices (out-degree <= 64),
// largest first.  The items of a run are decoded side by side, a lane each.
//
// Engines.  Light work -- subgraphs with at most 64 vertices, one 64-bit
// word per row -- is searched by the light engine: one depth-first search
// per lane (a whole arc, or one branch below an arc in deep counts), rows in
// the wave's LDS
// buffer, stacks in registers (k <= 7), LDS (k <= 12) or device memory.
// A heavy arc is walked by the whole wave in step (lane q holding word q of
// each mask).  A node with at most 256 candidates is copied to the wave's
// LDS, compacted to ceil(c/64) words per row; a node with at most 64
// candidates is compacted to one word per row and queued for the light
// engine; a node with two levels left and more than 64 candidates is
// finished lane-per-child from the LDS copy (need3_lanes).
//
// Exact arithmetic: per-lane uint64 accumulators (lane_sum.h: small additions
// as they are, the binomials of complete nodes through a carry check that
// leaves room for them; 32-bit partial sums are bounded where they are
// used); wave sums and the global accumulator are carry-checked, and a carry
// sets the query's overflow flag.
#include "items.h"
#include "lane_sum.h"
#include "wave.h"

namespace citron {

constexpr int kMaxBlock = 512;          // threads per count workgroup (8 waves)
constexpr int kWaveBufRows = 128;       // one-word rows queued per wave
constexpr int kLdsStackLevels = 7;      // deeper stacks (k > 12) live in device memory
constexpr int kArcMaxC = kArcLdsMax;    // LDS subgraph copies hold at most this many rows
constexpr int kDonateMinIdle = 16;      // idle lanes that trigger work donation
// A unit with at least this many vertices to choose is dealt branch by branch:
// a wave's queue holds few units of a deep count (two arcs per part of a split
// vertex), which kept lanes idle or trading work.  Units of less than
// kBranchMin candidates are dealt whole where the stacks are deep enough
// (below heavy nodes): such units come many at a time.
constexpr int kBranchNeed = 4;
constexpr int kBranchMin = 24;
// A node with at least this many vertices to choose has its edges counted
// before it is searched: when every pair is adjacent its count is a binomial.
// The probe costs one word operation per candidate, against a subtree of
// about c^3 / 24 in a dense subgraph; in graphs with planted cliques most
// such nodes are complete (Chung-Lu 2^14, k = 9: 12.0 -> 6.4 ms; R-MAT 16,
// k = 7, where they hardly ever are: no change).  A wave goes on probing
// while one node in kProbeRate is complete, after kProbeTrial tries; later it
// tries kProbeAgain more per queue.
constexpr int kProbeNeed = 4;
constexpr int kProbeTrial = 256;
constexpr int kProbeRate = 16;
constexpr int kProbeAgain = 8;
constexpr int kDeepClaim = 8;           // items a wave claims at once, at most, for k >= 7
constexpr int kBurstIters = 32;         // last-level steps of one leaf burst at most
constexpr int kBurstMinLanes = 32;      // lanes at a last-level node to keep a burst going
constexpr int kN3Burst = 8;             // two-level steps between refills of idle lanes
// donation mailbox per lane: M, R, (need, base), and the arc tag of per-arc launches
__host__ __device__ constexpr int mbox_words(bool per_arc) { return per_arc ? 4 : 3; }
constexpr int kPosList = 3 * kWave * 2; // candidate positions the smaller mailbox area holds (1.5 KB)
static_assert(kArcMaxC <= kPosList, "candidate positions of an LDS node fit the mailbox area");

// ------------------------------------------------------------------ layout

// Open levels of a heavy search (nodes with 3 .. k - 2 vertices to choose) and
// of a light one, which starts a branch below its unit.
__host__ __device__ inline int heavy_levels(int max_k) { return max_k > 4 ? max_k - 4 : 1; }
__host__ __device__ inline int light_levels(int max_k) { return max_k > 6 ? max_k - 5 : 1; }

// Where the light stacks live, by the largest k of a launch: registers (one
// level for k <= 6, two for k = 7), LDS (k <= 12) or device memory.  Each
// access to registers selects among the levels, since the lanes sit at
// different depths: with four, 16 selects a push, k = 8 of G(70, 0.8) took 1.88
// ms, with LDS 1.44 (R-MAT 12: 11.1 and 9.4 ms).  The heavy stacks are always in
// device memory: they are touched only when a heavy node is pushed or popped,
// and keeping them out of LDS lets more waves share a CU.
constexpr int kRegLevels = 2;
enum StackMode { kStackOne, kStackReg, kStackLds, kStackGlobal };
__host__ __device__ inline int stack_mode(int max_k)
{
    const int l = light_levels(max_k);
    return l <= 1 ? kStackOne : l <= kRegLevels ? kStackReg : (l <= kLdsStackLevels ? kStackLds : kStackGlobal);
}
// device-memory stack words per wave: heavy M and R, and for the deepest
// counts light M and R in as many levels
__host__ __device__ inline int64_t wave_global_stack_words(int max_k)
{
    return (stack_mode(max_k) == kStackGlobal ? 4ll : 2ll) * heavy_levels(max_k) * kWave;
}

// Largest LDS subgraph copy of a launch: nodes with 64 < c <= arc_max
// candidates, ceil(arc_max / 64) words per row.
__host__ __device__ inline int clamp_arc_max(int arc_max)
{
    return arc_max < kWave ? kWave : (arc_max > kArcMaxC ? kArcMaxC : arc_max);
}
__host__ __device__ inline int arc_copy_words(int arc_max)
{
    const int a = clamp_arc_max(arc_max);
    return a * ((a + 63) / 64);
}

// Per-wave LDS, in this order: queued rows (u64), their meta (i32), their
// arc tags (i32, per-arc launches only), the subgraph copy (u64), the
// donation mailbox (u64 per lane), the unit list (i32), the claimed items
// (i32 fields), the stacks kept in LDS.  Every part starts 8-byte aligned; the size is rounded to 16 bytes.
// The LDS per wave bounds the waves per CU (160 KB per CU), and the count
// kernel is latency-bound, so the layout is sized by what a launch uses.
__host__ __device__ inline int wave_lds_bytes(int max_k, int arc_max, bool per_arc)
{
    int b = 8 * kWaveBufRows + 4 * kWaveBufRows + (per_arc ? 4 * kWaveBufRows : 0);
    b += 8 * arc_copy_words(arc_max);
    b += 8 * mbox_words(per_arc) * kWave;
    b += 4 * kWaveBufRows;
    b += 4 * kItFields * kMaxClaim;
    if (stack_mode(max_k) == kStackLds) b += 8 * 2 * light_levels(max_k) * kWave;
    return (b + 15) & ~15;
}

// ------------------------------------------------------------ light engine
//
// Depth-first search with one 64-bit mask per level and one independent
// search per lane.  A unit is one row of a queued subgraph: choosing the
// row's vertex leaves `need` more vertices to choose from the row's mask.
// A lane that finishes a unit takes the next one at once.

struct Acc {
    u64 acc;             // with ovf, the lane's sum (lane_sum.h)
    int ovf;
    u64 st[kNumStats];   // per-lane work counters (instrumented launches only)
};

struct WaveBuf {
    u64* arc;        // LDS copy of one heavy arc's subgraph (multi-word rows)
    u64* mbox;       // donation mailbox: per lane M, R, and (need, base, tag)
    u64* rows;
    int32_t* meta;   // (first row of the subgraph << 8) | need
    int32_t* tags;   // arc of the unit (per-arc output)
    u64* sM;         // light stacks
    u64* sR;
    u64* hM;         // heavy stacks
    u64* hR;
    int32_t* units;  // search roots: row | sub-part << 8 | (one of kLightSubs sub-parts) << 16
    int n;           // rows in use (wave-uniform)
    int nu;          // units in use (wave-uniform)
    int arc_max;     // nodes with 64 < c <= arc_max are copied to LDS
    int whole_need;  // the light stacks hold units of up to this many vertices to choose whole
    int tried, hits; // probed nodes, and complete ones among them (wave-uniform)
};

// Per-lane light stack: slot s holds the (M, R) pair of level s + 1.  In
// registers (L > 0 levels) or in memory, one word per lane per level.
template <int L>
struct LightStack;

template <>
struct LightStack<2> {
    u64 m0 = 0, m1 = 0, r0 = 0, r1 = 0;
    __device__ __forceinline__ LightStack(const WaveBuf&) {}
    __device__ __forceinline__ void put(int s, u64 M, u64 R)
    {
        m0 = s == 0 ? M : m0;
        m1 = s == 0 ? m1 : M;
        set_r(s, R);
    }
    __device__ __forceinline__ void set_r(int s, u64 R)
    {
        r0 = s == 0 ? R : r0;
        r1 = s == 0 ? r1 : R;
    }
    __device__ __forceinline__ u64 get_m(int s) const { return s == 0 ? m0 : m1; }
    __device__ __forceinline__ u64 get_r(int s) const { return s == 0 ? r0 : r1; }
};
static_assert(kRegLevels == 2, "LightStack<2> holds the register levels");

template <>
struct LightStack<1> {
    u64 m = 0, r = 0;
    __device__ __forceinline__ LightStack(const WaveBuf&) {}
    __device__ __forceinline__ void put(int, u64 M, u64 R)
    {
        m = M;
        r = R;
    }
    __device__ __forceinline__ void set_r(int, u64 R) { r = R; }
    __device__ __forceinline__ u64 get_m(int) const { return m; }
    __device__ __forceinline__ u64 get_r(int) const { return r; }
};

template <>
struct LightStack<0> {
    u64* __restrict__ sM;
    u64* __restrict__ sR;
    int lane;
    __device__ __forceinline__ LightStack(const WaveBuf& wb) : sM(wb.sM), sR(wb.sR), lane(lane_of()) {}
    __device__ __forceinline__ void put(int s, u64 M, u64 R)
    {
        sM[s * kWave + lane] = M;
        sR[s * kWave + lane] = R;
    }
    __device__ __forceinline__ void set_r(int s, u64 R) { sR[s * kWave + lane] = R; }
    __device__ __forceinline__ u64 get_m(int s) const { return sM[s * kWave + lane]; }
    __device__ __forceinline__ u64 get_r(int s) const { return sR[s * kWave + lane]; }
};

// C(n, r) for n <= 64 and r <= 30 (k <= 32, two vertices chosen by the arc):
// below 2^61.
struct Binomials {
    u64 c[kWave + 1][kKMax - 1];
};
constexpr Binomials make_binomials()
{
    Binomials b = {};
    for (int n = 0; n <= kWave; ++n)
        for (int r = 0; r < kKMax - 1; ++r)
            b.c[n][r] = r == 0 ? 1 : (n == 0 ? 0 : b.c[n - 1][r - 1] + b.c[n - 1][r]);
    return b;
}
__device__ const Binomials binomials = make_binomials();

// One degrees-only step on a last-level node: the next two candidates x of
// R (R != 0) leave R, and the result is the sum of popcount(M AND row_x).
// Without a second candidate the first row is read twice and counted once
// (no branch).
__device__ __forceinline__ unsigned leaf_step(const u64* __restrict__ rows, int base, u64 M, u64& R)
{
    const int x1 = __builtin_ctzll(R);
    R &= R - 1;
    const bool two = R != 0ull;
    const int x2 = two ? __builtin_ctzll(R) : x1;
    R &= R - 1;                        // stays 0 when it was 0
    const u64 r1 = rows[base + x1];
    const u64 r2 = rows[base + x2];
    return (unsigned)__popcll(M & r1) + (two ? (unsigned)__popcll(M & r2) : 0u);
}

template <bool kStats, bool kPerArc, int kRegL>
__device__ __forceinline__ void light_engine(WaveBuf& wb, Acc& A, u64* __restrict__ per_arc)
{
    const int lane = lane_of();
    const u64 lt_mask = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    const u64* __restrict__ rows = wb.rows;
    LightStack<kRegL> stk(wb);
    constexpr bool kProbe = kRegL != 1;   // k <= 6 has no node that is probed
    const int nunits = wb.nu;
    int next = 0;                      // wave-uniform unit counter
    u64 branches = 0ull;               // first-level branches left of the unit before it (wave-uniform)
    int urow = 0, uneed = 0, ubase = 0;
    int tried = 0, hits = 0;           // probes and complete nodes among them (wave-uniform)
    if (kProbe) {
        tried = wb.tried > kProbeTrial ? wb.tried - kProbeAgain : wb.tried;
        hits = wb.hits;
    }
    bool active = false;
    int scan = 0;                      // 1 at a last-level node, or counting a node's edges before searching it
    unsigned sum = 0;                  // of the node scanned: cliques, or edges (below 2^12)
    u64 M = 0, R = 0, uacc = 0;
    int t = 0, need = 0, base = 0, tag = 0;
    auto probes = [&](int n) { return kProbe && n >= kProbeNeed && tried <= kProbeTrial + kProbeRate * hits; };
    for (;;) {
        u64 want = __ballot(!active);
        while (want && (branches || next < nunits)) {
            if (branches == 0ull) {
                // the next units, a wanting lane each, up to the first that is
                // dealt branch by branch; units too small for the rest of the
                // clique are passed over
                const int u = next + __popcll(want & lt_mask);
                const bool mine = !active && u < nunits;
                const int uw = wb.units[min(u, nunits - 1)];
                const int row = uw & 0xff;
                const int mt = wb.meta[row];
                const u64 m1 = rows[row];
                const int n = mt & 255, c = __popcll(m1);
                const bool viable = mine && c >= n;
                const u64 deal = __ballot(viable && n >= kBranchNeed &&
                                           (c >= kBranchMin || n > wb.whole_need || uw >> 16));
                const u64 take = deal ? want & ((1ull << __builtin_ctzll(deal)) - 1ull) : want;
                next += deal ? __popcll(take) + 1 : __popcll(take);
                if (viable && ((take >> lane) & 1)) {
                    base = mt >> 8;
                    need = n;
                    if (kStats) A.st[kStatLightUnits] += 1;
                    if (kPerArc) tag = wb.tags[row];
                    if (n == 1) {
                        A.acc += (u64)c;
                        if (kPerArc && c) atomicAdd(per_arc + tag, (u64)c);
                    } else {
                        M = m1;
                        R = m1;
                        t = 1;
                        scan = n == 2 || probes(n);
                        uacc = 0;
                        active = true;
                    }
                }
                if (deal) {
                    const int l = __builtin_ctzll(deal);
                    const int uwl = __builtin_amdgcn_readlane(uw, l), mtl = __builtin_amdgcn_readlane(mt, l);
                    urow = uwl & 0xff;
                    uneed = mtl & 255;
                    ubase = mtl >> 8;
                    // a sub-part takes the branches at positions q mod kLightSubs
                    static_assert(kLightSubs == 16, "mask of every 16th position");
                    branches = readlane64(m1, l) & ((uwl >> 16 ? 0x0001000100010001ull : ~0ull) << ((uwl >> 8) & 0xff));
                }
            } else {
                const int r = __popcll(want & lt_mask);
                const int left = __popcll(branches);
                const u64 m1 = readlane64(rows[urow], 0);
                if (!active && r < left) {
                    const u64 nm = m1 & rows[ubase + select64(branches, r)];
                    if (kStats) A.st[kStatLightUnits] += 1;
                    if (__popcll(nm) >= uneed - 1) {
                        M = nm;
                        R = nm;
                        t = 1;
                        need = uneed - 1;
                        base = ubase;
                        scan = probes(need);
                        if (kPerArc) tag = wb.tags[urow];
                        uacc = 0;
                        active = true;
                    }
                }
                const int taken = __popcll(want);
                if (taken >= left) {
                    branches = 0ull;
                } else {
                    const int last = __builtin_amdgcn_readfirstlane(select64(branches, taken - 1));
                    branches &= ~0ull << last << 1;
                }
            }
            want = __ballot(!active);
        }
        const u64 act = __ballot(active);
        if (act == 0ull) {
            break;               // no lane holds work and no unit is left
        }
        if (next >= nunits && branches == 0ull && __popcll(~act) >= kDonateMinIdle) {
            // work donation: no unit is left and lanes are idle, so every busy
            // lane offers the upper half of the remaining candidates of its
            // shallowest level that still holds real work; idle lanes take
            // them as new search roots (counts only depend on the subtree)
            int lvl = 0;
            u64 Ml = 0ull, Rl = 0ull;
            if (active) {
                // (what a probe has left is no part of the search)
                for (int l = 1; l <= t - (scan != 0 && need != 2 ? 1 : 0); ++l) {
                    const u64 r = (l == t) ? R : stk.get_r(l - 1);
                    const int pc = __popcll(r);
                    if (pc >= 2 && (need + (t - l) >= 3 || pc >= 8)) {
                        lvl = l;
                        Rl = r;
                        Ml = (l == t) ? M : stk.get_m(l - 1);
                        break;
                    }
                }
            }
            const u64 donors = __ballot(lvl > 0);
            if (donors) {
                const u64 idle = ~act;
                const int np = min(__popcll(donors), __popcll(idle));
                if (lvl > 0) {
                    const int r = __popcll(donors & lt_mask);
                    if (r < np) {
                        const int recv = select64(idle, r);
                        const int p = select64(Rl, __popcll(Rl) / 2);
                        const u64 low = Rl & ((1ull << p) - 1);
                        if (lvl == t) R = low;
                        else stk.set_r(lvl - 1, low);
                        u64* mb = wb.mbox + mbox_words(kPerArc) * recv;
                        mb[0] = Ml;
                        mb[1] = Rl & ~low;
                        mb[2] = ((u64)(unsigned)base << 32) | (unsigned)(need + (t - lvl));
                        if (kPerArc) mb[3] = (u64)(unsigned)tag;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (!active && __popcll(idle & lt_mask) < np) {
                    const u64* mb = wb.mbox + mbox_words(kPerArc) * lane;
                    M = mb[0];
                    R = mb[1];
                    need = (int)(unsigned)mb[2];
                    base = (int)(mb[2] >> 32);
                    if (kPerArc) tag = (int)(unsigned)mb[3];
                    t = 1;
                    uacc = 0;
                    active = true;
                    scan = need == 2;
                    if (kStats) A.st[kStatDonations] += 1;
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        if (kStats && lane == 0) {
            A.st[kStatLightIters] += 1;
            A.st[kStatLightActive] += (u64)__popcll(act);
        }
        bool probed = false, complete = false;
        if (active) {
            if (R != 0ull) {
                if (scan) {
                    // degrees-only last level (or a probe's edge count), two
                    // candidates per step
                    sum += leaf_step(rows, base, M, R);
                    if (kStats) A.st[kStatWordOps] += 2;
                } else {
                    const int x = __builtin_ctzll(R);
                    R &= R - 1;
                    const u64 nm = M & rows[base + x];
                    if (__popcll(nm) >= need - 1) {
                        stk.put(t - 1, M, R);
                        M = nm;
                        R = nm;
                        ++t;
                        --need;
                        scan = need == 2 || probes(need);
                        if (kStats) A.st[kStatPushes] += 1;
                    }
                }
            }
            if (scan && R != 0ull) {
                // leaf burst: while most lanes scan a node, run only such
                // steps, two candidates at a time
                for (int it = 0; it < kBurstIters; ++it) {
                    const bool leaf = R != 0ull;
                    if (__popcll(__ballot(leaf)) < kBurstMinLanes) break;
                    if (leaf) {
                        sum += leaf_step(rows, base, M, R);
                        if (kStats) A.st[kStatWordOps] += 2;
                    }
                }
            }
            if (R == 0ull) {
                if (kProbe && scan && need != 2) {
                    // every pair adjacent: the node's cliques are its subsets
                    // of `need`; otherwise it is searched
                    const int c = __popcll(M);
                    probed = true;
                    complete = 2 * sum == (unsigned)(c * (c - 1));
                    if (complete) {
                        const u64 b = binomials.c[c][need];
                        add_big(A.acc, A.ovf, b);
                        if (kPerArc) uacc += b;
                    } else {
                        R = M;
                    }
                } else {
                    A.acc += (u64)sum;         // 0 unless the node was scanned
                    if (kPerArc) uacc += (u64)sum;
                }
                scan = false;
                sum = 0;
            }
            if (R == 0ull) {
                if (t == 1) {
                    active = false;
                    if (kPerArc && uacc) atomicAdd(per_arc + tag, uacc);
                } else {
                    --t;
                    ++need;
                    if (kStats) A.st[kStatLightPops] += 1;
                    M = stk.get_m(t - 1);
                    R = stk.get_r(t - 1);
                }
            }
        }
        if (kProbe) {
            const u64 p = __ballot(probed);
            if (p) {
                tried += __popcll(p);
                hits += __popcll(__ballot(complete));
                if (tried > 16 * kProbeTrial) {
                    tried >>= 1;
                    hits >>= 1;
                }
            }
        }
    }
    if (kProbe) {
        wb.tried = tried;
        wb.hits = hits;
    }
}

template <bool kStats, bool kPerArc, int kRegL>
__device__ __forceinline__ void flush_tasks(WaveBuf& wb, Acc& A, u64* per_arc)
{
    if (wb.n == 0) return;
    if (kStats && lane_of() == 0) A.st[kStatFlushes] += 1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const u64 c0 = kStats ? __builtin_readcyclecounter() : 0ull;
    light_engine<kStats, kPerArc, kRegL>(wb, A, per_arc);
    if (kStats && lane_of() == 0) A.st[kStatCycLight] += __builtin_readcyclecounter() - c0;
    __builtin_amdgcn_wave_barrier();
    wb.n = 0;
    wb.nu = 0;
}

// ------------------------------------------------------------ heavy engine

typedef __attribute__((address_space(3))) u64 lds_u64;
typedef __attribute__((address_space(3))) int32_t lds_i32;
typedef __attribute__((address_space(1))) const u64 glb_u64;
typedef __attribute__((address_space(1))) const unsigned char glb_u8;

// Rows of a heavy subgraph: the source vertex's rows in device memory
// (kGlobal), addressed with 32-bit offsets from a wave-uniform base, or a
// compacted copy in the wave's LDS.
template <bool kGlobal>
struct RowRef;
template <>
struct RowRef<true> {
    glb_u64* p;
    __device__ __forceinline__ u64 operator()(unsigned i) const
    {
        return *reinterpret_cast<glb_u64*>(reinterpret_cast<glb_u8*>(p) + (i << 3));
    }
};
template <>
struct RowRef<false> {
    const lds_u64* p;
    __device__ __forceinline__ u64 operator()(unsigned i) const { return p[i]; }
};

template <bool kGlobal>
struct HeavyCtx {
    RowRef<kGlobal> rows;
    int W;     // words per row
    int L;     // vertices of the clique inside the subgraph (k - 1)
    int tag;   // the arc (per-arc output)
};

// Row x of H restricted to the candidates of M (lane q holds word q of M)
// and packed: bit i of the result is candidate i.  At most 256 candidates
// (four words o0..o3).  Uniform control flow: the whole wave calls it.
template <bool kGlobal>
__device__ __forceinline__ void pack_row(const HeavyCtx<kGlobal>& H, u64 M, int x, bool valid, u64& o0, u64& o1,
                                         u64& o2, u64& o3)
{
    o0 = o1 = o2 = o3 = 0ull;
    const unsigned base = valid ? (unsigned)(x * H.W) : 0u;
    int off = 0;
    for (int w0 = 0; w0 < H.W; w0 += 4) {
        // four source words in flight at a time
        u64 src[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) src[i] = (valid && w0 + i < H.W) ? H.rows(base + w0 + i) : 0ull;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (w0 + i >= H.W) break;
            const u64 mw = readlane64(M, w0 + i);
            if (mw == 0ull) continue;
            const u64 p = pext_apply(src[i], pext_prep(mw));
            const int wi = off >> 6, sh = off & 63;
            const u64 lo = p << sh;
            const u64 hi = sh ? (p >> (64 - sh)) : 0ull;
            // wi is wave-uniform; selects keep o0..o3 in registers
            o0 |= wi == 0 ? lo : 0ull;
            o1 |= (wi == 1 ? lo : 0ull) | (wi == 0 ? hi : 0ull);
            o2 |= (wi == 2 ? lo : 0ull) | (wi == 1 ? hi : 0ull);
            o3 |= (wi == 3 ? lo : 0ull) | (wi == 2 ? hi : 0ull);
            off += __popcll(mw);
        }
    }
}

// Copy the subgraph induced on the c candidates of M to dst in LDS,
// compacted to W2 = ceil(c / 64) words per row; c <= kArcMaxC.
__device__ __forceinline__ int copy_to_lds(const HeavyCtx<true>& H, u64 M, int c, lds_u64* dst)
{
    const int q = lane_of();
    const int W2 = (c + 63) >> 6;
    for (int a0 = 0; a0 < c; a0 += kWave) {
        const int a = a0 + q;
        const int xa = wave_select(M, a, H.W);
        u64 o0, o1, o2, o3;
        pack_row<true>(H, M, xa, a < c, o0, o1, o2, o3);
        if (a < c) {
            lds_u64* d = dst + a * W2;
            d[0] = o0;
            if (W2 > 1) d[1] = o1;
            if (W2 > 2) d[2] = o2;
            if (W2 > 3) d[3] = o3;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return W2;
}

// Two levels left on a node of the LDS copy with more than 64 candidates
// (W words per row, W = 2..4): every lane takes a candidate x, forms its
// child mask m AND row_x in registers and sums the last level of that
// child itself, two vertices y of the child per step; a lane that finishes
// takes the next candidate (positions listed in pos), so lanes stay busy
// however uneven the children are.  Returns this lane's sum (< 2^24).
template <int W, bool kStats>
__device__ __forceinline__ unsigned need3_lanes(const HeavyCtx<false>& H, const u64* mw, int nj,
                                                const lds_i32* pos, unsigned& took, unsigned& ops)
{
    const int lane = lane_of();
    const u64 lt = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    int next = 0;                 // wave-uniform: candidates handed out
    bool act = false;
    u64 ch[W];
#pragma unroll
    for (int i = 0; i < W; ++i) ch[i] = 0ull;
    u64 r = 0ull;
    int w = 0;
    unsigned sum = 0;
    for (;;) {
        const u64 idle = __ballot(!act);
        if (next < nj && (__popcll(idle) >= 8 || idle == ~0ull)) {
            const int jj = next + __popcll(idle & lt);
            next += __popcll(idle);
            if (!act && jj < nj) {
                const unsigned b = (unsigned)(pos[jj] * W);
#pragma unroll
                for (int i = 0; i < W; ++i) ch[i] = mw[i] & H.rows(b + i);
                r = ch[0];
                w = 0;
                act = true;
                if (kStats) ++took;
            }
        } else if (idle == ~0ull) {
            break;
        }
        // a burst of steps between refills: lanes that finish early wait
        // for the next refill (at most kN3Burst - 1 steps)
        for (int it = 0; it < kN3Burst; ++it) {
            if (act) {
                if (r == 0ull) {
#pragma unroll
                    for (int i = 1; i < W; ++i)
                        if (r == 0ull && w < i) {
                            w = i;
                            r = ch[i];
                        }
                    if (r == 0ull) act = false;
                }
            }
            if (act) {
                const int y1 = w * 64 + __builtin_ctzll(r);
                r &= r - 1;
                const bool two = r != 0ull;   // a second vertex of the same word
                const int y2 = two ? w * 64 + __builtin_ctzll(r) : y1;
                if (two) r &= r - 1;
                const unsigned b1 = (unsigned)(y1 * W), b2 = (unsigned)(y2 * W);
                u64 a1[W], a2[W];
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    a1[i] = H.rows(b1 + i);
                    a2[i] = H.rows(b2 + i);
                }
                unsigned c1 = 0, c2 = 0;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    c1 += __popcll(ch[i] & a1[i]);
                    c2 += __popcll(ch[i] & a2[i]);
                }
                sum += c1 + (two ? c2 : 0u);
                if (kStats) ops += two ? 2 * W : W;
            }
        }
    }
    return sum;
}

template <bool kStats, bool kPerArc, bool kGlobal, int kRegL>
__device__ __forceinline__ void heavy_search(const HeavyCtx<kGlobal>& H, u64 ch, int need0, int lvl0, int part, int P,
                                             WaveBuf& wb, Acc& A, u64& uacc, u64* per_arc);

// Handle a node with mask m (c candidates, `need` more vertices to choose;
// rows in device memory when kGlobal, else in the wave's LDS copy).  Returns
// true when the caller must search it depth first.  lvl is the first free
// level of the heavy stacks.  Only first-level branches j = part (mod P)
// of the node are taken; P > 1 only at the root of a split arc, which has
// need >= 4 (arc_parts is 1 for k <= 5).
template <bool kStats, bool kPerArc, bool kGlobal, int kRegL>
__device__ __forceinline__ bool heavy_node(const HeavyCtx<kGlobal>& H, u64 m, int c, int need, int lvl, int part,
                                           int P, WaveBuf& wb, Acc& A, u64& uacc, u64* per_arc)
{
    const int lane = lane_of();
    if (c < need) return false;
    if (need == 1) {
        if (lane == 0) {
            A.acc += (u64)c;
            if (kPerArc) uacc += (u64)c;
        }
        return false;
    }
    if (need == 2) {
        // degrees-only last level on multi-word rows: lanes over candidates
        for (int j0 = 0; j0 < c; j0 += kWave) {
            const int j = j0 + lane;
            const int x = wave_select(m, j, H.W);
            unsigned s = 0;
            const unsigned b = (unsigned)((j < c ? x : 0) * H.W);
            for (int w = 0; w < H.W; ++w) {
                const u64 mw = readlane64(m, w);
                if (j < c && mw) s += __popcll(mw & H.rows(b + w));
            }
            A.acc += (u64)s;
            if (kPerArc) uacc += (u64)s;
            if (kStats && j < c) {
                A.st[kStatWordOps] += H.W;
                A.st[kStatHeavyLeafCand] += 1;
            }
        }
        return false;
    }
    if constexpr (kGlobal) {
    if (c <= wb.arc_max && c > kWave) {
        // continue from an LDS copy of this node's subgraph
        const u64 c0 = kStats ? __builtin_readcyclecounter() : 0ull;
        lds_u64* arc = (lds_u64*)wb.arc;
        const int W2 = copy_to_lds(H, m, c, arc);
        if (kStats && lane == 0) A.st[kStatCycCopy] += __builtin_readcyclecounter() - c0;
        const HeavyCtx<false> HL{RowRef<false>{arc}, W2, H.L, H.tag};
        const int rem = c - 64 * lane;
        const u64 all = lane < W2 ? (rem >= 64 ? ~0ull : ((1ull << rem) - 1)) : 0ull;
        if (kStats && lane == 0) A.st[kStatArcLds] += 1;
        heavy_search<kStats, kPerArc, false, kRegL>(HL, all, need, lvl, part, P, wb, A, uacc, per_arc);
        __builtin_amdgcn_wave_barrier();
        return false;
    }
    }
    if constexpr (!kGlobal) {
    if (need == 3 && c > kWave) {
        const u64 c0 = kStats ? __builtin_readcyclecounter() : 0ull;
        const int nj = (c - part + P - 1) / P;
        // positions of the candidates taken, in the mailbox area (idle while
        // the light engine is not running); nj <= c <= arc_max <= kArcMaxC <= kPosList
        lds_i32* pos = (lds_i32*)wb.mbox;
        for (int j0 = 0; j0 < nj; j0 += kWave) {
            const int jj = j0 + lane;
            const int x = wave_select(m, jj < nj ? part + P * jj : c, H.W);
            if (jj < nj) pos[jj] = x;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        u64 mw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mw[i] = i < H.W ? readlane64(m, i) : 0ull;
        unsigned took = 0, ops = 0, sum;
        if (H.W == 2) sum = need3_lanes<2, kStats>(H, mw, nj, pos, took, ops);
        else if (H.W == 3) sum = need3_lanes<3, kStats>(H, mw, nj, pos, took, ops);
        else sum = need3_lanes<4, kStats>(H, mw, nj, pos, took, ops);
        if (kStats) {
            A.st[kStatNeed3MinOps] += (u64)(ops / H.W) * (u64)((c + 63) >> 6);
            if (lane == 0) A.st[kStatNeed3Nodes] += 1;
        }
        __builtin_amdgcn_wave_barrier();
        A.acc += (u64)sum;
        if (kPerArc) uacc += (u64)sum;
        if (kStats) {
            A.st[kStatWordOps] += ops;
            A.st[kStatNeed3Lanes] += took;
            if (lane == 0) A.st[kStatCycNeed3] += __builtin_readcyclecounter() - c0;
        }
        return false;
    }
    }
    if (c <= kWave) {
        // compaction: lane a packs row a over the c candidates into one
        // word and the node goes to the light engine's queue
        if (wb.n + c > kWaveBufRows) flush_tasks<kStats, kPerArc, kRegL>(wb, A, per_arc);
        const u64 c0 = kStats ? __builtin_readcyclecounter() : 0ull;
        const int xa = wave_select(m, lane, H.W);
        u64 o0, o1, o2, o3;
        pack_row<kGlobal>(H, m, xa, lane < c, o0, o1, o2, o3);
        if (lane < c) {
            wb.rows[wb.n + lane] = o0;
            wb.meta[wb.n + lane] = (wb.n << 8) | (need - 1);
            if (kPerArc) wb.tags[wb.n + lane] = H.tag;
        }
        const bool unit = lane < c && (P == 1 || lane % P == part);
        const u64 um = __ballot(unit);
        if (unit) wb.units[wb.nu + __popcll(um & (lane == 0 ? 0ull : (~0ull >> (kWave - lane))))] = wb.n + lane;
        wb.nu += __popcll(um);
        wb.n += c;
        if (kStats && lane == 0) {
            A.st[kStatCompactions] += 1;
            A.st[kStatCompactRows] += (u64)c;
            A.st[kStatCycCopy] += __builtin_readcyclecounter() - c0;
        }
        return false;
    }
    return true;
}

// Depth-first search, all lanes in step, of a node with mask ch (need0 more
// vertices to choose), rows in H; stack levels from lvl0.  One call site for
// every node, the root among them: the engines below a node are inlined
// there, and each further copy costs instruction cache and registers.
template <bool kStats, bool kPerArc, bool kGlobal, int kRegL>
__device__ __forceinline__ void heavy_search(const HeavyCtx<kGlobal>& H, u64 ch, int need0, int lvl0, int part, int P,
                                             WaveBuf& wb, Acc& A, u64& uacc, u64* per_arc)
{
    const int q = lane_of();
    u64 M = 0ull, R = 0ull;
    int t = 0;                 // open levels: M, R is level t's, the others' are on the stack
    int jroot = 0;
    for (;;) {
        const int cc = wave_sum_small(__popcll(ch));
        const bool root = t == 0;
        if (heavy_node<kStats, kPerArc, kGlobal, kRegL>(H, ch, cc, need0 - t, lvl0 + t, root ? part : 0, root ? P : 1,
                                                        wb, A, uacc, per_arc)) {
            if (t > 0) {
                wb.hM[(lvl0 + t - 1) * kWave + q] = M;
                wb.hR[(lvl0 + t - 1) * kWave + q] = R;
                if (kStats && q == 0) A.st[kStatPushes] += 1;
            }
            M = ch;
            R = ch;
            ++t;
        }
        // the next node: a child of the deepest open level with candidates left
        int x = -1;
        while (t > 0) {
            const u64 b = __ballot(R != 0ull);
            if (b == 0ull) {
                if (--t > 0) {
                    M = wb.hM[(lvl0 + t - 1) * kWave + q];
                    R = wb.hR[(lvl0 + t - 1) * kWave + q];
                }
                continue;
            }
            const int f = __builtin_ctzll(b);
            const u64 Rf = readlane64(R, f);
            if (q == f) R &= R - 1;
            if (t == 1) {
                const int jr = jroot++;
                if (P > 1 && jr % P != part) continue;
            }
            x = f * 64 + __builtin_ctzll(Rf);
            break;
        }
        if (x < 0) break;
        ch = M & (q < H.W ? H.rows((unsigned)(x * H.W + q)) : 0ull);
        if (kStats && q == 0) A.st[kStatHeavySteps] += 1;
    }
}

// --------------------------------------------------------------- the kernel

struct KParams {
    ItemSpace items;        // the items the dense kernel does not take
    u64* scratch;
    int64_t scratch_words;
    int32_t max_k;
    int32_t flush_rows;     // a wave runs its queue once it holds this many rows
    int32_t arc_lds_max;    // representation switch of heavy nodes (64..kArcMaxC)
    int32_t* progress;      // host-mapped word: items claimed, updated every 512 (nullable)
    int32_t progress_base;  // items the launch claimed before this kernel
};

template <int kMode, bool kStats, bool kPerArc>
__global__ void __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(kMode <= kStackReg ? 4 : kMode == kStackLds ? 3 : 2))) count_kernel(KParams P)
{
    constexpr int kRegL = kMode == kStackOne ? 1 : kMode == kStackReg ? kRegLevels : 0;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_of();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nwaves = blockDim.x / kWave;
    const int levels = heavy_levels(P.max_k);
    unsigned char* wbase = smem + wid * wave_lds_bytes(P.max_k, P.arc_lds_max, kPerArc);
    WaveBuf wb;
    int off = 0;
    wb.rows = reinterpret_cast<u64*>(wbase + off);
    off += 8 * kWaveBufRows;
    wb.meta = reinterpret_cast<int32_t*>(wbase + off);
    off += 4 * kWaveBufRows;
    wb.tags = reinterpret_cast<int32_t*>(wbase + off);     // per-arc launches only
    if (kPerArc) off += 4 * kWaveBufRows;
    wb.arc = reinterpret_cast<u64*>(wbase + off);
    off += 8 * arc_copy_words(P.arc_lds_max);
    wb.mbox = reinterpret_cast<u64*>(wbase + off);
    off += 8 * mbox_words(kPerArc) * kWave;
    wb.units = reinterpret_cast<int32_t*>(wbase + off);
    off += 4 * kWaveBufRows;
    int32_t* item = reinterpret_cast<int32_t*>(wbase + off);
    off += 4 * kItFields * kMaxClaim;
    u64* stacks = P.scratch + (int64_t)blockIdx.x * P.scratch_words + (int64_t)wid * wave_global_stack_words(P.max_k);
    wb.hM = stacks;
    wb.hR = stacks + (int64_t)levels * kWave;
    wb.sM = nullptr;
    wb.sR = nullptr;
    if (kMode == kStackLds) {
        wb.sM = reinterpret_cast<u64*>(wbase + off);
        wb.sR = wb.sM + light_levels(P.max_k) * kWave;
    } else if (kMode == kStackGlobal) {
        wb.sM = stacks + 2ll * levels * kWave;
        wb.sR = stacks + 3ll * levels * kWave;
    }
    wb.n = 0;
    wb.nu = 0;
    wb.arc_max = P.arc_lds_max;
    wb.whole_need = light_levels(P.max_k) + 2;
    wb.tried = 0;
    wb.hits = 0;

    Acc A;
    A.acc = 0ull;
    A.ovf = 0;
#pragma unroll
    for (int i = 0; i < kNumStats; ++i) A.st[i] = 0ull;
    int cur = -1;                      // query whose work the wave holds
    u64* per_arc = nullptr;
    const u64 t_start = kStats ? wall_clock64() : 0ull;
    const u64 cyc_start = kStats ? __builtin_readcyclecounter() : 0ull;
    if (kStats && lane == 0) {
        const u64 now = atomicAdd(P.items.queries[0].stats + kStatResidentNow, 1ull) + 1;
        atomicMax(P.items.queries[0].stats + kStatResidentMax, now);
    }
    u64 item_max = 0ull;

    const int wave = blockIdx.x * nwaves + wid;
    const int waves = gridDim.x * nwaves;
    const int acc_slot = (wave & (kAccSlots - 1)) * kAccStride;
    int shard = wave % kClaimShards;
    bool fresh = true;
    int g0 = 0, j = 0, nj = 0;         // the wave's run of items, decoded
    for (;;) {
        bool end = false;
        if (j >= nj) {
            g0 = claim_run(P.items, wave, waves, shard, fresh);
            end = g0 < 0;
            nj = end ? 0 : run_length(P.items, g0);
            j = 0;
            __builtin_amdgcn_wave_barrier();
            decode_run<kRestSpace>(P.items, g0, nj, item);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // progress for the host, read without any HIP call while the launch runs
            if (P.progress && !end && lane == 0 && (((g0 + nj - 1) ^ (g0 - 1)) & ~511))
                __hip_atomic_store(P.progress, P.progress_base + g0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        auto field = [&](int f) { return __builtin_amdgcn_readfirstlane(item[f * kMaxClaim + j]); };
        const int qi = end ? -1 : field(kItQuery);
        const int kind = end ? kItemHeavyArc : field(kItKind);
        const int d = end ? 0 : field(kItDegree);
        const bool heavy = kind != kItemLightVertex && kind != kItemDeepVertex && kind != kItemLightRoot;
        // run the queue before an item whose rows it cannot take, once it is
        // full enough, and before the query changes
        if (wb.n + (heavy ? 0 : d + 1) > kWaveBufRows || wb.n >= P.flush_rows || qi != cur) {
            flush_tasks<kStats, kPerArc, kRegL>(wb, A, per_arc);
            if (qi != cur) {
                if (cur >= 0) {
                    const QueryDesc& oq = P.items.queries[cur];
                    const u64 total = lane_total(A.acc, A.ovf);
                    wave_flush(total, A.ovf, oq.acc + acc_slot, oq.overflow);
                    if (kStats) wave_flush_stats(A.st, oq.stats);
                    A.acc = 0ull;
                    A.ovf = 0;
#pragma unroll
                    for (int i = 0; i < kNumStats; ++i) A.st[i] = 0ull;
                }
                if (end) break;
                cur = qi;
                per_arc = P.items.queries[qi].per_arc;
            }
        }
        if (end) break;
        const QueryDesc& q = P.items.queries[qi];
        const int k = q.k;
        const u64 t_item = kStats ? wall_clock64() : 0ull;
        const int r = field(kItRow), tag = field(kItTag), pw = field(kItPart);
        const int part = pw & 0xffff, nparts = pw >> 16;
        const u64* rows = q.rows.rows + field(kItRowsOff);
        const int g = g0 + j;
        if (heavy) {
            // a part of an arc, searched below its row, or (vertex-rooted
            // unit, Algorithm 2 per vertex) a whole vertex: all d positions
            // are candidates and its first level walks its arcs in turn
            const HeavyCtx<true> H{RowRef<true>{(glb_u64*)rows}, (d + 63) >> 6, k - 1, tag};
            const bool whole = kind == kItemHeavyVertex || kind == kItemDenseVertex;
            const int rem = d - 64 * lane;
            u64 M = 0ull;
            if (lane < H.W) {
                if (whole) M = rem >= 64 ? ~0ull : ((1ull << rem) - 1ull);
                else M = H.rows((unsigned)(r * H.W + lane));
            }
            u64 uacc = 0;
            heavy_search<kStats, kPerArc, true, kRegL>(H, M, whole ? H.L : H.L - 1, 0, part, nparts,
                                                       wb, A, uacc, per_arc);
            if (kPerArc) {
                const u64 s = wave_sum_u64(uacc);
                if (lane == 0 && s && tag >= 0) atomicAdd(per_arc + tag, s);
            }
        } else {
            // rows of the vertex into the wave's buffer; the searched arcs
            // (every nparts-th one, or the one listed) become units, or, for
            // a vertex-rooted light vertex, one unit rooted at the vertex
            // itself (mask of all d positions, k - 1 to choose)
            const bool from_root = kind == kItemLightRoot;
            if (lane < d) {
                wb.rows[wb.n + lane] = rows[lane];
                wb.meta[wb.n + lane] = (wb.n << 8) | (k - 2);
                if (kPerArc) wb.tags[wb.n + lane] = tag < 0 ? field(kItArc0) + lane : tag;
            }
            if (from_root && lane == 0) {
                wb.rows[wb.n + d] = d >= 64 ? ~0ull : ((1ull << d) - 1ull);
                wb.meta[wb.n + d] = (wb.n << 8) | (k - 1);
                wb.units[wb.nu] = wb.n + d;
            }
            // part = arc residue + light_arcs * sub-part
            const int subs = kind == kItemDeepVertex ? kLightSubs : 1;
            const int every = nparts / subs, sub = part / every;
            const bool unit = !from_root && lane < d && (r >= 0 ? lane == r : lane % every == part - sub * every);
            const u64 um = __ballot(unit);
            if (unit)
                wb.units[wb.nu + __popcll(um & (lane == 0 ? 0ull : (~0ull >> (kWave - lane))))] =
                    (wb.n + lane) | (sub << 8) | (subs > 1 ? 1 << 16 : 0);
            wb.nu += __popcll(um) + (from_root ? 1 : 0);
            wb.n += d + (from_root ? 1 : 0);
        }
        ++j;
        if (kStats && lane == 0) {
            const u64 dt = wall_clock64() - t_item;
            if (dt > (item_max >> 32)) item_max = (dt << 32) | (u64)(unsigned)g;
        }
    }
    if (kStats && lane == 0) {
        // wave timing (instrumented single-query launches)
        const u64 t_end = wall_clock64();
        u64* st = P.items.queries[0].stats;
        atomicAdd(st + kStatWaveBusy, t_end - t_start);
        atomicMin(st + kStatWaveFirst, t_start);
        atomicMax(st + kStatWaveLast, t_end);
        atomicAdd(st + kStatWaves, 1ull);
        atomicMax(st + kStatWaveBusyMax, t_end - t_start);
        atomicMax(st + kStatItemMax, item_max);
        atomicAdd(st + kStatCycTotal, __builtin_readcyclecounter() - cyc_start);
        atomicAdd(st + kStatResidentNow, ~0ull);   // minus one
    }
}

template <int kMode, bool kStats, bool kPerArc>
static hipError_t launch_variant(const KParams& P, const CountLaunch& cl, hipStream_t s)
{
    const void* fn = (const void*)count_kernel<kMode, kStats, kPerArc>;
    if (cl.lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, cl.lds_bytes);
        if (e != hipSuccess) return e;
    }
    count_kernel<kMode, kStats, kPerArc><<<cl.blocks, cl.wg_waves * kWave, cl.lds_bytes, s>>>(P);
    return hipGetLastError();
}

template <int kMode>
hipError_t launch_mode(const KParams& P, const CountLaunch& cl, hipStream_t s)
{
    const int v = (cl.stats ? 2 : 0) | (cl.per_arc ? 1 : 0);
    switch (v) {
    case 0: return launch_variant<kMode, false, false>(P, cl, s);
    case 1: return launch_variant<kMode, false, true>(P, cl, s);
    case 2: return launch_variant<kMode, true, false>(P, cl, s);
    default: return launch_variant<kMode, true, true>(P, cl, s);
    }
}

// One translation unit per stack mode, so that they compile side by side:
// this file by itself holds the host functions and the variants of k <= 6,
// and is included with CITRON_COUNT_UNIT set to another mode by
// kernels_count_reg.hip, kernels_count_lds.hip and kernels_count_deep.hip.
#ifdef CITRON_COUNT_UNIT
template hipError_t launch_mode<CITRON_COUNT_UNIT>(const KParams&, const CountLaunch&, hipStream_t);
#else
template hipError_t launch_mode<kStackOne>(const KParams&, const CountLaunch&, hipStream_t);
extern template hipError_t launch_mode<kStackReg>(const KParams&, const CountLaunch&, hipStream_t);
extern template hipError_t launch_mode<kStackLds>(const KParams&, const CountLaunch&, hipStream_t);
extern template hipError_t launch_mode<kStackGlobal>(const KParams&, const CountLaunch&, hipStream_t);

int64_t count_scratch_words(int32_t, int32_t max_k, int32_t wg_waves)
{
    return ((int64_t)wg_waves * wave_global_stack_words(max_k) + 31) & ~31ll;
}

int64_t count_deep_scratch_words(int32_t max_k, int32_t wg_waves)
{
    if (stack_mode(max_k) != kStackGlobal) return 0;
    return ((int64_t)wg_waves * wave_global_stack_words(max_k) + 31) & ~31ll;
}

int32_t count_lds_bytes(int32_t arc_max, int32_t max_k, int32_t wg_waves, bool per_arc)
{
    return wg_waves * wave_lds_bytes(max_k, arc_max, per_arc);
}

hipError_t launch_count(const CountLaunch& cl, hipStream_t s)
{
    if (launch_items(cl) <= 0) return hipSuccess;
    if (cl.wg_waves < 1 || cl.wg_waves * kWave > kMaxBlock) return hipErrorInvalidValue;
    // the dense arcs first (the costliest items of a launch), then the rest
    hipError_t e = launch_dense(cl, s);
    if (e != hipSuccess) return e;
    const int32_t rest = cl.space_items[kRestSpace];
    if (rest <= 0) return hipSuccess;
    KParams P;
    P.items.queries = cl.queries;
    P.items.n_queries = cl.n_queries;
    P.items.total = rest;
    P.items.cursors = cl.item_ctr + kRestSpace * kClaimInts;
    P.scratch = cl.scratch;
    P.scratch_words = cl.scratch_words;
    P.max_k = cl.max_k;
    // a wave runs its queue once it holds flush_rows rows (at most its buffer)
    P.flush_rows = cl.flush_rows > kWaveBufRows ? kWaveBufRows : cl.flush_rows;
    P.arc_lds_max = clamp_arc_max(cl.arc_lds_max);
    P.progress = cl.progress;
    P.progress_base = (int32_t)(launch_items(cl) - rest);
    // a launch is no wider than its items
    CountLaunch c2 = cl;
    const int64_t need = ((int64_t)rest + cl.wg_waves - 1) / cl.wg_waves;
    if (need < c2.blocks) c2.blocks = (int32_t)need;
    // deep counts: an item's cost is far from what its key says, so runs stay
    // shorter (Chung-Lu 2^17, k = 8, runs of 2, 4 and 8: 1.10, 0.87 and 0.74
    // ms, for their decoding; with planted cliques, k = 10, 1.23, 0.98 and 0.85;
    // R-MAT 12, k = 10, whose light vertices are deep, 73.3, 75.3 and 76.6)
    set_runs(P.items, (int64_t)c2.blocks * cl.wg_waves, cl.max_k <= 6 ? kMaxClaim : kDeepClaim);
    switch (stack_mode(cl.max_k)) {
    case kStackOne: return launch_mode<kStackOne>(P, c2, s);
    case kStackReg: return launch_mode<kStackReg>(P, c2, s);
    case kStackLds: return launch_mode<kStackLds>(P, c2, s);
    default: return launch_mode<kStackGlobal>(P, c2, s);
    }
}

__global__ void check_arcs_kernel(const int32_t* __restrict__ arcs, int32_t n, int64_t m, int32_t* __restrict__ err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && (arcs[i] < 0 || (int64_t)arcs[i] >= m)) atomicOr(err, 1);
}

__global__ void gather_arc_c_kernel(const int32_t* __restrict__ arcs, int32_t n, const int32_t* __restrict__ arc_c,
                                    u64* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (u64)arc_c[arcs[i]];
}

// parts of each listed arc (heavy sources split as in the full schedule)
__global__ void list_parts_kernel(const int32_t* __restrict__ arcs, int32_t n, const int32_t* __restrict__ dag_src,
                                  const int32_t* __restrict__ dag_ptr, const int32_t* __restrict__ arc_c, int32_t k,
                                  int32_t pct, int32_t* __restrict__ parts)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int e = arcs[i];
    const int u = dag_src[e];
    const int d = dag_ptr[u + 1] - dag_ptr[u];
    parts[i] = d > kLightMaxDeg ? arc_parts(arc_c[e], k, pct) : 1;
}

__global__ void list_items_kernel(int32_t n, const int32_t* __restrict__ parts, const int32_t* __restrict__ offs,
                                  int32_t* __restrict__ items)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int P = parts[i];
    const int o = offs[i];
    for (int p = 0; p < P; ++p) {
        items[2 * (o + p)] = (int32_t)i;
        items[2 * (o + p) + 1] = p | (P << 16);
    }
}

hipError_t launch_list_parts(const int32_t* arcs, int32_t n, const int32_t* dag_src, const int32_t* dag_ptr,
                             const int32_t* arc_c, int32_t k, int32_t pct, int32_t* parts, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    list_parts_kernel<<<(n + 255) / 256, 256, 0, s>>>(arcs, n, dag_src, dag_ptr, arc_c, k, pct, parts);
    return hipGetLastError();
}

hipError_t launch_list_items(int32_t n, const int32_t* parts, const int32_t* offs, int32_t* items, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    list_items_kernel<<<(n + 255) / 256, 256, 0, s>>>(n, parts, offs, items);
    return hipGetLastError();
}

hipError_t launch_check_arcs(const int32_t* arcs, int32_t n, int64_t m, int32_t* err, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    check_arcs_kernel<<<(n + 255) / 256, 256, 0, s>>>(arcs, n, m, err);
    return hipGetLastError();
}

hipError_t launch_gather_arc_c(const int32_t* arcs, int32_t n, const int32_t* arc_c, u64* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    gather_arc_c_kernel<<<(n + 255) / 256, 256, 0, s>>>(arcs, n, arc_c, out);
    return hipGetLastError();
}

__global__ void fill_i32_kernel(int32_t* p, int32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void fill_u64_kernel(u64* p, u64 v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    fill_i32_kernel<<<(unsigned)blocks, 256, 0, s>>>(p, v, n);
    return hipGetLastError();
}

hipError_t launch_fill_u64(u64* p, u64 v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    fill_u64_kernel<<<(unsigned)blocks, 256, 0, s>>>(p, v, n);
    return hipGetLastError();
}
#endif  // CITRON_COUNT_UNIT

}  // namespace citron
