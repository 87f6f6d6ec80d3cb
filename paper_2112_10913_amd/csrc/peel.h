// One step of the level-synchronous peeling, written once for the GPU
// (kernels_core.hip) and for a host that replays the workgroups of a launch in
// any order.
//
// Launch s of the peeling does the one phase that copy s & 1 of the control
// block names, and only its last workgroup writes: the other copy, which
// launch s + 1 reads.  So whenever a workgroup of launch s starts, also after
// the last one has set up the next phase, it reads the phase of its own launch
// and leaves if that phase has no work for it.  (With one copy a workgroup
// that started late, on a device busy with other streams, joined the next
// phase, which the next launch then did again.)  The counters are changed by
// the workgroups that the phase needs, and are not read by the others.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define PEEL_FN __device__ __forceinline__
#else
#define PEEL_FN inline
#endif

namespace citron {

enum PeelPhase { kPeelRelax, kPeelMark, kPeelMin, kPeelCollect, kPeelDone };
struct PeelCtl {
    int32_t phase;       // what the launch does
    int32_t t, r;        // threshold, round
    int32_t remaining;   // vertices not yet relaxed
    int32_t cur, n_cur;  // the round's frontier: list and size
    int32_t side, n_alive;   // list of the vertices left at the last rise of t, and its size
};
// Zero (min_deg: INT_MAX) at the start of every launch.
struct PeelCounters {
    int32_t n_frontier;  // appended to the next frontier
    int32_t n_left;      // appended to the next list of vertices left
    int32_t min_deg;     // smallest degree found
    int32_t done;        // workgroups of the launch that have finished
};
struct PeelParams {
    const int32_t* row_ptr;
    const int32_t* col;
    int32_t* deg;        // n
    int32_t* round;      // n: the round each vertex leaves in
    int32_t* frontier[2];    // n each
    int32_t* alive[2];       // n each
    PeelCtl* ctl;        // two copies
    PeelCounters* cnt;
};

constexpr int32_t kNoDegree = 0x7fffffff;

// Vertices of `alive` still present: those of degree <= t become the round's
// frontier (marked), the others the next list of vertices left.
template <class Group>
PEEL_FN void peel_collect(Group& G, const PeelParams& P, const int32_t* alive, int n_alive, int t, int r,
                          int32_t* frontier, int32_t* left, int first, int step)
{
    for (int i0 = first; i0 < n_alive; i0 += step) {       // uniform over a wave
        const int i = i0 + G.lane();
        const int32_t v = i < n_alive ? alive[i] : -1;
        const bool here = v >= 0 && P.round[v] < 0;
        const bool now = here && P.deg[v] <= t;
        if (now) P.round[v] = r;
        G.append(now, v, frontier, &P.cnt->n_frontier);
        G.append(here && !now, v, left, &P.cnt->n_left);
    }
}

// Workgroup `block` of the `grid` of a launch that reads *now and leaves the
// next launch's control block in *next.  Group: the workgroup (its lanes,
// barriers and atomics).
template <class Group>
PEEL_FN void peel_step(Group& G, const PeelParams& P, const PeelCtl* now, PeelCtl* next_ctl, int block, int grid)
{
    constexpr int kWaves = Group::kBlock / Group::kWave;
    PeelCtl c = *now;
    if (c.phase == kPeelDone) {
        if (block == 0 && G.thread() == 0) *next_ctl = c;
        return;
    }
    PeelCounters* const cnt = P.cnt;
    const int nf = c.n_cur, n_alive = c.n_alive;
    int32_t* const frontier = P.frontier[c.cur];
    int32_t* const next = P.frontier[1 - c.cur];
    const int32_t* const alive = P.alive[c.side];
    int32_t* const left = P.alive[1 - c.side];
    // workgroups the phase needs; the others leave at once
    const int items = c.phase == kPeelRelax || c.phase == kPeelMark ? nf : n_alive;
    const int per_block = c.phase == kPeelRelax ? kWaves : Group::kBlock * Group::kPerThread;
    const int need = (items + per_block - 1) / per_block;
    const int groups = need < 1 ? 1 : (need < grid ? need : grid);
    if (block >= groups) return;
    const int first = block * Group::kBlock + G.thread(), step = groups * Group::kBlock;
    const int wave = block * kWaves + G.wave(), waves = groups * kWaves;
    if (c.phase == kPeelRelax) {
        // one wave per frontier vertex, lanes over its neighbours
        for (int i = wave; i < nf; i += waves) {
            const int32_t v = frontier[i];
            const int32_t a = P.row_ptr[v], b = P.row_ptr[v + 1];
            for (int32_t e0 = a; e0 < b; e0 += Group::kWave) {
                const int32_t e = e0 + G.lane();
                const int32_t w = e < b ? P.col[e] : -1;
                // gone, or leaving in this round, when its round is set
                const bool join = w >= 0 && P.round[w] < 0 && G.add(&P.deg[w], -1) == c.t + 1;
                G.append(join, w, next, &cnt->n_frontier);
            }
        }
    } else if (c.phase == kPeelMark) {
        for (int i = first; i < nf; i += step) P.round[frontier[i]] = c.r;
    } else if (c.phase == kPeelMin) {
        int m = kNoDegree;
        for (int i = first; i < n_alive; i += step) {
            const int32_t v = alive[i];
            if (P.round[v] < 0 && P.deg[v] < m) m = P.deg[v];
        }
        m = G.min_of(m);
        if (G.thread() == 0 && m != kNoDegree) G.min(&cnt->min_deg, m);
    } else {
        peel_collect(G, P, alive, n_alive, c.t, c.r, frontier, left, wave * Group::kWave, waves * Group::kWave);
    }
    // the workgroup that finishes last sets up the next phase
    if (!G.last_of(&cnt->done, groups)) return;
    const bool one = G.thread() == 0;
    const int joined = G.load(&cnt->n_frontier), n_left = G.load(&cnt->n_left), min_deg = G.load(&cnt->min_deg);
    G.sync();                           // every thread has read what thread 0 clears below
    if (one) {
        G.store(&cnt->n_frontier, 0);
        G.store(&cnt->n_left, 0);
        G.store(&cnt->min_deg, kNoDegree);
        G.store(&cnt->done, 0);
    }
    if (c.phase == kPeelMin) {
        c.t = min_deg;
        c.phase = kPeelCollect;
        if (one) *next_ctl = c;
        return;
    }
    if (c.phase == kPeelMark) {
        c.phase = kPeelRelax;
        if (one) *next_ctl = c;
        return;
    }
    if (c.phase == kPeelCollect) {
        c.n_cur = joined;
        c.n_alive = n_left;
        c.side = 1 - c.side;
        c.phase = kPeelRelax;
        if (one) *next_ctl = c;
        return;
    }
    // a round is over
    c.remaining -= nf;
    c.r += 1;
    if (c.remaining == 0) {
        c.phase = kPeelDone;
        if (one) *next_ctl = c;
        return;
    }
    if (joined > 0) {
        const bool mark = joined <= Group::kInline;
        if (mark)
            for (int i = G.thread(); i < joined; i += Group::kBlock) P.round[G.load(&next[i])] = c.r;
        c.cur = 1 - c.cur;
        c.n_cur = joined;
        c.phase = mark ? kPeelRelax : kPeelMark;
        if (one) *next_ctl = c;
        return;
    }
    // no vertex at or below t is left: t rises to the smallest degree present
    if (n_alive > Group::kInline) {
        c.phase = kPeelMin;
        if (one) *next_ctl = c;
        return;
    }
    int m = kNoDegree;
    for (int i = G.thread(); i < n_alive; i += Group::kBlock) {
        const int32_t v = alive[i];
        if (G.load(&P.round[v]) < 0 && G.load(&P.deg[v]) < m) m = G.load(&P.deg[v]);
    }
    m = G.min_of(m);
    G.sync();
    // (the counters were just cleared by thread 0, before the barriers)
    peel_collect(G, P, alive, n_alive, m, c.r, frontier, left, G.wave() * Group::kWave, kWaves * Group::kWave);
    G.sync();
    if (one) {
        c.t = m;
        c.n_cur = G.load(&cnt->n_frontier);
        c.n_alive = G.load(&cnt->n_left);
        c.side = 1 - c.side;
        c.phase = kPeelRelax;
        G.store(&cnt->n_frontier, 0);
        G.store(&cnt->n_left, 0);
        *next_ctl = c;
    }
}

}  // namespace citron
