// Replays the launches of the peeling (csrc/peel.h) on the host, one workgroup
// after the other, in an order that a busy device may come to.
#include <algorithm>
#include <numeric>
#include <random>
#include <vector>

#include "../paper_2112_10913_amd/csrc/peel.h"

namespace {

struct HostGroup {
    static constexpr int kWave = 1;
    static constexpr int kBlock = 1;
    static constexpr int kPerThread = 2;
    static constexpr int kInline = 3;
    int capacity;        // entries a list holds
    bool* overrun;
    int thread() const { return 0; }
    int lane() const { return 0; }
    int wave() const { return 0; }
    void sync() const {}
    int add(int32_t* p, int v) const
    {
        const int old = *p;
        *p += v;
        return old;
    }
    void min(int32_t* p, int v) const { *p = std::min(*p, v); }
    int32_t load(const int32_t* p) const { return *p; }
    void store(int32_t* p, int32_t v) const { *p = v; }
    int min_of(int v) const { return v; }
    void append(bool take, int32_t v, int32_t* list, int32_t* cnt) const
    {
        if (!take) return;
        const int at = (*cnt)++;
        if (at >= capacity) *overrun = true;
        else list[at] = v;
    }
    bool last_of(int32_t* done, int groups) const { return add(done, 1) == groups - 1; }
};

}  // namespace

// order 0: ascending (the workgroups a phase needs before the others),
// 1: descending, 2: shuffled.  copies: 2, or 1 for launches that read and
// write the same control block.  Returns 0 when the peeling ended, 1 when it
// did not, 2 when a list would have been written past its end.
extern "C" int peel_replay(int32_t n, const int32_t* row_ptr, const int32_t* col, int grid, int order, int seed,
                           int copies, int32_t* round, int32_t* rounds)
{
    using namespace citron;
    std::vector<int32_t> deg(n), lists(4 * (size_t)(n + 1)), block(grid);
    PeelCtl ctl[2] = {};
    ctl[0].phase = kPeelMin;
    ctl[0].remaining = ctl[0].n_alive = n;
    PeelCounters cnt = {};
    cnt.min_deg = kNoDegree;
    PeelParams P;
    P.row_ptr = row_ptr;
    P.col = col;
    P.deg = deg.data();
    P.round = round;
    for (int i = 0; i < 2; ++i) {
        P.frontier[i] = lists.data() + i * (size_t)(n + 1);
        P.alive[i] = lists.data() + (2 + i) * (size_t)(n + 1);
    }
    P.ctl = ctl;
    P.cnt = &cnt;
    for (int32_t v = 0; v < n; ++v) {
        deg[v] = row_ptr[v + 1] - row_ptr[v];
        round[v] = -1;
        P.alive[0][v] = v;
    }
    bool overrun = false;
    HostGroup G{n + 1, &overrun};
    std::mt19937 rng(seed);
    std::iota(block.begin(), block.end(), 0);
    if (order == 1) std::reverse(block.begin(), block.end());
    for (int64_t s = 0; s < 4ll * n + 8; ++s) {
        PeelCtl* now = ctl + (copies == 2 ? (s & 1) : 0);
        PeelCtl* next = ctl + (copies == 2 ? 1 - (s & 1) : 0);
        if (order == 2) std::shuffle(block.begin(), block.end(), rng);
        for (int b : block) {
            peel_step(G, P, now, next, b, grid);
            if (overrun) return 2;
        }
        // the host looks at the copy that the next launch reads, and later
        // launches leave it as it is
        if (s % 5 == 4 && next->phase == kPeelDone) {
            *rounds = next->r;
            return 0;
        }
    }
    return 1;
}
