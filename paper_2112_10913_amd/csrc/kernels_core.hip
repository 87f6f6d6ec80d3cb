// Core ordering on the GPU (Section III, Algorithm 1 and the discussion of
// its cost in Section IV): the paper's Algorithm 1 removes one vertex of
// smallest current degree at a time, a sequential process.  Here all
// vertices whose current degree is at most a threshold t leave in one round
// (level-synchronous peeling): a round marks its frontier, then lowers the
// degree of every neighbour still present by one per edge; a neighbour whose
// degree falls from t + 1 to t joins the next round's frontier (exactly one
// decrement sees that step, so it is appended once).  When a round's
// frontier is empty, t rises to the smallest degree still present.  The
// round numbers are the order key (ties by id): every out-degree of the
// resulting DAG is at most the t of its vertex's round, which never exceeds
// the degeneracy.
//
// The device drives itself: each launch of peel_step_kernel does one phase
// that the control block names, and the workgroup that finishes last sets up
// the next one, so the host only queues launches and looks at the control
// block once per batch.  No workgroup ever waits for another.  Small steps
// (marking a short frontier, raising t over a short list of the vertices
// left) are done by that last workgroup at once.  Bound by latency: a round
// is one launch of about 11 us, most of it a chain of dependent loads and
// atomics (128, 256 and 1,024 workgroups are alike).  (With the host reading each round's
// frontier size and launching four kernels for it, a round took 38 us:
// R-MAT 16, 314 rounds: 12.5 ms for load, ordering and DAG, now 5.8 ms.)
#include "kernels.h"

namespace citron {

namespace {

constexpr int kPeelBlock = 512;
constexpr int kPeelWaves = kPeelBlock / kWave;
constexpr int kPeelBlocks = 128;
constexpr int kPerThread = 8;                  // list entries a thread takes before another workgroup starts
constexpr int kInlineMark = 16 * kPeelBlock;   // lists the last workgroup handles itself
constexpr int kInlineRaise = 16 * kPeelBlock;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Smallest v over the workgroup, in every thread.
__device__ int block_min(int v)
{
    __shared__ int wmin[kPeelWaves];
    const int lane = lane_id(), wid = threadIdx.x / kWave;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, kWave));
    __syncthreads();
    if (lane == 0) wmin[wid] = v;
    __syncthreads();
    int m = wmin[0];
#pragma unroll
    for (int w = 1; w < kPeelWaves; ++w) m = min(m, wmin[w]);
    return m;
}

// Appends the lanes' v with `take` to list at *cnt: one atomic per wave.
__device__ __forceinline__ void wave_append(bool take, int32_t v, int32_t* list, int32_t* cnt)
{
    const unsigned long long mask = __ballot(take);
    if (!mask) return;
    const int lane = lane_id();
    int base = 0;
    if (lane == 0) base = atomicAdd(cnt, __popcll(mask));
    base = __shfl(base, 0, kWave);
    const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    if (take) list[base + __popcll(mask & below)] = v;
}

// Vertices of `alive` still present: those of degree <= t become the round's
// frontier (marked), the others the next list of vertices left.
__device__ void peel_collect(const PeelParams& P, PeelCtl* c, const int32_t* alive, int n_alive, int t, int r,
                             int32_t* frontier, int32_t* left, int first, int step)
{
    for (int i0 = first; i0 < n_alive; i0 += step) {       // uniform over a wave
        const int i = i0 + lane_id();
        const int32_t v = i < n_alive ? alive[i] : -1;
        const bool here = v >= 0 && P.round[v] < 0;
        const bool now = here && P.deg[v] <= t;
        if (now) P.round[v] = r;
        wave_append(now, v, frontier, &c->n_frontier);
        wave_append(here && !now, v, left, &c->n_left);
    }
}

}  // namespace

__global__ void peel_init_kernel(int32_t n, PeelParams P)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) {
        P.deg[v] = P.row_ptr[v + 1] - P.row_ptr[v];
        P.round[v] = -1;
        P.alive[0][v] = (int32_t)v;
    }
    if (v == 0) {
        PeelCtl c = {};
        c.phase = kPeelMin;
        c.remaining = n;
        c.n_alive = n;
        c.min_deg = 0x7fffffff;
        *P.ctl = c;
    }
}

__global__ void __launch_bounds__(kPeelBlock) peel_step_kernel(PeelParams P)
{
    __shared__ int last;
    PeelCtl* const c = P.ctl;
    const int phase = c->phase;
    if (phase == kPeelDone) return;
    const int cur = c->cur, side = c->side, t = c->t, r = c->r;
    const int nf = c->n_cur, n_alive = c->n_alive;
    int32_t* const frontier = P.frontier[cur];
    int32_t* const next = P.frontier[1 - cur];
    const int32_t* const alive = P.alive[side];
    // workgroups the phase needs; the others leave at once
    const int items = phase == kPeelRelax ? nf : phase == kPeelMark ? nf : n_alive;
    const int per_block = phase == kPeelRelax ? kPeelWaves : kPeelBlock * kPerThread;
    const int groups = min((int)gridDim.x, max(1, (items + per_block - 1) / per_block));
    if ((int)blockIdx.x >= groups) return;
    const int wid = threadIdx.x / kWave, lane = lane_id();
    const int wave = blockIdx.x * kPeelWaves + wid, waves = groups * kPeelWaves;
    if (phase == kPeelRelax) {
        // one wave per frontier vertex, lanes over its neighbours
        for (int i = wave; i < nf; i += waves) {
            const int32_t v = frontier[i];
            const int32_t a = P.row_ptr[v], b = P.row_ptr[v + 1];
            for (int32_t e0 = a; e0 < b; e0 += kWave) {
                const int32_t e = e0 + lane;
                const int32_t w = e < b ? P.col[e] : -1;
                // gone, or leaving in this round, when its round is set
                const bool join = w >= 0 && P.round[w] < 0 && atomicSub(&P.deg[w], 1) == t + 1;
                wave_append(join, w, next, &c->n_frontier);
            }
        }
    } else if (phase == kPeelMark) {
        for (int i = blockIdx.x * kPeelBlock + threadIdx.x; i < nf; i += groups * kPeelBlock) P.round[frontier[i]] = r;
    } else if (phase == kPeelMin) {
        int m = 0x7fffffff;
        for (int i = blockIdx.x * kPeelBlock + threadIdx.x; i < n_alive; i += groups * kPeelBlock) {
            const int32_t v = alive[i];
            if (P.round[v] < 0) m = min(m, P.deg[v]);
        }
        m = block_min(m);
        if (threadIdx.x == 0 && m != 0x7fffffff) atomicMin(&c->min_deg, m);
    } else {
        peel_collect(P, c, alive, n_alive, t, r, frontier, P.alive[1 - side], wave * kWave, waves * kWave);
    }
    // the workgroup that finishes last sets up the next phase
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(&c->done, 1) == groups - 1;
        __threadfence();
    }
    __syncthreads();
    if (!last) return;
    auto read = [](const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (phase == kPeelMin) {
        if (threadIdx.x == 0) {
            c->t = read(&c->min_deg);
            c->min_deg = 0x7fffffff;
            c->phase = kPeelCollect;
            c->done = 0;
        }
        return;
    }
    if (phase == kPeelMark) {
        if (threadIdx.x == 0) {
            c->phase = kPeelRelax;
            c->done = 0;
        }
        return;
    }
    if (phase == kPeelCollect) {
        if (threadIdx.x == 0) {
            c->n_cur = read(&c->n_frontier);
            c->n_alive = read(&c->n_left);
            c->n_frontier = 0;
            c->n_left = 0;
            c->side = 1 - side;
            c->phase = kPeelRelax;
            c->done = 0;
        }
        return;
    }
    // a round is over
    const int joined = read(&c->n_frontier);
    const int remaining = c->remaining - nf;
    __syncthreads();                    // every thread has read what thread 0 writes below
    if (threadIdx.x == 0) {
        c->remaining = remaining;
        c->r = r + 1;
        c->n_frontier = 0;
        c->done = 0;
    }
    if (remaining == 0) {
        if (threadIdx.x == 0) c->phase = kPeelDone;
        return;
    }
    if (joined > 0) {
        if (threadIdx.x == 0) {
            c->cur = 1 - cur;
            c->n_cur = joined;
            c->phase = joined <= kInlineMark ? kPeelRelax : kPeelMark;
        }
        if (joined <= kInlineMark)
            for (int i = threadIdx.x; i < joined; i += kPeelBlock) P.round[read(&next[i])] = r + 1;
        return;
    }
    // no vertex at or below t is left: t rises to the smallest degree present
    if (n_alive > kInlineRaise) {
        if (threadIdx.x == 0) c->phase = kPeelMin;
        return;
    }
    int m = 0x7fffffff;
    for (int i = threadIdx.x; i < n_alive; i += kPeelBlock) {
        const int32_t v = alive[i];
        if (read(&P.round[v]) < 0) m = min(m, read(&P.deg[v]));
    }
    m = block_min(m);
    __syncthreads();
    // (n_frontier was just cleared by thread 0, before the barriers)
    peel_collect(P, c, alive, n_alive, m, r + 1, frontier, P.alive[1 - side], wid * kWave, kPeelWaves * kWave);
    __syncthreads();
    if (threadIdx.x == 0) {
        c->t = m;
        c->n_cur = read(&c->n_frontier);
        c->n_alive = read(&c->n_left);
        c->n_frontier = 0;
        c->n_left = 0;
        c->side = 1 - side;
        c->phase = kPeelRelax;
    }
}

hipError_t launch_peel_init(int32_t n, const PeelParams& P, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    peel_init_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, P);
    return hipGetLastError();
}

hipError_t launch_peel_steps(const PeelParams& P, int32_t steps, hipStream_t s)
{
    for (int32_t i = 0; i < steps; ++i) peel_step_kernel<<<kPeelBlocks, kPeelBlock, 0, s>>>(P);
    return hipGetLastError();
}

}  // namespace citron
