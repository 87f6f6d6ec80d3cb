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
// the next one (peel.h), so the host only queues launches and looks at the
// control block once per batch.  No workgroup ever waits for another, and none
// reads what another one of its launch writes to the control block.  Small
// steps (marking a short frontier, raising t over a short list of the vertices
// left) are done by that last workgroup at once.  Bound by latency: a round
// is one launch of about 11 us, most of it a chain of dependent loads and
// atomics (128, 256 and 1,024 workgroups are alike).  (With the host reading each round's
// frontier size and launching four kernels for it, a round took 38 us:
// R-MAT 16, 314 rounds: 12.5 ms for load, ordering and DAG, now 5.8 ms.)
#include "kernels.h"

namespace citron {

namespace {

constexpr int kPeelBlocks = 128;

// A workgroup of the peeling on the device.
struct DeviceGroup {
    static constexpr int kWave = citron::kWave;
    static constexpr int kBlock = 512;
    static constexpr int kPerThread = 8;           // list entries a thread takes before another workgroup starts
    static constexpr int kInline = 16 * kBlock;    // lists the last workgroup handles itself
    static constexpr int kWaves = kBlock / kWave;
    int* shared;                                   // kWaves words

    __device__ __forceinline__ int thread() const { return threadIdx.x; }
    __device__ __forceinline__ int lane() const { return threadIdx.x & (kWave - 1); }
    __device__ __forceinline__ int wave() const { return threadIdx.x / kWave; }
    __device__ __forceinline__ void sync() const { __syncthreads(); }
    __device__ __forceinline__ int add(int32_t* p, int v) const { return atomicAdd(p, v); }
    __device__ __forceinline__ void min(int32_t* p, int v) const { atomicMin(p, v); }
    __device__ __forceinline__ int32_t load(const int32_t* p) const
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void store(int32_t* p, int32_t v) const
    {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Smallest v over the workgroup, in every thread.
    __device__ int min_of(int v) const
    {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) v = ::min(v, __shfl_xor(v, o, kWave));
        __syncthreads();
        if (lane() == 0) shared[wave()] = v;
        __syncthreads();
        int m = shared[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) m = ::min(m, shared[w]);
        return m;
    }
    // Appends the lanes' v with `take` to list at *cnt: one atomic per wave.
    __device__ __forceinline__ void append(bool take, int32_t v, int32_t* list, int32_t* cnt) const
    {
        const unsigned long long mask = __ballot(take);
        if (!mask) return;
        int base = 0;
        if (lane() == 0) base = atomicAdd(cnt, __popcll(mask));
        base = __shfl(base, 0, kWave);
        const unsigned long long below = lane() == 0 ? 0ull : (~0ull >> (kWave - lane()));
        if (take) list[base + __popcll(mask & below)] = v;
    }
    // Whether this is the last of `groups` workgroups to get here; what the
    // others wrote before is then visible.
    __device__ __forceinline__ bool last_of(int32_t* done, int groups) const
    {
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();
            shared[0] = atomicAdd(done, 1) == groups - 1;
            __threadfence();
        }
        __syncthreads();
        return shared[0] != 0;
    }
};

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
        P.ctl[0] = c;
        PeelCounters k = {};
        k.min_deg = kNoDegree;
        *P.cnt = k;
    }
}

__global__ void __launch_bounds__(DeviceGroup::kBlock) peel_step_kernel(PeelParams P, int parity)
{
    __shared__ int shared[DeviceGroup::kWaves];
    DeviceGroup G{shared};
    peel_step(G, P, P.ctl + parity, P.ctl + 1 - parity, blockIdx.x, gridDim.x);
}

hipError_t launch_peel_init(int32_t n, const PeelParams& P, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    peel_init_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, P);
    return hipGetLastError();
}

hipError_t launch_peel_steps(const PeelParams& P, int64_t first, int32_t steps, hipStream_t s)
{
    for (int64_t i = first; i < first + steps; ++i)
        peel_step_kernel<<<kPeelBlocks, DeviceGroup::kBlock, 0, s>>>(P, (int)(i & 1));
    return hipGetLastError();
}

}  // namespace citron
