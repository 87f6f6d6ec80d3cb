// Input validation, device-wide exclusive scan and the ordering phase
// (Section IV, Algorithm 3 of Lonkar & Beamer): count the out-degree of
// every vertex under the degree ordering, prefix-sum the counts into the
// DAG row offsets, and place the kept neighbours of each row in their input
// (ascending id) order.
#include "kernels.h"

namespace citron {

// ------------------------------------------------------------ wave helpers

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// ------------------------------------------------------- order and row walks

// omega(u) < omega(v): lower key first, ties by lower id.  The key is the
// undirected degree for the degree ordering (Section IV), or the round in
// which a vertex left the peeling for the core ordering.
__device__ __forceinline__ bool keeps(int32_t du, int32_t u, int32_t dv, int32_t v)
{
    return du < dv || (du == dv && u < v);
}

// key of v: its degree, or key[v] when a key array is given
__device__ __forceinline__ int32_t key_of(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ key,
                                          int32_t v)
{
    return key ? key[v] : row_ptr[v + 1] - row_ptr[v];
}

// Largest v and sum of s over the block, then one atomic each per block
// (sum_out may be null): all vertices of a graph meet at these two words,
// whose atomics the device serialises at about 12 ns (one per vertex took
// 11.9 ms of the 12.3 ms of the out-degree pass on 2^20 vertices).
__device__ void block_max_sum_to(int v, unsigned long long s, int32_t* max_out, unsigned long long* sum_out)
{
    __shared__ int wmax[1024 / kWave];
    __shared__ unsigned long long wsum[1024 / kWave];
    const int lane = lane_id(), wid = threadIdx.x / kWave;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        v = max(v, __shfl_xor(v, o, kWave));
        s += __shfl_xor(s, o, kWave);
    }
    if (lane == 0) {
        wmax[wid] = v;
        wsum[wid] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int m = wmax[0];
        unsigned long long t = wsum[0];
        for (int w = 1; w < (int)(blockDim.x / kWave); ++w) {
            m = max(m, wmax[w]);
            t += wsum[w];
        }
        if (m > 0) atomicMax(max_out, m);
        if (sum_out && t) atomicAdd(sum_out, t);
    }
}

// Rows of a sparse graph are short (25 entries on average in the power-law
// families), so a whole wave per row leaves most lanes idle: 16 lanes walk a
// row of up to kGroupMaxRow entries, and the longer rows among a wave's four
// are then walked by all 64 lanes in turn.  visit(u, a, b, lane, step, du)
// takes every step-th entry of row u from a + lane; done(u, v) is called by
// the first lane of the row's group with the group's sum of visit's results.
constexpr int kRowGroup = 16;
constexpr int kGroupsPerWave = kWave / kRowGroup;
constexpr int kGroupMaxRow = 256;
constexpr int kWalkBlock = 512;

template <typename Visit, typename Done>
__device__ __forceinline__ void walk_rows(int32_t n, const int32_t* __restrict__ row_ptr,
                                          const int32_t* __restrict__ key, Visit visit, Done done)
{
    const int lane = lane_id();
    const int sub = lane & (kRowGroup - 1);
    const int64_t waves = (int64_t)gridDim.x * blockDim.x / kWave;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    for (int64_t u0 = wave * kGroupsPerWave; u0 < n; u0 += waves * kGroupsPerWave) {
        const int64_t u = u0 + lane / kRowGroup;
        const bool in = u < n;
        const int32_t a = in ? row_ptr[u] : 0, b = in ? row_ptr[u + 1] : 0;
        const int32_t du = in ? (key ? key[u] : b - a) : 0;
        const bool big = b - a > kGroupMaxRow;
        int cnt = big ? 0 : visit((int32_t)u, a, b, sub, kRowGroup, du);
#pragma unroll
        for (int o = kRowGroup / 2; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, kWave);
        unsigned long long rest = __ballot(big && sub == 0);
        while (rest) {
            const int src = __builtin_ctzll(rest);
            rest &= rest - 1;
            const int32_t bu = (int32_t)(u0 + src / kRowGroup);
            int c = visit(bu, __shfl(a, src, kWave), __shfl(b, src, kWave), lane, kWave, __shfl(du, src, kWave));
#pragma unroll
            for (int o = kWave / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
            if (lane == src) cnt = c;
        }
        if (in && sub == 0) done((int32_t)u, cnt);
    }
}

// Blocks of a row walk: one pass over the rows, or the 32 waves per CU that
// 256 CUs hold, whichever is less (each block ends with an atomic or two).
static unsigned walk_blocks(int32_t n)
{
    const int64_t need = ((int64_t)n + kWalkBlock / kRowGroup - 1) / (kWalkBlock / kRowGroup);
    return (unsigned)(need < 1024 ? need : 1024);
}

// ------------------------------------------------------------- validation

// err bits: 1 row_ptr out of range or decreasing, 2 column id out of range,
// 4 self-loop, 8 row not strictly ascending, 16 asymmetric, 32 row_ptr[0]
// not 0 or row_ptr[n] not nnz.
__global__ void validate_row_ptr_kernel(int32_t n, int64_t nnz, const int32_t* __restrict__ row_ptr,
                                        int32_t* __restrict__ err)
{
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u == 0 && (row_ptr[0] != 0 || (int64_t)row_ptr[n] != nnz)) atomicOr(err, 32);
    if (u >= n) return;
    int32_t a = row_ptr[u], b = row_ptr[u + 1];
    if (a < 0 || b < a || (int64_t)b > nnz) atomicOr(err, 1);
}

// Entries, once the offsets are known to be in range (*err is read first: a
// bad offset ends the kernel before it follows one).  The degrees that the
// degree ordering compares are at hand here, so the pass also leaves every
// vertex's out-degree under it, the largest of them and their sum.
//
// Symmetry: of the two entries of an edge, only the one in the row of the
// higher endpoint searches for its mirror, in the row of the lower endpoint
// (the shorter row).  Searched entries map to distinct unsearched ones, so
// the graph is symmetric iff every search succeeds and the unsearched ones
// (the sum of the out-degrees) are exactly half: the caller compares
// *kept with nnz / 2.  Searching for every entry in the other row, long or
// short, took 2.27 ms on 2^20 vertices and 25.8 M entries.
__global__ void __launch_bounds__(kWalkBlock) validate_entries_kernel(int32_t n, const int32_t* __restrict__ row_ptr,
                                        const int32_t* __restrict__ col, int32_t* __restrict__ err,
                                        int32_t* __restrict__ outdeg, int32_t* __restrict__ max_outdeg,
                                        unsigned long long* __restrict__ kept)
{
    if (*(volatile int32_t*)err & 33) return;   // set by the offsets' kernel only: the same for all waves
    int bits = 0, mx = 0;
    unsigned long long sum = 0;
    walk_rows(n, row_ptr, nullptr,
        [&](int32_t u, int32_t a, int32_t b, int lane, int step, int32_t du) {
            int cnt = 0;
            for (int32_t e = a + lane; e < b; e += step) {
                const int32_t v = col[e];
                if (v < 0 || v >= n) { bits |= 2; continue; }
                if (v == u) { bits |= 4; continue; }
                if (e > a && col[e - 1] >= v) bits |= 8;
                int32_t lo = row_ptr[v];
                const int32_t end = row_ptr[v + 1];
                if (keeps(du, u, end - lo, v)) { ++cnt; continue; }
                // u must appear in row v (row v is checked for order by its
                // own walk; a binary search on an unsorted row may miss u,
                // which is then reported as asymmetric, still an error)
                int32_t hi = end;
                while (lo < hi) {
                    const int32_t mid = lo + ((hi - lo) >> 1);
                    if (col[mid] < u) lo = mid + 1;
                    else hi = mid;
                }
                if (lo >= end || col[lo] != u) bits |= 16;
            }
            return cnt;
        },
        [&](int32_t u, int cnt) {
            outdeg[u] = cnt;
            mx = max(mx, cnt);
            sum += (unsigned long long)cnt;
        });
    if (bits) atomicOr(err, bits);
    block_max_sum_to(mx, sum, max_outdeg, kept);
}

// ------------------------------------------------------------------- scan
//
// Exclusive prefix sum of n int32 values into out[0..n], out[n] = total,
// by reduce-then-scan over tiles of kScanTile values (recursive on the tile
// sums).  The totals must fit int32 (they are CSR offsets).

constexpr int kScanBlock = 256;
constexpr int kScanPer = 16;
constexpr int kScanTile = kScanBlock * kScanPer;

__device__ int block_exclusive_scan(int v, int* total)
{
    __shared__ int wsum[kScanBlock / kWave];
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    int inc = wave_inclusive_scan(v);
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / kWave; ++w) {
        if (w < wid) off += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__global__ void scan_tile_sums_kernel(const int32_t* __restrict__ in, int64_t n, int32_t* __restrict__ sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int s = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i)
        if (base + i < n) s += in[base + i];
    int tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void scan_tiles_kernel(const int32_t* __restrict__ in, int64_t n,
                                  const int32_t* __restrict__ tile_off, int32_t* __restrict__ out)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int vals[kScanPer];
    int s = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        vals[i] = (base + i < n) ? in[base + i] : 0;
        s += vals[i];
    }
    int tot;
    int run = block_exclusive_scan(s, &tot) + (tile_off ? tile_off[blockIdx.x] : 0);
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        if (base + i < n) out[base + i] = run;
        run += vals[i];
    }
    // the thread holding element n-1 writes the total into out[n]
    if (n > 0 && base <= n - 1 && n - 1 < base + kScanPer) out[n] = run;
    if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) out[0] = tile_off ? tile_off[0] : 0;
    (void)tot;
}

size_t scan_workspace_ints(int64_t n)
{
    if (n <= kScanTile) return 1;
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    return (size_t)(2 * tiles + 1) + scan_workspace_ints(tiles);
}

// in and out may not alias; out receives n + 1 values.
// ws: scan_workspace_ints(n) ints: [tile sums | scanned tile sums | deeper].
hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int32_t* ws, hipStream_t s)
{
    if (n <= kScanTile) {
        scan_tiles_kernel<<<1, kScanBlock, 0, s>>>(in, n, nullptr, out);
        return hipGetLastError();
    }
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    int32_t* sums = ws;
    int32_t* offs = ws + tiles;
    scan_tile_sums_kernel<<<(unsigned)tiles, kScanBlock, 0, s>>>(in, n, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = scan_exclusive(sums, offs, tiles, ws + 2 * tiles + 1, s);
    if (e != hipSuccess) return e;
    scan_tiles_kernel<<<(unsigned)tiles, kScanBlock, 0, s>>>(in, n, offs, out);
    return hipGetLastError();
}

// --------------------------------------------------------------- ordering

// Out-degree of every vertex (first loop of Algorithm 3) under a given key,
// and the largest out-degree.
__global__ void __launch_bounds__(kWalkBlock) orient_count_kernel(int32_t n, const int32_t* __restrict__ row_ptr,
                                    const int32_t* __restrict__ col, const int32_t* __restrict__ key,
                                    int32_t* __restrict__ outdeg, int32_t* __restrict__ max_outdeg)
{
    int mx = 0;
    walk_rows(n, row_ptr, key,
        [&](int32_t u, int32_t a, int32_t b, int lane, int step, int32_t du) {
            int cnt = 0;
            for (int32_t e = a + lane; e < b; e += step) {
                const int32_t v = col[e];
                cnt += keeps(du, u, key_of(row_ptr, key, v), v) ? 1 : 0;
            }
            return cnt;
        },
        [&](int32_t u, int cnt) {
            outdeg[u] = cnt;
            mx = max(mx, cnt);
        });
    block_max_sum_to(mx, 0, max_outdeg, nullptr);
}

// Place the kept neighbours (second loop of Algorithm 3).  One wavefront per
// vertex walks its row in 64-entry steps; a ballot marks the kept entries and
// each lane writes at the count of kept entries before it, so the row keeps
// its ascending order.  dag_src (may be null) receives the source vertex of
// every arc.
__global__ void orient_scatter_kernel(int32_t n, const int32_t* __restrict__ row_ptr,
                                      const int32_t* __restrict__ col, const int32_t* __restrict__ key,
                                      const int32_t* __restrict__ dag_ptr,
                                      int32_t* __restrict__ dag_col, int32_t* __restrict__ dag_src)
{
    const int64_t u = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (u >= n) return;
    const int lane = lane_id();
    const int32_t a = row_ptr[u], b = row_ptr[u + 1];
    const int32_t du = key_of(row_ptr, key, (int32_t)u);
    int32_t out = dag_ptr[u];
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    for (int32_t e0 = a; e0 < b; e0 += kWave) {
        const int32_t e = e0 + lane;
        int32_t v = -1;
        bool keep = false;
        if (e < b) {
            v = col[e];
            keep = keeps(du, (int32_t)u, key_of(row_ptr, key, v), v);
        }
        const unsigned long long mask = __ballot(keep);
        if (keep) {
            const int32_t pos = out + __popcll(mask & below);
            dag_col[pos] = v;
            if (dag_src) dag_src[pos] = (int32_t)u;
        }
        out += __popcll(mask);
    }
}

// ------------------------------------------------------------ host wrappers

hipError_t launch_validate(int32_t n, int64_t nnz, const int32_t* row_ptr, const int32_t* col, int32_t* err,
                           int32_t* outdeg, int32_t* max_outdeg, unsigned long long* kept, hipStream_t s)
{
    validate_row_ptr_kernel<<<(unsigned)(((int64_t)n + 256) / 256), 256, 0, s>>>(n, nnz, row_ptr, err);
    if (n > 0)
        validate_entries_kernel<<<walk_blocks(n), kWalkBlock, 0, s>>>(n, row_ptr, col, err, outdeg, max_outdeg, kept);
    return hipGetLastError();
}

hipError_t launch_orient(int32_t n, const int32_t* row_ptr, const int32_t* col, int32_t* outdeg,
                         int32_t* dag_ptr, int32_t* dag_col, int32_t* dag_src, int32_t* max_outdeg,
                         int32_t* scan_ws, hipStream_t s, const int32_t* key, bool count)
{
    if (n == 0) return hipSuccess;
    const int64_t threads = (int64_t)n * kWave;
    const unsigned blocks = (unsigned)((threads + 255) / 256);
    hipError_t e;
    if (count) {
        orient_count_kernel<<<walk_blocks(n), kWalkBlock, 0, s>>>(n, row_ptr, col, key, outdeg, max_outdeg);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    e = scan_exclusive(outdeg, dag_ptr, n, scan_ws, s);
    if (e != hipSuccess) return e;
    orient_scatter_kernel<<<blocks, 256, 0, s>>>(n, row_ptr, col, key, dag_ptr, dag_col, dag_src);
    return hipGetLastError();
}

}  // namespace citron
