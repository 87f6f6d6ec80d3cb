// Subgraph construction of the counting phase (Lonkar & Beamer, Section V-B,
// Algorithm 5) and the schedule of the count kernel.
//
// For every vertex u with out-list N->(u) = (v_0 < ... < v_{d-1}) the rows
// of the subgraph induced on N->(u) are built once per graph: row i is
// N->(v_i) cap N->(u), a bitmap over the positions 0..d-1 of N->(u) with
// W(u) = ceil(d/64) words.  Row i is also the candidate set C_uv of the arc
// u -> v_i, so its popcount |C_uv| is the arc's triangle count and the arc's
// cost estimate.  The rows do not depend on k; every count reuses them.
//
// Vertices are sorted by out-degree (descending): a workgroup per heavy
// vertex (out-degree > 64), and batches of light vertices of about
// `light_rows` rows.
#include "kernels.h"
#include "wave.h"

namespace citron {

namespace {

constexpr int kWave_ = kWave;

__device__ __forceinline__ int wave_incl_scan(int v)
{
    const int lane = lane_of();
#pragma unroll
    for (int o = 1; o < kWave_; o <<= 1) {
        int t = __shfl_up(v, o, kWave_);
        if (lane >= o) v += t;
    }
    return v;
}

__device__ __forceinline__ int upper_bound_i32(const int32_t* a, int n, int32_t x)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int lower_bound_i32(const int32_t* a, int n, int32_t x)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

constexpr int kLightBlock = 256;
constexpr int kLightWaves = kLightBlock / kWave;
constexpr int kProbeRatio = 4;
constexpr int kHeavyBlock = 512;
constexpr int kHeavyWaves = kHeavyBlock / kWave;

// Adds a workgroup's triangles and build counters to the graph's (tri,
// entries: every thread's; verts, rows, bytes: thread 0's).
template <int kBlock>
__device__ __forceinline__ void flush_build(const BuildParams& P, u64 tri, u64 verts, u64 rows, u64 bytes, u64 entries)
{
    __shared__ u64 part[kBlock / kWave_][2];
#pragma unroll
    for (int o = kWave_ / 2; o > 0; o >>= 1) {
        tri += __shfl_xor(tri, o, kWave_);
        entries += __shfl_xor(entries, o, kWave_);
    }
    if (lane_of() == 0) {
        part[threadIdx.x / kWave_][0] = tri;
        part[threadIdx.x / kWave_][1] = entries;
    }
    __syncthreads();
    if (threadIdx.x != 0 || !verts) return;
    for (int w = 1; w < kBlock / kWave_; ++w) {
        tri += part[w][0];       // a workgroup's triangles: below 2^31 arcs x 2^12
        entries += part[w][1];
    }
    BuildSums* s = P.sums + (blockIdx.x & (kBuildSlots - 1));
    if (tri) {
        const u64 old = atomicAdd(&s->tri, tri);
        if (old + tri < old) atomicOr(&s->tri_ovf, 1);
    }
    atomicAdd(&s->verts, verts);
    atomicAdd(&s->rows, rows);
    atomicAdd(&s->entries, entries);
    atomicAdd(&s->bytes, bytes + 4ull * entries);
}

}  // namespace

__host__ __device__ inline int build_rows_cap(int light_rows) { return light_rows + kLightMaxDeg; }

static int32_t light_lds_bytes(int32_t light_rows)
{
    const int Dc = build_rows_cap(light_rows);
    const int Vc = Dc / 2 + 2;
    int b = 4 * kLightWaves + 5 * 4 * (Dc + 4) + 4 * 4 * Vc;
    b = (b + 15) & ~15;
    return b + 8 * Dc;
}

// Batches of light vertices.  The (row, entry) pairs of a batch are one
// sequence cut into a contiguous range per wave, so that a wave finds its
// first row by one search and the rows of the next 64 entries by stepping on;
// each entry of N->(v_i) is then searched in N->(u) (at most 64 ids, in LDS).
// Where N->(v_i) is more than kProbeRatio times as long as N->(u), the row's
// entries are those of N->(u) instead, each searched in N->(v_i) in device
// memory (about 9 dependent reads): a vertex with few out-neighbours does not
// read a hub's whole list for each.  Ratios of 4, 8, 16 and never: 3.3, 3.7,
// 4.0 and 3.9 ms on a Chung-Lu graph of 2^20 vertices.
__global__ void __launch_bounds__(kLightBlock) build_light_kernel(BuildParams P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = kLightBlock, tid = threadIdx.x, lane = lane_of(), wid = tid / kWave_;
    const int nwaves = kLightWaves;
    const int Dc = build_rows_cap(P.plan.light_rows);
    const int Vc = Dc / 2 + 2;
    int32_t* wsum = reinterpret_cast<int32_t*>(smem);       // a word per wave
    int32_t* row_v = wsum + kLightWaves;
    int32_t* row_owner = row_v + (Dc + 4);
    int32_t* row_begin = row_owner + (Dc + 4);
    int32_t* row_n = row_begin + (Dc + 4);       // length of N->(v) for a row that probes it, else 0
    int32_t* pre = row_n + (Dc + 4);
    int32_t* vert_u = pre + (Dc + 4);
    int32_t* vert_base = vert_u + Vc;
    int32_t* vert_deg = vert_base + Vc;
    int32_t* vert_arc0 = vert_deg + Vc;
    size_t off = (size_t)((unsigned char*)(vert_arc0 + Vc) - smem);
    off = (off + 15) & ~(size_t)15;
    u64* bm = reinterpret_cast<u64*>(smem + off);
    const int32_t* __restrict__ dag_ptr = P.dag_ptr;
    const int32_t* __restrict__ dag_col = P.dag_col;
    u64 tri = 0, st_entries = 0, st_rows = 0, st_verts = 0, st_bytes = 0;

    for (int b0 = blockIdx.x; b0 < P.plan.n_batches; b0 += gridDim.x) {
        const int s0 = P.batch_start[b0], s1 = P.batch_start[b0 + 1];
        const int base0 = P.light_pre[s0];
        const int nb = s1 - s0, R = P.light_pre[s1] - base0;
        for (int j = tid; j < nb; j += T) {
            const int u = P.order[P.plan.n_heavy + s0 + j];
            vert_u[j] = u;
            vert_base[j] = P.light_pre[s0 + j] - base0;
            vert_deg[j] = P.light_pre[s0 + j + 1] - P.light_pre[s0 + j];
            vert_arc0[j] = dag_ptr[u];
        }
        __syncthreads();
        // rows: v = N->(u)[i] and the length of N->(v)
        for (int r = tid; r < R; r += T) {
            const int b = upper_bound_i32(vert_base, nb, r) - 1;
            const int v = dag_col[vert_arc0[b] + (r - vert_base[b])];
            row_v[r] = v;
            row_owner[r] = b;
            const int a0 = dag_ptr[v];
            row_begin[r] = a0;
            const int n = dag_ptr[v + 1] - a0, du = vert_deg[b];
            const bool probe = n > kProbeRatio * du;
            row_n[r] = probe ? n : 0;
            pre[r] = probe ? du : n;
            bm[r] = 0ull;
            st_entries += (u64)n;
        }
        __syncthreads();
        {   // block-wide exclusive scan of the row lengths, pre[R] = total
            int carry = 0;
            for (int base = 0; base < R; base += T) {
                const int r = base + tid;
                const int v = r < R ? pre[r] : 0;
                const int inc = wave_incl_scan(v);
                if (lane == kWave_ - 1) wsum[wid] = inc;
                __syncthreads();
                int o = 0, tot = 0;
                for (int w = 0; w < nwaves; ++w) {
                    const int x = wsum[w];
                    if (w < wid) o += x;
                    tot += x;
                }
                if (r < R) pre[r] = carry + o + inc - v;
                __syncthreads();
                carry += tot;
            }
            if (tid == 0) pre[R] = carry;
        }
        __syncthreads();
        const int total = pre[R];
        if (tid == 0) {
            st_verts += (u64)nb;
            st_rows += (u64)R;
            st_bytes += 4ull * ((u64)R + 2ull * nb) + 8ull * R;
        }
        // Algorithm 5: each entry x of N->(v_r) looked up in N->(u), or the
        // other way round
        const int span = ((total + nwaves - 1) / nwaves + kWave_ - 1) & ~(kWave_ - 1);
        const int t_end = min(total, (wid + 1) * span);
        int r0 = wid * span < total ? upper_bound_i32(pre, R + 1, wid * span) - 1 : 0;
        for (int t0 = wid * span; t0 < t_end; t0 += kWave_) {
            const int t = t0 + lane;
            int r = r0;
            if (t < t_end) {
                while (pre[r + 1] <= t) ++r;
                const int b = row_owner[r];
                const int32_t* nu = row_v + vert_base[b];
                const int n = row_n[r], i = t - pre[r];
                if (n == 0) {
                    const int x = dag_col[row_begin[r] + i];
                    const int du = vert_deg[b];
                    const int p = lower_bound_i32(nu, du, x);
                    if (p < du && nu[p] == x) atomicOr(&bm[r], 1ull << p);
                } else {
                    const int x = nu[i];
                    const int32_t* __restrict__ nv = dag_col + row_begin[r];
                    const int p = lower_bound_i32(nv, n, x);
                    if (p < n && nv[p] == x) atomicOr(&bm[r], 1ull << i);
                }
            }
            r0 = __shfl(r, min(kWave_ - 1, t_end - 1 - t0), kWave_);
        }
        __syncthreads();
        for (int r = tid; r < R; r += T) {
            const u64 bits = bm[r];
            const int b = row_owner[r];
            const int li = r - vert_base[b];
            const int c = __popcll(bits);
            P.rows[(int64_t)P.rows_off[vert_u[b]] + li] = bits;
            P.arc_c[vert_arc0[b] + li] = c;
            tri += (u64)c;
        }
        __syncthreads();
    }
    flush_build<kLightBlock>(P, tri, st_verts, st_rows, st_bytes, st_entries);
}

// LDS of the heavy build for out-degrees up to max_deg: a hash table of
// N->(u) at most a quarter full (ids, positions), the rows' list bounds, and
// a row of bits per wave.
__host__ __device__ inline int heavy_table_size(int max_deg)
{
    int s = 512;
    while (s < 4 * max_deg) s *= 2;
    return s;
}
static int32_t heavy_lds_bytes(int32_t max_deg)
{
    const int s = heavy_table_size(max_deg), w = (max_deg + 63) / 64;
    return s * 6 + 8 * max_deg + 8 * kHeavyWaves * w + 64;
}

// One workgroup per heavy vertex u, one wave per row: lanes take the entries
// of N->(v_i), four at a time, and look each up in a hash table of N->(u) in
// LDS (nine of ten entries miss, most on their first probe); the row's bits
// gather in the wave's buffer and go out in one coalesced store.  Bound by
// the reads of the neighbours' lists (4 bytes per entry, from L2 and the
// memory-side cache).  R-MAT 20: 4.5 ms here and 2.5 ms for the light
// batches; a search of each entry's row and of its position by bisection, 17
// dependent LDS reads per entry, took 22.4 ms for both.
__global__ void __launch_bounds__(kHeavyBlock) build_heavy_kernel(BuildParams P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int S = heavy_table_size(P.max_deg);
    const int shift = __builtin_clz((unsigned)S) + 1;          // 32 - log2(S)
    int32_t* tab = reinterpret_cast<int32_t*>(smem);
    int32_t* begin = tab + S;
    int32_t* len = begin + P.max_deg;
    u64* bits = reinterpret_cast<u64*>(((uintptr_t)(len + P.max_deg) + 7) & ~(uintptr_t)7);
    const int wmax = (P.max_deg + 63) >> 6;
    uint16_t* pos = reinterpret_cast<uint16_t*>(bits + kHeavyWaves * wmax);
    const int tid = threadIdx.x, lane = lane_of();
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave_);
    u64* mine = bits + wid * wmax;
    const int32_t* __restrict__ dag_ptr = P.dag_ptr;
    const int32_t* __restrict__ dag_col = P.dag_col;
    u64 tri = 0, st_entries = 0, st_rows = 0, st_verts = 0;
    for (int g = blockIdx.x; g < P.plan.n_heavy; g += gridDim.x) {
        const int u = P.order[g];
        const int a0 = dag_ptr[u], d = dag_ptr[u + 1] - a0;
        const int W = (d + 63) >> 6;
        for (int i = tid; i < S; i += kHeavyBlock) tab[i] = -1;
        __syncthreads();
        for (int i = tid; i < d; i += kHeavyBlock) {
            const int v = dag_col[a0 + i];
            unsigned h = (unsigned)v * 0x9E3779B1u >> shift;
            while (atomicCAS(&tab[h], -1, v) != -1) h = (h + 1) & (S - 1);
            pos[h] = (uint16_t)i;
            const int b = dag_ptr[v], n = dag_ptr[v + 1] - b;
            begin[i] = b;
            len[i] = n;
            st_entries += (u64)n;
        }
        __syncthreads();
        u64* __restrict__ out = P.rows + P.rows_off[u];
        for (int r = wid; r < d; r += kHeavyWaves) {
            const int b = begin[r], n = len[r];
            if (lane < W) mine[lane] = 0ull;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int e0 = 0; e0 < n; e0 += 4 * kWave_) {
                int32_t x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int e = e0 + j * kWave_ + lane;
                    x[j] = e < n ? dag_col[b + e] : -2;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (x[j] < 0) continue;
                    unsigned h = (unsigned)x[j] * 0x9E3779B1u >> shift;
                    int32_t key = tab[h];
                    while (key != x[j] && key != -1) {
                        h = (h + 1) & (S - 1);
                        key = tab[h];
                    }
                    if (key == x[j]) {
                        const int p = pos[h];
                        atomicOr(&mine[p >> 6], 1ull << (p & 63));
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const u64 word = lane < W ? mine[lane] : 0ull;
            if (lane < W) out[(int64_t)r * W + lane] = word;
            int c = __popcll(word);
#pragma unroll
            for (int o = kWave_ / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave_);
            if (lane == 0) {
                P.arc_c[a0 + r] = c;
                tri += (u64)c;
            }
        }
        if (tid == 0) {
            st_verts += 1;
            st_rows += (u64)d;
        }
        __syncthreads();
    }
    flush_build<kHeavyBlock>(P, tri, st_verts, st_rows, 4ull * (st_rows + 2ull * st_verts) + 8ull * st_rows, st_entries);
}

// rows_len[u] = d(u) * W(u), the words of u's rows
__global__ void rows_len_kernel(int32_t n, const int32_t* __restrict__ dag_ptr, int32_t min_deg,
                                int32_t* __restrict__ len)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    const int d = dag_ptr[u + 1] - dag_ptr[u];
    len[u] = d >= min_deg ? d * ((d + 63) >> 6) : 0;
}

// The rows of a heavy vertex once more, with rows and bits in the order of
// the DAG instead of ascending id: row and bit i stand for the i-th
// out-neighbour by (key, id).  An out-neighbour's own out-neighbours all come
// later, so the matrix is strictly upper triangular: the tile kernel skips
// the lower half, and the row walks meet zero words.  One workgroup per
// vertex sorts by counting smaller keys (d^2 compares); then a wave per row
// gathers the bits of 64 sorted positions, one per lane, and a ballot is the
// word.
__global__ void __launch_bounds__(256) sorted_rows_kernel(SortedRowsParams P)
{
    __shared__ int32_t key[kMaxDeg];
    __shared__ uint16_t pos[kMaxDeg];     // sorted index -> position
    const int tid = threadIdx.x, lane = lane_of(), wid = tid / kWave_;
    for (int b = blockIdx.x; b < P.n_heavy; b += gridDim.x) {
        const int u = P.order[b];
        const int a0 = P.dag_ptr[u];
        const int d = P.dag_ptr[u + 1] - a0;
        const int W = (d + 63) >> 6;
        for (int i = tid; i < d; i += blockDim.x) {
            const int v = P.dag_col[a0 + i];
            key[i] = P.key ? P.key[v] : P.row_ptr[v + 1] - P.row_ptr[v];
        }
        __syncthreads();
        for (int i = tid; i < d; i += blockDim.x) {
            const int ki = key[i];
            int rank = 0;
            // positions ascend with the id, so ties keep their order
            for (int j = 0; j < d; ++j) rank += (key[j] < ki || (key[j] == ki && j < i)) ? 1 : 0;
            pos[rank] = (uint16_t)i;
            P.hpos[a0 + i] = (uint16_t)rank;
            P.hinv[a0 + rank] = (uint16_t)i;
        }
        __syncthreads();
        const u64* __restrict__ src = P.rows + P.rows_off[u];
        u64* __restrict__ dst = P.hrows + P.hoff[u];
        for (int a = wid; a < d; a += blockDim.x / kWave_) {
            const u64* __restrict__ row = src + (int64_t)pos[a] * W;
            u64 mine = 0;
            for (int w = a >> 6; w < W; ++w) {
                const int i = w * 64 + lane;
                const int s = i < d ? pos[i] : 0;
                const u64 bits = __ballot(i < d && ((row[s >> 6] >> (s & 63)) & 1));
                if (lane == w) mine = bits;
            }
            if (lane < W) dst[(int64_t)a * W + lane] = mine;
        }
        __syncthreads();
    }
}

// Class of every heavy vertex (density_class): of each four of its sorted rows
// one wave takes one, and there the largest arc that the dense kernel could
// take; of its candidates kSampled at even distances, and of each the pairs of
// its neighbours among the candidates that are adjacent.
constexpr int kSampled = 8;
__global__ void __launch_bounds__(256) density_kernel(SortedRowsParams P, const int32_t* __restrict__ arc_c,
                                                      uint8_t* __restrict__ density)
{
    __shared__ unsigned found[4][2];      // adjacent pairs and pairs, per wave
    const int tid = threadIdx.x, lane = lane_of(), wid = __builtin_amdgcn_readfirstlane(tid / kWave_);
    for (int b = blockIdx.x; b < P.n_heavy; b += gridDim.x) {
        const int u = P.order[b];
        const int a0 = P.dag_ptr[u];
        const int d = P.dag_ptr[u + 1] - a0;
        const int W = (d + 63) >> 6;
        int best = 0;                     // |C_uv| << 16 | row
        for (int a = 4 * lane + wid; a < d; a += 4 * kWave_) {
            const int c = arc_c[a0 + P.hinv[a0 + a]];
            if (dense_size(c)) best = max(best, c << 16 | a);
        }
#pragma unroll
        for (int o = kWave_ / 2; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, kWave_));
        const int c = __builtin_amdgcn_readfirstlane(best >> 16), row = __builtin_amdgcn_readfirstlane(best & 0xffff);
        const u64* __restrict__ rows = P.hrows + P.hoff[u];
        const u64 m = lane < W && c ? rows[(int64_t)row * W + lane] : 0ull;
        // the sampled candidates, a lane each
        const int xs = wave_select(m, (2 * (lane & (kSampled - 1)) + 1) * c / (2 * kSampled), W);
        unsigned edges = 0, pairs = 0;
        for (int i = 0; c && i < kSampled; ++i) {
            const int x = __builtin_amdgcn_readlane(xs, i);
            const u64 near = lane < W ? m & rows[(int64_t)x * W + lane] : 0ull;
            const int r = wave_sum_small(__popcll(near));
            pairs += (unsigned)(r * (r - 1) / 2);
            for (int j0 = 0; j0 < r; j0 += kWave_) {
                const int y = wave_select(near, j0 + lane, W);   // any position past the last
                const bool in = j0 + lane < r;
                const u64* __restrict__ ry = rows + (int64_t)(in ? y : 0) * W;
                for (int w0 = x >> 6; w0 < W; w0 += 4) {         // four words in flight
                    u64 q[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) q[t] = ry[min(w0 + t, W - 1)];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const u64 nw = w0 + t < W ? readlane64(near, w0 + t) : 0ull;
                        edges += in ? __popcll(nw & q[t]) : 0;
                    }
                }
            }
        }
#pragma unroll
        for (int o = kWave_ / 2; o > 0; o >>= 1) edges += __shfl_xor(edges, o, kWave_);
        if (lane == 0) {
            found[wid][0] = edges;
            found[wid][1] = pairs;
        }
        __syncthreads();
        if (tid == 0) {
            const unsigned all = found[0][1] + found[1][1] + found[2][1] + found[3][1];
            density[u] = (uint8_t)(all ? density_class(found[0][0] + found[1][0] + found[2][0] + found[3][0], all) : 0);
        }
        __syncthreads();
    }
}

hipError_t launch_density(const SortedRowsParams& P, const int32_t* arc_c, uint8_t* density, hipStream_t s)
{
    if (P.n_heavy <= 0) return hipSuccess;
    density_kernel<<<P.n_heavy < 2048 ? P.n_heavy : 2048, 256, 0, s>>>(P, arc_c, density);
    return hipGetLastError();
}

hipError_t launch_sorted_rows(const SortedRowsParams& P, hipStream_t s)
{
    if (P.n_heavy <= 0) return hipSuccess;
    const int blocks = P.n_heavy < 2048 ? P.n_heavy : 2048;
    sorted_rows_kernel<<<blocks, 256, 0, s>>>(P);
    return hipGetLastError();
}

// per_arc[e] = |C_uv| (the k = 3 per-arc counts)
__global__ void arc_c_to_u64_kernel(int64_t m, const int32_t* __restrict__ arc_c, u64* __restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < m) out[e] = (u64)arc_c[e];
}

hipError_t launch_rows_len(int32_t n, const int32_t* dag_ptr, bool heavy_only, int32_t* len, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    rows_len_kernel<<<(n + 255) / 256, 256, 0, s>>>(n, dag_ptr, heavy_only ? kLightMaxDeg + 1 : 0, len);
    return hipGetLastError();
}

hipError_t launch_build_rows(const BuildParams& P, int32_t blocks, hipStream_t s)
{
    if (P.plan.n_heavy > 0) {
        const int32_t lds = heavy_lds_bytes(P.max_deg);
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute((const void*)build_heavy_kernel,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
        }
        const int32_t n = P.plan.n_heavy < blocks ? P.plan.n_heavy : blocks;
        build_heavy_kernel<<<n, kHeavyBlock, lds, s>>>(P);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (P.plan.n_batches > 0) {
        // twice the workgroups of the heavy build: they are half as wide
        const int32_t n = P.plan.n_batches < 2 * blocks ? P.plan.n_batches : 2 * blocks;
        build_light_kernel<<<n, kLightBlock, light_lds_bytes(P.plan.light_rows), s>>>(P);
    }
    return hipGetLastError();
}

hipError_t launch_arc_c_to_u64(int64_t m, const int32_t* arc_c, u64* out, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    arc_c_to_u64_kernel<<<(unsigned)((m + 255) / 256), 256, 0, s>>>(m, arc_c, out);
    return hipGetLastError();
}

}  // namespace citron
