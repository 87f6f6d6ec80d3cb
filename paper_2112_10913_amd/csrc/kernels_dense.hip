// Dense kernel: k-clique counts of heavy arcs and vertices on the matrix cores.
//
// A work item is an arc u -> v with kDenseMin <= c = |C_uv| <= kDenseMax of a
// count with k >= 6 (dense_arc), or a heavy vertex of up to kDenseMax
// out-neighbours of a count with k = 4 or 5 (dense_vertex), whose subgraph
// takes the place of the arc's below.  These subgraphs are dense (about 0.9 of all
// pairs adjacent in the power-law families), and the search below an arc
// ends, k - 5 levels down, in triangle counts of induced subgraphs
//     T(M) = sum over x, y in M, A[x][y] = 1, of |row x & row y & M|,
// a matrix product: P = A_M A_M^T summed where A is 1, with A_M the rows of M
// masked by M.  One workgroup lays an arc's subgraph out in LDS once, and its
// waves count T(M) for every M the search reaches.
//
//  - Layout.  The c candidates in the order of the DAG (sorted rows, packed
//    like everywhere by parallel bit extract), so A is strictly upper
//    triangular; in three forms: bit rows (the search), 4-bit operand tiles
//    (1.0 is 0b0010 in e2m1) of 32 rows x 64 bits in the operand order of
//    v_mfma_f32_32x32x64_f8f6f4, and for every pair of 32-tiles the bytes
//    A[x][y] in the order of the accumulators.
//  - T(M).  For 32-row tiles x <= y from M's first tile on: the x operand is
//    the tile AND M's 4-bit pattern, with the rows outside M cleared; the y
//    operand is the plain tile; the products are small integers (at most
//    254), exact in fp32.  Sixteen v_cvt_pk_u8_f32 pack the accumulators to
//    bytes and four v_dot4_u32_u8 take them times A; columns outside M are
//    dropped last.  Tiles before M's first and below the diagonal are never
//    touched: a mask that starts at tile t of n costs (n - t)(n - t + 1) / 2
//    tile pairs, whatever its size.
//  - A mask's own pattern is its last vertex's tile row AND its parent's, so
//    nothing is expanded from bits inside the search.
//
// What bounds it: VALU issue, 20 instructions per tile pair (80 of its about
// 150 cycles), then LDS reads (1 KB per operand tile and per byte tile); the
// products themselves take 32 cycles per 32 x 32 x 64.
#include "items.h"
#include "wave.h"

namespace citron {

namespace {

// Waves of a workgroup, and on a CU at most by registers (64 to 185 of the 512
// a SIMD lane has).  Two and three row words leave LDS for several workgroups
// of four waves on a CU (two waves for two words: 41 -> 43 ms); larger
// subgraphs share a workgroup's tiles among more waves.  One-word subgraphs
// are packed by one wave, and at k <= 6 searched in microseconds, so there
// each wave has its own (R-MAT 20, k = 6: their 24 ms fell to 18 against four
// waves and their barriers); deeper searches are worth sharing (R-MAT 16,
// k = 7: 33.3 ms against 32.7).
__host__ __device__ constexpr int dense_waves(int K, int max_k)
{
    return K == 1 ? (max_k <= 6 ? 1 : 4) : (K <= 3 ? 4 : (K == 5 ? 12 : 8));
}
__host__ __device__ constexpr int dense_cu_waves(int K) { return K == 1 ? 28 : (K == 2 ? 20 : (K <= 4 ? 16 : (K == 5 ? 12 : 8))); }
constexpr int kDenseClaim = 8;              // items a workgroup claims at once, at most

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

struct DenseParams {
    ItemSpace items;
    int32_t max_k;
    int32_t* progress;       // host-mapped word (nullable)
    int32_t progress_base;   // items the launch claimed before this kernel
};

// Operand tiles of K row words (K tiles of 64 bits, 2K tiles of 32 rows): row
// tile t holds bit tiles t/2 .. K-1, stored in that order.
__host__ __device__ constexpr int tile_base(int K, int t)
{
    return 2 * (t >> 1) * K - (t >> 1) * ((t >> 1) - 1) + (t & 1) * (K - (t >> 1));
}
__host__ __device__ constexpr int n_tiles(int K) { return tile_base(K, 2 * K); }
// byte tiles of row-tile pairs x <= y
__host__ __device__ constexpr int pair_base(int K, int x) { return x * 2 * K - x * (x - 1) / 2; }
__host__ __device__ constexpr int n_pairs(int K) { return K * (2 * K + 1); }
static_assert(tile_base(4, 8) == 20 && n_pairs(4) == 36, "upper triangles of 8 x 4 and 8 x 8 tiles");
static_assert(1024 * (n_tiles(6) + n_pairs(6)) + 8 * 64 * 36 + 8 * dense_waves(6, 32) * 26 * 12 + 2048 <= 160 * 1024,
              "the largest instance fits LDS at k = 32");

// LDS of a workgroup: [operand tiles 1 KB each][byte tiles 1 KB each][bit
// rows][stacks: per wave, levels x (mask, rest)][items][branch counter].
__host__ __device__ constexpr int dense_stack_words(int K, int max_k)
{
    return (max_k > 6 ? max_k - 6 : 0) * 2 * K;
}
__host__ __device__ constexpr int dense_lds_bytes(int K, int max_k)
{
    return 1024 * (n_tiles(K) + n_pairs(K)) + 8 * 64 * K * K +
           8 * dense_waves(K, max_k) * dense_stack_words(K, max_k) + 4 * kItFields * kMaxClaim + 16;
}

__device__ __forceinline__ u64 uniform64(u64 v)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return ((u64)hi << 32) | lo;
}

// true in the lanes (mod 32) whose bit is set
__device__ __forceinline__ bool lanes32(unsigned m)
{
    return __builtin_amdgcn_inverse_ballot_w64(((u64)m << 32) | m);
}

// Eight bits to eight 4-bit values, 2 (1.0 in e2m1) for a set bit.
__device__ __forceinline__ int spread4(unsigned b)
{
    b = (b | (b << 12)) & 0x001E001Eu;      // the byte comes shifted up by one
    b = (b | (b << 6)) & 0x06060606u;
    b = (b | (b << 3)) & 0x22222222u;
    return (int)b;
}

template <int K>
struct Dense {
    const v4i* tiles;        // operand tiles
    const v4i* bytes;        // byte tiles
    const u64* rows;         // bit rows, K words each
    int nt;                  // 32-row tiles in use, ceil(c / 32)

    __device__ __forceinline__ void row(int x, u64 (&r)[K]) const
    {
#pragma unroll
        for (int w = 0; w < K; ++w) r[w] = uniform64(rows[x * K + w]);
    }

    // T(M), this lane's share.  pat: M's 4-bit patterns (per bit tile, the
    // lane's half).  kSplit: the row tiles x = first mod kSplit only.
    template <int kSplit>
    __device__ __forceinline__ unsigned triangles(const u64 (&M)[K], const v4i (&pat)[K], int first) const
    {
        const int lane = lane_of();
        unsigned sum = 0, s[2 * K];      // per row tile y: its columns outside M are dropped at the end
#pragma unroll
        for (int y = 0; y < 2 * K; ++y) s[y] = 0;
#pragma unroll
        for (int x = 0; x < 2 * K; ++x) {
            const unsigned mx = (unsigned)(M[x >> 1] >> (32 * (x & 1)));
            if (mx == 0u || (kSplit > 1 && x % kSplit != first)) continue;
            const int in = lanes32(mx) ? -1 : 0;
            v4i a[K];
#pragma unroll
            for (int z = 0; z < K; ++z) {
                if (z < (x >> 1)) continue;
                a[z] = tiles[(tile_base(K, x) + z - (x >> 1)) * kWave + lane] & pat[z] & in;
            }
#pragma unroll
            for (int y = 0; y < 2 * K; ++y) {
                if (y < x || y >= nt) continue;
                const v4i m = bytes[(pair_base(K, x) + y - x) * kWave + lane];
                // chains of at most four bit tiles: with bit y itself never
                // set, a product is then at most 255, what a byte holds
#pragma unroll
                for (int chain = 0; chain < 2; ++chain) {
                    const int z0 = (y >> 1) + 4 * chain;
                    if (z0 >= K) continue;
                    v16f p = {};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int z = z0 + i;
                        if (z >= K) continue;
                        const v4i b = tiles[(tile_base(K, y) + z - (y >> 1)) * kWave + lane];
                        const v8i a8 = {a[z][0], a[z][1], a[z][2], a[z][3], 0, 0, 0, 0};
                        const v8i b8 = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
                        p = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, p, 4, 4, 0, 0, 0, 0);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        unsigned w = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) w = __builtin_amdgcn_cvt_pk_u8_f32(p[4 * q + j], j, w);
                        s[y] = __builtin_amdgcn_udot4(w, (unsigned)m[q], s[y], false);
                    }
                }
            }
        }
#pragma unroll
        for (int y = 0; y < 2 * K; ++y) {
            const unsigned my = (unsigned)(M[y >> 1] >> (32 * (y & 1)));
            sum += lanes32(my) ? s[y] : 0u;
        }
        return sum;
    }

    // Sum of T(P & row x) over x in R (R within P).  all: P is the whole
    // subgraph (its pattern is all ones).
    __device__ __forceinline__ u64 last_levels(const u64 (&P)[K], u64 (&R)[K], bool all) const
    {
        const int lane = lane_of();
        const int half = lane >> 5;
        v4i pp[K];
#pragma unroll
        for (int z = 0; z < K; ++z) {
            const unsigned b = half ? (unsigned)(P[z] >> 32) : (unsigned)P[z];
#pragma unroll
            for (int i = 0; i < 4; ++i) pp[z][i] = all ? 0x22222222 : spread4(((b >> (8 * i)) & 0xffu) << 1);
        }
        unsigned sum = 0;      // at most 384 masks of 78 tile pairs, 2 x 16 x 255 each: below 2^28
#pragma unroll
        for (int w = 0; w < K; ++w) {
            u64 r = R[w];
            while (r) {
                const int x = w * 64 + __builtin_ctzll(r);
                r &= r - 1;
                u64 M[K];
                row(x, M);
                int c = 0;
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    M[i] &= P[i];
                    c += __popcll(M[i]);
                }
                if (c < 3) continue;
                v4i pat[K];
#pragma unroll
                for (int z = 0; z < K; ++z) {
                    if (z < w) {
                        pat[z] = v4i{0, 0, 0, 0};     // row x starts after bit x
                        continue;
                    }
                    pat[z] = tiles[(tile_base(K, x >> 5) + z - w) * kWave + half * 32 + (x & 31)] & pp[z];
                }
                sum += triangles<1>(M, pat, 0);
            }
        }
        return (u64)sum;
    }

    // Depth-first search below a node with mask M, r >= 4 vertices still to
    // choose; this lane's share.  stack: (r - 4) levels of (mask, rest).
    __device__ __forceinline__ u64 search(const u64 (&M0)[K], int r, u64* stack) const
    {
        const int lane = lane_of();
        u64 sum = 0;
        u64 M[K], R[K];
#pragma unroll
        for (int w = 0; w < K; ++w) M[w] = R[w] = M0[w];
        if (r == 4) return last_levels(M, R, false);
        int t = 0;             // levels on the stack; r - t vertices to choose at this node
        for (;;) {
            int x = -1;
#pragma unroll
            for (int w = 0; w < K; ++w)
                if (x < 0 && R[w]) {
                    x = w * 64 + __builtin_ctzll(R[w]);
                    R[w] &= R[w] - 1;
                }
            if (x < 0) {
                if (t == 0) break;
                --t;
#pragma unroll
                for (int w = 0; w < K; ++w) {
                    M[w] = uniform64(stack[t * 2 * K + w]);
                    R[w] = uniform64(stack[t * 2 * K + K + w]);
                }
                continue;
            }
            u64 ch[K];
            row(x, ch);
            int c = 0;
#pragma unroll
            for (int w = 0; w < K; ++w) {
                ch[w] &= M[w];
                c += __popcll(ch[w]);
            }
            const int need = r - t - 1;
            if (c < need) continue;
            if (need == 4) {
                u64 rest[K];
#pragma unroll
                for (int w = 0; w < K; ++w) rest[w] = ch[w];
                sum += last_levels(ch, rest, false);
                continue;
            }
#pragma unroll
            for (int w = 0; w < K; ++w) {
                if (lane == 0) {
                    stack[t * 2 * K + w] = M[w];
                    stack[t * 2 * K + K + w] = R[w];
                }
                M[w] = R[w] = ch[w];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            ++t;
        }
        return sum;
    }
};

// Bit rows of the subgraph of mask M (lane q holds word q, W words) over the
// sorted rows `src`, packed to K words each: the waves take 64 rows at a
// time.  Rows c .. 64 K - 1 are zero.
template <int K, int kWaves>
__device__ void pack_rows(const u64* __restrict__ src, int W, u64 M, int c, u64* __restrict__ dst)
{
    const int lane = lane_of();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (int a0 = wid * kWave; a0 < 64 * K; a0 += kWaves * kWave) {
        const int a = a0 + lane;
        const bool valid = a < c;
        const int xa = a0 < c ? wave_select(M, a, W) : 0;
        // rows are strictly upper triangular: nothing before the first row's word
        const int w0 = a0 < c ? __builtin_amdgcn_readfirstlane(xa) >> 6 : W;
        const u64* __restrict__ row = src + (int64_t)(valid ? xa : 0) * W;
        u64 out = 0;
        int off = 0;
        for (int w = 0; w < W; ++w) {
            const u64 mw = readlane64(M, w);
            if (mw == 0ull) continue;
            const int pc = __popcll(mw), sh = off & 63;
            const u64 p = w >= w0 && valid ? pext_apply(row[w], pext_prep(mw)) : 0ull;
            out |= p << sh;
            if (sh + pc >= 64) {
                dst[a * K + (off >> 6)] = out;
                out = sh ? p >> (64 - sh) : 0ull;
            }
            off += pc;
        }
        if (off & 63) dst[a * K + (off >> 6)] = out;
    }
}

// Operand and byte tiles of the bit rows.
template <int K, int kWaves>
__device__ void build_tiles(const u64* __restrict__ rows, v4i* __restrict__ tiles, v4i* __restrict__ bytes, int nt)
{
    const int lane = lane_of();
    const int wid = threadIdx.x / kWave;
    const int half = lane >> 5, l = lane & 31;
    const unsigned* __restrict__ rows32 = reinterpret_cast<const unsigned*>(rows);
    int f = 0;
    for (int x = 0; x < 2 * K; ++x)
        for (int z = x >> 1; z < K; ++z, ++f) {
            if (f % kWaves != wid) continue;
            const unsigned b = rows32[((32 * x + l) * K + z) * 2 + half];
            v4i v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = spread4(((b >> (8 * i)) & 0xffu) << 1);
            tiles[f * kWave + lane] = v;
        }
    for (int x = 0; x < nt; ++x)
        for (int y = x; y < nt; ++y) {
            const int p = pair_base(K, x) + y - x;
            if (p % kWaves != wid) continue;
            // accumulator 4 q + j of this lane: row 8 q + 4 half + j of tile x, column l of tile y
            v4i v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned d = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned b = rows32[(32 * x + 8 * q + 4 * half + j) * K * 2 + y];
                    d |= ((b >> l) & 1u) << (8 * j);
                }
                v[q] = (int)d;
            }
            bytes[p * kWave + lane] = v;
        }
}

// One item: an arc's subgraph (mask row r of its source's rows, packed) or a
// whole vertex's (its rows as they are), laid out once; then its first level
// is shared among the waves.  need: vertices to choose from the subgraph, 3
// (one triangle count, k = 4) or more.  per_arc (vertices only): counts per
// first vertex x go to per_arc[inv[x]].  Returns this lane's
// share of the count.
template <int K, int kWaves>
__device__ __forceinline__ u64 dense_item(const u64* __restrict__ src, int W, int d, int r, int need, int part, int P,
                                          int max_k, unsigned char* smem, u64* stacks, int* branch, u64* per_arc,
                                          const uint16_t* inv)
{
    v4i* tiles = reinterpret_cast<v4i*>(smem);
    v4i* bytes = tiles + n_tiles(K) * kWave;
    u64* rows = reinterpret_cast<u64*>(bytes + n_pairs(K) * kWave);
    const int lane = lane_of();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int c = d;
    if (threadIdx.x == 0) *branch = 0;
    if (r < 0) {
        // W = K: the vertex's class is that of its out-degree
        for (int i = threadIdx.x; i < 64 * K * K; i += kWaves * kWave) rows[i] = i < d * K ? src[i] : 0ull;
    } else {
        const u64 M = lane < W ? src[(int64_t)r * W + lane] : 0ull;
        c = wave_sum_small(__popcll(M));
        // rows past the last candidate, and words past a row's last, read as zero
        for (int i = threadIdx.x; i < 64 * K * K; i += kWaves * kWave) rows[i] = 0ull;
        __syncthreads();
        pack_rows<K, kWaves>(src, W, M, c, rows);
    }
    const int nt = (c + 31) >> 5;
    __syncthreads();
    build_tiles<K, kWaves>(rows, tiles, bytes, nt);
    __syncthreads();
    const Dense<K> D{tiles, bytes, rows, nt};
    u64 all[K];
#pragma unroll
    for (int w = 0; w < K; ++w) {
        const int rem = c - 64 * w;
        all[w] = rem >= 64 ? ~0ull : (rem > 0 ? (1ull << rem) - 1ull : 0ull);
    }
    u64 sum = 0;
    if (need == 3 && !per_arc) {
        v4i pat[K];
#pragma unroll
        for (int z = 0; z < K; ++z) pat[z] = v4i{0x22222222, 0x22222222, 0x22222222, 0x22222222};
        sum = D.template triangles<kWaves>(all, pat, wid);
        __syncthreads();
        return sum;
    }
    for (;;) {
        int j = 0;
        if (lane == 0) j = atomicAdd(branch, 1);
        const int x = part + P * __builtin_amdgcn_readfirstlane(j);
        if (x >= c) break;
        u64 s = 0;
        if (need == 3) {
            // per-arc counts of k = 4 want row x's own sum: lanes over its y
            u64 rx[K];
            D.row(x, rx);
            for (int y = lane; y < c; y += kWave)
                if ((rows[x * K + (y >> 6)] >> (y & 63)) & 1)
#pragma unroll
                    for (int w = 0; w < K; ++w) s += (u64)__popcll(rx[w] & rows[y * K + w]);
        } else if (need == 4) {
            u64 R[K];
#pragma unroll
            for (int w = 0; w < K; ++w) R[w] = (x >> 6) == w ? 1ull << (x & 63) : 0ull;
            s = D.last_levels(all, R, true);
        } else {
            u64 ch[K];
            D.row(x, ch);
            int cc = 0;
#pragma unroll
            for (int w = 0; w < K; ++w) cc += __popcll(ch[w]);
            if (cc >= need - 1) s = D.search(ch, need - 1, stacks + wid * dense_stack_words(K, max_k));
        }
        sum += s;
        if (per_arc) {
            const u64 t = wave_sum_u64(s);
            if (lane == 0 && t) atomicAdd(per_arc + inv[x], t);
        }
    }
    __syncthreads();
    return sum;
}

}  // namespace

template <int K, int kWaves>
__global__ void __launch_bounds__(kWaves * kWave)
    __attribute__((amdgpu_waves_per_eu(dense_cu_waves(K) / 4))) dense_kernel(DenseParams P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_of();
    u64* stacks = reinterpret_cast<u64*>(smem + 1024 * (n_tiles(K) + n_pairs(K)) + 8 * 64 * K * K);
    int32_t* item = reinterpret_cast<int32_t*>(stacks + kWaves * dense_stack_words(K, P.max_k));
    int* shared = item + kItFields * kMaxClaim;      // [0] branch counter, [1] first item of the run
    u64 acc = 0ull;
    int cur = -1;
    int shard = blockIdx.x % kClaimShards;
    bool fresh = true;
    const int acc_slot = (int)((blockIdx.x * kWaves + threadIdx.x / kWave) & (kAccSlots - 1)) * kAccStride;
    for (;;) {
        if (threadIdx.x < kWave) {
            const int g = claim_run(P.items, blockIdx.x, gridDim.x, shard, fresh);
            const int n = g < 0 ? 0 : run_length(P.items, g);
            decode_run<kDenseClasses - K>(P.items, g, n, item);
            if (lane == 0) {
                shared[1] = g;
                if (P.progress && g >= 0 && (((g + n - 1) ^ (g - 1)) & ~511))
                    __hip_atomic_store(P.progress, P.progress_base + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        __syncthreads();
        const int g0 = __builtin_amdgcn_readfirstlane(shared[1]);
        if (g0 < 0) break;
        const int n = run_length(P.items, g0);
        for (int j = 0; j < n; ++j) {
            auto field = [&](int f) { return __builtin_amdgcn_readfirstlane(item[f * kMaxClaim + j]); };
            const int qi = field(kItQuery);
            if (qi != cur) {
                if (cur >= 0) wave_flush(acc, 0, P.items.queries[cur].acc + acc_slot, P.items.queries[cur].overflow);
                acc = 0ull;
                cur = qi;
            }
            const QueryDesc& q = P.items.queries[qi];
            const int tag = field(kItTag), r = field(kItRow), pw = field(kItPart);
            const int W = (field(kItDegree) + 63) >> 6;
            const u64* src = q.rows.hrows + field(kItRowsOff);
            const bool vertex = field(kItKind) == kItemDenseVertex;
            const int a0 = field(kItArc0);
            const u64 s = dense_item<K, kWaves>(src, W, field(kItDegree), r, vertex ? q.k - 1 : q.k - 2, pw & 0xffff, pw >> 16,
                                        P.max_k, smem, stacks, shared, vertex && q.per_arc ? q.per_arc + a0 : nullptr,
                                        q.rows.hinv + a0);
            acc += s;            // a lane adds at most 2^28 per mask's children: 2^36 of them before it could wrap
            if (q.per_arc && !vertex) {
                const u64 t = wave_sum_u64(s);
                if (lane == 0 && t) atomicAdd(q.per_arc + tag, t);
            }
        }
        // the last item's closing barrier separates its reads of the run from the next claim
    }
    if (cur >= 0) wave_flush(acc, 0, P.items.queries[cur].acc + acc_slot, P.items.queries[cur].overflow);
}

template <int K, int kWaves>
static hipError_t launch_class(const CountLaunch& cl, int cus, int32_t base, hipStream_t s)
{
    const int space = kDenseClasses - K;
    const int32_t n = cl.space_items[space];
    if (n <= 0) return hipSuccess;
    const int lds = dense_lds_bytes(K, cl.max_k);
    DenseParams P;
    P.items.queries = cl.queries;
    P.items.n_queries = cl.n_queries;
    P.items.total = n;
    P.items.cursors = cl.item_ctr + space * kClaimInts;
    P.max_k = cl.max_k;
    P.progress = cl.progress;
    P.progress_base = base;
    // as many workgroups as LDS and registers hold, no more than items
    const int by_lds = 160 * 1024 / lds, by_regs = dense_cu_waves(K) / kWaves;
    int64_t blocks = (int64_t)cus * (by_lds < by_regs ? by_lds : by_regs);
    if (blocks > n) blocks = n;
    set_runs(P.items, blocks, kDenseClaim);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)dense_kernel<K, kWaves>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    dense_kernel<K, kWaves><<<(unsigned)blocks, kWaves * kWave, lds, s>>>(P);
    return hipGetLastError();
}

hipError_t launch_dense(const CountLaunch& cl, hipStream_t s)
{
    if (launch_items(cl) == cl.space_items[kRestSpace]) return hipSuccess;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    int32_t base = 0;
    if (e == hipSuccess) e = launch_class<6, dense_waves(6, 6)>(cl, cus, base, s);
    base += cl.space_items[0];
    if (e == hipSuccess) e = launch_class<5, dense_waves(5, 6)>(cl, cus, base, s);
    base += cl.space_items[1];
    if (e == hipSuccess) e = launch_class<4, dense_waves(4, 6)>(cl, cus, base, s);
    base += cl.space_items[2];
    if (e == hipSuccess) e = launch_class<3, dense_waves(3, 6)>(cl, cus, base, s);
    base += cl.space_items[3];
    if (e == hipSuccess) e = launch_class<2, dense_waves(2, 6)>(cl, cus, base, s);
    base += cl.space_items[4];
    if (e == hipSuccess)
        e = cl.max_k <= 6 ? launch_class<1, dense_waves(1, 6)>(cl, cus, base, s)
                          : launch_class<1, dense_waves(1, 7)>(cl, cus, base, s);
    return e;
}

}  // namespace citron
