// Dense kernel: k-clique counts of heavy arcs and vertices on the matrix cores.
//
// A work item is an arc u -> v with kDenseMin <= c = |C_uv| <= kDenseMax of a
// count with k >= 6 (dense_arc: from k = 7 on of a dense enough subgraph), or k
// = 5 for u of more than kDenseMax out-neighbours and in per-arc counts, or a
// heavy vertex of at most kDenseMax out-neighbours of a count with k = 4 or 5
// (dense_vertex), whose subgraph takes the place of the arc's below.  The
// search below an arc ends, k - 5 levels down, in triangle counts of induced
// subgraphs
//     T(M) = sum over x, y in M, A[x][y] = 1, of |row x & row y & M|,
// a matrix product: P = A_M A_M^T summed where A is 1, with A_M the rows of M
// masked by M.  A is the same for every M of an item, so the products of all
// its masks are added up in the accumulators, and summed where A is 1 once.
//
//  - Layout.  The c candidates in the order of the DAG (sorted rows, packed
//    like everywhere by parallel bit extract), so A is strictly upper
//    triangular; in two forms in LDS: bit rows (the search), and 4-bit
//    operand tiles (1.0 is 0b0010 in e2m1) of 32 rows x 64 bits in the
//    operand order of v_mfma_f32_32x32x64_f8f6f4.
//  - A mask.  For 32-row tiles x <= y from M's first tile on: both operands
//    are the tile AND M's 4-bit pattern, with the rows outside M cleared (one
//    v_bitop3 per register); a tile serves as x and as y.  A mask's own
//    pattern is its last vertex's tile row AND its node's, so nothing is
//    expanded from bits inside the search.  A mask that starts at tile t of n
//    costs (n - t)(n - t + 1) / 2 tile pairs, whatever its size.
//  - Accumulators hold small integers, exact in fp32: they are summed before
//    any could reach 2^20.
//
// What bounds it (R-MAT 20, k = 6, counters): the matrix cores are busy 0.63 to
// 0.72 of the time for two to six row words, with vector instructions issued in
// 0.47 to 0.56 of the cycles beside them and two waves of 255 registers per
// SIMD to hide the latency of the rest; for one row word 0.49, beside 0.71 for
// layout and search.  LDS is read in 0.15 to 0.23 of the cycles, with hardly a
// bank conflict.  With every mask's products packed to bytes and summed on
// their own, 20 VALU instructions per tile pair, R-MAT 20, k = 6 took 165 ms
// and R-MAT 16, k = 7 32.7 ms; now 94 and 20.8 ms.
#include "items.h"
#include "wave.h"

namespace citron {

namespace {

// Waves of a workgroup, and on a CU at most by registers (100 for one row
// word, else up to 256 of the 512 a SIMD lane has).  A workgroup of one wave
// waits at no barrier, so up to three words, where LDS holds all eight waves'
// subgraphs, each wave has an item of its own (two words with 1, 2 and 4
// waves: 22.1, 26.6 and 34.2 ms of R-MAT 20, k = 6; three words with 2 and 4:
// 28.9 and 31.5 ms; four with 4 and 8: 14.8 and 19.4 ms).
__host__ __device__ constexpr int dense_waves(int K) { return K <= 3 ? 1 : (K == 4 ? 2 : 4); }
__host__ __device__ constexpr int dense_cu_waves(int K) { return K == 1 ? 16 : 8; }
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
static_assert(tile_base(4, 8) == 20, "upper triangle of 8 x 4 tiles");
static_assert(1024 * n_tiles(6) + 8 * 64 * 36 + 8 * dense_waves(6) * 26 * 12 + 2048 <= 160 * 1024,
              "the largest instance fits LDS at k = 32");

// The tile pairs of a pass over an item's masks: K = 1 and 2 hold all of
// theirs in accumulators (3 and 10 of 16 registers) at once; larger
// subgraphs go over the masks once per block of at most 10, what 256
// registers hold beside the operands (blocks of up to 11 spill and cost 41
// instead of 32 ms for three words and 53 instead of 19 for four).
struct Block {
    int x0, x1, y0, y1;
};
constexpr int n_passes(int K) { return K <= 2 ? 1 : (K == 3 ? 3 : (K == 4 ? 5 : (K == 5 ? 8 : 11))); }
constexpr Block block_of(int K, int p)
{
    constexpr Block k3[] = {{0, 2, 0, 4}, {0, 2, 4, 6}, {2, 6, 2, 6}};
    constexpr Block k4[] = {{0, 2, 0, 4}, {0, 2, 4, 8}, {2, 4, 2, 6}, {2, 4, 6, 8}, {4, 8, 4, 8}};
    constexpr Block k5[] = {{0, 2, 0, 4}, {0, 2, 4, 7}, {0, 2, 7, 10}, {2, 4, 2, 6},
                            {2, 4, 6, 10}, {4, 6, 4, 7}, {4, 6, 7, 10}, {6, 10, 6, 10}};
    constexpr Block k6[] = {{0, 2, 0, 4}, {0, 2, 4, 8}, {0, 2, 8, 12}, {2, 4, 2, 6}, {2, 4, 6, 10}, {2, 4, 10, 12},
                            {4, 6, 4, 8}, {4, 6, 8, 12}, {6, 8, 6, 9}, {6, 8, 9, 12}, {8, 12, 8, 12}};
    return K <= 2 ? Block{0, 2 * K, 0, 2 * K} : (K == 3 ? k3[p] : (K == 4 ? k4[p] : (K == 5 ? k5[p] : k6[p])));
}
// masks a pass adds up before it sums: an accumulator stays below 2^20, so
// that sixteen of them are exact in fp32
constexpr int max_masks(int K) { return (1 << 20) / (64 * K); }

// LDS of a workgroup: [operand tiles 1 KB each][bit rows][stacks: per wave,
// levels x (mask, rest)][items][first item of the run, branch counters].
__host__ __device__ constexpr int dense_stack_words(int K, int max_k)
{
    return (max_k > 6 ? max_k - 6 : 0) * 2 * K;
}
__host__ __device__ constexpr int dense_lds_bytes(int K, int max_k)
{
    return 1024 * n_tiles(K) + 8 * 64 * K * K +
           8 * dense_waves(K) * dense_stack_words(K, max_k) + 4 * kItFields * kMaxClaim + 64;
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
    const u64* rows;         // bit rows, K words each
    int nt;                  // 32-row tiles in use, ceil(c / 32)

    __device__ __forceinline__ void row(int x, u64 (&r)[K]) const
    {
#pragma unroll
        for (int w = 0; w < K; ++w) r[w] = uniform64(rows[x * K + w]);
    }

    // A[x tile][y tile] in the order of the accumulators: 4 q + j of this lane
    // is row 8 q + 4 half + j of tile x, column l of tile y.
    __device__ __forceinline__ unsigned bit(int x, int y, int i) const
    {
        const int lane = lane_of();
        const unsigned* rows32 = reinterpret_cast<const unsigned*>(rows) + 4 * (lane >> 5) * K * 2;
        return (rows32[(32 * x + 8 * (i >> 2) + (i & 3)) * K * 2 + y] >> (lane & 31)) & 1u;
    }
    __device__ __forceinline__ v4i adjacency(int x, int y) const
    {
        v4i v;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = (int)(bit(x, y, 4 * q) | bit(x, y, 4 * q + 1) << 8 | bit(x, y, 4 * q + 2) << 16 |
                         bit(x, y, 4 * q + 3) << 24);
        return v;
    }

    // The whole subgraph's triangles, this lane's share: the row tiles x =
    // first mod the waves only.  With one mask there is nothing to add up, so
    // the products go to bytes (sixteen v_cvt_pk_u8_f32 and four
    // v_dot4_u32_u8 per tile pair).
    __device__ __forceinline__ unsigned triangles(int first) const
    {
        const int lane = lane_of();
        unsigned sum = 0;
#pragma unroll
        for (int x = 0; x < 2 * K; ++x) {
            if (x >= nt || x % dense_waves(K) != first) continue;
            v4i a[K];
#pragma unroll
            for (int z = 0; z < K; ++z) {
                if (z < (x >> 1)) continue;
                a[z] = tiles[(tile_base(K, x) + z - (x >> 1)) * kWave + lane];
            }
#pragma unroll
            for (int y = 0; y < 2 * K; ++y) {
                if (y < x || y >= nt) continue;
                const v4i m = adjacency(x, y);
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
                        sum = __builtin_amdgcn_udot4(w, (unsigned)m[q], sum, false);
                    }
                }
            }
        }
        return sum;
    }

    // The pattern of all of P's bits (per bit tile, the lane's half).
    __device__ __forceinline__ void spread(const u64 (&P)[K], v4i (&pp)[K]) const
    {
        const int half = lane_of() >> 5;
#pragma unroll
        for (int z = 0; z < K; ++z) {
            const unsigned b = half ? (unsigned)(P[z] >> 32) : (unsigned)P[z];
#pragma unroll
            for (int i = 0; i < 4; ++i) pp[z][i] = spread4(((b >> (8 * i)) & 0xffu) << 1);
        }
    }
};

// The accumulators of one pass: tile pairs x <= y with x in [x0, x1), y in
// [y0, y1).
template <int K, int kPass>
struct Pass {
    static constexpr Block B = block_of(K, kPass);
    static constexpr int index(int x, int y)
    {
        int n = 0;
        for (int i = B.x0; i < x; ++i)
            for (int j = B.y0; j < B.y1; ++j) n += j >= i;
        for (int j = B.y0; j < y; ++j) n += j >= x;
        return n;
    }
    static constexpr int kPairs = index(B.x1, B.y0);
    static constexpr int kFirst = B.x0 >> 1;      // first bit tile of any operand
    v16f acc[kPairs];

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) acc[i] = v16f{};
    }

    static constexpr bool kHeld = K <= 2;      // the operand tiles, masked by the node's pattern, stay in registers
    v4i held[kHeld ? n_tiles(K) : 1];

    // Adds A_M A_M^T of this pass's tile pairs for the masks M = N & row x,
    // x in N, x = first mod stride.  Tile by tile of x: rows of tile t have no bit before it, so
    // the code for each first tile is straight, operand reads first.
    template <int kTile = B.x0>
    __device__ __forceinline__ void add(const Dense<K>& D, const u64 (&N)[K], const v4i (&pp)[K], int stride, int first)
    {
        if constexpr (kTile < B.x1) {
            if constexpr (kHeld && kTile == B.x0)
#pragma unroll
                for (int x = 0; x < 2 * K; ++x)
#pragma unroll
                    for (int z = x >> 1; z < K; ++z) {
                        const int f = tile_base(K, x) + z - (x >> 1);
                        held[f] = D.tiles[f * kWave + lane_of()] & pp[z];
                    }
            for (int t = kTile == B.x0 ? 0 : kTile; t <= kTile; ++t) {
                unsigned r = 0;
#pragma unroll
                for (int w = 0; w < K; ++w)
                    if (w == (t >> 1)) r = (unsigned)(N[w] >> (32 * (t & 1)));
                if (stride > 1) r &= (unsigned)__ballot((32 * t + lane_of()) % stride == first);
                if (r) add_tile<kTile>(D, N, pp, t, r);
            }
            add<kTile + 1>(D, N, pp, stride, first);
        }
    }

    template <int kTile>
    __device__ __forceinline__ void add_tile(const Dense<K>& D, const u64 (&N)[K], const v4i (&pp)[K], int t, unsigned r)
    {
        constexpr int X = B.x1 - B.x0;
        constexpr int kY = kTile > B.y0 ? kTile : B.y0;
        constexpr int kZ = kTile >> 1;             // first bit tile
        const int lane = lane_of();
        const u64* rows = D.rows + 32 * t * K;
        const v4i* pats = D.tiles + (tile_base(K, t) - (t >> 1)) * kWave + (lane & 32);
        u64 row[K];
        v4i rpat[K];
        int x = __builtin_ctz(r);
        auto fetch = [&] {
#pragma unroll
            for (int z = kZ; z < K; ++z) {
                row[z] = rows[x * K + z];
                rpat[z] = pats[z * kWave + x];
            }
        };
        fetch();
        for (;;) {
            u64 M[K];
            v4i pat[K];
#pragma unroll
            for (int z = kZ; z < K; ++z) {
                M[z] = uniform64(row[z]) & N[z];
                pat[z] = kHeld ? rpat[z] : rpat[z] & pp[z];
            }
            // the next row's words and pattern are read beside the products
            r &= r - 1;
            if (r) x = __builtin_ctz(r);
            fetch();
            v4i ax[X][K];
            auto operand = [&](int x, int z0, v4i (&a)[K]) {
                const int in = lanes32((unsigned)(M[x >> 1] >> (32 * (x & 1)))) ? -1 : 0;
#pragma unroll
                for (int z = 0; z < K; ++z)
                    if (z >= z0) {
                        const int f = tile_base(K, x) + z - (x >> 1);
                        a[z] = (kHeld ? held[kHeld ? f : 0] : D.tiles[f * kWave + lane]) & pat[z] & in;
                    }
            };
            // x tiles that are none of the y tiles
#pragma unroll
            for (int x = kTile; x < B.x1; ++x)
                if (x < kY) operand(x, kY >> 1, ax[x - B.x0]);
#pragma unroll
            for (int y = kY; y < B.y1; ++y) {
                v4i own[K];
                v4i (&ay)[K] = y < B.x1 ? ax[y < B.x1 ? y - B.x0 : 0] : own;
                operand(y, y >> 1, ay);
#pragma unroll
                for (int z = 0; z < K; ++z) {
                    if (z < (y >> 1)) continue;
#pragma unroll
                    for (int x = kTile; x < B.x1; ++x) {
                        if (x > y) continue;
                        v16f& p = acc[index(x, y)];
                        const v4i a = ax[x - B.x0][z], b = ay[z];
                        const v8i a8 = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
                        const v8i b8 = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
                        p = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, p, 4, 4, 0, 0, 0, 0);
                    }
                }
            }
            if (!r) break;
        }
    }

    // The accumulators where A is 1, this lane's share.
    __device__ __forceinline__ u64 sum(const Dense<K>& D) const
    {
        const int lane = lane_of();
        unsigned s = 0;          // at most 10 pairs x 16 x 2^20
#pragma unroll
        for (int x = B.x0; x < B.x1; ++x) {
#pragma unroll
            for (int y = B.y0; y < B.y1; ++y) {
                if (y < x || y >= D.nt) continue;
                const v16f& p = acc[index(x, y)];
                float f = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) f = fmaf((float)D.bit(x, y, i), p[i], f);
                s += (unsigned)f;
            }
        }
        return (u64)s;
    }
};

// Bit rows of the subgraph of mask M (lane q holds word q, W words) over the
// sorted rows `src`, packed to K words each: the waves take 64 rows at a
// time.  Rows c .. 64 K - 1 are zero.
template <int K>
__device__ void pack_rows(const u64* __restrict__ src, int W, u64 M, int c, u64* __restrict__ dst)
{
    const int lane = lane_of();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (int a0 = wid * kWave; a0 < 64 * K; a0 += dense_waves(K) * kWave) {
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

// Operand tiles of the bit rows.
template <int K>
__device__ void build_tiles(const u64* __restrict__ rows, v4i* __restrict__ tiles)
{
    const int lane = lane_of();
    const int wid = threadIdx.x / kWave;
    const int half = lane >> 5, l = lane & 31;
    const unsigned* __restrict__ rows32 = reinterpret_cast<const unsigned*>(rows);
    int f = 0;
    for (int x = 0; x < 2 * K; ++x)
        for (int z = x >> 1; z < K; ++z, ++f) {
            if (f % dense_waves(K) != wid) continue;
            const unsigned b = rows32[((32 * x + l) * K + z) * 2 + half];
            v4i v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = spread4(((b >> (8 * i)) & 0xffu) << 1);
            tiles[f * kWave + lane] = v;
        }
}

// Takes the lowest bit of R, or -1.
template <int K>
__device__ __forceinline__ int take(u64 (&R)[K])
{
    int x = -1;
#pragma unroll
    for (int w = 0; w < K; ++w)
        if (x < 0 && R[w]) {
            x = w * 64 + __builtin_ctzll(R[w]);
            R[w] &= R[w] - 1;
        }
    return x;
}

// The nodes with four vertices to choose that one wave comes to, one after
// the other.
template <int K>
struct Nodes {
    u64 N[K];            // the node; its rows x = first mod stride are to add
    int stride, first;
    v4i pp[K];           // its pattern
    int t;               // levels on the stack
    bool started;

    __device__ __forceinline__ void start(int c)
    {
        t = -1;
        started = false;
        stride = 1;
        first = 0;
#pragma unroll
        for (int w = 0; w < K; ++w) {
            const int rem = c - 64 * w;
            N[w] = rem >= 64 ? ~0ull : (rem > 0 ? (1ull << rem) - 1ull : 0ull);
            pp[w] = v4i{0x22222222, 0x22222222, 0x22222222, 0x22222222};
        }
    }

    __device__ __forceinline__ bool next(const Dense<K>& D, int c, int need, int part, int P, int wid, u64* stack,
                                         int* branch)
    {
        const int lane = lane_of();
        auto claim = [&] {
            int j = 0;
            if (lane == 0) j = atomicAdd(branch, 1);
            return part + P * __builtin_amdgcn_readfirstlane(j);
        };
        if (need == 4) {
            if (started) return false;
            started = true;
            stride = P * dense_waves(K);
            first = part + P * wid;
            return true;
        }
        for (;;) {
            // stack[t]: (node, its branches left); r vertices to choose at
            // the node that x is taken from
            int r = need, x, n = 0;
            u64* top = stack + t * 2 * K;
            if (t < 0) {
                x = claim();
                if (x >= c) return false;
                D.row(x, N);
            } else {
                u64 S[K];
#pragma unroll
                for (int w = 0; w < K; ++w) S[w] = uniform64(top[K + w]);
                x = take<K>(S);
                if (x < 0) {
                    --t;
                    continue;
                }
                r = need - 1 - t;
                D.row(x, N);
#pragma unroll
                for (int w = 0; w < K; ++w) {
                    N[w] &= uniform64(top[w]);
                    if (lane == 0) top[K + w] = S[w];
                }
            }
#pragma unroll
            for (int w = 0; w < K; ++w) n += __popcll(N[w]);
            const bool deeper = n >= r - 1 && r > 5;
            if (deeper) {
                ++t;
#pragma unroll
                for (int w = 0; w < K; ++w)
                    if (lane == 0) stack[t * 2 * K + w] = stack[t * 2 * K + K + w] = N[w];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (n < r - 1 || deeper) continue;
            D.spread(N, pp);
            return true;
        }
    }
};

// One wave's share of one pass, and of those after it.  need == 4: the masks
// are the rows x = part mod P, dealt to the waves in turn.  Deeper:
// first-level branches x = part mod P are claimed, and a depth-first search below each comes to the nodes
// whose rows are the masks; stack: need - 5 levels of (node, branches left).
template <int K, int kPass>
__device__ __forceinline__ void dense_passes(const Dense<K>& D, int c, int need, int part, int P, int wid, u64* stack,
                                             int* branch, u64& sum)
{
    if constexpr (kPass < n_passes(K)) {
        using Acc = Pass<K, kPass>;
        if (Acc::B.x0 < D.nt && Acc::B.y0 < D.nt) {
            Nodes<K> node;
            node.start(c);
            bool more = true;
            do {
                Acc A;
                A.clear();
                int masks = 0;
                for (;;) {
                    more = node.next(D, c, need, part, P, wid, stack, branch + kPass);
                    if (!more) break;
                    A.add(D, node.N, node.pp, node.stride, node.first);
#pragma unroll
                    for (int w = 0; w < K; ++w) masks += __popcll(node.N[w]);
                    if (masks > max_masks(K) - 64 * K) break;
                }
                sum += A.sum(D);
            } while (more);
        }
        dense_passes<K, kPass + 1>(D, c, need, part, P, wid, stack, branch, sum);
    }
}

// One item: an arc's subgraph (mask row r of its source's rows, packed) or a
// whole vertex's (its rows as they are), laid out once; then its first level
// is shared among the waves.  need: vertices to choose from the subgraph, 3
// (one triangle count) or more.  per_arc (vertices at k = 4 only): counts
// per first vertex x go to per_arc[inv[x]].  Returns this lane's share.
template <int K>
__device__ __forceinline__ u64 dense_item(const u64* __restrict__ src, int W, int d, int r, int need, int part, int P,
                                          int max_k, unsigned char* smem, u64* stacks, int* branch, u64* per_arc,
                                          const uint16_t* inv)
{
    v4i* tiles = reinterpret_cast<v4i*>(smem);
    u64* rows = reinterpret_cast<u64*>(tiles + n_tiles(K) * kWave);
    const int lane = lane_of();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int c = d;
    if (threadIdx.x < n_passes(K)) branch[threadIdx.x] = 0;
    if (r < 0) {
        // W = K: the vertex's class is that of its out-degree
        for (int i = threadIdx.x; i < 64 * K * K; i += dense_waves(K) * kWave) rows[i] = i < d * K ? src[i] : 0ull;
    } else {
        const u64 M = lane < W ? src[(int64_t)r * W + lane] : 0ull;
        c = __builtin_amdgcn_readfirstlane(wave_sum_small(__popcll(M)));
        // rows past the last candidate, and words past a row's last, read as zero
        for (int i = threadIdx.x; i < 64 * K * K; i += dense_waves(K) * kWave) rows[i] = 0ull;
        __syncthreads();
        pack_rows<K>(src, W, M, c, rows);
    }
    const int nt = (c + 31) >> 5;
    __syncthreads();
    build_tiles<K>(rows, tiles);
    __syncthreads();
    const Dense<K> D{tiles, rows, nt};
    u64 sum = 0;
    if (need == 3 && !per_arc) {
        sum = D.triangles(wid);
        __syncthreads();
        return sum;
    }
    if (need == 3) {
        // per-arc counts of k = 4 want row x's own sum: lanes over its y
        for (int x = part + P * wid; x < c; x += P * dense_waves(K)) {
            u64 rx[K], s = 0;
            D.row(x, rx);
            for (int y = lane; y < c; y += kWave)
                if ((rows[x * K + (y >> 6)] >> (y & 63)) & 1)
#pragma unroll
                    for (int w = 0; w < K; ++w) s += (u64)__popcll(rx[w] & rows[y * K + w]);
            sum += s;
            const u64 t = wave_sum_u64(s);
            if (lane == 0 && t) atomicAdd(per_arc + inv[x], t);
        }
        __syncthreads();
        return sum;
    }
    u64* stack = stacks + wid * dense_stack_words(K, max_k);
    dense_passes<K, 0>(D, c, need, part, P, wid, stack, branch, sum);
    __syncthreads();
    return sum;
}

}  // namespace

template <int K>
__global__ void __launch_bounds__(dense_waves(K) * kWave)
    __attribute__((amdgpu_waves_per_eu(dense_cu_waves(K) / 4))) dense_kernel(DenseParams P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_of();
    u64* stacks = reinterpret_cast<u64*>(smem + 1024 * n_tiles(K) + 8 * 64 * K * K);
    int32_t* item = reinterpret_cast<int32_t*>(stacks + dense_waves(K) * dense_stack_words(K, P.max_k));
    int* shared = item + kItFields * kMaxClaim;      // first item of the run, then a branch counter per pass
    u64 acc = 0ull;
    int cur = -1;
    int shard = blockIdx.x % kClaimShards;
    bool fresh = true;
    const int acc_slot = (int)((blockIdx.x * dense_waves(K) + threadIdx.x / kWave) & (kAccSlots - 1)) * kAccStride;
    for (;;) {
        if (threadIdx.x < kWave) {
            const int g = claim_run(P.items, blockIdx.x, gridDim.x, shard, fresh);
            const int n = g < 0 ? 0 : run_length(P.items, g);
            decode_run<kDenseClasses - K>(P.items, g, n, item);
            if (lane == 0) {
                shared[0] = g;
                if (P.progress && g >= 0 && (((g + n - 1) ^ (g - 1)) & ~511))
                    __hip_atomic_store(P.progress, P.progress_base + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        __syncthreads();
        const int g0 = __builtin_amdgcn_readfirstlane(shared[0]);
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
            const u64 s = dense_item<K>(src, W, field(kItDegree), r, vertex ? q.k - 1 : q.k - 2, pw & 0xffff, pw >> 16,
                                        P.max_k, smem, stacks, shared + 1, vertex && q.per_arc ? q.per_arc + a0 : nullptr,
                                        q.rows.hinv + a0);
            acc += s;            // a lane adds below 2^28 per 2^9 masks or more
            if (q.per_arc && !vertex) {
                const u64 t = wave_sum_u64(s);
                if (lane == 0 && t) atomicAdd(q.per_arc + tag, t);
            }
        }
        // the last item's closing barrier separates its reads of the run from the next claim
    }
    if (cur >= 0) wave_flush(acc, 0, P.items.queries[cur].acc + acc_slot, P.items.queries[cur].overflow);
}

template <int K>
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
    const int by_lds = 160 * 1024 / lds, by_regs = dense_cu_waves(K) / dense_waves(K);
    int64_t blocks = (int64_t)cus * (by_lds < by_regs ? by_lds : by_regs);
    if (blocks > n) blocks = n;
    set_runs(P.items, blocks, kDenseClaim);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)dense_kernel<K>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    dense_kernel<K><<<(unsigned)blocks, dense_waves(K) * kWave, lds, s>>>(P);
    return hipGetLastError();
}

hipError_t launch_dense(const CountLaunch& cl, hipStream_t s)
{
    if (launch_items(cl) == cl.space_items[kRestSpace]) return hipSuccess;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    int32_t base = 0;
    if (e == hipSuccess) e = launch_class<6>(cl, cus, base, s);
    base += cl.space_items[0];
    if (e == hipSuccess) e = launch_class<5>(cl, cus, base, s);
    base += cl.space_items[1];
    if (e == hipSuccess) e = launch_class<4>(cl, cus, base, s);
    base += cl.space_items[2];
    if (e == hipSuccess) e = launch_class<3>(cl, cus, base, s);
    base += cl.space_items[3];
    if (e == hipSuccess) e = launch_class<2>(cl, cus, base, s);
    base += cl.space_items[4];
    if (e == hipSuccess) e = launch_class<1>(cl, cus, base, s);
    return e;
}

}  // namespace citron
