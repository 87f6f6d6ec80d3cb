// k-clique listing through the counting recursion (the paper's conclusion
// names listing as a small change of the counting method): for each listed
// arc u -> v, the k-cliques whose two lowest vertices in the ordering are u
// and v are written out as k vertex ids each, in increasing order of the
// ordering -- u, v, then the chosen candidates level by level.  Within an
// arc the cliques come in the order of a depth-first search that takes the
// candidates of every level in ascending position (= ascending id) order.
//
// One wave per arc at a time (a persistent grid).  The search state is wave-uniform, lane q holding word q of each
// candidate mask over the positions of N->(u), as in the heavy count engine;
// the masks of the open levels live in the wave's LDS, k - 2 levels of one
// word per lane (3 KB per wave at k = 5, 14 KB at k = 16).  The last two
// levels are written at once: a lane per candidate x counts the y that
// complete a clique with it, a wave scan places them, and then the lanes take
// the node's cliques 64 at a time in output order, each finding its x in the
// scan and its y by rank, so the stores are full and in sequence.  (With one
// step per x, about 13 of 64 lanes wrote, and each step waited for its row.)
// Arcs are claimed from sharded cursors in runs decoded a lane each: 71,000
// claims of one cursor alone were 0.85 ms of the 1.16 ms that the 35 M
// 4-cliques of R-MAT 14, 566 MB, took; now 0.46 ms.  The offsets of the arcs' output come from their exact counts (a scan of the
// per-arc counts of the count kernel), so no atomics order the output;
// every write is checked against the arc's slot and a mismatch raises a
// flag instead of writing outside it.
#include "items.h"
#include "wave.h"

#include <numeric>

namespace citron {

namespace {

constexpr int kListBlock = 256;                 // 4 waves
constexpr int kListWaves = kListBlock / kWave;

// Levels whose masks are kept for the way back: a node at level t is
// pushed only while k - 2 - t >= 3 vertices remain to choose, so levels
// 0 .. k - 5 are stored; k - 2 (at least 1) bounds them.
__host__ __device__ __forceinline__ int list_levels(int k) { return k > 3 ? k - 2 : 1; }

}  // namespace

__global__ void __launch_bounds__(kListBlock) list_arcs_kernel(ListParams P)
{
    // the open levels' masks, k - 2 levels per wave (sized at launch, so
    // that small k leaves LDS for more resident waves)
    extern __shared__ u64 lds_levels[];
    __shared__ int32_t sPre[kListWaves][kListMaxK];
    const int lane = lane_of();
    const int wid = threadIdx.x / kWave;
    const int k = P.k;
    const int levels = list_levels(k);
    u64* const sM = lds_levels + (size_t)wid * levels * kWave;
    u64* const sR = lds_levels + (size_t)(kListWaves + wid) * levels * kWave;
    const int wave = blockIdx.x * kListWaves + wid, waves = gridDim.x * kListWaves;
    int shard = wave % kClaimShards;
    bool fresh = true;
    int jj = 0, nj = 0;                 // the wave's run of arcs, decoded a lane each
    int l_u = 0, l_v = 0, l_a0 = 0, l_d = 0, l_r = 0, l_off = 0;
    long long l_slot0 = 0, l_slot1 = 0;
    for (;;) {
        if (jj >= nj) {
            const int j0 = claim_run(P.items, wave, waves, shard, fresh);
            if (j0 < 0) break;
            nj = run_length(P.items, j0);
            jj = 0;
            if (lane < nj) {
                // claim j lists arc j * stride mod n_arcs (stride coprime to
                // n_arcs): a run of claims spreads over the list, so the arcs
                // of one heavy vertex, adjacent in DAG order, do not land in
                // one wave's run
                const int i = (int)(((long long)(j0 + lane) * P.stride) % P.n_arcs);
                const int e = P.arcs[i];
                l_slot0 = P.offsets[i];
                l_slot1 = P.offsets[i + 1];
                l_u = P.dag_src[e];
                l_v = P.dag_col[e];
                l_a0 = P.dag_ptr[l_u];
                l_d = P.dag_ptr[l_u + 1] - l_a0;
                l_r = e - l_a0;
                l_off = P.rows_off[l_u];
            }
        }
        const int u = __builtin_amdgcn_readlane(l_u, jj), v = __builtin_amdgcn_readlane(l_v, jj);
        const int a0 = __builtin_amdgcn_readlane(l_a0, jj), d = __builtin_amdgcn_readlane(l_d, jj);
        const int r = __builtin_amdgcn_readlane(l_r, jj), row0 = __builtin_amdgcn_readlane(l_off, jj);
        const long long slot0 = (long long)readlane64((u64)l_slot0, jj);
        const long long slot_n = (long long)readlane64((u64)l_slot1, jj) - slot0;
        ++jj;
        if (slot_n == 0) continue;              // no clique starts with this arc
        long long done = 0;                     // cliques of this arc written so far
        if (lane == 0) {
            sPre[wid][0] = u;
            sPre[wid][1] = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (k == 2) {
            if (lane == 0) {
                if (slot_n >= 1) {
                    P.out[2 * slot0] = u;
                    P.out[2 * slot0 + 1] = v;
                } else {
                    atomicOr(P.err, 1);
                }
            }
            done = 1;
        } else {
            const int W = (d + 63) >> 6;
            const u64* __restrict__ rows = P.rows + row0;
            // level 0: the arc's candidate set C_uv, k - 2 vertices to choose
            u64 M = lane < W ? rows[(long long)r * W + lane] : 0ull;
            u64 R = M;
            int t = 0;                          // level; k - 2 - t vertices still to choose
            for (;;) {
                const int need = k - 2 - t;
                if (need == 1) {
                    // every candidate of M completes a clique
                    int before = 0;
                    for (int w = 0; w < W; ++w) {
                        const u64 mw = readlane64(M, w);
                        const int pc = __popcll(mw);
                        for (int j0 = 0; j0 < pc; j0 += kWave) {
                            const int j = j0 + lane;
                            if (j < pc) {
                                const long long idx = done + before + j;
                                const int x = w * 64 + select64(mw, j);
                                if (idx < slot_n) {
                                    int32_t* o = P.out + (slot0 + idx) * k;
                                    for (int c = 0; c < k - 1; ++c) o[c] = sPre[wid][c];
                                    o[k - 1] = P.dag_col[a0 + x];
                                } else {
                                    atomicOr(P.err, 1);
                                }
                            }
                        }
                        before += pc;
                    }
                    done += before;
                    R = 0ull;                   // node finished
                }
                if (need == 2) {
                    int c = __popcll(M);
#pragma unroll
                    for (int o = kWave / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
                    for (int j0 = 0; j0 < c; j0 += kWave) {
                        // the j-th candidate x, its id, and the cliques it leads to
                        const int j = j0 + lane;
                        const int sel = wave_select(M, j, W);       // any position past the last
                        const int x = j < c ? sel : 0;
                        const int xid = j < c ? P.dag_col[a0 + x] : 0;
                        int cnt = 0;
                        for (int w = 0; w < W; ++w) {
                            const u64 mw = readlane64(M, w);
                            if (j < c && mw) cnt += __popcll(mw & rows[(long long)x * W + w]);
                        }
                        int inc = cnt;
#pragma unroll
                        for (int o = 1; o < kWave; o <<= 1) {
                            const int v = __shfl_up(inc, o, kWave);
                            if (lane >= o) inc += v;
                        }
                        const int tot = __shfl(inc, kWave - 1, kWave);
                        for (int o0 = 0; o0 < tot; o0 += kWave) {
                            const int o = o0 + lane;
                            // the first lane whose inclusive sum passes o
                            int s = 0;
#pragma unroll
                            for (int h = kWave / 2; h > 0; h >>= 1)
                                if (__shfl(inc, s + h - 1, kWave) <= o) s += h;
                            s = min(s, kWave - 1);
                            const int xs = __shfl(x, s, kWave), xsid = __shfl(xid, s, kWave);
                            int r2 = o - __shfl(inc - cnt, s, kWave);
                            int y = -1;
                            for (int w = 0; w < W; ++w) {
                                const u64 mw = readlane64(M, w);
                                if (mw == 0ull) continue;
                                if (o < tot && y < 0) {
                                    const u64 word = mw & rows[(long long)xs * W + w];
                                    const int pc = __popcll(word);
                                    if (r2 < pc) y = w * 64 + select64(word, r2);
                                    r2 -= pc;
                                }
                            }
                            if (o < tot) {
                                const long long idx = done + o;
                                if (idx < slot_n && y >= 0) {
                                    const int yid = P.dag_col[a0 + y];
                                    int32_t* out = P.out + (slot0 + idx) * k;
                                    if (P.wide) {           // k = 4, output aligned to 16 bytes
                                        *reinterpret_cast<int4*>(out) = make_int4(sPre[wid][0], sPre[wid][1], xsid, yid);
                                    } else {
                                        for (int c2 = 0; c2 < k - 2; ++c2) out[c2] = sPre[wid][c2];
                                        out[k - 2] = xsid;
                                        out[k - 1] = yid;
                                    }
                                } else {
                                    atomicOr(P.err, 1);
                                }
                            }
                        }
                        done += tot;
                    }
                    R = 0ull;                   // node finished
                }
                // next candidate of this level, or back up
                const u64 b = __ballot(R != 0ull);
                if (b == 0ull) {
                    if (t == 0) break;
                    --t;
                    M = sM[t * kWave + lane];
                    R = sR[t * kWave + lane];
                    continue;
                }
                const int f = __builtin_ctzll(b);
                const u64 Rf = readlane64(R, f);
                const int x = f * 64 + __builtin_ctzll(Rf);
                if (lane == f) R &= R - 1;
                const u64 ch = M & (lane < W ? rows[(long long)x * W + lane] : 0ull);
                int cc = __popcll(ch);
#pragma unroll
                for (int o = kWave / 2; o > 0; o >>= 1) cc += __shfl_xor(cc, o, kWave);
                if (cc >= need - 1) {
                    // descend: the level's state is kept for the way back
                    sM[t * kWave + lane] = M;
                    sR[t * kWave + lane] = R;
                    if (lane == 0) sPre[wid][2 + t] = P.dag_col[a0 + x];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    ++t;
                    M = ch;
                    R = ch;
                }
            }
        }
        if (lane == 0 && done != slot_n) atomicOr(P.err, 2);
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t launch_list_arcs(const ListParams& P, int32_t blocks, hipStream_t s)
{
    if (P.n_arcs <= 0) return hipSuccess;
    if (P.k < 2 || P.k > kListMaxK) return hipErrorInvalidValue;
    const size_t lds = 2 * (size_t)kListWaves * list_levels(P.k) * kWave * sizeof(u64);
    ListParams Q = P;
    Q.wide = P.k == 4 && (reinterpret_cast<uintptr_t>(P.out) & 15) == 0;
    const int64_t need = (P.n_arcs + kListWaves - 1) / kListWaves;
    if (need < blocks) blocks = (int32_t)need;
    Q.items = {};
    Q.items.total = P.n_arcs;
    Q.items.cursors = P.cursors;
    set_runs(Q.items, (int64_t)blocks * kListWaves, kMaxClaim);
    // a stride near 0.618 n_arcs (consecutive claims then land far apart,
    // as in Fibonacci hashing) that shares no factor with n_arcs
    int64_t st = 1;
    if (Q.items.chunk > 1) {
        for (int64_t t = (int64_t)(0.6180339887 * P.n_arcs); t < P.n_arcs; ++t)
            if (std::gcd(t, (int64_t)P.n_arcs) == 1) {
                st = t;
                break;
            }
    }
    Q.stride = (int32_t)st;
    list_arcs_kernel<<<blocks, kListBlock, lds, s>>>(Q);
    return hipGetLastError();
}

// ------------------------------------------------------- 64-bit exclusive scan

namespace {
constexpr int kScan64Block = 256;
constexpr int kScan64Per = 8;
constexpr int kScan64Tile = kScan64Block * kScan64Per;

__device__ long long block_exclusive_scan64(long long v, long long* total)
{
    __shared__ long long wsum[kScan64Block / kWave];
    const int lane = lane_of(), wid = threadIdx.x / kWave;
    long long inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const long long t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    long long off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kScan64Block / kWave; ++w) {
        if (w < wid) off += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}
}  // namespace

__global__ void scan64_tile_sums_kernel(const u64* __restrict__ in, int64_t n, long long* __restrict__ sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScan64Tile + (int64_t)threadIdx.x * kScan64Per;
    long long s = 0;
#pragma unroll
    for (int i = 0; i < kScan64Per; ++i)
        if (base + i < n) s += (long long)in[base + i];
    long long tot;
    block_exclusive_scan64(s, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void scan64_tiles_kernel(const u64* __restrict__ in, int64_t n, const long long* __restrict__ tile_off,
                                    long long* __restrict__ out)
{
    const int64_t base = (int64_t)blockIdx.x * kScan64Tile + (int64_t)threadIdx.x * kScan64Per;
    long long vals[kScan64Per];
    long long s = 0;
#pragma unroll
    for (int i = 0; i < kScan64Per; ++i) {
        vals[i] = (base + i < n) ? (long long)in[base + i] : 0;
        s += vals[i];
    }
    long long tot;
    long long run = block_exclusive_scan64(s, &tot) + (tile_off ? tile_off[blockIdx.x] : 0);
#pragma unroll
    for (int i = 0; i < kScan64Per; ++i) {
        if (base + i < n) out[base + i] = run;
        run += vals[i];
    }
    if (n > 0 && base <= n - 1 && n - 1 < base + kScan64Per) out[n] = run;
    if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) out[0] = tile_off ? tile_off[0] : 0;
}

size_t scan64_workspace(int64_t n)
{
    if (n <= kScan64Tile) return 1;
    const int64_t tiles = (n + kScan64Tile - 1) / kScan64Tile;
    return (size_t)(2 * tiles + 1) + scan64_workspace(tiles);
}

// out[0..n] = exclusive prefix sums of in[0..n) (out[n] = total); in holds
// non-negative counts below 2^63 in total.  ws: scan64_workspace(n) words.
hipError_t scan_exclusive64(const u64* in, long long* out, int64_t n, long long* ws, hipStream_t s)
{
    if (n <= kScan64Tile) {
        scan64_tiles_kernel<<<1, kScan64Block, 0, s>>>(in, n, nullptr, out);
        return hipGetLastError();
    }
    const int64_t tiles = (n + kScan64Tile - 1) / kScan64Tile;
    long long* sums = ws;
    long long* offs = ws + tiles;
    scan64_tile_sums_kernel<<<(unsigned)tiles, kScan64Block, 0, s>>>(in, n, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the tile sums are scanned as unsigned words holding non-negative values
    e = scan_exclusive64(reinterpret_cast<const u64*>(sums), offs, tiles, ws + 2 * tiles + 1, s);
    if (e != hipSuccess) return e;
    scan64_tiles_kernel<<<(unsigned)tiles, kScan64Block, 0, s>>>(in, n, offs, out);
    return hipGetLastError();
}

}  // namespace citron
