// Wave-wide helpers shared by the count kernels: cross-lane reads, sums,
// selection in bit masks, parallel bit extract.
#pragma once

#include "internal.h"

namespace citron {

typedef unsigned long long u64;

__device__ __forceinline__ int lane_of() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ u64 shfl64(u64 v, int src)
{
    unsigned lo = __shfl((unsigned)v, src, kWave);
    unsigned hi = __shfl((unsigned)(v >> 32), src, kWave);
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 readlane64(u64 v, int lane)
{
    unsigned lo = __builtin_amdgcn_readlane((unsigned)v, lane);
    unsigned hi = __builtin_amdgcn_readlane((unsigned)(v >> 32), lane);
    return ((u64)hi << 32) | lo;
}

// Sum over the wave of per-lane values in 0..127, from seven ballots (no
// LDS traffic, no cross-lane shuffles).
__device__ __forceinline__ int wave_sum_small(int v)
{
    int s = 0;
#pragma unroll
    for (int b = 0; b < 7; ++b) s += __popcll(__ballot((v >> b) & 1)) << b;
    return s;
}

__device__ __forceinline__ u64 wave_sum_u64(u64 v)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += shfl64(v, lane_of() ^ o);
    return v;
}

// Wave-wide carry-checked reduction; lane 0 adds the total to *dst.
__device__ __forceinline__ void wave_flush(u64 acc, int ovf, u64* dst, int32_t* ovf_dst)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const u64 other = shfl64(acc, lane_of() ^ o);
        ovf |= __shfl_xor(ovf, o, kWave);
        const u64 s = acc + other;
        ovf |= (s < acc) ? 1 : 0;
        acc = s;
    }
    if (lane_of() == 0) {
        if (acc) {
            const u64 old = atomicAdd(dst, acc);
            if (old + acc < old) ovf = 1;
        }
        if (ovf) atomicOr(ovf_dst, 1);
    }
}

__device__ __forceinline__ void wave_flush_stats(const u64* vals, u64* dst)
{
#pragma unroll
    for (int i = 0; i < kNumStats; ++i) {
        // written once per wave at its end
        if ((i >= kStatWaveBusy && i <= kStatWaves) || (i >= kStatWaveBusyMax && i <= kStatCycTotal)) continue;
        const u64 v = wave_sum_u64(vals[i]);
        if (lane_of() == 0 && v) atomicAdd(dst + i, v);
    }
}

// Position of the r-th (0-based) set bit of v; always in 0..63.
__device__ __forceinline__ int select64(u64 v, int r)
{
    int pos = 0;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const u64 low = v & ((1ull << s) - 1);
        const int c = __popcll(low);
        if (r >= c) {
            r -= c;
            v >>= s;
            pos += s;
        } else {
            v = low;
        }
    }
    return pos;
}

// A W-word mask held one word per lane (lane w holds word w, lanes >= W
// hold 0).  Returns, in lane j, the position of the j-th set bit (for j
// below the popcount).  Uniform control flow: the whole wave calls it.
__device__ __forceinline__ int wave_select(u64 m, int j, int W)
{
    int before = 0, my_w = 0, my_r = 0;
    u64 my_word = 0;
    for (int w = 0; w < W; ++w) {
        const u64 mw = readlane64(m, w);
        const int pc = __popcll(mw);
        const bool here = j >= before && j < before + pc;
        my_w = here ? w : my_w;
        my_r = here ? j - before : my_r;
        my_word = here ? mw : my_word;
        before += pc;
    }
    return my_w * 64 + select64(my_word, my_r);
}

// Parallel bit extract with a wave-uniform mask (Hacker's Delight, section
// 7-4, "compress"): the masks are prepared once per mask word (scalar
// work), then each lane packs its own word in six shift-and-merge steps.
struct Pext {
    u64 m, v0, v1, v2, v3, v4, v5;
};

__device__ __forceinline__ u64 prefix_xor64(u64 x)
{
    x ^= x << 1;
    x ^= x << 2;
    x ^= x << 4;
    x ^= x << 8;
    x ^= x << 16;
    x ^= x << 32;
    return x;
}

__device__ __forceinline__ Pext pext_prep(u64 m)
{
    Pext p;
    p.m = m;
    u64 mk = ~m << 1;
    u64 v[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const u64 mp = prefix_xor64(mk);
        v[i] = mp & m;
        m = (m ^ v[i]) | (v[i] >> (1 << i));
        mk &= ~mp;
    }
    p.v0 = v[0];
    p.v1 = v[1];
    p.v2 = v[2];
    p.v3 = v[3];
    p.v4 = v[4];
    p.v5 = v[5];
    return p;
}

__device__ __forceinline__ u64 pext_apply(u64 x, const Pext& p)
{
    u64 t;
    x &= p.m;
    t = x & p.v0; x = (x ^ t) | (t >> 1);
    t = x & p.v1; x = (x ^ t) | (t >> 2);
    t = x & p.v2; x = (x ^ t) | (t >> 4);
    t = x & p.v3; x = (x ^ t) | (t >> 8);
    t = x & p.v4; x = (x ^ t) | (t >> 16);
    t = x & p.v5; x = (x ^ t) | (t >> 32);
    return x;
}

}  // namespace citron
