// A lane's sum in the count kernel, exact modulo 2^64 with a carry flag.
//
// Most additions are small (popcounts, 2^24 at most at once): a lane cannot
// run the 2^58 steps it would take them to reach 2^62, so they are added to
// `acc` as they are.  The binomials of complete nodes are large (below 2^61)
// and go through add_big, which keeps `acc` below 2^63 by moving that bit to
// `flags`, and from there, the second time, to the carry.  So neither kind can
// wrap `acc`, whatever the order they come in.
#pragma once

#ifdef __HIPCC__
#define LANE_FN __device__ __forceinline__
#else
#define LANE_FN inline
#endif

namespace citron {

enum LaneSumFlag { kSumCarry = 1, kSumHalf = 2 };   // the sum passed 2^64; 2^63 beside acc

LANE_FN void add_big(unsigned long long& acc, int& flags, unsigned long long b)
{
    constexpr unsigned long long top = 1ull << 63;
    acc += b;
    if (acc & top) {
        acc ^= top;
        flags = flags & kSumHalf ? kSumCarry : flags | kSumHalf;
    }
}

// The sum modulo 2^64; flags keeps the carry alone.
LANE_FN unsigned long long lane_total(unsigned long long acc, int& flags)
{
    const unsigned long long s = acc + (flags & kSumHalf ? 1ull << 63 : 0ull);
    flags = (flags & kSumCarry) | (s < acc ? kSumCarry : 0);
    return s;
}

}  // namespace citron
