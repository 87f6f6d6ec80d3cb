"""The count kernel's lane sums (csrc/lane_sum.h) on the CPU: the value modulo
2^64 and the carry of any mix of small additions and binomials, against whole
numbers."""
import ctypes
import math
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "%s/paper_2112_10913_amd/csrc/lane_sum.h"
extern "C" unsigned long long lane_sum(const unsigned long long* v, const int* big, int n, int* carry)
{
    unsigned long long acc = 0;
    int flags = 0;
    for (int i = 0; i < n; ++i) {
        if (big[i]) citron::add_big(acc, flags, v[i]);
        else acc += v[i];
    }
    const unsigned long long s = citron::lane_total(acc, flags);
    *carry = flags;
    return s;
}
""" % ROOT


@pytest.fixture(scope="module")
def lane_sum(tmp_path_factory):
    d = tmp_path_factory.mktemp("lane")
    (d / "lane.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", str(d / "lane.cpp"), "-o", str(d / "lane.so")])
    fn = ctypes.CDLL(str(d / "lane.so")).lane_sum
    fn.restype = ctypes.c_uint64

    def run(values):
        n = len(values)
        carry = ctypes.c_int(-1)
        v = fn((ctypes.c_uint64 * n)(*[x for x, _ in values]), (ctypes.c_int * n)(*[int(b) for _, b in values]), n,
               ctypes.byref(carry))
        return v, carry.value
    return run


def _check(lane_sum, values):
    total = sum(x for x, _ in values)
    assert lane_sum(values) == (total % 2 ** 64, int(total >= 2 ** 64))


@pytest.mark.parametrize("below", [0, 1, 63, 64, 4095, 1 << 24])
def test_a_small_addition_at_the_edge(lane_sum, below):
    """Binomials up to 2^64 - 1 - below, then a small addition that just
    carries or just does not."""
    rest = 2 ** 64 - 1 - below
    values = []
    while rest:
        b = min(rest, math.comb(64, 30))
        values.append((b, True))
        rest -= b
    for c in (below, below + 1):
        _check(lane_sum, values + [(c, False)])
        _check(lane_sum, [(c, False)] + values)
        _check(lane_sum, values[:3] + [(c, False)] + values[3:])


def test_random_mixes(lane_sum):
    rng = random.Random(5)
    for _ in range(300):
        values = []
        for _ in range(rng.randrange(1, 60)):
            big = rng.random() < 0.5
            values.append((math.comb(64, rng.randrange(4, 31)) if big else rng.randrange(1 << rng.choice([3, 7, 24])), big))
        _check(lane_sum, values)
