"""The device-driven peeling replayed on the CPU: every order in which the
workgroups of a launch may run gives the oracle's rounds.  On a device that
other streams keep busy, a workgroup can start after the others of its launch
have set up the next phase."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import graphgen as gg
import oracle

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("peel") / "peel_replay.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "peel_replay.cpp"),
                           "-o", so])
    fn = ctypes.CDLL(so).peel_replay
    fn.restype = ctypes.c_int

    def run(g, grid, order, seed=0, copies=2):
        key = np.zeros(max(g.n, 1), np.int32)
        rounds = ctypes.c_int32(-1)
        rp, col = (np.ascontiguousarray(a, np.int32) for a in (g.row_ptr, g.col))
        st = fn(ctypes.c_int32(g.n), ctypes.c_void_p(rp.ctypes.data), ctypes.c_void_p(col.ctypes.data), grid, order, seed,
                copies, ctypes.c_void_p(key.ctypes.data), ctypes.byref(rounds))
        return st, key[:g.n], rounds.value
    return run


def _graphs():
    return [gg.rmat(7, 8, seed=1), gg.rmat(9, 16, seed=2), gg.erdos_renyi(300, 12, seed=3), gg.complete(17),
            gg.grid(13, 7), gg.hypercube(6), gg.disjoint_cliques([3, 7, 12, 5]), gg.empty(9)]


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("grid", [1, 3, 16, 128])
def test_rounds_for_every_order_of_workgroups(replay, grid, order):
    for g in _graphs():
        want = oracle.peel_rounds(g.n, g.row_ptr, g.col)
        st, key, rounds = replay(g, grid, order, seed=grid)
        assert st == 0, g.name
        assert np.array_equal(key, want) and rounds == int(want.max()) + 1, g.name


def test_the_replay_sees_a_control_block_that_is_read_and_written_in_one_launch(replay):
    """With a single copy, workgroups that run late join the next phase and the
    next launch does their share again (in ascending order it does not: those
    that joined are then the ones that come late again)."""
    g = gg.rmat(9, 16, seed=2)
    want = oracle.peel_rounds(g.n, g.row_ptr, g.col)
    wrong = 0
    for seed in range(8):
        st, key, _ = replay(g, 128, 2, seed=seed, copies=1)
        wrong += st != 0 or not np.array_equal(key, want)
    assert wrong == 8
    st, key, _ = replay(g, 128, 1, copies=1)      # surplus workgroups first: harmless
    assert st == 0 and np.array_equal(key, want)
