"""The block pool (csrc/pool.cpp) on the CPU, over a device that only counts
bytes: what it holds, when it gives memory back, what a search costs."""
import ctypes
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2112_10913_amd", "csrc")
MIB = 1 << 20


@pytest.fixture
def pool(tmp_path):
    so = str(tmp_path / "pool_replay.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-shared", "-fPIC",
                           os.path.join(HERE, "pool_replay.cpp"), os.path.join(CSRC, "pool.cpp"), "-o", so])
    lib = ctypes.CDLL(so, mode=os.RTLD_NOW | getattr(os, "RTLD_DEEPBIND", 0))
    for name in ("pool_malloc", "device_malloc", "host_malloc"):
        f = getattr(lib, "replay_" + name)
        f.argtypes, f.restype = [ctypes.c_size_t], ctypes.c_void_p
    lib.replay_used.restype = ctypes.c_size_t
    lib.replay_capacity.argtypes = [ctypes.c_size_t]
    lib.replay_pool_free.argtypes = lib.replay_device_free.argtypes = [ctypes.c_void_p]
    lib.replay_host_free.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    return lib


def test_idle_blocks_make_room_for_the_librarys_other_memory(pool):
    """A batch's or a server's memory comes through device_malloc: idle blocks
    of the pool do not make it fail."""
    blocks = [pool.replay_pool_malloc(10 * MIB) for _ in range(5)]
    assert all(blocks)
    for b in blocks:
        pool.replay_pool_free(b)
    assert pool.replay_used() >= 50 * MIB                   # kept
    big = pool.replay_device_malloc(60 * MIB)
    assert big
    assert pool.replay_pool_malloc(8 * MIB) is None         # and a real lack of memory is reported
    pool.replay_device_free(big)
    assert pool.replay_used() == 0


def test_idle_blocks_make_room_for_a_block_of_another_size(pool):
    for b in [pool.replay_pool_malloc(s * MIB) for s in (5, 9, 13, 17)]:
        pool.replay_pool_free(b)
    assert pool.replay_pool_malloc(48 * MIB)


def test_release_gives_everything_idle_back(pool):
    keep = pool.replay_pool_malloc(3 * MIB)
    for b in [pool.replay_pool_malloc(s) for s in (1, 100, 5000, MIB, 7 * MIB)]:
        pool.replay_pool_free(b)
    host = [pool.replay_host_malloc(1000) for _ in range(3)]
    for h in host[1:]:
        pool.replay_host_free(h, 1000)
    pool.replay_release()
    assert 3 * MIB <= pool.replay_used() < 4 * MIB and pool.replay_pinned() == 1
    pool.replay_release()
    pool.replay_pool_free(keep)
    pool.replay_release()
    assert pool.replay_used() == 0


def test_all_device_memory_comes_through_the_pools_file():
    """So that idle blocks are given back whichever allocation fails."""
    for name in os.listdir(CSRC):
        text = re.sub(r"//.*", "", open(os.path.join(CSRC, name)).read())
        assert name == "pool.cpp" or not re.search(r"\bhipMalloc\w*\s*\(", text), name


def test_blocks_too_large_to_keep_are_as_large_as_asked(pool):
    pool.replay_capacity(1024 * MIB)
    for mib in (257, 300, 577, 1000, 1024):
        b = pool.replay_pool_malloc(mib * MIB)
        assert b and pool.replay_used() == mib * MIB
        pool.replay_pool_free(b)
        assert pool.replay_used() == 0                      # nothing idle
    b = pool.replay_pool_malloc(256 * MIB)                  # the largest that is kept
    pool.replay_pool_free(b)
    assert pool.replay_used() == 256 * MIB


def test_small_blocks_count_the_page_they_take(pool):
    """The bound of 1 GiB holds for what the device has given, also for many
    blocks of a few bytes."""
    pool.replay_capacity(4096 * MIB)
    blocks = [pool.replay_pool_malloc(64 + i % 512) for i in range(400_000)]
    for b in blocks:
        pool.replay_pool_free(b)
    assert pool.replay_used() <= 1024 * MIB


def test_a_search_does_not_look_at_every_idle_block(pool):
    """A program that drops many graphs goes on at the speed of one that has
    none: 100,000 idle blocks, then blocks of sizes that are not among them."""
    import time
    pool.replay_capacity(4096 * MIB)
    blocks = [pool.replay_pool_malloc(4096) for i in range(100_000)]
    for b in blocks:
        pool.replay_pool_free(b)
    t = time.perf_counter()
    held = [pool.replay_pool_malloc(10_000) for _ in range(20_000)]
    assert all(held) and time.perf_counter() - t < 2.0      # 2,000,000,000 steps when each search walks the list


def test_the_newest_of_a_size_is_reused_and_the_oldest_goes_first(pool):
    pool.replay_capacity(4096 * MIB)
    a, b = pool.replay_pool_malloc(9000), pool.replay_pool_malloc(9000)
    pool.replay_pool_free(a)
    pool.replay_pool_free(b)
    assert pool.replay_pool_malloc(8900) == b               # one size class
    pool.replay_pool_free(b)
    calls = pool.replay_calls()
    assert {pool.replay_pool_malloc(9000), pool.replay_pool_malloc(9000)} == {a, b}
    assert pool.replay_calls() == calls
    big = [pool.replay_pool_malloc(200 * MIB) for _ in range(6)]
    pool.replay_pool_free(a)                                # the oldest idle block
    for x in big:
        pool.replay_pool_free(x)
    assert pool.replay_used() <= 1024 * MIB + 8192
    assert pool.replay_pool_malloc(9000) is not None and pool.replay_calls() == calls + 7
