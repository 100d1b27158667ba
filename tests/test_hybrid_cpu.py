"""The hybrid partition of the eight-wave kernels as the planner gives it, on
the CPU: every work-group has a share of the shared tiles, the arrivals a tile
waits for are the work-groups that arrive, its counter returns to zero, and
together with the whole tiles every block is computed once.

A work-group with an empty range never arrives; with fewer shared blocks than
work-groups such gaps lay between a tile's contributors, its count was never
complete, its outputs were not written and its counter stayed non-zero for
later calls (4096 x 11008 at 353..384, 705..768, 1409..1536 and 2177..2304
rows, among others).
"""
import ctypes
import os
import random
import subprocess

import pytest

from test_partition_cpu import model, range_start

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_11743_amd", "csrc")
PROBE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "plan_probe.cpp")
FREE = 1 << 62
SCRATCH = (1 << 20) + (32 << 20)


@pytest.fixture(scope="module")
def partition(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plan") / "libplan_probe.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", CSRC, "-o", out,
                    os.path.join(CSRC, "plan.cpp"), PROBE], check=True)
    lib = ctypes.CDLL(out)
    lib.probe_partition.restype = None
    lib.probe_partition.argtypes = [ctypes.c_int] * 5 + [ctypes.c_uint64, ctypes.c_char_p, ctypes.POINTER(ctypes.c_int)]

    def call(M, N, K, gu=1, cus=256, ws=FREE, force=None):
        v = (ctypes.c_int * 9)()
        lib.probe_partition(M, N, K, gu, cus, ws, force, v)
        return dict(zip(("kind", "whole", "hybrid", "grid", "tiles", "units", "gran", "per_wg", "extra"), v))
    return call


def check(p, K, seen, where):
    KU = K // 128
    assert p["per_wg"] >= 1, (where, p)  # every work-group has a share
    if not p["hybrid"]:
        return 0
    grid, shared = p["grid"], p["units"] // KU
    assert shared == p["tiles"] % grid and p["gran"] == 1 and not p["whole"]
    assert (p["tiles"] - shared) % grid == 0  # whole tiles come out even
    if (shared, KU, grid) not in seen:
        seen.add((shared, KU, grid))
        model(shared, KU, grid, 1, random.Random(shared * 1000 + KU))
    return 1


LAYERS = [(4096, 4096), (4096, 11008), (11008, 4096), (8192, 10240), (8192, 8192), (8192, 28672), (28672, 8192),
          (5120, 5120), (5120, 13824), (3584, 18944), (4096, 22016)]


@pytest.mark.parametrize("K,N", LAYERS)
def test_every_plan_of_a_layer(partition, K, N):
    seen, n = set(), 0
    for gu in (0, 1):
        for M in range(65, 4097, 1 if N > 8192 else 5):
            n += check(partition(M, N, K, gu), K, seen, (M, N, K, gu))
    assert n > 0  # the hybrid is in use on each of them


def test_drawn_shapes_devices_and_scratch(partition):
    rng, seen, n = random.Random(7), set(), 0
    for _ in range(20000):
        K, N = 128 * rng.randint(1, 224), 64 * rng.randint(1, 448)
        M = round(2 ** rng.uniform(0, 12))
        gu = rng.choice([g for g in (0, 1, 2, 4) if g == 0 or K // 128 % g == 0])
        cus, ws = rng.choice([256, 256, 256, 304, 128, 100, 38, 7]), rng.choice([FREE, FREE, SCRATCH, 1 << 20])
        n += check(partition(M, N, K, gu, cus, ws), K, seen, (M, N, K, gu, cus, ws))
    assert n > 1000


@pytest.mark.parametrize("kind", ["wide", "tile8,nb=4", "tile8,nb=2"])
def test_forced_partitions(partition, kind):
    rng, seen, n = random.Random(8), set(), 0
    for _ in range(3000):
        K, N, M = 128 * rng.randint(1, 40), 64 * rng.randint(1, 200), rng.randint(1, 4096)
        grid = rng.choice([0, 1, 2, 3, 7, 29, 64, 250, 256, 512])
        force = ("kind=%s,whole=%d" % (kind, rng.choice([0, 1, 2, 2])) + (",grid=%d" % grid if grid else "")).encode()
        n += check(partition(M, N, K, 1, force=force), K, seen, (M, N, K, force))
    assert n > 100


def test_the_broken_row_counts_now_have_no_empty_range(partition):
    # two, four and six tiles of 32 blocks left over: fewer than work-groups
    for M in (353, 360, 384, 705, 768, 1409, 1536, 2177, 2304):
        p = partition(M, 11008, 4096)
        assert p["per_wg"] >= 1 and (not p["hybrid"] or p["units"] >= p["grid"]), (M, p)
        starts = [range_start(w, p["units"] // p["gran"], p["grid"]) for w in range(p["grid"] + 1)]
        assert all(a < b for a, b in zip(starts, starts[1:]))
