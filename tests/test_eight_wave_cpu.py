"""Host side of the eight-wave tile and wide kernels: their compiled load
groups, the hybrid partition, and the rule that keeps fp32 group scales."""
import os
import re
import subprocess

import pytest

import paper_2408_11743_amd as mk
from paper_2408_11743_amd import build as B
from test_partition_cpu import range_start, unit_owner

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_11743_amd", "csrc")


@pytest.mark.parametrize("src,loads,count", [("tile8.hip", (7, 6), 4), ("wide.hip", (7, 6), 2), ("pair.hip", (7, 6), 2)])
def test_loads_come_in_whole_stages(tmp_path, src, loads, count):
    # The kernels count the direct-to-LDS loads issued after a stage's, so a
    # stage's loads are all of them, and no other buffer load but the partial
    # tiles' (device-coherent, outside the loop) may mix in; spilled registers
    # would add memory operations of their own.
    out = str(tmp_path / "k.s")
    flags = B.SOURCE_FLAGS.get(src, B.DEVICE_FLAGS)
    subprocess.run([B.hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, *flags, "--cuda-device-only", "-S", "-o", out, os.path.join(CSRC, src)], check=True,
                   capture_output=True)
    text = open(out).read()
    n = 0
    for m in re.finditer(r"^(_ZN6marlin\S*w4a16_(?:(?:tile|wide)_kernel\S*EightWaves|pair_kernel)ILb(\d)E\S*):", text, re.M):
        body = text[m.end():text.index(".Lfunc_end", m.end())]
        lines = [l.strip() for l in body.splitlines() if l.strip() and not l.strip().startswith(";")]
        n += 1
        stage = loads[int(m.group(2))]
        if src == "tile8.hip" and "Li8ELi1E" in m.group(1):
            stage -= 2  # 64-row tiles: two row loads per wave instead of four
        dma = [l for l in lines if l.startswith("buffer_load") and l.endswith("lds")]
        other = [l for l in lines if l.startswith("buffer_load") and not l.endswith("lds")]
        assert dma and len(dma) % stage == 0, (m.group(1), len(dma))
        assert all(l.endswith("sc1") for l in other), m.group(1)
        assert all(l.endswith("sc1") for l in lines if l.startswith("buffer_store")), m.group(1)
        assert not [l for l in lines if l.startswith("scratch_")], m.group(1)
        assert not [l for l in lines if l.split()[0] in ("buffer_wbl2", "buffer_inv")]
    assert n == count


@pytest.mark.parametrize("tiles,KU,grid", [(344, 32, 256), (320, 64, 256), (308, 5, 256), (511, 64, 256), (7, 3, 2),
                                           (896, 64, 256)])
def test_hybrid_covers_every_unit_once(tiles, KU, grid):
    # (coverage alone: which of these the planner may take, and that every
    # arrival a tile waits for happens, is checked in test_hybrid_cpu.py)
    shared = tiles % grid
    total = shared * KU
    seen = {}
    for w in range(grid):
        u0, u1 = (range_start(w, total, grid), range_start(w + 1, total, grid)) if total else (0, 0)
        for u in range(u0, u1):
            seen[divmod(u, KU)] = seen.get(divmod(u, KU), 0) + 1
            assert unit_owner(u, total, grid) == w
        c = shared + w
        n = 0
        while c < tiles:
            for k in range(KU):
                seen[(c, k)] = seen.get((c, k), 0) + 1
            c += grid
            n += 1
        assert n == (tiles - shared) // grid  # the stage count the kernel uses
    assert len(seen) == tiles * KU and set(seen.values()) == {1}


def test_group_scales_stay_in_fp32():
    # Up to 128 rows, and at widths that no 256-column kernel with fp16-rounded
    # weights served, group scales multiply fp32 products: never the wide kernel.
    for M in (65, 100, 128, 200, 1000, 4096):
        for K, N in ((8192, 28672), (28672, 8192), (4096, 4160), (8192, 12096), (4096, 1472)):
            if M > 128 and N % 256 == 0:
                continue
            assert not mk.marlin_describe(M, N, K, 128).startswith("w4a16_wide"), (M, N, K)
    # per-channel scales multiply the sums in every kernel
    assert mk.marlin_describe(2384, 16960, 3328, -1).startswith("w4a16_wide")
    # prefill on the 7B and 70B layers
    for K, N in ((4096, 4096), (4096, 11008), (8192, 28672), (28672, 8192)):
        assert mk.marlin_describe(4096, N, K, 128).startswith("w4a16_wide"), (K, N)
