"""GPU parity of the eight-wave tile and wide kernels against the fp64 oracle:
ragged row groups and column tiles (N of one and five packed tiles), fewer
128-row blocks than ring slots, whole tiles, Stream-K ranges with several tiles
per work-group and several work-groups per tile, and the hybrid (whole tiles
after ranges of shared ones), grouped and per-channel.

Tolerance: |error| <= 2e-3 + 1e-2 |C|, the bar of the other parity tests (fp16
output rounding 2^-11 relative, fp16 weights of the wide kernel, fp32 sums).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11743_amd as m
    return m


SHAPES = [(128, 64, -1), (256, 320, 128), (384, 512, 128), (1280, 1088, 256), (1408, 768, -1)]
PARTS = ["whole=1", "whole=0,grid=7", "whole=0,grid=29", "whole=2,grid=2", "whole=2,grid=3", ""]


@pytest.mark.parametrize("kind", ["kind=tile8,nb=4", "kind=tile8,nb=2", "kind=wide"])
@pytest.mark.parametrize("part", PARTS)
@pytest.mark.parametrize("K,N,g", SHAPES)
def test_eight_wave_kernels(mk, monkeypatch, kind, part, K, N, g):
    monkeypatch.setenv("MARLIN_FORCE_CONFIG", kind + ("," + part if part else ""))
    q, s = synth.weights(21, K, N, None if g == -1 else g)
    wp, sp = mk.pack(torch.from_numpy(q).cuda(), torch.from_numpy(s).cuda(), group=g)
    ws = mk.Workspace("cuda")
    for M in (1, 16, 63, 64, 65, 127, 128, 129, 200, 385):
        name = "w4a16_wide_kernel<" if "wide" in kind else "w4a16_tile_kernel<"
        assert mk.marlin_describe(M, N, K, g).startswith(name)
        A = synth.activations(21, M, K)
        got = mk.gemm(torch.from_numpy(A).cuda(), wp, sp, K, N, group=g, workspace=ws).cpu().numpy().astype(np.float64)
        ref = oracle.gemm(A, q, s, g)
        bad = np.abs(got - ref) > 2e-3 + 1e-2 * np.abs(ref)
        assert not bad.any(), "%s %s M=%d: %d wrong, first at %s" % (kind, part, M, bad.sum(), np.argwhere(bad)[:3])
    # every launch leaves the arrival counters at zero
    assert int(ws.buf[: 1 << 20].view(torch.int32).abs().max()) == 0


def problem(mk, K, N, M, g=128):
    q, s = synth.weights(22, K, N, None if g == -1 else g)
    wp, sp = mk.pack(torch.from_numpy(q).cuda(), torch.from_numpy(s).cuda(), group=g)
    A = synth.activations(22, M, K)
    ws = mk.Workspace("cuda", mk.marlin_workspace_bytes(M, N, K, g))
    return torch.from_numpy(A).cuda(), wp, sp, ws, oracle.gemm(A, q, s, g)


def check(out, ref, ws, what):
    got = out.cpu().numpy().astype(np.float64)
    bad = ~(np.abs(got - ref) <= 2e-3 + 1e-2 * np.abs(ref))  # an output nobody wrote is NaN
    assert not bad.any(), "%s: %d wrong, first at %s" % (what, bad.sum(), np.argwhere(bad)[:3])
    assert int(ws.buf[: 1 << 20].view(torch.int32).abs().max()) == 0, what


@pytest.mark.parametrize("K,N,M,g", [(4096, 11008, 353, 128), (4096, 11008, 705, -1), (4096, 11008, 1409, 128),
                                     (4096, 11008, 2177, 128), (5120, 5120, 800, -1), (3584, 18944, 400, 128),
                                     (4096, 22016, 129, 128), (4096, 11008, 1000, 128), (1024, 28672, 700, -1)])
def test_few_tiles_left_over(mk, monkeypatch, K, N, M, g):
    # the library's own choice at row counts with from one to a few tiles more
    # than a multiple of the work-groups, then the same workspace again
    monkeypatch.delenv("MARLIN_FORCE_CONFIG", raising=False)
    A, wp, sp, ws, ref = problem(mk, K, N, M, g)
    d = mk.marlin_describe(M, N, K, g)
    for _ in range(2):
        out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        mk.gemm(A, wp, sp, K, N, group=g, out=out, workspace=ws)
        check(out, ref, ws, "%s M=%d" % (d, M))


@pytest.mark.parametrize("K,N,M", [(4096, 11008, 1000), (8192, 10240, 1000)])
def test_hybrid_in_a_replayed_graph(mk, monkeypatch, K, N, M):
    # the library's own choice, repeated in a graph, is right at every replay
    # and equals the eager result bit for bit
    monkeypatch.delenv("MARLIN_FORCE_CONFIG", raising=False)
    assert " hybrid=" in mk.marlin_describe(M, N, K, 128)
    A, wp, sp, ws, ref = problem(mk, K, N, M)
    first = mk.gemm(A, wp, sp, K, N, workspace=ws).clone()
    check(first, ref, ws, "eager")
    out = torch.empty_like(first)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mk.gemm(A, wp, sp, K, N, out=out, workspace=ws)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        assert torch.equal(out, first)
        assert torch.equal(mk.gemm(A, wp, sp, K, N, workspace=ws), first)
    check(out, ref, ws, "replayed")
