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


@pytest.mark.parametrize("K,N,M", [(1024, 10240, 500), (512, 4160, 2100)])
def test_hybrid_in_a_replayed_graph(mk, K, N, M):
    # the library's own choice, repeated in a graph, equals the eager result bit for bit
    q, s = synth.weights(22, K, N, 128)
    wp, sp = mk.pack(torch.from_numpy(q).cuda(), torch.from_numpy(s).cuda(), group=128)
    A = torch.from_numpy(synth.activations(22, M, K)).cuda()
    ws = mk.Workspace("cuda")
    first = mk.gemm(A, wp, sp, K, N, workspace=ws).clone()
    out = torch.empty_like(first)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mk.gemm(A, wp, sp, K, N, out=out, workspace=ws)
    for _ in range(3):
        out.zero_()
        graph.replay()
        assert torch.equal(out, first)
        assert torch.equal(mk.gemm(A, wp, sp, K, N, workspace=ws), first)
