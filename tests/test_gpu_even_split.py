"""GPU parity of column tiles split evenly over several work-groups (up to 64
rows: the planner's own choice, dense and 2:4 sparse) against the fp64 oracle,
at numbers of 128-row blocks that the split does not divide, a ragged last row
group, grouped and per-channel scales.

Tolerance: |error| <= 2e-3 + 1e-2 |C|, the bar of the other parity tests.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,g,sparse", [(8320, 640, 128, False), (8320, 1280, -1, False), (6272, 2560, 128, False),
                                          (8320, 640, -1, True), (5248, 1088, 128, True), (6272, 2560, 128, True)])
def test_even_splits(monkeypatch, K, N, g, sparse):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11743_amd as mk
    monkeypatch.delenv("MARLIN_FORCE_CONFIG", raising=False)
    groups = None if g == -1 else g
    if sparse:
        q, _, s = synth.sparse24_weights(51, K, N, groups)
    else:
        q, s = synth.weights(51, K, N, groups)
    wp, sp = mk.pack(torch.from_numpy(q).cuda(), torch.from_numpy(s).cuda(), group=g, sparse=sparse)
    ws = mk.Workspace("cuda")
    describe = mk.marlin_describe_sparse if sparse else mk.marlin_describe
    split = 0
    for M in (8, 16, 17, 32, 33, 64):
        d = describe(M, N, K, g)
        cols, rg, grid = (int(d.split(k + "=")[1].split()[0]) for k in ("cols", "rg", "grid"))
        tiles = N // cols * rg
        split += "streamk" in d and grid % tiles == 0 and grid > tiles and (K // 128) % (grid // tiles) != 0
        A = synth.activations(51, M, K)
        ref = oracle.gemm(A, q, s, g)
        for _ in range(2):
            got = mk.gemm(torch.from_numpy(A).cuda(), wp, sp, K, N, group=g, workspace=ws, sparse=sparse)
            bad = np.abs(got.cpu().numpy().astype(np.float64) - ref) > 2e-3 + 1e-2 * np.abs(ref)
            assert not bad.any(), "%s M=%d: %d wrong, first at %s" % (d, M, bad.sum(), np.argwhere(bad)[:3])
    assert split >= 4
    # every launch leaves the arrival counters at zero
    assert int(ws.buf[: 1 << 20].view(torch.int32).abs().max()) == 0
