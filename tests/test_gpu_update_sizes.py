"""The per-iteration update at the edges of its launches: particle counts
around the 64 that one workgroup sums and point counts around the 1024 that
one workgroup tests (several workgroups write their parts of the list in
order, one at stride 6 the whole list), for one and several resolution levels
and with every point kept.  The frame equals the oracle's: valid points, overlap
and APS sizes per iteration, pose; a second run of the same frame equals the
first bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def small(orc):
    from paper_2105_05600_amd import rose
    w = synth.small_frame()
    vol = rose.Tsdf(w.dims, w.vox, w.mu, w.origin)
    psi = np.ones(w.dims[::-1], np.float32)
    wt = np.zeros_like(psi)
    for p, d in zip(w.fuse_poses, w.fuse_depths):
        vol.integrate(torch.from_numpy(d).cuda(), w.K, p.q, p.t)
        orc.integrate(psi, wt, w.vox, w.origin, w.mu, d, w.K, p.q, p.t, prec=orc.F32)
    pst, _ = orc.pst_sample(1100, 5600)
    return w, vol, psi, pst


def _frame(w, points, stride):
    """The frame with valid depth at its first `points` samples only."""
    d = np.zeros_like(w.depth)
    H, W = d.shape
    left = points
    for v in range(0, H, stride):
        for u in range(0, W, stride):
            if left > 0 and w.depth[v, u] > 0:
                d[v, u] = w.depth[v, u]
                left -= 1
    return d


@pytest.mark.parametrize("n,points,stride,flags,levels", [
    (2, 1, 3, 0, None), (63, 1023, 3, 0, None), (64, 1024, 3, 0, None), (65, 1025, 3, 0, None),
    (1025, 2048, 2, 0, None), (1100, 2049, 2, 0, None), (1088, 4800, 2, 1, None), (500, 19200, 1, 0, None),
    (900, 4000, 2, 0, [(900, 4), (300, 2), (65, 3)]), (300, 2160, 3, 2, None), (200, 500, 6, 0, None)])
def test_update_sizes(orc, small, n, points, stride, flags, levels):
    from paper_2105_05600_amd import rose
    w, vol, psi, pst = small
    prev = w.fuse_poses[-1]
    depth = _frame(w, points, stride if levels is None else 1)
    # the centre threshold: no ties that the rounding order decides
    flags |= rose.FLAG_CENTRE_THRESHOLD
    params = rose.track_params(max_iters=7, stride=stride, flags=flags, levels=levels)
    runs = []
    for _ in range(2):
        st = rose.track_state(prev.q, prev.t, [0.1] * 6)
        runs.append(rose.track_frame(vol, torch.from_numpy(depth).cuda(), w.K, torch.from_numpy(pst[:n].copy()).cuda(),
                                     params, st))
    g = runs[0]
    assert all(np.array_equal(np.array(g[k]), np.array(runs[1][k])) for k in g)
    o = orc.track_frame(psi, w.vox, w.origin, depth, w.K, pst[:n], prev.q, prev.t, np.full(6, 0.1), max_iters=7,
                        stride=stride, flags=flags, prec=orc.F32, levels=levels)
    assert g["n_points"] == o["n_points"]
    assert list(g["n_overlap"]) == list(o["n_overlap"])
    assert list(g["aps"]) == list(o["aps"])
    assert np.linalg.norm(np.array(g["t"]) - o["t"]) <= 1e-9
    assert np.allclose(g["r1"], o["r1"], rtol=1e-9, atol=0)
