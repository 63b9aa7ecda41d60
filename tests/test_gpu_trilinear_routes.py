"""Interpolated lookups by every route: corners in pairs, in pairs with the
boundary loads skipped (a tracked frame's particles one per lane), one by one
(16-bit volumes with few points per slice or few poses).  The sums are exact
on their grid, so all routes give the same bits."""
import numpy as np
import pytest

import synth
from test_gpu_fitness_paths import _coords, _inputs, _trilinear_F, _volume

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("m,n", [(1024, 300), (1025, 300), (1537, 300), (4000, 16), (4000, 17), (4000, 64), (4000, 65), (90, 1), (3, 700)])
def test_fitness_routes(m, n, fmt):
    from paper_2105_05600_amd import rose
    vol, psi = _volume((72, 40, 56), 0.02, fmt, m + n)
    pts, T = _inputs((72, 40, 56), 0.02, m, n, 0.5, m + n)
    F = []
    for shape in ((4, 2), (8, 2), (64, 8)):
        vol.set_fitness_shape(*shape)
        F.append(rose.fitness_eval(vol, pts, T, rose.TRILINEAR)[0])
    assert torch.equal(F[0], F[1]) and torch.equal(F[0], F[2])
    # the bound of test_gpu_fitness_paths.py
    assert float((F[0].double() - _trilinear_F(psi, _coords(vol, pts, T))).abs().max()) <= 29 * 2.0 ** -24


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("n,stride,r", [(1, 3, 0.1), (70, 3, 0.02), (513, 2, 0.1), (1000, 1, 0.01)])
def test_track_routes(fmt, n, stride, r):
    from paper_2105_05600_amd import rose
    w = synth.small_frame()
    vol = rose.Tsdf(w.dims, w.vox, w.mu, w.origin, fmt=fmt)
    for p, d in zip(w.fuse_poses, w.fuse_depths):
        vol.integrate(torch.from_numpy(d).cuda(), w.K, p.q, p.t)
    prev, pst = w.fuse_poses[-1], rose.pst_sample(n, 7)
    params = rose.track_params(max_iters=6, stride=stride, lookup=rose.TRILINEAR)
    out = []
    for shape in ((4, 2), (8, 2), (64, 8), (0, 0)):  # the last switches by the footprint
        vol.set_fitness_shape(*shape)
        st = rose.track_state(prev.q, prev.t, [r] * 6)
        out.append(rose.track_frame(vol, torch.from_numpy(w.depth).cuda(), w.K, pst, params, st))
    for o in out[1:]:
        assert all(np.array_equal(np.array(o[k]), np.array(out[0][k])) for k in o if k != "fit_mode")


def _best(f, reps):
    t = 1e9
    for _ in range(8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            f()
        e1.record()
        e1.synchronize()
        t = min(t, e0.elapsed_time(e1))
    return t


def test_few_points_in_16_bits():
    """4096 poses x 300 points in a binary16 volume: at most 1.12 times the binary32 volume's time."""
    from paper_2105_05600_amd import rose
    t = []
    for fmt in (0, 1):
        vol, _ = _volume((64, 64, 64), 0.02, fmt, 1)
        vol.set_fitness_shape(4, 2)
        pts, T = _inputs((64, 64, 64), 0.02, 300, 4096, 0.1, 5)
        t.append(_best(lambda: rose.fitness_eval(vol, pts, T, rose.TRILINEAR), 50))
    assert t[1] < 1.12 * t[0]


def test_few_poses_one_per_lane():
    """64 poses x 4000 points with one pose per lane: at most 1.6 times the time with the points across the lanes."""
    from paper_2105_05600_amd import rose
    vol, _ = _volume((64, 64, 64), 0.02, 0, 1)
    pts, T = _inputs((64, 64, 64), 0.02, 4000, 64, 0.1, 5)
    t = []
    for shape in ((4, 2), (64, 8)):
        vol.set_fitness_shape(*shape)
        t.append(_best(lambda: rose.fitness_eval(vol, pts, T, rose.TRILINEAR), 50))
    assert t[1] < 1.6 * t[0]


def test_alike_poses_one_per_lane():
    """A tracked binary32 frame, one particle per lane: under 0.95 times the binary16 frame's time."""
    import time

    from paper_2105_05600_amd import rose
    w, t = synth.small_frame(), []
    pst, depth = rose.pst_sample(70, 7), torch.from_numpy(w.depth).cuda()
    params = rose.track_params(max_iters=20, stride=1, lookup=rose.TRILINEAR)
    for fmt in (0, 1):
        vol = rose.Tsdf(w.dims, w.vox, w.mu, w.origin, fmt=fmt)
        for p, d in zip(w.fuse_poses, w.fuse_depths):
            vol.integrate(torch.from_numpy(d).cuda(), w.K, p.q, p.t)
        vol.set_fitness_shape(64, 8)
        best = 1e9
        for _ in range(30):
            st = rose.track_state(w.fuse_poses[-1].q, w.fuse_poses[-1].t, [0.01] * 6)
            torch.cuda.synchronize()
            start = time.perf_counter()
            rose.track_frame(vol, depth, w.K, pst, params, st)
            best = min(best, time.perf_counter() - start)
        t.append(best)
    assert t[0] < 0.95 * t[1]
