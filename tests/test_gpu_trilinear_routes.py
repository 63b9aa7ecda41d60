"""Interpolated lookups by every route: corners in pairs, one by one
(16-bit volumes with few points per slice or few poses).  The sums are exact
on their grid, so all routes give the same bits."""
import pytest

from test_gpu_fitness_paths import _coords, _inputs, _trilinear_F, _volume

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("m,n", [(1535, 300), (1536, 300), (1537, 300), (4000, 16), (4000, 17), (4000, 64), (4000, 65), (90, 1), (3, 700)])
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
