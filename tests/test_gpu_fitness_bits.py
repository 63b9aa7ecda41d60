"""Points-across nearest fitness at the edges of how its launches read the
brick bits (from memory; from LDS, copied in a burst or a word at a time, by
4 or 8 wavefronts): points per slice around the least that large launches
stage for, few and many particles, bit counts that fill no whole 16 bytes.
Exact against plain torch, as in test_gpu_fitness_paths.py."""
import pytest

from test_gpu_fitness_paths import _coords, _inputs, _nearest_F, _volume

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# bits of 23, 8192 and 35 words
@pytest.mark.parametrize("fmt", [0, 2])
@pytest.mark.parametrize("shape", [(4, 2), (8, 4)])
@pytest.mark.parametrize("dims", [(72, 72, 72), (512, 512, 512), (264, 264, 8)])
@pytest.mark.parametrize("m,n", [(1535, 4096), (1536, 4097), (1537, 8200), (1536, 1000), (511, 4096), (512, 4096), (90, 4096), (5000, 3), (5000, 130)])
def test_bits_paths(dims, m, n, shape, fmt):
    from paper_2105_05600_amd import rose
    vol, psi = _volume(dims, 0.02, fmt, m + n)
    vol.set_fitness_shape(*shape)
    pts, T = _inputs(dims, 0.02, m, n, 0.4, m * 3 + n)
    F, _ = rose.fitness_eval(vol, pts, T)
    for i in range(0, n, 1024):  # (the reference holds n x m values)
        assert torch.equal(F[i:i + 1024], _nearest_F(psi, _coords(vol, pts, T[i:i + 1024]), m))


def test_few_points_in_a_large_volume():
    """300 points under 10240 poses: within 1.1 times of a volume whose bits are not staged at all."""
    from paper_2105_05600_amd import rose
    t = []
    for nx in (520, 512):  # the first has more bits than the LDS holds
        vol = rose.Tsdf((nx, 512, 512), 0.01, 0.1, (0.0, 0.0, 0.0), fmt=rose.SN16)
        vol.set_fitness_shape(4, 2)
        pts, T = _inputs((512, 512, 512), 0.01, 300, 10240, 0.1, 5)
        best = 1e9
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(50):
                rose.fitness_eval(vol, pts, T)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1))
        t.append(best)
        vol.close()
    assert t[1] < 1.1 * t[0]
