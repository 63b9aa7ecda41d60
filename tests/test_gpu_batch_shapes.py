"""The batched tracker's fixed shapes, with the brick bits staged in LDS and,
for the shapes of 32 evaluations per lane and step, in memory: the same poses
bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

COUNT = 32


@pytest.fixture(scope="module")
def runs():
    from paper_2105_05600_amd import rose
    w = synth.small_frame()
    prev, depth = w.fuse_poses[-1], torch.from_numpy(w.depth).cuda()
    vols = []
    for _ in range(COUNT):
        vol = rose.Tsdf(w.dims, w.vox, w.mu, w.origin)
        for p, d in zip(w.fuse_poses, w.fuse_depths):
            vol.integrate(torch.from_numpy(d).cuda(), w.K, p.q, p.t)
        vols.append(vol)
    psts = [rose.pst_sample(700 + 64 * (i % 4), 50 + i) for i in range(COUNT)]
    params = [rose.track_params(max_iters=8, stride=1 + i % 2) for i in range(COUNT)]
    out = {}
    for shape in ((4, 2), (4, 4), (8, 2), (4, 8), (8, 4)):
        for v in vols:
            v.set_fitness_shape(*shape)
        torch.cuda.synchronize()
        batch = rose.Batch(vols, [w.K] * COUNT, psts, params)
        states = (rose.TrackState * COUNT)(*[rose.track_state(prev.q, prev.t, [0.1] * 6) for _ in range(COUNT)])
        out[shape] = batch.track([depth] * COUNT, states, stream=torch.cuda.Stream())
        batch.close()
    return out


@pytest.mark.parametrize("shape", [(4, 4), (8, 2), (4, 8), (8, 4)])
def test_shapes_agree(runs, shape):
    for a, b in zip(runs[(4, 2)], runs[shape]):
        assert all(np.array_equal(np.array(a[k]), np.array(b[k])) for k in ("q", "t", "r1", "aps", "n_overlap"))
