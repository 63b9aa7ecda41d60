"""The first tracked frame of a handle allocates its scratch, and waits for
its own stream only: work that another stream has queued is still running
when the call returns."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_first_frame_waits_for_its_stream_only():
    from paper_2105_05600_amd import rose
    w = synth.small_frame()
    depth, pst = torch.from_numpy(w.depth).cuda(), rose.pst_sample(w.n_particles, 3)
    prev, params = w.fuse_poses[-1], rose.track_params(max_iters=4, stride=w.stride)
    ours, other = torch.cuda.Stream(), torch.cuda.Stream()

    def first_frame():
        with torch.cuda.stream(ours):
            vol = rose.Tsdf(w.dims, w.vox, w.mu, w.origin)
            for p, d in zip(w.fuse_poses, w.fuse_depths):
                vol.integrate(torch.from_numpy(d).cuda(), w.K, p.q, p.t)
            st = rose.track_state(prev.q, prev.t, [0.1] * 6)
            return vol, rose.track_frame(vol, depth, w.K, pst, params, st)

    torch.cuda.synchronize()
    alone, ref = first_frame()  # loads the kernels
    busy = torch.cuda.Event()
    with torch.cuda.stream(other):
        torch.zeros(1, device="cuda")
        torch.cuda._sleep(int(2e8))  # 84 ms at the 2.4 GHz that it counts
        busy.record()
    vol, r = first_frame()
    still_busy = not busy.query()
    torch.cuda.synchronize()
    assert all(np.array_equal(np.array(r[k]), np.array(ref[k])) for k in ref)
    assert still_busy
    vol.close()
    alone.close()
