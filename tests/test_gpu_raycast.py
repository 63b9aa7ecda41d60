"""tsdf_raycast against the oracle's serial march, bit for bit (binary64
geometry on both sides), over what decides its path: the pixel count (1, 4 or
16 pixels per wavefront, image sizes that are no multiple of the patch), the
storage format, cameras inside and outside the volume, steps from a fraction
of a voxel to many voxels, and volumes with NaN, zero and all-positive
bricks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


class _K:
    def __init__(self, w, h, f):
        self.width, self.height, self.fx, self.fy, self.cx, self.cy = w, h, f, f, w / 2 - 0.5, h / 2 - 0.5


def _volume(rng, dims, special):
    """A noisy ball of free space in a solid, noise near its surface."""
    nx, ny, nz = dims
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    d = np.sqrt((x - nx * 0.45) ** 2 + (y - ny * 0.5) ** 2 + (z - nz * 0.55) ** 2)
    psi = np.clip((0.38 * min(dims) - d) / 4.0, -1, 1)
    psi = np.where(np.abs(psi) < 1, psi + 0.2 * rng.standard_normal(psi.shape), psi)
    psi = np.where(psi < -0.9, 1.0, psi).clip(-1, 1).astype(np.float32)
    if special:
        psi[rng.random(psi.shape) < 0.01] = np.float32(0.0)
        psi[rng.random(psi.shape) < 0.002] = np.float32("nan")
    return psi


CASES = [(1, 1, 0.5, False), (37, 29, 0.5, False), (131, 119, 0.37, False), (203, 151, 0.5, True), (520, 505, 0.5, False),
         (64, 48, 3.0, False), (150, 140, 11.0, True)]


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("w,h,step_vox,special", CASES)
def test_raycast_equals_serial_march(orc, w, h, step_vox, special, fmt):
    from paper_2105_05600_amd import rose
    if special and fmt == 2:
        special = False  # the integer format has no NaN
    rng = np.random.default_rng(w * 1000 + h)
    dims, vox, org = (56, 48, 64), 0.03, (-0.4, 0.2, 0.1)
    vol = rose.Tsdf(dims, vox, 0.12, org, fmt=fmt)
    vol.load(torch.from_numpy(_volume(rng, dims, special)).cuda())
    psi = vol.export()[0].cpu().numpy()
    K = _K(w, h, 0.9 * w)
    q = rng.standard_normal(4)
    q /= np.linalg.norm(q)
    centre = np.array(org) + vox * np.array([0.45 * 56, 0.5 * 48, 0.55 * 64])
    for t in (centre, centre + np.array([0.3, 0.1, -0.2]), np.array(org) - 1.0):
        if np.allclose(t, np.array(org) - 1.0):  # outside, looking in
            f = (centre - t) / np.linalg.norm(centre - t)
            x = np.cross(f, [0, 0, 1.0])
            x /= np.linalg.norm(x)
            R = np.stack([x, np.cross(f, x), f], axis=1)
            q = np.array([np.sqrt(max(0.0, 1 + np.trace(R))) / 2, 0, 0, 0])
            q[1:] = np.array([R[2, 1] - R[1, 2], R[0, 2] - R[2, 0], R[1, 0] - R[0, 1]]) / (4 * q[0])
        g = rose.raycast(vol, q, t, K, near=0.05, far=6.0, step=step_vox * vox).cpu().numpy()
        o = orc.raycast(psi, vox, np.array(org), q, t, K, near=0.05, far=6.0, step=step_vox * vox)
        assert np.array_equal(g, np.asarray(o, np.float32).reshape(g.shape))
