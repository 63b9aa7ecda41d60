"""16-bit volumes at any address that their elements allow: a psi buffer two
bytes past a 4-byte boundary gives the results of an aligned one, bit for
bit, for both lookups, both kinds of launch shape and the raycast; and the
volume's last cell, whose pairs end at the buffer's end, is read right."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DIMS, VOX = (16, 24, 8), 0.05


def _volume(fmt, shift):
    """A volume whose psi lies `shift` elements past an aligned address, with the buffer's own end at psi's end."""
    from paper_2105_05600_amd import rose
    nx, ny, nz = DIMS
    n = nx * ny * nz
    v = rose.Tsdf.__new__(rose.Tsdf)
    v.dims, v.voxel, v.trunc, v.origin, v.fmt = DIMS, VOX, 0.1, (0.0, 0.0, 0.0), fmt
    pd, wd = rose.Tsdf._dtypes[fmt]
    v.psi = torch.empty(n + shift, dtype=pd, device="cuda")[shift:]
    v.weight = torch.empty(n, dtype=wd, device="cuda")
    assert v.psi.data_ptr() % 4 == 2 * (shift % 2)
    h, org = C.c_void_p(), (C.c_float * 3)(0.0, 0.0, 0.0)
    rose._check("tsdf_create", rose._lib.tsdf_create(nx, ny, nz, VOX, 0.1, org, fmt, 128.0, rose._ptr(v.psi),
                                                     rose._ptr(v.weight), rose._stream(), C.byref(h)))
    v.handle = h
    rng = np.random.default_rng(7 + fmt)
    psi = rng.uniform(-1, 1, (nz, ny, nx)).astype(np.float32)
    v.load(torch.from_numpy(psi).cuda())
    return v


def _points(rng):
    """Points over the whole volume, and a third of them in its last cell."""
    ext = np.array(DIMS) * VOX
    pts = rng.uniform(-0.02, 1.02, (700, 3)) * ext
    pts[::3] = (np.array(DIMS) - 1.5 + rng.uniform(0.02, 0.98, (len(pts[::3]), 3))) * VOX
    return pts.astype(np.float32)


def _poses(n):
    T = np.zeros((n, 3, 4), np.float32)
    T[:, :, :3] = np.eye(3)
    T[1:, :, 3] = np.random.default_rng(3).uniform(-0.001, 0.001, (n - 1, 3))
    return T


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("shape", [(4, 2), (64, 8)])
@pytest.mark.parametrize("lookup", [0, 1])
def test_fitness_of_an_odd_buffer(orc, fmt, shape, lookup):
    from paper_2105_05600_amd import rose
    pts, T = _points(np.random.default_rng(11)), _poses(70)
    F = []
    for shift in (0, 1):
        v = _volume(fmt, shift)
        v.set_fitness_shape(*shape)
        F.append(rose.fitness_eval(v, torch.from_numpy(pts).cuda(), torch.from_numpy(T).cuda(), lookup)[0].cpu().numpy())
        psi = v.export()[0].cpu().numpy()
    assert np.array_equal(F[0], F[1])
    o = orc.fitness(psi, VOX, np.zeros(3, np.float32), pts, T.astype(np.float64), lookup=lookup, prec=orc.F32)
    assert np.max(np.abs(F[0] - o) / np.abs(o)) <= 1e-5


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("w,h", [(31, 23), (160, 121), (530, 500)])
def test_raycast_of_an_odd_buffer(orc, fmt, w, h):
    """1, 4 and 16 pixels per wavefront; most rays leave through the far corner."""
    from paper_2105_05600_amd import rose

    class K:
        width, height, fx, fy, cx, cy = w, h, 1.3 * w, 1.3 * w, w / 2 - 0.5, h / 2 - 0.5

    c = (np.array(DIMS) - 1.0) * VOX
    t = c - np.array([0.5, 0.7, 0.6])
    f = (c - t) / np.linalg.norm(c - t)
    x = np.cross(f, [0, 0, 1.0])
    x /= np.linalg.norm(x)
    R = np.stack([x, np.cross(f, x), f], axis=1)
    q = np.array([np.sqrt(1 + np.trace(R)) / 2, 0, 0, 0])
    q[1:] = np.array([R[2, 1] - R[1, 2], R[0, 2] - R[2, 0], R[1, 0] - R[0, 1]]) / (4 * q[0])
    out = []
    for shift in (0, 1):
        v = _volume(fmt, shift)
        out.append(rose.raycast(v, q, t, K, near=0.05, far=3.0, step=0.5 * VOX).cpu().numpy())
        psi = v.export()[0].cpu().numpy()
    assert np.array_equal(out[0], out[1])
    o = orc.raycast(psi, VOX, np.zeros(3), q, t, K, near=0.05, far=3.0, step=0.5 * VOX)
    assert np.array_equal(out[0], np.asarray(o, np.float32).reshape(out[0].shape))
    assert float((out[0] > 0).mean()) > 0.1
