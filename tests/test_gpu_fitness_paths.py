"""fitness_eval at the edges of the fitness kernels' paths against plain torch:
nearest fitness exactly (integer sums on the 2^-39 grid), trilinear within
its arithmetic, for every storage format and a shape of each kind (points
across the lanes, with the brick bits in LDS or, for volumes of more than
8192 x 32 bricks, in memory; one particle per lane, with steps wholly inside
the grid and not).  The poses put points inside, on the faces, far outside,
and across brick boundaries in every axis."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _inputs(dims, vox, m, n, spread, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    ext = torch.tensor(dims, device="cuda", dtype=torch.float32) * vox
    pts = (torch.rand((m, 3), generator=g, device="cuda") - 0.5) * ext * 0.9
    T = torch.zeros((n, 3, 4), device="cuda")
    a = torch.rand(n, generator=g, device="cuda") * 0.3
    T[:, 0, 0], T[:, 0, 1], T[:, 1, 0], T[:, 1, 1], T[:, 2, 2] = a.cos(), -a.sin(), a.sin(), a.cos(), 1.0
    T[:, :, 3] = ext / 2 + (torch.rand((n, 3), generator=g, device="cuda") - 0.5) * spread * ext
    return pts.contiguous(), T.contiguous()


def _volume(dims, vox, fmt, seed):
    from paper_2105_05600_amd import rose
    g = torch.Generator(device="cuda").manual_seed(seed)
    nx, ny, nz = dims
    psi = torch.rand((nz, ny, nx), generator=g, device="cuda") * 2 - 1
    b = torch.rand((nz // 8, ny // 8, nx // 8), generator=g, device="cuda") < 0.4  # bricks that hold only +1
    psi[b.repeat_interleave(8, 0).repeat_interleave(8, 1).repeat_interleave(8, 2)] = 1.0
    vol = rose.Tsdf(dims, vox, 0.1, (0.0, 0.0, 0.0), fmt=fmt)
    vol.load(psi)
    return vol, vol.export()[0]


def _coords(vol, pts, T):
    inv = 1.0 / float(np.float32(vol.voxel))
    V = T.double().clone()
    V = (V * inv).float()  # folded in binary64, rounded once (origin 0)
    x = [pts[:, d].double() for d in range(3)]
    out = []
    for r in range(3):  # each fmaf: exact in binary64 up to its own rounding
        acc = V[:, r, 3, None].double()
        for d in range(3):
            acc = (V[:, r, d, None].double() * x[d] + acc).float().double()
        out.append(acc.float())
    return out


def _nearest_F(psi, c, m):
    nz, ny, nx = psi.shape
    ok = torch.ones_like(c[0], dtype=torch.bool)
    for v, n in zip(c, (nx, ny, nz)):
        ok &= (v >= 0) & (v < n)
    i = [torch.where(ok, v, torch.zeros_like(v)).long() for v in c]
    v = torch.where(ok, psi.reshape(-1)[(i[2] * ny + i[1]) * nx + i[0]], torch.ones_like(c[0])).double()
    k = torch.round(v * v * 2.0 ** 39)  # ties to even, exact below 2^53
    return (k.sum(1) * 2.0 ** -39 / m).float()


def _trilinear_F(psi, c):
    nz, ny, nx = psi.shape
    h = [v.float() - 0.5 for v in c]
    ok = torch.ones_like(h[0], dtype=torch.bool)
    for v, n in zip(h, (nx, ny, nz)):
        ok &= (v >= 0) & (v < n - 1)
    i = [torch.where(ok, v, torch.zeros_like(v)).long() for v in h]
    f = [torch.where(ok, v, torch.zeros_like(v)).double() - b for v, b in zip(h, i)]
    flat, acc = psi.reshape(-1).double(), torch.zeros_like(f[0])
    for e in range(8):
        d = (e & 1, (e >> 1) & 1, e >> 2)
        w = torch.ones_like(acc)
        for a in range(3):
            w = w * (f[a] if d[a] else 1 - f[a])
        acc += w * flat[((i[2] + d[2]) * ny + i[1] + d[1]) * nx + i[0] + d[0]]
    return (torch.where(ok, acc, torch.ones_like(acc)) ** 2).mean(1)


# (dims, points, poses, spread): the brick bits of 520^3 exceed the LDS limit,
# all others fit; the spreads take poses from all inside to mostly outside
CASES = [((64, 72, 40), 1, 1, 0.0), ((64, 72, 40), 7, 65, 0.1), ((64, 72, 40), 513, 130, 1.5), ((128, 64, 96), 2160, 1024, 0.3),
         ((512, 512, 512), 1029, 700, 0.05), ((520, 520, 520), 700, 257, 0.6)]


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("shape", [(4, 2), (8, 2), (64, 8), (64, 16)])
@pytest.mark.parametrize("dims,m,n,spread", CASES)
def test_nearest_exact(dims, m, n, spread, shape, fmt):
    from paper_2105_05600_amd import rose
    vol, psi = _volume(dims, 0.02, fmt, m + n)
    vol.set_fitness_shape(*shape)
    pts, T = _inputs(dims, 0.02, m, n, spread, m * 3 + n)
    F, _ = rose.fitness_eval(vol, pts, T)
    assert torch.equal(F, _nearest_F(psi, _coords(vol, pts, T), m))


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("shape", [(4, 2), (64, 8)])
@pytest.mark.parametrize("dims,m,n,spread", CASES[:5])
def test_trilinear(dims, m, n, spread, shape, fmt):
    from paper_2105_05600_amd import rose
    vol, psi = _volume(dims, 0.02, fmt, m + n)
    vol.set_fitness_shape(*shape)
    pts, T = _inputs(dims, 0.02, m, n, spread, m * 3 + n)
    F, _ = rose.fitness_eval(vol, pts, T, rose.TRILINEAR)
    # seven binary32 interpolations of values in [-1, 1] per term: each term
    # within 2 x 14 x 2^-24 of its exact square, F rounded once more
    assert float((F.double() - _trilinear_F(psi, _coords(vol, pts, T))).abs().max()) <= 28 * 2.0 ** -24 + 2.0 ** -24
