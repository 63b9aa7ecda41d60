"""What a user of this framework has it do, as a list of timed cases.

Every case is one call (or one training step) through the public binding
(paper_2105_05600_amd.rose), on synthetic rooms made here with torch: a box
room with spheres and boxes standing in it, seen by a depth camera that moves
by some centimetres and degrees per frame, depth noise 0.002 z^2.

Kinds:
* track:     pso_track_frame -- the pose search of one frame in a volume
             fused from the frames before it (the tracker's inner loop).
* learned:   pso_track_frame_learned -- the same with the learned proposal.
* batch:     pso_batch_track -- many small sequences in lockstep (a server).
* fitness:   fitness_eval -- many candidate poses against a loaded map
             (relocalisation, and the call that other optimisers build on).
* integrate: tsdf_integrate -- fusion of one frame.
* raycast:   tsdf_raycast -- a depth image rendered from the model.
* forward:   rose_mlp_forward -- the proposal network, one row per sequence.
* train:     rose_mlp_loss_grad and rose_mlp_adam -- one training step.
* gemm:      rose_gemm_bf16 -- the matrix-core product on its own.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_2105_05600_amd import rose

FMT = {"f32": rose.F32, "f16": rose.F16, "sn16": rose.SN16}
LOOKUP = {"nearest": rose.NEAREST, "trilinear": rose.TRILINEAR}
# the multi-resolution schedule of the benchmark, as (share of the template, stride)
LEVELS = ((1.0, 6), (0.3, 4), (0.1, 3))
NET_IN, NET_HID, NET_OUT = 1216, 256, 12


class _Camera:
    def __init__(self, width, height):
        self.width, self.height = width, height
        self.fx = self.fy = float(np.float32(525.0 * width / 640.0))
        self.cx, self.cy = width / 2.0 - 0.5, height / 2.0 - 0.5


# ----------------------------------------------------------------- the cases
def listed():
    return [
        # the benchmark's frame: 512^3 at 1 cm, 640x480 at stride 4, 10240
        # particles, 20 iterations, the switching launch mode
        dict(name="track_room", kind="track", nx=512, ny=512, nz=512, vox=0.01, mu=0.15, w=640, h=480, stride=4,
             n=10240, iters=20, fmt="f32", lookup="nearest", switch=True, levels=False, first=False),
        # the smallest tracked frame: 64^3 at 2 cm, 160x120, as on a small
        # robot; default launch shape
        dict(name="track_small", kind="track", nx=64, ny=64, nz=64, vox=0.02, mu=0.06, w=160, h=120, stride=3,
             n=1024, iters=10, fmt="f32", lookup="nearest", switch=False, levels=False, first=False),
        # half-precision map, interpolated lookups, an odd volume; the second
        # frame of a sequence: one fused frame, the widest search
        dict(name="track_f16_trilinear", kind="track", nx=384, ny=392, nz=248, vox=0.01, mu=0.15, w=320, h=240,
             stride=4, n=4096, iters=20, fmt="f16", lookup="trilinear", switch=True, levels=False, first=True),
        # the learned proposal at 320x240 with the committed weights
        dict(name="learned_320", kind="learned", nx=512, ny=512, nz=512, vox=0.01, mu=0.15, w=320, h=240, stride=4,
             n=6144, iters=12, fmt="f32", lookup="nearest", switch=True, levels=False, first=False),
        # a server's frame step: 64 small sequences at once (captured graph)
        dict(name="batch_64", kind="batch", count=64, nx=128, ny=128, nz=128, vox=0.04, mu=0.15, w=160, h=120,
             stride=3, n=1024, iters=20, fmt="f32", lookup="nearest", switch=False, levels=False, first=False),
        # relocalisation: candidate poses scattered over half a metre
        dict(name="fitness_reloc", kind="fitness", nx=512, ny=512, nz=512, vox=0.01, mu=0.15, w=640, h=480, stride=4,
             n=10240, spread=0.15, fmt="f32", lookup="nearest"),
        # fusion of the benchmark's frame, and of a small one in 16 bits
        dict(name="integrate_room", kind="integrate", nx=512, ny=512, nz=512, vox=0.01, mu=0.15, w=640, h=480,
             fmt="f32"),
        dict(name="integrate_f16", kind="integrate", nx=256, ny=256, nz=256, vox=0.02, mu=0.15, w=320, h=240,
             fmt="f16"),
        # the model seen from the camera, at half the sensor's resolution
        dict(name="raycast_320", kind="raycast", nx=512, ny=512, nz=512, vox=0.01, mu=0.15, w=320, h=240, fmt="f32"),
        # one proposal: a single row through the network
        dict(name="forward_1", kind="forward", batch=1),
        # a training step of the proposal network
        dict(name="train_1024", kind="train", batch=1024),
        # the matrix product away from the network's small shapes
        dict(name="gemm_4096", kind="gemm", m=4096, n=4096, k=4096, ta=False, tb=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    """Volume dimensions (multiples of 8), each its own, and a voxel size for a room of 1.3 to 5.2 m."""
    d = 8 * _log_int(rng, lo // 8, hi // 8)
    nx, ny, nz = (max(lo, min(hi, 8 * round(d * rng.uniform(0.85, 1.0) / 8))) for _ in range(3))
    vox = round(rng.uniform(1.28, 5.12) / max(nx, ny, nz), 4)
    return dict(nx=nx, ny=ny, nz=nz, vox=max(0.008, vox))


def draw(rng):
    kind = rng.choice(["track", "track", "learned", "batch", "fitness", "integrate", "integrate", "raycast", "forward",
                       "train", "gemm"])
    fmt = rng.choice(["f32", "f32", "f16", "sn16"])
    lookup = rng.choice(["nearest", "nearest", "trilinear"])
    w = _log_int(rng, 160, 640)
    h = max(120, int(w * rng.uniform(0.7, 0.8)))
    if kind == "forward":
        return dict(kind=kind, batch=_log_int(rng, 1, 1024))
    if kind == "train":
        return dict(kind=kind, batch=_log_int(rng, 64, 1024))
    if kind == "gemm":
        return dict(kind=kind, m=_log_int(rng, 32, 4096), n=_log_int(rng, 32, 4096), k=_log_int(rng, 32, 4096),
                    ta=rng.random() < 0.3, tb=rng.random() < 0.3)
    if kind == "learned":
        g = _grid(rng, 256, 512)
        return dict(kind=kind, **g, mu=max(0.06, round(8 * g["vox"], 3)), w=320, h=240, stride=4, n=_log_int(rng, 1024, 6144),
                    iters=rng.randint(6, 12), fmt=fmt, lookup="nearest", switch=rng.random() < 0.7, levels=False, first=False)
    if kind == "batch":
        g = _grid(rng, 64, 128)
        return dict(kind=kind, count=_log_int(rng, 4, 64), **g, mu=max(0.06, round(4 * g["vox"], 3)), w=160, h=120,
                    stride=rng.choice([3, 4, 5]), n=_log_int(rng, 300, 1024), iters=rng.randint(5, 20), fmt=fmt,
                    lookup="nearest", switch=rng.random() < 0.5, levels=False, first=False)
    g = _grid(rng, 64, 512)
    g["mu"] = max(0.06, round(10 * g["vox"], 3))
    if kind == "track":
        tri = lookup == "trilinear"  # eight reads per evaluation: fewer evaluations
        if tri:
            w, h = max(160, w // 2), max(120, h // 2)
        return dict(kind=kind, **g, w=w, h=h, stride=rng.choice([4, 5, 6] if tri else [4, 4, 5, 6]),
                    n=_log_int(rng, 500, 4096 if tri else 10240), iters=rng.randint(5, 20), fmt=fmt, lookup=lookup,
                    switch=rng.random() < 0.6, levels=(not tri) and rng.random() < 0.25, first=rng.random() < 0.25)
    if kind == "fitness":
        return dict(kind=kind, **g, w=w, h=h, stride=rng.choice([4, 5, 6]), n=_log_int(rng, 64, 10240),
                    spread=round(math.exp(rng.uniform(math.log(0.005), math.log(0.15))), 4), fmt=fmt, lookup=lookup)
    if kind == "raycast":
        w = _log_int(rng, 40, 320)
        return dict(kind=kind, **g, w=w, h=max(30, int(w * 0.75)), fmt=fmt)
    return dict(kind=kind, **g, w=w, h=h, fmt=fmt)


# ------------------------------------------------------------ rooms and views
def _room(case, seed):
    """A seeded room that fills the volume: walls, spheres and boxes that keep
    clear of the volume's middle, where the camera is."""
    r = np.random.default_rng([seed, 1])
    ext = np.array([case["nx"], case["ny"], case["nz"]], float) * case["vox"]
    s = float(ext.min())
    lo, hi = np.full(3, 0.02 * s), ext - 0.02 * s
    spheres, boxes = [], []
    for i in range(5):
        a = r.uniform(0, 2 * math.pi)
        c = ext / 2 + np.array([0.33 * ext[0] * math.cos(a), 0.33 * ext[1] * math.sin(a), ext[2] * r.uniform(-0.3, 0.3)])
        spheres.append((c, s * r.uniform(0.04, 0.1)))
    for i in range(6):
        a = r.uniform(0, 2 * math.pi)
        c = ext[:2] / 2 + np.array([0.33 * ext[0] * math.cos(a), 0.33 * ext[1] * math.sin(a)])
        e = s * r.uniform(0.03, 0.1, 2)
        boxes.append((np.array([*(c - e), lo[2]]), np.array([*(c + e), lo[2] + s * r.uniform(0.1, 0.4)])))
    return dict(ext=ext, lo=lo, hi=hi, spheres=spheres, boxes=boxes, a0=r.uniform(0, 2 * math.pi),
                y0=r.uniform(0, 2 * math.pi))


def _pose(room, k):
    """Camera (R, t) of frame k: 2-10 cm and 3.5 degrees per frame."""
    ext = room["ext"]
    s = float(ext.min())
    a = room["a0"] + 0.2 * k
    t = ext / 2 + np.array([0.1 * s * math.cos(a), 0.1 * s * math.sin(a), 0.03 * s * math.sin(0.7 * a)])
    yaw, pitch = room["y0"] + 0.06 * k, -0.25 + 0.1 * math.sin(0.3 * k + room["a0"])
    f = np.array([math.cos(yaw) * math.cos(pitch), math.sin(yaw) * math.cos(pitch), math.sin(pitch)])
    x = np.cross(f, [0.0, 0.0, 1.0])
    x /= np.linalg.norm(x)
    return np.stack([x, np.cross(f, x), f], axis=1), t


def _quat(R):
    """Rotation matrix -> quaternion (w, x, y, z), w >= 0 (the eigenvector of the standard 4x4 form)."""
    K = np.array([[R[0, 0] + R[1, 1] + R[2, 2], R[2, 1] - R[1, 2], R[0, 2] - R[2, 0], R[1, 0] - R[0, 1]],
                  [0, R[0, 0] - R[1, 1] - R[2, 2], R[0, 1] + R[1, 0], R[0, 2] + R[2, 0]],
                  [0, 0, R[1, 1] - R[0, 0] - R[2, 2], R[1, 2] + R[2, 1]],
                  [0, 0, 0, R[2, 2] - R[0, 0] - R[1, 1]]])
    q = np.linalg.eigh(K, UPLO="U")[1][:, -1]
    return q if q[0] >= 0 else -q


def _render(room, K, R, t, seed):
    """The depth frame (h x w float32) of the room with sensor noise."""
    u = torch.arange(K.width, dtype=torch.float64, device="cuda")
    v = torch.arange(K.height, dtype=torch.float64, device="cuda")
    dc = [((u - K.cx) / K.fx)[None, :].expand(K.height, K.width), ((v - K.cy) / K.fy)[:, None].expand(K.height, K.width)]
    d = [R[i, 0] * dc[0] + R[i, 1] * dc[1] + R[i, 2] for i in range(3)]
    z = torch.full((K.height, K.width), math.inf, dtype=torch.float64, device="cuda")
    for i in range(3):
        z = torch.minimum(z, torch.where(d[i] > 0, room["hi"][i] - t[i], room["lo"][i] - t[i]) / d[i])
    dd = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
    for c, r in room["spheres"]:
        oc = t - c
        b = d[0] * oc[0] + d[1] * oc[1] + d[2] * oc[2]
        disc = b * b - dd * float(oc @ oc - r * r)
        zs = (-b - disc.clamp(min=0).sqrt()) / dd
        z = torch.where((disc > 0) & (zs > 0), torch.minimum(z, zs), z)
    for blo, bhi in room["boxes"]:
        near = torch.full_like(z, -math.inf)
        far = torch.full_like(z, math.inf)
        for i in range(3):
            a, b = (blo[i] - t[i]) / d[i], (bhi[i] - t[i]) / d[i]
            near, far = torch.maximum(near, torch.minimum(a, b)), torch.minimum(far, torch.maximum(a, b))
        z = torch.where((near <= far) & (near > 0), torch.minimum(z, near), z)
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = z + 0.002 * z * z * torch.randn(z.shape, generator=g, dtype=torch.float64, device="cuda")
    z = torch.where((z > 0.05) & (z < 6.0), z, 0.0)
    return torch.where(torch.rand(z.shape, generator=g, device="cuda") < 0.02, 0.0, z).float().contiguous()


def _map(case, room):
    """A saved map of the room: the truncated distance at voxel centres (+1
    where nothing was seen, behind the surfaces) and the weights."""
    nx, ny, nz, vox, mu = (case[k] for k in ("nx", "ny", "nz", "vox", "mu"))
    c = [(torch.arange(n, device="cuda", dtype=torch.float32) + 0.5) * vox for n in (nx, ny, nz)]
    psi = torch.empty((nz, ny, nx), device="cuda")
    for k0 in range(0, nz, 64):
        x, y, z = c[0][None, None, :], c[1][None, :, None], c[2][k0:k0 + 64, None, None]
        lo, hi = room["lo"], room["hi"]
        d = torch.minimum(torch.minimum(x - lo[0], hi[0] - x), torch.minimum(y - lo[1], hi[1] - y))
        d = torch.minimum(d, torch.minimum(z - lo[2], hi[2] - z))
        for p, r in room["spheres"]:
            d = torch.minimum(d, ((x - p[0]) ** 2 + (y - p[1]) ** 2 + (z - p[2]) ** 2).sqrt() - r)
        for blo, bhi in room["boxes"]:
            q = [(v - 0.5 * (blo[i] + bhi[i])).abs() - 0.5 * (bhi[i] - blo[i]) for i, v in enumerate((x, y, z))]
            out = (q[0].clamp(min=0) ** 2 + q[1].clamp(min=0) ** 2 + q[2].clamp(min=0) ** 2).sqrt()
            d = torch.minimum(d, out + torch.maximum(torch.maximum(q[0], q[1]), q[2]).clamp(max=0))
        psi[k0:k0 + 64] = torch.where(d < -mu, 1.0, (d / mu).clamp(-1, 1))
    g = torch.Generator(device="cuda").manual_seed(case["nx"])
    wt = torch.randint(1, 40, psi.shape, generator=g, device="cuda").float()
    return psi, wt


def _volume(case):
    return rose.Tsdf((case["nx"], case["ny"], case["nz"]), case["vox"], case["mu"], (0.0, 0.0, 0.0),
                     fmt=FMT[case["fmt"]])


def _params(case):
    levels = [(max(1, int(s * case["n"])), st) for s, st in LEVELS] if case["levels"] else None
    return rose.track_params(max_iters=case["iters"], stride=case["stride"], lookup=LOOKUP[case["lookup"]],
                             levels=levels)


def _copy_state(st):
    return rose.TrackState.from_buffer_copy(st)


def _poses_about(case, seed):
    """n candidate poses (3x4 float32) about the camera, the first exact."""
    room = _room(case, seed)
    R, t = _pose(room, 8)
    g = torch.Generator(device="cuda").manual_seed(seed + 17)
    u = torch.randn((case["n"], 6), generator=g, device="cuda", dtype=torch.float64) * case["spread"] / 2
    u[0] = 0
    a = u[:, :3]
    th = a.norm(dim=1, keepdim=True).clamp(min=1e-12)
    k = a / th
    Kx = torch.zeros((case["n"], 3, 3), device="cuda", dtype=torch.float64)
    Kx[:, 0, 1], Kx[:, 0, 2], Kx[:, 1, 2] = -k[:, 2], k[:, 1], -k[:, 0]
    Kx = Kx - Kx.transpose(1, 2)
    KK = (Kx[:, :, :, None] * Kx[:, None, :, :]).sum(2)
    E = torch.eye(3, device="cuda", dtype=torch.float64) + torch.sin(th)[:, :, None] * Kx + (1 - torch.cos(th))[:, :, None] * KK
    Rt = torch.tensor(R, device="cuda")
    Rn = (Rt[None, :, :, None] * E[:, None, :, :]).sum(2)
    tn = torch.tensor(t, device="cuda") + u[:, 3:]
    return torch.cat([Rn, tn[:, :, None]], dim=2).float().contiguous()


# -------------------------------------------------------------------- prepare
def _prepare_tracker(case, seed, fused=10):
    """A volume fused from the frames so far, the state carried from the last
    tracked one, and the next frame; in a sequence's second frame one fused
    frame and the axis lengths that the first frame's rule gives."""
    fused = 1 if case["first"] else fused
    room, K = _room(case, seed), _Camera(case["w"], case["h"])
    vol = _volume(case)
    if case["switch"]:
        vol.set_fitness_shape(0, 0)
    poses = [_pose(room, k) for k in range(fused + 2)]
    depths = [_render(room, K, *p, seed * 100 + k) for k, p in enumerate(poses)]
    for k in range(fused):
        vol.integrate(depths[k], K, _quat(poses[k][0]), poses[k][1])
    pst = rose.pst_sample(case["n"], 5600 + seed)
    params = _params(case)
    st = rose.track_state(_quat(poses[fused - 1][0]), poses[fused - 1][1], [0.55 if case["first"] else 0.1] * 6)
    if case["first"]:
        return dict(case=case, vol=vol, K=K, pst=pst, params=params, start=st, depth=depths[1], vel=[0.0] * 6)
    before = list(st.pose.q), list(st.pose.t)
    rose.track_frame(vol, depths[fused], K, pst, params, st)
    vol.integrate(depths[fused], K, st.pose.q, st.pose.t)
    vel = rose.chart_log(*before, st.pose.q, st.pose.t)
    return dict(case=case, vol=vol, K=K, pst=pst, params=params, start=st, depth=depths[fused + 1], vel=vel)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "track":
        return _prepare_tracker(case, seed)
    if kind == "learned":
        s = _prepare_tracker(case, seed)
        z = np.load(os.path.join(os.path.dirname(rose.__file__), "weights", "proposal.npz"))
        s["net"] = rose.Mlp(NET_IN, NET_HID, NET_OUT, max_batch=64)
        s["weights"] = s["net"].pack({k: z[k] for k in ("W1", "b1", "W2", "b2", "W3", "b3")})
        s["plain_pst"] = rose.pst_sample(10240, 5600 + seed)
        s["work"] = torch.zeros(40 * 30 + NET_IN + NET_OUT, device="cuda")
        s["plain"] = rose.track_params(max_iters=20, stride=case["stride"], lookup=LOOKUP[case["lookup"]])
        s["lp"] = rose.learned_params(scale=8, kappa=3.0, delta=0.01, iters=case["iters"])
        return s
    if kind == "batch":
        K, vols, depths, psts = _Camera(case["w"], case["h"]), [], [], []
        states = (rose.TrackState * case["count"])()
        maps = []
        for i in range(case["count"]):
            if i < 8:  # eight rooms; the others are further cameras in them
                room = _room(case, seed * 1000 + i)
                maps.append((room, *_map(case, room)))
            room, psi, wt = maps[i % 8]
            vol = _volume(case)
            if case["switch"]:
                vol.set_fitness_shape(0, 0)
            vol.load(psi, wt)
            R, t = _pose(room, 3 * i)
            states[i] = rose.track_state(_quat(R), t, [0.1] * 6)
            vols.append(vol)
            depths.append(_render(room, K, *_pose(room, 3 * i + 1), seed * 100 + i))
            psts.append(rose.pst_sample(case["n"], 5600 + i))
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        b = rose.Batch(vols, [K] * case["count"], psts, [_params(case)] * case["count"])
        return dict(case=case, batch=b, depths=depths, start=states, stream=stream, keep=(vols, psts))
    if kind == "forward" or kind == "train":
        g = torch.Generator(device="cuda").manual_seed(seed)
        net = rose.Mlp(NET_IN, NET_HID, NET_OUT, max_batch=case["batch"])
        P = _net_params(seed)
        X = _features(case["batch"], g)
        s = dict(case=case, net=net, P=P, X=X)
        if kind == "train":
            s["Y"], s["m"], s["v"] = _train_extra(case["batch"], P.numel(), g)
            s["grads"], s["loss"], s["step"] = torch.zeros_like(P), torch.zeros(1, device="cuda"), 1000
        return s
    if kind == "gemm":
        return dict(case=case, **dict(zip("AB", _gemm_inputs(case, seed))))
    room, K = _room(case, seed), _Camera(case["w"], case["h"])
    vol = _volume(case)
    vol.load(*_map(case, room))
    R, t = _pose(room, 8)
    s = dict(case=case, vol=vol, K=K, q=_quat(R), t=t)
    if kind != "raycast":
        s["depth"] = _render(room, K, R, t, seed)
    if kind == "fitness":
        s["pts"] = _points(s["depth"], K, case["stride"])
        s["T"] = _poses_about(case, seed)
    return s


def _points(depth, K, stride):
    """The frame's samples as camera-frame points, in 8x8-sample tiles as the tracker takes them."""
    return rose.depth_unproject(depth, K, stride, tiled=True).clone()


def _net_params(seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 5)
    part = []
    for i, o in ((NET_IN, NET_HID), (NET_HID, NET_HID), (NET_HID, NET_OUT)):
        part.append(torch.randn(i * o, generator=g, device="cuda") * math.sqrt(2.0 / i))
        part.append(torch.randn(o, generator=g, device="cuda") * 0.05)
    return torch.cat(part)


def _features(batch, g):
    """Depth residuals (many exactly zero), the previous motion, zero padding."""
    X = torch.randn((batch, NET_IN), generator=g, device="cuda") * 0.1
    X = X.clamp(-0.5, 0.5) * (torch.rand((batch, NET_IN), generator=g, device="cuda") > 0.2)
    X[:, 1206:] = 0
    return X


def _train_extra(batch, n, g):
    Y = torch.randn((batch, 6), generator=g, device="cuda") * 0.05
    m = torch.randn(n, generator=g, device="cuda") * 1e-3
    v = torch.rand(n, generator=g, device="cuda") * 1e-4 + 1e-6
    return Y, m, v


def _gemm_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    m, n, k = case["m"], case["n"], case["k"]
    A = torch.randn((k, m) if case["ta"] else (m, k), generator=g, device="cuda")
    B = torch.randn((n, k) if case["tb"] else (k, n), generator=g, device="cuda")
    return (A.t() if case["ta"] else A), (B.t() if case["tb"] else B)


# ------------------------------------------------------------------------ run
def _track_out(r):
    out = {k: np.array(r[k], np.float64) for k in ("q", "t", "r1")}
    out["rho"] = float(r["rho"])
    for k in ("aps", "n_overlap"):
        out[k] = np.array(r[k], np.int64)
    return out


def run(s):
    kind = s["case"]["kind"]
    if kind == "track":
        st = _copy_state(s["start"])
        r = rose.track_frame(s["vol"], s["depth"], s["K"], s["pst"], s["params"], st)
        out = _track_out(r)
        out["rho_iter"] = np.array(r["rho_iter"])
        out["rho_centre"] = np.array(r["rho_centre"])
        return out
    if kind == "learned":
        st = _copy_state(s["start"])
        r = rose.track_frame_learned(s["vol"], s["depth"], s["K"], s["pst"], s["plain_pst"], s["net"], s["weights"],
                                     s["work"], s["vel"], s["params"], s["lp"], st)
        out = _track_out(r)
        out["fallback"] = int(r["fallback"])
        return out
    if kind == "batch":
        n = s["case"]["count"]
        states = (rose.TrackState * n).from_buffer_copy(s["start"])
        rs = s["batch"].track(s["depths"], states, stream=s["stream"])
        return {k: np.array([r[k] for r in rs]) for k in ("q", "t", "r1", "rho", "aps", "n_overlap")}
    if kind == "fitness":
        F, rho = rose.fitness_eval(s["vol"], s["pts"], s["T"], LOOKUP[s["case"]["lookup"]])
        return {"F": F, "rho": rho}
    if kind == "integrate":
        s["vol"].integrate(s["depth"], s["K"], s["q"], s["t"])
        return {"psi": s["vol"].psi, "weight": s["vol"].weight}
    if kind == "raycast":
        return {"depth": rose.raycast(s["vol"], s["q"], s["t"], s["K"])}
    if kind == "forward":
        return {"out": s["net"].forward(s["P"], s["X"])}
    if kind == "train":
        s["net"].loss_grad(s["P"], s["X"], s["Y"], s["grads"], s["loss"])
        s["step"] += 1
        rose.Mlp.adam(s["P"], s["grads"], s["m"], s["v"], s["step"], 1e-4)
        return {k: s[k] for k in ("P", "grads", "loss", "m", "v")}
    return {"C": rose.gemm_bf16(s["A"], s["B"])}


# ----------------------------------------------------------------------- work
def work(case):
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4.0 * (m * k + k * n + m * n), "flops": 2.0 * m * n * k}
    net = NET_IN * NET_HID + NET_HID * NET_HID + NET_HID * NET_OUT
    if kind == "forward":
        return {"bytes": 4.0 * (net + case["batch"] * (NET_IN + NET_OUT)), "flops": 2.0 * net * case["batch"]}
    if kind == "train":
        # parameters, both moments read and written, gradients written and read
        return {"bytes": 4.0 * (8 * net + case["batch"] * (NET_IN + 6)),
                "flops": case["batch"] * (4.0 * net + 2.0 * (NET_HID * NET_HID + NET_HID * NET_OUT)) + 12.0 * net}
    vox = float(case["nx"]) * case["ny"] * case["nz"]
    elem = 4.0 if case["fmt"] == "f32" else 2.0
    if kind == "integrate":
        # about a quarter of the volume is in view and not behind a surface:
        # value and weight read and written there
        return {"bytes": 4.0 * case["w"] * case["h"] + 0.25 * vox * 4 * elem, "flops": 0.25 * vox * 30}
    if kind == "raycast":
        rays = float(case["w"]) * case["h"]
        steps = 0.5 * min(case["nx"], case["ny"], case["nz"]) / 0.5  # half the room at half a voxel
        return {"bytes": 4.0 * rays + min(vox, rays * steps) * elem, "flops": rays * steps * 60}

    def evals_flops(n, m, tri):
        return n * m * (22.0 + (14.0 if tri else 0.0))

    def points(stride):
        return math.ceil(case["w"] / stride) * math.ceil(case["h"] / stride)

    tri = case["lookup"] == "trilinear"
    reads = 8.0 if tri else 1.0
    if kind == "fitness":
        n, m = case["n"], points(case["stride"])
        return {"bytes": 12.0 * m + 56.0 * n + min(vox, n * m * reads) * elem, "flops": evals_flops(n, m, tri)}
    it = case["iters"]
    if case["levels"]:
        per = [(max(1, int(s * case["n"])), points(st)) for s, st in LEVELS]
        evals = sum(per[k % 3][0] * per[k % 3][1] for k in range(it))
    else:
        evals = float(case["n"]) * points(case["stride"]) * it
    one = {"bytes": 4.0 * points(case["stride"]) + 24.0 * case["n"] + min(vox, evals * reads) * elem,
           "flops": evals_flops(1, evals, tri)}
    c = case.get("count", 1)
    return {"bytes": c * one["bytes"], "flops": c * one["flops"]}


# ---------------------------------------------------------------------- exact
def _stored(case, psi):
    """What the volume's format keeps of a loaded map, in 64 bits."""
    if case["fmt"] == "f16":
        return psi.half().double()
    if case["fmt"] == "sn16":
        return torch.round(psi.double().clamp(-1, 1) * 32767.0) / 32767.0
    return psi.double()


def _bricks(v):
    """A linear [k][j][i] volume in 8x8x8 bricks, x-fastest throughout."""
    nz, ny, nx = v.shape
    return v.reshape(nz // 8, 8, ny // 8, 8, nx // 8, 8).permute(0, 2, 4, 1, 3, 5).reshape(-1)


def _corners(vol, g):
    """Trilinear psi at voxel coordinates g (3 tensors), +1 where a corner is outside."""
    nz, ny, nx = vol.shape
    h = [c - 0.5 for c in g]
    ok = torch.ones_like(h[0], dtype=torch.bool)
    for c, n in zip(h, (nx, ny, nz)):
        ok &= (c >= 0) & (c < n - 1)
    i = [torch.where(ok, c, 0.0).floor().long() for c in h]
    f = [torch.where(ok, c, 0.0) - b for c, b in zip(h, i)]
    flat = vol.reshape(-1)
    acc = torch.zeros_like(h[0])
    for dz in (0, 1):
        for dy in (0, 1):
            for dx in (0, 1):
                w = (f[0] if dx else 1 - f[0]) * (f[1] if dy else 1 - f[1]) * (f[2] if dz else 1 - f[2])
                acc += w * flat[((i[2] + dz) * ny + i[1] + dy) * nx + i[0] + dx]
    return torch.where(ok, acc, 1.0)


def _nearest(vol, g):
    nz, ny, nx = vol.shape
    ok = torch.ones_like(g[0], dtype=torch.bool)
    for c, n in zip(g, (nx, ny, nz)):
        ok &= (c >= 0) & (c < n)
    i = [torch.where(ok, c, 0.0).long() for c in g]
    return torch.where(ok, vol.reshape(-1)[(i[2] * ny + i[1]) * nx + i[0]], 1.0)


def exact(case, seed):
    kind = case["kind"]
    # a search takes discrete decisions (voxels, which particles beat the
    # threshold) that are defined in 32 bits: its result has no 64-bit value
    if kind in ("track", "learned", "batch"):
        return None
    if kind == "gemm":
        A, B = _gemm_inputs(case, seed)
        return {"C": (A.double() @ B.double())}
    if kind in ("forward", "train"):
        g = torch.Generator(device="cuda").manual_seed(seed)
        P = _net_params(seed).double()
        X = _features(case["batch"], g).double()
        if kind == "forward":
            return {"out": _net(P, X)}
        Y, m, v = (t.double() for t in _train_extra(case["batch"], P.numel(), g))
        P.requires_grad_(True)
        o = _net(P, X)
        loss = ((Y - o[:, :6]) ** 2 / (2 * torch.exp(2 * o[:, 6:])) + o[:, 6:]).sum(1).mean()
        (gr,) = torch.autograd.grad(loss, P)
        m2, v2 = 0.9 * m + 0.1 * gr, 0.999 * v + 0.001 * gr * gr
        upd = 1e-4 * (m2 / (1 - 0.9 ** 1001)) / ((v2 / (1 - 0.999 ** 1001)).sqrt() + 1e-8)
        return {"P": P.detach() - upd, "grads": gr, "loss": loss.detach().reshape(1), "m": m2, "v": v2}
    room, K = _room(case, seed), _Camera(case["w"], case["h"])
    psi, wt = _map(case, room)
    vol = _stored(case, psi)
    R, t = _pose(room, 8)
    if kind == "integrate":
        depth = _render(room, K, R, t, seed).double()
        nz, ny, nx = vol.shape
        mu, vox = float(np.float32(case["mu"])), float(np.float32(case["vox"]))
        wt = wt.double()
        for k0 in range(0, nz, 32):
            z, y, x = (torch.arange(a, b, device="cuda", dtype=torch.float64) for a, b in
                       ((k0, min(nz, k0 + 32)), (0, ny), (0, nx)))
            X = [((x + 0.5) * vox - t[0])[None, None, :], ((y + 0.5) * vox - t[1])[None, :, None],
                 ((z + 0.5) * vox - t[2])[:, None, None]]
            c = [R[0, i] * X[0] + R[1, i] * X[1] + R[2, i] * X[2] for i in range(3)]
            u = torch.floor(K.fx * c[0] / c[2] + K.cx + 0.5)
            v = torch.floor(K.fy * c[1] / c[2] + K.cy + 0.5)
            ok = (c[2] > 0) & (u >= 0) & (u < K.width) & (v >= 0) & (v < K.height)
            D = depth.reshape(-1)[torch.where(ok, v * K.width + u, 0.0).long()]
            ok &= (D > 0) & (D - c[2] >= -mu)
            d = ((D - c[2]) / mu).clamp(max=1.0)
            p, w = vol[k0:k0 + 32], wt[k0:k0 + 32]
            p.copy_(torch.where(ok, (w * p + d) / (w + 1), p))
            w.copy_(torch.where(ok, (w + 1).clamp(max=128.0), w))
        psi64 = _bricks(vol)
        if case["fmt"] == "sn16":
            return None  # whole numbers throughout
        return {"psi": psi64, "weight": _bricks(wt) if case["fmt"] == "f32" else None}
    vox = float(np.float32(case["vox"]))
    if kind == "raycast":
        u = torch.arange(K.width, dtype=torch.float64, device="cuda")
        v = torch.arange(K.height, dtype=torch.float64, device="cuda")
        fx, cx, cy = (float(np.float32(a)) for a in (K.fx, K.cx, K.cy))
        dx = ((u - cx) / fx)[None, :].expand(K.height, K.width)
        dy = ((v - cy) / fx)[:, None].expand(K.height, K.width)
        d = [R[i, 0] * dx + R[i, 1] * dy + R[i, 2] for i in range(3)]
        step = case["vox"] / 2
        out = torch.zeros_like(dx)
        prev, done = torch.ones_like(dx), torch.zeros_like(dx, dtype=torch.bool)
        far = min(8.0, 2.0 * float(room["ext"].max()))  # every ray has left the volume by then
        k = 0
        while 0.2 + k * step <= far:
            z = 0.2 + k * step
            s = _corners(vol, [(t[i] + z * d[i]) / vox for i in range(3)])
            if k:
                hit = ~done & (prev > 0) & (s <= 0) & (prev < 1) & (s > -1)
                out = torch.where(hit, (z - step) + step * prev / (prev - s), out)
                done |= hit
            prev = s
            k += 1
        return {"depth": out}
    # fitness
    depth = _render(room, K, R, t, seed)
    pts = _points64(depth, K, case["stride"])
    T = _poses_about(case, seed).double()
    look = _nearest if case["lookup"] == "nearest" else _corners
    F = []
    step = max(1, 8_000_000 // max(1, pts.shape[0]))
    for i in range(0, T.shape[0], step):
        Tc = T[i:i + step]
        g = [(Tc[:, a, 0, None] * pts[:, 0] + Tc[:, a, 1, None] * pts[:, 1] + Tc[:, a, 2, None] * pts[:, 2]
              + Tc[:, a, 3, None]) / vox for a in range(3)]
        F.append((look(vol, g) ** 2).mean(dim=1))
    F = torch.cat(F)
    return {"F": F, "rho": torch.exp(-F)}


def _points64(depth, K, stride):
    d = depth.double()[::stride, ::stride]
    v, u = torch.meshgrid(torch.arange(0, K.height, stride, device="cuda", dtype=torch.float64),
                          torch.arange(0, K.width, stride, device="cuda", dtype=torch.float64), indexing="ij")
    p = torch.stack([(u - K.cx) * d / K.fx, (v - K.cy) * d / K.fy, d], dim=-1)
    return p[d > 0]


def _net(P, X):
    i = 0
    h = X
    for a, b, last in ((NET_IN, NET_HID, False), (NET_HID, NET_HID, False), (NET_HID, NET_OUT, True)):
        W = P[i:i + a * b].reshape(a, b)
        h = h @ W + P[i + a * b:i + a * b + b]
        i += a * b + b
        if not last:
            h = 0.5 * h * (1 + torch.erf(h / math.sqrt(2.0)))
    return h
