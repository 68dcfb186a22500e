"""Performance cases of the bundle adjuster: the calls that a mapping backend makes.

Every case is one call sequence through the package's public entry points on
inputs that a frontend would hand it: keyframe windows (one at a time and in
batches), the adjoint and the differentiable solve, motion-only frames,
triangulation, pose graphs and visual-inertial windows.  ``listed`` names the
cases, ``draw`` gives others of the same ranges, ``prepare`` makes what the
caller has in hand, ``run`` is one pass, ``work`` the bytes and operations the
pass cannot do without, and ``exact`` the same answer by plain torch in 64 bits.

Inputs are synthetic: EuRoC-like mono windows (752x480, f = 458), a KITTI-like
stereo pair (1241x376, f = 718, 0.54 m) and a 32-camera outward-facing rig, with
pixel noise, some gross mismatches under the Huber kernel, and starts a few
centimetres and degrees off.  Mono windows hold their two oldest keyframes (a
sliding window's gauge: one pose leaves the scale free).
"""
import math

import numpy as np
import torch

import paper_2506_04359_amd as ba

DELTA, LAM0, MIN_DEPTH = 1.0, 1e-3, 1e-3
IMU_NOISE = (1.7e-4, 2.0e-3, 2.0e-5, 3.0e-3)   # gyro, accel, gyro walk, accel walk densities
IMU_RATE = 200.0
F64 = torch.float64


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _win(name, op="solve", rig="mono", windows=1, kf_lo=5, kf_hi=5, lm_lo=200, lm_hi=200, track="subset",
         iters=10, precision="fp64", weighted=False):
    c = dict(kind="window", op=op, rig=rig, windows=windows, kf_lo=kf_lo, kf_hi=kf_hi, lm_lo=lm_lo, lm_hi=lm_hi,
             track=track, iters=iters, precision=precision, weighted=weighted)
    return dict(c, name=name) if name else c


def _pnp(name, rig="stereo", frames=1, lm=300, uneven=False, map_frame=False, weighted=False, iters=10,
         precision="fp64"):
    c = dict(kind="pnp", rig=rig, frames=frames, lm=lm, uneven=uneven, map_frame=map_frame, weighted=weighted,
             iters=iters, precision=precision)
    return dict(c, name=name) if name else c


def _tri(name, rig="mono", windows=1, kf=20, lm=4000, iters=10, precision="fp64"):
    c = dict(kind="tri", rig=rig, windows=windows, kf=kf, lm=lm, iters=iters, precision=precision)
    return dict(c, name=name) if name else c


def _pgo(name, laps=3, per_lap=500, weighted=False, iters=10):
    c = dict(kind="pgo", laps=laps, per_lap=per_lap, weighted=weighted, iters=iters)
    return dict(c, name=name) if name else c


def _vi(name, kf=10, lm=400, samples=50, iters=10, precision="fp64"):
    c = dict(kind="vi", kf=kf, lm=lm, samples=samples, iters=iters, precision=precision)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest window: a mono frontend's last five keyframes, in the library's default precision
        _win("window-mono-5kf"),
        # one stereo SLAM backend's local map, solved after each keyframe
        _win("window-stereo-20kf", rig="stereo", kf_lo=20, kf_hi=20, lm_lo=5000, lm_hi=5000, precision="mixed"),
        # a 32-camera rig's window: few poses, 300 k observations
        _win("window-rig-32cam", rig="rig", kf_lo=10, kf_hi=10, lm_lo=20000, lm_hi=20000, precision="mixed"),
        # a mapping server: many uneven windows of many robots in one call
        _win("batch-256-mono", windows=256, kf_lo=5, kf_hi=30, lm_lo=500, lm_hi=8000, iters=15, precision="mixed"),
        # a small batch with observation weights in the default precision
        _win("batch-16-weighted", windows=16, kf_lo=5, kf_hi=30, lm_lo=500, lm_hi=3000, weighted=True),
        # gradients of a pose loss to the keypoints of a training batch, at converged windows
        _win("adjoint-64", op="adjoint", windows=64, kf_lo=10, kf_hi=10, lm_lo=2000, lm_hi=2000, track="long",
             precision="mixed", weighted=True),
        # one step of training through the differentiable solve: forward, loss, backward
        _win("train-4", op="train", windows=4, kf_lo=8, kf_hi=10, lm_lo=400, lm_hi=700, track="long", iters=15,
             weighted=True),
        # the tracker's call for one stereo frame against the map
        _pnp("pnp-1-stereo"),
        # relocalisation or log replay: many stereo frames at once
        _pnp("pnp-4096-stereo", frames=4096, precision="mixed"),
        # every landmark of many windows triangulated from its tracks
        _tri("tri-1m-mono", windows=256, kf=18, lm=4100, precision="mixed"),
        # loop closing over a 1500-keyframe trajectory
        _pgo("pgo-1500"),
        # a visual-inertial window: preintegration of its samples, then the solve
        _vi("vi-10kf"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["window", "window", "window", "batch", "adjoint", "train", "pnp", "pnp", "tri", "pgo", "vi"])
    prec = rng.choice(["mixed", "fp64"])
    w = rng.random() < 0.4
    if kind == "window":
        rig = rng.choice(["mono", "mono", "stereo", "rig"])
        if rig == "rig":
            lm = _log(rng, 1000, 20000)
            kf = rng.randint(4, 10)
        else:
            lm = _log(rng, 150, 8000)
            kf = rng.randint(4, 30 if rig == "mono" else 24)
        return _win(None, rig=rig, kf_lo=kf, kf_hi=kf, lm_lo=lm, lm_hi=lm, iters=rng.randint(5, 15), precision=prec,
                    weighted=w)
    if kind == "batch":
        n = _log(rng, 2, 160)
        lo = rng.randint(200, 1500)
        return _win(None, windows=n, kf_lo=rng.randint(4, 9), kf_hi=rng.randint(10, 30), lm_lo=lo,
                    lm_hi=lo + rng.randint(100, 5000 if n < 64 else 2500), iters=rng.randint(5, 15), precision=prec,
                    weighted=w)
    if kind == "adjoint":
        n, kf = _log(rng, 1, 64), rng.randint(5, 14)
        lm = _log(rng, 200, 2000)
        return _win(None, op="adjoint", windows=n, kf_lo=kf, kf_hi=kf + rng.randint(0, 2), lm_lo=lm,
                    lm_hi=lm + rng.randint(0, 300), track="long", precision=prec, weighted=w)
    if kind == "train":
        kf = rng.randint(6, 12)
        lm = _log(rng, 200, 1000)
        return _win(None, op="train", windows=_log(rng, 1, 8), kf_lo=kf, kf_hi=kf + rng.randint(0, 2), lm_lo=lm,
                    lm_hi=lm + rng.randint(0, 200), track="long", iters=15, weighted=w)
    if kind == "pnp":
        rig = rng.choice(["stereo", "stereo", "rig"])
        return _pnp(None, rig=rig, frames=_log(rng, 1, 4096 if rig == "stereo" else 512), lm=_log(rng, 40, 300),
                    uneven=rng.random() < 0.5, map_frame=rng.random() < 0.3, weighted=w, iters=rng.randint(5, 10),
                    precision=prec)
    if kind == "tri":
        rig = rng.choice(["mono", "mono", "stereo"])
        return _tri(None, rig=rig, windows=_log(rng, 1, 128), kf=rng.randint(6, 30), lm=_log(rng, 200, 4100),
                    iters=rng.randint(5, 10), precision=prec)
    if kind == "pgo":
        return _pgo(None, laps=rng.randint(2, 4), per_lap=_log(rng, 30, 375), weighted=w, iters=rng.randint(6, 10))
    return _vi(None, kf=rng.randint(4, 20), lm=_log(rng, 120, 800), samples=rng.randint(20, 60),
               iters=rng.randint(6, 12), precision=prec)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

class _Rand:
    """Random numbers on the GPU from one seed."""

    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(int(seed) * 7919 + 13)

    def u(self, lo, hi, *shape):
        return torch.rand(*shape, generator=self.g, device=self.dev, dtype=F64) * (hi - lo) + lo

    def n(self, *shape):
        return torch.randn(*shape, generator=self.g, device=self.dev, dtype=F64)

    def ints(self, lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=self.g, device=self.dev)

    def unit(self, *shape):
        v = self.n(*shape, 3)
        return v / v.norm(dim=-1, keepdim=True)


def _skew(v):
    z = torch.zeros_like(v[..., 0])
    return torch.stack([torch.stack([z, -v[..., 2], v[..., 1]], -1), torch.stack([v[..., 2], z, -v[..., 0]], -1),
                        torch.stack([-v[..., 1], v[..., 0], z], -1)], -2)


def _rot(phi):
    """Rotation matrices of rotation vectors (..., 3)."""
    th = phi.norm(dim=-1)[..., None, None]
    K = _skew(phi)
    s = torch.where(th < 1e-6, 1 - th * th / 6, torch.sin(th) / th.clamp_min(1e-300))
    h = torch.sin(0.5 * th)
    c = torch.where(th < 1e-6, 0.5 - th * th / 24, 2 * h * h / (th * th).clamp_min(1e-300))
    return torch.eye(3, dtype=phi.dtype, device=phi.device) + s * K + c * (K @ K)


def _pose(R_wc, centre):
    R = R_wc.transpose(-1, -2)
    return torch.cat([R, -(R @ centre[..., None])], -1)


def _rig(name, rand):
    """Intrinsics (C, 4), extrinsics (C, 3, 4) and image size of a rig."""
    dev = rand.dev
    eye = torch.cat([torch.eye(3, dtype=F64, device=dev), torch.zeros(3, 1, dtype=F64, device=dev)], 1)[None]
    if name == "mono":
        return torch.tensor([[458.0, 458.0, 367.0, 248.0]], dtype=F64, device=dev), eye, (752.0, 480.0)
    if name == "stereo":
        E = eye.repeat(2, 1, 1)
        E[1, 0, 3] = -0.54
        return torch.tensor([[718.0, 718.0, 607.0, 185.0]] * 2, dtype=F64, device=dev), E, (1241.0, 376.0)
    z, a = rand.unit(32), rand.unit(32)
    x = torch.linalg.cross(a, z)
    x = x / x.norm(dim=-1, keepdim=True)
    R = torch.stack([x, torch.linalg.cross(z, x), z], 1)   # camera-from-base
    E = torch.cat([R, -(R @ (0.3 * z)[..., None])], -1)
    return torch.tensor([[400.0, 400.0, 320.0, 240.0]] * 32, dtype=F64, device=dev), E, (640.0, 480.0)


def _project(K, x):
    return torch.stack([K[..., 0] * x[..., 0] / x[..., 2] + K[..., 2], K[..., 1] * x[..., 1] / x[..., 2] + K[..., 3]], -1)


def _views(pts, poses, K, E, size):
    """Visibility (n, poses, cameras) of points."""
    xb = torch.einsum("fab,nb->nfa", poses[:, :, :3], pts) + poses[:, :, 3]
    xc = torch.einsum("cab,nfb->nfca", E[:, :, :3], xb) + E[:, :, 3]
    uv = _project(K, torch.where(xc[..., 2:] > 0.1, xc, torch.ones_like(xc)))
    return (xc[..., 2] > 0.1) & (uv[..., 0] >= 0) & (uv[..., 0] < size[0]) & (uv[..., 1] >= 0) & (uv[..., 1] < size[1])


def _pixels(rand, pts, poses, K, E, i, j, k, sigma, mismatch):
    xb = (poses[i][:, :, :3] @ pts[j][..., None])[..., 0] + poses[i][:, :, 3]
    xc = (E[k][:, :, :3] @ xb[..., None])[..., 0] + E[k][:, :, 3]
    s = torch.full((i.numel(), 1), sigma, dtype=F64, device=rand.dev)
    if mismatch > 0:   # matches the frontend should not have kept: several pixels off
        s = torch.where(rand.u(0, 1, i.numel(), 1) < mismatch, 8 * s, s)
    return _project(K[k], xc) + s * rand.n(i.numel(), 2)


def _scene(rand, rig, n_kf, n_lm, track, K, E, size):
    """Poses (n_kf, 3, 4), points (n_lm, 3) and observation lists (pose, point, camera)."""
    dev = rand.dev
    k = torch.arange(n_kf, device=dev, dtype=F64)
    pts, chosen, have = [], [], 0
    if rig == "mono":
        ang = torch.zeros(n_kf, 3, dtype=F64, device=dev)
        ang[:, 1] = rand.u(-1, 1, n_kf) * math.radians(5.0)
        centre = torch.stack([0.5 * k, 0 * k, 0 * k], 1)
        poses = _pose(_rot(ang), centre)
        # "subset": a random 2 (3 in the shortest windows) to 10 of the visible frames; "long":
        # tracks through most of the window
        lo = (3 if n_kf <= 5 else 2) if track == "subset" else max(3, n_kf - 2)
        while have < n_lm:
            m = 2 * (n_lm - have) + 256
            p = torch.stack([rand.u(-4.0, 0.5 * (n_kf - 1) + 4.0, m), rand.u(-3, 3, m), rand.u(2, 20, m)], 1)
            v = _views(p, poses, K, E, size)[:, :, 0]
            nv = v.sum(1)
            key = torch.where(v, rand.u(0, 1, m, n_kf), torch.full((), 2.0, dtype=F64, device=dev))
            rank = key.argsort(1).argsort(1)
            if track == "subset":
                v = v & (rank < (lo + (rand.u(0, 1, m) * (nv.clamp_max(10) - lo + 1)).long())[:, None])
            ok = torch.nonzero(nv >= lo)[: n_lm - have, 0]
            v = v[ok]
            if track == "long":   # the same number of observations for every seed
                v = v & (rank[ok] < (lo - (have + torch.arange(ok.numel(), device=dev)) % 2)[:, None])
            pts.append(p[ok])
            chosen.append(v[:, :, None])
            have += ok.numel()
    elif rig == "stereo":
        yaw = torch.cumsum(rand.u(-1, 1, n_kf) * math.radians(1.0), 0)
        ang = torch.zeros(n_kf, 3, dtype=F64, device=dev)
        ang[:, 1] = yaw
        R = _rot(ang)
        step = R[:, :, 2]
        centre = torch.cumsum(torch.cat([torch.zeros(1, 3, dtype=F64, device=dev), step[:-1]]), 0)
        poses = _pose(R, centre)
        while have < n_lm:
            m = 3 * (n_lm - have) + 256
            want = 2 + torch.floor(torch.log(rand.u(1e-12, 1, m)) / math.log(1 - 0.14)).long()
            want = want.clamp_max(min(15, n_kf))
            e = rand.ints(1, n_kf, m)
            d = torch.exp(rand.u(math.log(3.0), math.log(60.0), m))
            u, w = rand.u(0, size[0], m), rand.u(0, size[1], m)
            xc = torch.stack([(u - K[0, 2]) / K[0, 0] * d, (w - K[0, 3]) / K[0, 1] * d, d], 1)
            p = (poses[e][:, :, :3].transpose(1, 2) @ (xc - poses[e][:, :, 3])[..., None])[..., 0]
            v = _views(p, poses, K, E, size).all(2)
            back = (e[:, None] - torch.arange(15, device=dev)[None]).clamp_min(0)
            seen = torch.gather(v, 1, back) & (torch.arange(15, device=dev)[None] <= e[:, None])
            run = torch.cumprod(seen.long(), 1).sum(1)
            n = torch.minimum(run, want)
            fr = torch.arange(n_kf, device=dev)[None]
            v = (fr <= e[:, None]) & (fr > (e - n)[:, None])
            ok = torch.nonzero(n >= 2)[: n_lm - have, 0]
            pts.append(p[ok])
            chosen.append(v[ok][:, :, None].expand(-1, -1, 2))
            have += ok.numel()
    else:
        th = 0.2 * k
        centre = torch.stack([2 * torch.sin(th), 0 * th, 2 * torch.cos(th)], 1)
        fwd = torch.stack([torch.cos(th), 0 * th, -torch.sin(th)], 1)
        down = torch.tensor([0.0, 1.0, 0.0], dtype=F64, device=dev).expand(n_kf, 3)
        poses = _pose(torch.stack([torch.linalg.cross(down, fwd), down, fwd], 2), centre)
        while have < n_lm:
            m = (n_lm - have) + (n_lm - have) // 4 + 64
            p = rand.unit(m) * rand.u(12, 15, m, 1)
            v = _views(p, poses, K, E, size)
            q = min(1.0, 15.0 * m / max(1, int(v.sum())))   # about 15 observations per landmark
            v = v & (rand.u(0, 1, *v.shape) < q)
            ok = torch.nonzero(v.any(2).sum(1) >= 2)[: n_lm - have, 0]
            pts.append(p[ok])
            chosen.append(v[ok])
            have += ok.numel()
    j, i, c = torch.nonzero(torch.cat(chosen), as_tuple=True)
    return poses, torch.cat(pts), i, j, c


def _perturb(rand, poses, fixed, rot, trans):
    n = poses.shape[0]
    R = _rot(rot * rand.unit(n))
    out = R @ poses
    out[:, :, 3] += trans * rand.unit(n)
    return torch.where(fixed[:, None, None], poses, out)


def _sizes(case):
    """Keyframes and landmarks of each window: spread over the case's ranges, the same for every seed."""
    out = []
    for w in range(case["windows"]):
        a, b = (0.5 + 0.6180339887 * w) % 1.0, (0.5 + 0.7548776662 * w) % 1.0
        out.append((case["kf_lo"] + int(a * (case["kf_hi"] - case["kf_lo"] + 1)),
                    case["lm_lo"] + int(b * (case["lm_hi"] - case["lm_lo"] + 1))))
    return out


def _windows_data(case, seed):
    """Per window: everything a solve needs, on the GPU."""
    rand = _Rand(seed)
    out = []
    K, E, size = _rig(case["rig"], rand)
    for n_kf, n_lm in _sizes(case):
        poses, pts, i, j, c = _scene(rand, case["rig"], n_kf, n_lm, case["track"], K, E, size)
        mism = 0.02 if case["rig"] == "stereo" else 0.0
        uv = _pixels(rand, pts, poses, K, E, i, j, c, 0.7 if mism else 0.5, mism)
        perm = torch.argsort(rand.u(0, 1, i.numel()))
        i, j, c, uv = i[perm], j[perm], c[perm], uv[perm]
        fixed = torch.zeros(n_kf, dtype=torch.bool, device=rand.dev)
        fixed[: 2 if case["rig"] == "mono" else 1] = True
        start = 0.0 if case["op"] == "adjoint" else 1.0   # the adjoint's windows are at their solution
        out.append(dict(
            K=K, E=E, i=i, j=j, c=c, uv=uv, w=rand.u(0.5, 1.5, i.numel()) if case["weighted"] else None, fixed=fixed,
            poses_gt=poses, poses=_perturb(rand, poses, fixed, 0.05 * start, 0.05 * start),
            points=pts + start * 0.1 * rand.n(*pts.shape), target=_perturb(rand, poses, fixed, 0.01, 0.02)))
    return out


def _settings(case):
    return ba.Settings(max_iters=case["iters"], precision=ba.BA_MIXED if case.get("precision") == "mixed" else ba.BA_FP64,
                       lambda_init=LAM0, huber_delta=DELTA, min_depth=MIN_DEPTH)


def _cat(ws, key):
    return None if ws[0][key] is None else torch.cat([w[key] for w in ws]).contiguous()


def _plan(ws, batched):
    wins = []
    for w in ws:
        h = {k: w[k].cpu().numpy() for k in ("i", "j", "c", "fixed", "K", "E")}
        wins.append(ba.Window(w["poses"].shape[0], w["points"].shape[0], h["i"], h["j"], h["K"], obs_cam=h["c"],
                              pose_fixed=h["fixed"].astype(np.uint8), extrinsics=h["E"], host_only=batched))
    return ba.Batch(wins) if batched else wins[0]


def _bytes(n, m):
    return torch.zeros(ba.REPORT_DTYPE.itemsize * n * m, dtype=torch.uint8, device="cuda")


def _prepare_window(case, seed):
    ws = _windows_data(case, seed)
    s = _settings(case)
    plan = _plan(ws, case["windows"] > 1)
    st = dict(case=case, s=s, plan=plan, poses=_cat(ws, "poses"), points=_cat(ws, "points"), uv=_cat(ws, "uv"),
              w=_cat(ws, "w"), target=_cat(ws, "target"), rep=_bytes(len(ws), 1),
              ws=torch.empty(plan.workspace_size(s), dtype=torch.uint8, device="cuda"))
    if case["op"] == "adjoint":
        st["cot"] = 2 * (st["poses"] - st["target"])   # of the squared pose error
        st["cot_pts"] = torch.zeros_like(st["points"])
        st["guv"], st["gw"] = torch.empty_like(st["uv"]), torch.empty(st["uv"].shape[0], dtype=F64, device="cuda")
    if case["op"] == "train":
        st["uv"].requires_grad_(True)
        if st["w"] is not None:
            st["w"].requires_grad_(True)
    return st


def _prepare_pnp(case, seed):
    d = _pnp_data(case, seed)
    d["rig"] = ba.Rig(d["K"].cpu().numpy(), d["E"].cpu().numpy())
    d.update(case=case, s=_settings(case), rep=_bytes(case["frames"], 1))
    for k in ("begin", "j", "c"):
        d[k] = d[k].to(torch.int32).contiguous()
    return d


def _pnp_data(case, seed):
    rand = _Rand(seed)
    K, E, size = _rig(case["rig"], rand)
    F, n = case["frames"], case["lm"]
    per = torch.full((F,), n, device=rand.dev)
    if case["uneven"]:
        per = rand.ints(max(20, n // 2), n + 1, F)
    fr = torch.repeat_interleave(torch.arange(F, device=rand.dev), per)
    ang = torch.zeros(F, 3, dtype=F64, device=rand.dev)
    ang[:, 1] = rand.u(-math.pi, math.pi, F)
    R = _rot(ang) @ _rot(0.1 * rand.u(0, 1, F, 1) * rand.unit(F))
    centre = rand.u(-50, 50, F, 3) * torch.tensor([1.0, 0.1, 1.0], dtype=F64, device=rand.dev)
    poses = _pose(R, centre)
    m = fr.numel()
    if case["rig"] == "stereo":
        d = torch.exp(rand.u(math.log(3.0), math.log(60.0), m))
        off = K[0, 0] * 0.54 / d   # seen by both cameras: right of the disparity
        u = off + rand.u(0, 1, m) * (size[0] - off)
        v = rand.u(0, size[1], m)
        xb = torch.stack([(u - K[0, 2]) / K[0, 0] * d, (v - K[0, 3]) / K[0, 1] * d, d], 1)
        lm = torch.arange(m, device=rand.dev).repeat_interleave(2)
        cam = torch.arange(2, device=rand.dev).repeat(m)
    else:
        xb = rand.unit(m) * rand.u(12, 15, m, 1)
        vis = _views(xb, torch.eye(4, dtype=F64, device=rand.dev)[None, :3], K, E, size)[:, 0]
        vis[torch.arange(m, device=rand.dev), (E[:, 2, :3] @ xb.T + E[:, 2, 3:]).argmax(0)] = True
        lm, cam = torch.nonzero(vis, as_tuple=True)
    pts = (R[fr] @ xb[..., None])[..., 0] + centre[fr]
    of = fr[lm]
    xc = (E[cam][:, :, :3] @ xb[lm][..., None])[..., 0] + E[cam][:, :, 3]
    sg = torch.where(rand.u(0, 1, lm.numel(), 1) < 0.02, 8 * 0.7, 0.7)
    uv = _project(K[cam], xc) + sg * rand.n(lm.numel(), 2)
    perm = torch.argsort(of.to(F64) + rand.u(0, 0.9, of.numel()))   # any order within a frame
    begin = torch.zeros(F + 1, dtype=torch.long, device=rand.dev)
    begin[1:] = torch.cumsum(torch.bincount(of, minlength=F), 0)
    M = None
    gt = poses
    if case["map_frame"]:   # the loop-closure pose against a neighbouring map
        M = _pose(_rot(rand.u(0, 0.5, F, 1) * rand.unit(F)), rand.u(-5, 5, F, 3))
        Ri = M[:, :, :3].transpose(1, 2)
        gt = torch.cat([poses[:, :, :3] @ Ri, poses[:, :, 3:] - poses[:, :, :3] @ (Ri @ M[:, :, 3:])], 2)
    init = _perturb(rand, gt, torch.zeros(F, dtype=torch.bool, device=rand.dev), 0.02, 0.05)
    return dict(K=K, E=E, begin=begin, frame=of[perm], j=lm[perm], c=cam[perm], uv=uv[perm].contiguous(),
                points=pts.contiguous(), poses=init.contiguous(), M=None if M is None else M.contiguous(),
                w=rand.u(0.5, 1.5, lm.numel()) if case["weighted"] else None)


def _tri_data(case, seed):
    rand = _Rand(seed)
    K, E, size = _rig(case["rig"], rand)
    out, pb, lb = [], 0, 0
    for w in range(case["windows"]):
        poses, pts, i, j, c = _scene(rand, case["rig"], case["kf"], case["lm"], "subset", K, E, size)
        uv = _pixels(rand, pts, poses, K, E, i, j, c, 0.5, 0.0)
        out.append((poses, i + pb, j + lb, c, uv))
        pb, lb = pb + poses.shape[0], lb + pts.shape[0]
    poses, i, j, c, uv = (torch.cat(x) for x in zip(*out))   # landmark-major already
    begin = torch.zeros(lb + 1, dtype=torch.long, device=rand.dev)
    begin[1:] = torch.cumsum(torch.bincount(j, minlength=lb), 0)
    return dict(K=K, E=E, poses=poses.contiguous(), i=i, j=j, c=c, uv=uv.contiguous(), begin=begin, n=lb)


def _prepare_tri(case, seed):
    d = _tri_data(case, seed)
    d["rig"] = ba.Rig(d["K"].cpu().numpy(), d["E"].cpu().numpy())
    d.update(case=case, s=_settings(case), rep=_bytes(d["n"], 1), points=torch.empty(d["n"], 3, dtype=F64, device="cuda"))
    for k in ("begin", "i", "c"):
        d[k] = d[k].to(torch.int32).contiguous()
    return d


def _np_rot(phi):
    return _rot(torch.as_tensor(phi, dtype=F64)).numpy()


def _np_mul(A, B):
    return np.concatenate([A[..., :3] @ B[..., :3], A[..., :3] @ B[..., 3:] + A[..., 3:]], -1)


def _pgo_data(case, seed):
    """A helix of several laps: odometry and loop-closure edges, poses world-from-base."""
    rng = np.random.default_rng(seed)
    per, n = case["per_lap"], case["laps"] * case["per_lap"]
    a = 2 * math.pi * np.arange(n) / per
    z = np.zeros(n)
    fwd = np.stack([-np.sin(a), z, np.cos(a)], 1)
    up = np.stack([z, z + 1, z], 1)
    radius = 10.0 * per / 500.0
    gt = np.stack([fwd, up, np.cross(fwd, up),
                   np.stack([radius * np.cos(a), 0.5 * np.arange(n) / per, radius * np.sin(a)], 1)], 2)
    k = np.repeat(np.arange(per, n), 3)
    j = k - per + np.tile([-1, 0, 1], n - per)
    ok = (j >= 0) & (j < k - 1) & (rng.random(k.size) < 0.5)
    ei = np.concatenate([np.arange(n - 1), j[ok]])
    ej = np.concatenate([np.arange(1, n), k[ok]])
    Ri = gt[ei, :, :3].transpose(0, 2, 1)
    D = np.concatenate([Ri @ gt[ej, :, :3], Ri @ (gt[ej, :, 3:] - gt[ei, :, 3:])], 2)
    noise = np.concatenate([_np_rot(rng.normal(0, 0.002, (ei.size, 3))), rng.normal(0, 0.01, (ei.size, 3, 1))], 2)
    D = _np_mul(noise, D)
    init = [gt[0]]
    for e in range(n - 1):
        init.append(_np_mul(init[-1], D[e]))
    w = rng.uniform(0.5, 1.5, ei.size) if case["weighted"] else None
    return dict(n=n, ei=ei.astype(np.int32), ej=ej.astype(np.int32), D=D, init=np.stack(init), w=w)


def _prepare_pgo(case, seed):
    d = _pgo_data(case, seed)
    g = ba.Graph(d["n"], d["ei"], d["ej"])
    dev = lambda x: None if x is None else torch.tensor(x, dtype=F64, device="cuda").contiguous()  # noqa: E731
    return dict(case=case, s=_settings(case), graph=g, poses=dev(d["init"]), deltas=dev(d["D"]), w=dev(d["w"]),
                rep=_bytes(1, 1), ws=torch.empty(g.workspace_size(), dtype=torch.uint8, device="cuda"))


def _vi_data(case, seed):
    """A mono camera on a base moving forward with its IMU; keyframes every `samples` samples."""
    rng = np.random.default_rng(seed + 17)
    n_kf, n_s, dt, g = case["kf"], case["samples"], 1.0 / IMU_RATE, np.array([0.0, 9.81, 0.0])
    bias_a, bias_g, ph = rng.normal(0, 0.05, 3), rng.normal(0, 0.01, 3), rng.uniform(0, 2 * math.pi, 6)
    R, p, v = np.eye(3), np.zeros(3), np.array([0.1, 0.0, 1.0])
    n = n_s * (n_kf - 1)
    t = np.arange(n)[:, None] * dt
    w = np.array([0.15, 0.3, 0.1]) * np.sin(np.array([0.9, 0.6, 1.1]) * t + ph[:3])
    aw = np.array([0.4, 0.2, 0.3]) * np.sin(np.array([0.8, 0.7, 0.5]) * t + ph[3:])
    dR = _np_rot(w * dt)
    poses, vels, acc = [], [], np.empty((n, 3))
    for q in range(n + 1):
        if q % n_s == 0:
            poses.append(np.concatenate([R.T, -(R.T @ p)[:, None]], 1))
            vels.append(v)
        if q == n:
            break
        acc[q] = R.T @ (aw[q] - g)
        p = p + v * dt + 0.5 * aw[q] * dt * dt
        v = v + aw[q] * dt
        R = R @ dR[q]
    gyro = w + bias_g + rng.normal(0, IMU_NOISE[0] / math.sqrt(dt), (n, 3))
    accel = acc + bias_a + rng.normal(0, IMU_NOISE[1] / math.sqrt(dt), (n, 3))
    rand = _Rand(seed)
    K, E, size = _rig("mono", rand)
    P = torch.tensor(np.stack(poses), dtype=F64, device=rand.dev)
    z_end = float(-(poses[-1][:, :3].T @ poses[-1][:, 3])[2])
    lo, have, pts, chosen = min(3, n_kf), 0, [], []
    while have < case["lm"]:
        m = 8 * (case["lm"] - have) + 64
        q = torch.stack([rand.u(-5, 5, m), rand.u(-3, 3, m), rand.u(z_end + 3, z_end + 20, m)], 1)
        vis = _views(q, P, K, E, size)[:, :, 0]
        nv = vis.sum(1)
        key = torch.where(vis, rand.u(0, 1, m, n_kf), torch.full((), 2.0, dtype=F64, device=rand.dev))
        cnt = lo + (rand.u(0, 1, m) * (nv.clamp_max(6) - lo + 1)).long()
        vis = vis & (key.argsort(1).argsort(1) < cnt[:, None])
        ok = torch.nonzero(nv >= lo)[: case["lm"] - have, 0]
        pts.append(q[ok])
        chosen.append(vis[ok])
        have += ok.numel()
    pts = torch.cat(pts)
    j, i = torch.nonzero(torch.cat(chosen), as_tuple=True)
    c = torch.zeros_like(i)
    uv = _pixels(rand, pts, P, K, E, i, j, c, 0.5, 0.0)
    fixed = torch.zeros(n_kf, dtype=torch.bool, device=rand.dev)
    fixed[0] = True
    states = torch.zeros(n_kf, 9, dtype=F64, device=rand.dev)
    states[:, :3] = torch.tensor(np.stack(vels), dtype=F64, device=rand.dev) + 0.05 * rand.n(n_kf, 3)
    win = dict(K=K, E=E, i=i, j=j, c=c, uv=uv, w=None, fixed=fixed, poses=_perturb(rand, P, fixed, 0.03, 0.03),
               points=pts + 0.1 * rand.n(*pts.shape))
    return win, states, gyro, accel, dt, g


def _prepare_vi(case, seed):
    w, states, gyro, accel, dt, g = _vi_data(case, seed)
    s = _settings(case)
    plan = _plan([w], False)
    dev = lambda x: torch.tensor(x, dtype=F64, device="cuda")  # noqa: E731
    n = case["kf"] - 1
    return dict(case=case, s=s, plan=plan, poses=w["poses"].contiguous(), points=w["points"].contiguous(),
                uv=w["uv"].contiguous(), states=states, gyro=dev(gyro), accel=dev(accel), dt=dt, g=g,
                begin=torch.arange(n + 1, device="cuda", dtype=torch.int32) * case["samples"],
                bias=torch.zeros(n, 6, dtype=F64, device="cuda"), rep=_bytes(1, 1),
                pre=torch.zeros(n, ba.VI_PREINT_DOUBLES, dtype=F64, device="cuda"),
                ws=torch.empty(ba.vi_workspace_size(plan, s), dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    return dict(window=_prepare_window, pnp=_prepare_pnp, tri=_prepare_tri, pgo=_prepare_pgo,
                vi=_prepare_vi)[case["kind"]](case, seed)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _outcome(rep):
    """Costs (start, end) and status of each report, as the caller reads them.  (How many
    of the last attempts are accepted is decided by the costs' last bits, so it is not kept.)"""
    return rep.view(F64).view(-1, 6)[:, :2], rep.view(torch.int32).view(-1, 12)[:, 10]


def run(st):
    kind = st["case"]["kind"]
    if kind == "window" and st["case"]["op"] == "train":
        uv, w = st["uv"], st["w"]
        P, L = ba.BASolve.apply(st["poses"], st["points"], uv, w, st["plan"], st["s"])
        loss = ((P - st["target"]) ** 2).sum()
        wrt = [uv] if w is None else [uv, w]
        return {"poses": P.detach(), "points": L.detach(), "loss": loss.detach(), "grads": list(torch.autograd.grad(loss, wrt))}
    if kind == "window" and st["case"]["op"] == "adjoint":
        ba.adjoint(st["plan"], st["s"], st["poses"], st["points"], st["uv"], st["w"], st["cot"], st["cot_pts"],
                   st["guv"], st["gw"], workspace=st["ws"], reports=st["rep"])
        return {"uv": st["guv"], "w": st["gw"]}
    if kind == "tri":
        ba.triangulate(st["rig"], st["s"], st["begin"], st["poses"], st["i"], st["uv"], st["points"], obs_cam=st["c"],
                       reports=st["rep"])
        cost, status = _outcome(st["rep"])
        return {"points": st["points"], "cost": cost, "status": status}
    P = st["poses"].clone()   # the solves work in place
    if kind == "pnp":
        ba.pnp_solve(st["rig"], st["s"], st["begin"], P, st["points"], st["j"], st["uv"], obs_cam=st["c"],
                     obs_w=st["w"], frame_transform=st["M"], reports=st["rep"])
        cost, status = _outcome(st["rep"])
        return {"poses": P, "cost": cost, "status": status}
    if kind == "pgo":
        ba.pgo_solve(st["graph"], st["s"], P, st["deltas"], st["ws"], edge_w=st["w"], report=st["rep"])
        cost, status = _outcome(st["rep"])
        return {"poses": P, "cost": cost, "status": status}
    L = st["points"].clone()
    if kind == "vi":
        x = st["states"].clone()
        pre = ba.vi_preintegrate(st["begin"], st["gyro"], st["accel"], st["dt"], st["bias"], IMU_NOISE, out=st["pre"])
        ba.vi_solve(st["plan"], st["s"], pre, st["g"], P, L, x, st["uv"], workspace=st["ws"], report=st["rep"])
        cost, status = _outcome(st["rep"])
        return {"poses": P, "points": L, "states": x, "preint": pre, "cost": cost, "status": status}
    if st["case"]["windows"] > 1:
        ba.solve_batched(st["plan"], st["s"], P, L, st["uv"], st["w"], workspace=st["ws"], reports=st["rep"])
    else:
        ba.solve(st["plan"], st["s"], P, L, st["uv"], st["w"], workspace=st["ws"], report=st["rep"])
    cost, status = _outcome(st["rep"])
    return {"poses": P, "points": L, "cost": cost, "status": status}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

# per observation and linearisation: transform 36, projection and Huber 20,
# Jacobians 60, block products 230; its candidate's cost: 60
_LIN, _COST = 350.0, 60.0


def _mean_track(rig, kf, track):
    """Observations per landmark and distinct keyframes per landmark (means of the generator)."""
    if rig == "stereo":
        n = min(6.0, 0.6 * kf + 0.8)
        return 2 * n, n
    if rig == "rig":
        return 15.0, min(7.0, 0.7 * kf)
    n = max(3, kf - 2) - 0.5 if track == "long" else min(5.5, 0.5 * (2 + 0.9 * kf))
    return n, n


def work(case):
    if case["kind"] == "window":
        by = fl = 0.0
        att = 1 if case["op"] == "adjoint" else case["iters"] + (1 if case["op"] == "train" else 0)
        for kf, lm in _sizes(case):
            o, p = _mean_track(case["rig"], kf, case["track"])
            n = 6.0 * (kf - 1)
            by += lm * o * (16 + 12 + (8 if case["weighted"] else 0)) + 48 * lm + 192 * kf
            if case["op"] != "solve":
                by += lm * o * 24
            fl += att * (lm * (o * (_LIN + _COST) + 150 * p + 120 + 234 * p * (p - 1) / 2) + n ** 3 / 3)
        return {"bytes": by, "flops": fl}
    if case["kind"] == "pnp":
        n = case["frames"] * case["lm"] * (2.0 if case["rig"] == "stereo" else 3.3) * (0.75 if case["uneven"] else 1)
        return {"bytes": n * (16 + 8 + (8 if case["weighted"] else 0)) + case["frames"] * (case["lm"] * 24 + 192 + 48),
                "flops": n * 209.0 * (case["iters"] + 1)}
    if case["kind"] == "tri":
        lm = case["windows"] * case["lm"]
        o, _ = _mean_track(case["rig"], case["kf"], "subset")
        return {"bytes": lm * (o * 24 + 4 + 24 + 48.0), "flops": lm * o * (81 + 95.0 * (case["iters"] + 1))}
    if case["kind"] == "pgo":
        n = case["laps"] * case["per_lap"]
        e = n + 1.5 * (n - case["per_lap"])
        return {"bytes": 192.0 * n + e * 104, "flops": case["iters"] * (2100.0 * e + 6000.0 * n)}
    p = min(4.5, 0.95 * case["kf"])
    n = 6.0 * (case["kf"] - 1)
    return {"bytes": case["lm"] * (48 + p * 24) + case["kf"] * (336 + case["samples"] * 48.0),
            "flops": case["kf"] * case["samples"] * 2500.0 + case["iters"] * (
                case["lm"] * (p * (_LIN + _COST + 150) + 120 + 117 * p * p) + n ** 3 / 3 + case["kf"] * (60000.0 + 200 * n * 9))}


# ---------------------------------------------------------------------------
# the same answers by plain torch in 64 bits
# ---------------------------------------------------------------------------

def _rho(s):
    out = s > DELTA * DELTA
    q = torch.sqrt(torch.where(out, s, torch.ones_like(s)))
    one, zero = torch.ones_like(s), torch.zeros_like(s)
    return (torch.where(out, 2 * DELTA * q - DELTA * DELTA, s), torch.where(out, DELTA / q, one),
            torch.where(out, -0.5 * DELTA / (q * q * q), zero))


def _exp(xi):
    """SE(3) exponential of (rho, phi) (..., 6) as (..., 3, 4)."""
    rho, phi = xi[..., :3], xi[..., 3:]
    t2 = (phi * phi).sum(-1)[..., None, None]
    a, b, c = torch.ones_like(t2), torch.ones_like(t2), torch.ones_like(t2)
    for k in range(14, -1, -1):
        n = 2.0 * k
        a = 1 - t2 / ((n + 2) * (n + 3)) * a
        b = 1 - t2 / ((n + 3) * (n + 4)) * b
        c = 1 - t2 / ((n + 4) * (n + 5)) * c
    K = _skew(phi)
    K2 = K @ K
    eye = torch.eye(3, dtype=xi.dtype, device=xi.device)
    V = eye + 0.5 * b * K + c / 6 * K2
    return torch.cat([eye + a * K + 0.5 * b * K2, V @ rho[..., None]], -1)


def _apply(D, T):
    return torch.cat([D[..., :3] @ T[..., :3], D[..., :3] @ T[..., 3:] + D[..., 3:]], -1)


class _Visual:
    """Residuals of one window and their derivatives."""

    def __init__(self, w):
        self.i, self.j, self.uv = w["i"], w["j"], w["uv"]
        self.K, self.R, self.t = w["K"][w["c"]], w["E"][w["c"]][:, :, :3], w["E"][w["c"]][:, :, 3]
        self.w = torch.ones_like(self.uv[:, 0]) if w["w"] is None else w["w"]
        self.slot = torch.cumsum((~w["fixed"]).long(), 0) - 1
        self.slot[w["fixed"]] = -1
        self.free = torch.nonzero(~w["fixed"])[:, 0]

    def residual(self, P, L):
        T = P[self.i]
        xb = (T[:, :, :3] @ L[self.j][..., None])[..., 0] + T[:, :, 3]
        xc = (self.R @ xb[..., None])[..., 0] + self.t
        return xb, xc, _project(self.K, xc) - self.uv

    def cost(self, P, L):
        _, xc, r = self.residual(P, L)
        return 0.5 * (self.w * _rho((r * r).sum(1))[0]).sum(), bool((xc[:, 2] > MIN_DEPTH).all())

    def jacobians(self, P, L):
        xb, xc, r = self.residual(P, L)
        iz = 1 / xc[:, 2]
        z = torch.zeros_like(iz)
        A = torch.stack([torch.stack([self.K[:, 0] * iz, z, -self.K[:, 0] * xc[:, 0] * iz * iz], 1),
                         torch.stack([z, self.K[:, 1] * iz, -self.K[:, 1] * xc[:, 1] * iz * iz], 1)], 1)
        A = A @ self.R
        Jp = torch.cat([A, -(A @ _skew(xb))], 2)
        return Jp, A @ P[self.i][:, :, :3], r


def _ldl_solve(V, B):
    """V^-1 B for symmetric 3x3 V (m, 3, 3), B (m, 3, n)."""
    d0 = V[:, 0, 0]
    l1, l2 = V[:, 0, 1] / d0, V[:, 0, 2] / d0
    d1 = V[:, 1, 1] - l1 * l1 * d0
    l3 = (V[:, 1, 2] - l2 * l1 * d0) / d1
    d2 = V[:, 2, 2] - l2 * l2 * d0 - l3 * l3 * d1
    l1, l2, l3 = l1[:, None], l2[:, None], l3[:, None]
    y0 = B[:, 0]
    y1 = B[:, 1] - l1 * y0
    y2 = B[:, 2] - l2 * y0 - l3 * y1
    x2 = y2 / d2[:, None]
    x1 = y1 / d1[:, None] - l3 * x2
    x0 = y0 / d0[:, None] - l1 * x1 - l2 * x2
    return torch.stack([x0, x1, x2], 1), bool(((d0 > 0) & (d1 > 0) & (d2 > 0)).all())


def _blocks(vis, HUU, HUV, HVV, gU, gV, M):
    """Sums of per-observation blocks per pose, pair and landmark."""
    nf, dev = vis.free.numel(), HVV.device
    s = vis.slot[vis.i]
    f = s >= 0
    U = torch.zeros(nf, 6, 6, dtype=F64, device=dev).index_add_(0, s[f], HUU[f])
    gp = torch.zeros(nf, 6, dtype=F64, device=dev).index_add_(0, s[f], gU[f])
    V = torch.zeros(M, 3, 3, dtype=F64, device=dev).index_add_(0, vis.j, HVV)
    gl = torch.zeros(M, 3, dtype=F64, device=dev).index_add_(0, vis.j, gV)
    W = torch.zeros(M * nf, 3, 6, dtype=F64, device=dev).index_add_(0, vis.j[f] * nf + s[f], HUV[f].transpose(1, 2))
    return U, gp, V, gl, W.view(M, nf, 3, 6).permute(0, 2, 1, 3).reshape(M, 3, nf * 6)


def _schur_solve(U, V, W, b, c):
    """[[U, W^T], [W, V]] (x, y) = (b, c) with the landmarks eliminated; None when not positive definite."""
    nf, M = U.shape[0], V.shape[0]
    Y, ok = _ldl_solve(V, torch.cat([W, c[..., None]], 2))
    S = torch.block_diag(*U) if nf else torch.zeros(0, 0, dtype=F64, device=V.device)
    red = W.reshape(3 * M, 6 * nf).T @ Y.reshape(3 * M, 6 * nf + 1)
    S = (S - red[:, :-1]).cpu().numpy()
    rhs = (b.reshape(-1) - red[:, -1]).cpu().numpy()
    try:
        if not ok:
            return None
        np.linalg.cholesky(S)
        x = torch.from_numpy(np.linalg.solve(S, rhs)).to(V.device)
    except np.linalg.LinAlgError:
        return None
    return x.view(nf, 6), Y[:, :, -1] - (Y[:, :, :-1] @ x)


def _exact_solve(w, iters):
    vis, P, L, lam = _Visual(w), w["poses"], w["points"], LAM0
    M = L.shape[0]
    F = F0 = vis.cost(P, L)[0]
    lin = None
    for _ in range(iters):
        if lin is None:
            Jp, Jl, r = vis.jacobians(P, L)
            w1 = (vis.w * _rho((r * r).sum(1))[1])[:, None, None]
            wp, wl, rc = (w1 * Jp).transpose(1, 2), (w1 * Jl).transpose(1, 2), r[..., None]
            lin = _blocks(vis, wp @ Jp, wp @ Jl, wl @ Jl, (wp @ rc)[..., 0], (wl @ rc)[..., 0], M)
        U, gp, V, gl, W = lin
        dU, dV = torch.diagonal(U, dim1=1, dim2=2), torch.diagonal(V, dim1=1, dim2=2)
        sol = _schur_solve(U + torch.diag_embed(lam * dU.clamp_min(1e-9)), V + torch.diag_embed(lam * dV.clamp_min(1e-9)),
                           W, -gp, -gl)
        accept = False
        if sol is not None:
            Pc = P.clone()
            Pc[vis.free] = _apply(_exp(sol[0]), P[vis.free])
            Lc = L + sol[1]
            Fc, deep = vis.cost(Pc, Lc)
            accept = deep and bool(Fc < F)
        if accept:
            P, L, F, lin = Pc, Lc, Fc, None
        lam = max(lam / 10, 1e-10) if accept else min(lam * 10, 1e10)
    return P, L, torch.stack([F0, F])


def _exact_adjoint(w, P, L, G, GL):
    """Gradients to the pixels and weights at the state (P, L), the exact Hessian by automatic differentiation."""
    vis = _Visual(w)

    def f(z, T, p, K, R, t, uv, wo):
        xb = T[:, :3] @ (p + z[6:]) + T[:, 3]
        k = torch.linalg.cross(z[3:6], xb)   # second order of Exp(z) x
        xb = xb + k + 0.5 * torch.linalg.cross(z[3:6], k) + z[:3] + 0.5 * torch.linalg.cross(z[3:6], z[:3])
        r = _project(K, R @ xb + t) - uv
        return 0.5 * wo * _rho((r * r).sum())[0]

    hess = torch.func.vmap(torch.func.hessian(f), in_dims=(None, 0, 0, 0, 0, 0, 0, 0))
    z = torch.zeros(9, dtype=F64, device=L.device)
    H = torch.cat([hess(z, P[vis.i[s]], L[vis.j[s]], vis.K[s], vis.R[s], vis.t[s], vis.uv[s], vis.w[s])
                   for s in torch.split(torch.arange(vis.i.numel(), device=L.device), 60000)])
    Jp, Jl, r = vis.jacobians(P, L)
    zero = torch.zeros_like(H[:, 0])
    U, _, V, _, W = _blocks(vis, H[:, :6, :6], H[:, :6, 6:], H[:, 6:, 6:], zero[:, :6], zero[:, 6:], L.shape[0])
    Tm, Gm = P[vis.free], G[vis.free]
    Mx = Gm[:, :, :3] @ Tm[:, :, :3].transpose(1, 2) + Gm[:, :, 3:] @ Tm[:, :, 3:].transpose(1, 2)
    c = torch.stack([Gm[:, 0, 3], Gm[:, 1, 3], Gm[:, 2, 3], Mx[:, 2, 1] - Mx[:, 1, 2], Mx[:, 0, 2] - Mx[:, 2, 0],
                     Mx[:, 1, 0] - Mx[:, 0, 1]], 1)
    sol = _schur_solve(U, V, W, c, GL)
    if sol is None:
        return None
    a = torch.zeros(P.shape[0], 6, dtype=F64, device=L.device)
    a[vis.free] = sol[0]
    Ja = (Jp @ a[vis.i][..., None] + Jl @ sol[1][vis.j][..., None])[..., 0]
    _, d1, d2 = _rho((r * r).sum(1))
    rJ = (r * Ja).sum(1)
    return vis.w[:, None] * (d1[:, None] * Ja + 2 * (d2 * rJ)[:, None] * r), -d1 * rJ


def _exact_window(case, seed):
    ws = _windows_data(case, seed)
    if case["op"] == "adjoint":
        g = [_exact_adjoint(w, w["poses"], w["points"], 2 * (w["poses"] - w["target"]), torch.zeros_like(w["points"]))
             for w in ws]
        return None if any(x is None for x in g) else {"uv": torch.cat([x[0] for x in g]), "w": torch.cat([x[1] for x in g])}
    sol = [_exact_solve(w, case["iters"]) for w in ws]
    P, L = torch.cat([x[0] for x in sol]), torch.cat([x[1] for x in sol])
    if case["op"] == "solve":
        return {"poses": P, "points": L, "cost": torch.stack([x[2] for x in sol]), "status": None}
    g = [_exact_adjoint(w, x[0], x[1], 2 * (x[0] - w["target"]), torch.zeros_like(x[1])) for w, x in zip(ws, sol)]
    if any(x is None for x in g):
        return None
    grads = [torch.cat([x[0] for x in g])] + ([torch.cat([x[1] for x in g])] if case["weighted"] else [])
    return {"poses": P, "points": L, "loss": ((P - _cat(ws, "target")) ** 2).sum(), "grads": grads}


def _chol_solve6(H, b):
    """Batched 6x6 solve by Cholesky; NaN rows where a pivot is not positive."""
    n = H.shape[-1]
    R = [[None] * n for _ in range(n)]
    y, x = [None] * n, [None] * n
    for a in range(n):
        d = torch.sqrt(H[:, a, a] - sum((R[m][a] ** 2 for m in range(a)), torch.zeros_like(H[:, 0, 0])))
        R[a][a] = d
        for c in range(a + 1, n):
            R[a][c] = (H[:, a, c] - sum((R[m][a] * R[m][c] for m in range(a)), torch.zeros_like(d))) / d
        y[a] = (b[:, a] - sum((R[m][a] * y[m] for m in range(a)), torch.zeros_like(d))) / d
    for a in range(n - 1, -1, -1):
        x[a] = (y[a] - sum((R[a][m] * x[m] for m in range(a + 1, n)), torch.zeros_like(y[a]))) / R[a][a]
    return torch.stack(x, 1)


def _sum_by(index, n, x):
    return torch.zeros(n, *x.shape[1:], dtype=F64, device=x.device).index_add_(0, index, x)


def _exact_many(iters, n, state, linearise, step):
    """LM on n independent small problems: state (n, ...), linearise -> (cost, bad, H, g), step(state, d)."""
    F, bad, H, g = linearise(state)
    F0, start_bad = F, bad
    lam = torch.full((n,), LAM0, dtype=F64, device=F.device)
    for _ in range(iters):
        dg = torch.diagonal(H, dim1=1, dim2=2)
        d = _chol_solve6(H + torch.diag_embed(lam[:, None] * dg.clamp_min(1e-9)), -g)
        solved = torch.isfinite(d).all(1)
        cand = step(state, torch.where(solved[:, None], d, torch.zeros_like(d)))
        Fc, badc, Hc, gc = linearise(cand)
        acc = solved & ~badc & (Fc < F)
        pick = lambda a, b: torch.where(acc.view(-1, *[1] * (a.dim() - 1)), a, b)  # noqa: E731
        state, F, H, g = pick(cand, state), pick(Fc, F), pick(Hc, H), pick(gc, g)
        lam = torch.where(acc, (lam / 10).clamp_min(1e-10), (lam * 10).clamp_max(1e10))
    return state, torch.stack([F0, F], 1), start_bad


def _exact_pnp(case, seed):
    d = _pnp_data(case, seed)
    n = case["frames"]
    w = torch.ones_like(d["uv"][:, 0]) if d["w"] is None else d["w"]
    K, R, t, f = d["K"][d["c"]], d["E"][d["c"]][:, :, :3], d["E"][d["c"]][:, :, 3], d["frame"]
    p = d["points"][d["j"]]
    if d["M"] is not None:
        p = (d["M"][f][:, :, :3] @ p[..., None])[..., 0] + d["M"][f][:, :, 3]

    def lin(T):
        xb = (T[f][:, :, :3] @ p[..., None])[..., 0] + T[f][:, :, 3]
        xc = (R @ xb[..., None])[..., 0] + t
        r = _project(K, xc) - d["uv"]
        rho, d1, _ = _rho((r * r).sum(1))
        iz = 1 / xc[:, 2]
        a0 = (K[:, 0] * iz)[:, None] * (R[:, 0] - (xc[:, 0] * iz)[:, None] * R[:, 2])
        a1 = (K[:, 1] * iz)[:, None] * (R[:, 1] - (xc[:, 1] * iz)[:, None] * R[:, 2])
        A = torch.stack([a0, a1], 1)
        J = torch.cat([A, torch.linalg.cross(xb[:, None].expand_as(A), A)], 2)
        wJ = (w * d1)[:, None, None] * J
        H = _sum_by(f, n, (wJ.transpose(1, 2) @ J))
        g = _sum_by(f, n, (wJ.transpose(1, 2) @ r[..., None])[..., 0])
        return 0.5 * _sum_by(f, n, w * rho), _sum_by(f, n, (~(xc[:, 2] > MIN_DEPTH)).to(F64)) > 0, H, g

    T, cost, _ = _exact_many(case["iters"], n, d["poses"], lin, lambda T, x: _apply(_exp(x), T))
    return {"poses": T, "cost": cost, "status": None}


def _exact_tri(case, seed):
    d = _tri_data(case, seed)
    n, j = d["n"], d["j"]
    K, E, T = d["K"][d["c"]], d["E"][d["c"]], d["poses"][d["i"]]
    C = _apply(E, T)
    R, t = C[:, :, :3].contiguous(), C[:, :, 3].contiguous()
    v = torch.stack([(d["uv"][:, 0] - K[:, 2]) / K[:, 0], (d["uv"][:, 1] - K[:, 3]) / K[:, 1], torch.ones_like(K[:, 0])], 1)
    ray = (R.transpose(1, 2) @ v[..., None])[..., 0]
    ray = ray / ray.norm(dim=1, keepdim=True)
    ctr = -(R.transpose(1, 2) @ t[..., None])[..., 0]
    Pj = torch.eye(3, dtype=F64, device=ray.device) - ray[:, :, None] * ray[:, None]
    p0, _ = _ldl_solve(_sum_by(j, n, Pj), _sum_by(j, n, (Pj @ ctr[..., None])[..., 0])[..., None])

    def lin(p):
        xc = (R @ p[j][..., None])[..., 0] + t
        r = _project(K, xc) - d["uv"]
        rho, d1, _ = _rho((r * r).sum(1))
        iz = 1 / xc[:, 2]
        J = torch.stack([(K[:, 0] * iz)[:, None] * (R[:, 0] - (xc[:, 0] * iz)[:, None] * R[:, 2]),
                         (K[:, 1] * iz)[:, None] * (R[:, 1] - (xc[:, 1] * iz)[:, None] * R[:, 2])], 1)
        wJ = d1[:, None, None] * J
        H = _sum_by(j, n, wJ.transpose(1, 2) @ J)
        g = _sum_by(j, n, (wJ.transpose(1, 2) @ r[..., None])[..., 0])
        return 0.5 * _sum_by(j, n, rho), _sum_by(j, n, (~(xc[:, 2] > MIN_DEPTH)).to(F64)) > 0, H, g

    p, cost, behind = _exact_many(case["iters"], n, p0[:, :, 0], lin, lambda p, x: p + x)
    p = torch.where(behind[:, None], p0[:, :, 0], p)   # a start behind a camera is not refined
    return {"points": p, "cost": torch.where(behind[:, None], torch.full_like(cost, math.nan), cost), "status": None}


def _log_rot(R):
    v = 0.5 * torch.stack([R[2, 1] - R[1, 2], R[0, 2] - R[2, 0], R[1, 0] - R[0, 1]])
    s2 = (v * v).sum()
    c = 0.5 * (R[0, 0] + R[1, 1] + R[2, 2] - 1)
    small = s2 < 1e-10
    s = torch.sqrt(torch.where(small, torch.ones_like(s2), s2))
    return torch.where(small, 1 + s2 / 6 + 3 * s2 * s2 / 40, torch.atan2(s, c) / s) * v


def _log_se3(T):
    phi = _log_rot(T[:, :3])
    t2 = (phi * phi).sum()
    small = t2 < 1e-4
    th = torch.sqrt(torch.where(small, torch.ones_like(t2), t2))
    d = torch.where(small, 1 / 12 + t2 * (1 / 720 + t2 / 30240), 1 / (th * th) - torch.cos(0.5 * th) / (2 * th * torch.sin(0.5 * th)))
    K = _skew(phi)
    Ji = torch.eye(3, dtype=F64, device=T.device) - 0.5 * K + d * (K @ K)
    return torch.cat([Ji @ T[:, 3], phi])


def _exp1(xi):
    """Exp to second order, enough for first derivatives at zero."""
    K = _skew(xi[3:])
    eye = torch.eye(3, dtype=F64, device=xi.device)
    return torch.cat([eye + K + 0.5 * K @ K, ((eye + 0.5 * K) @ xi[:3])[:, None]], 1)


def _exact_pgo(case, seed):
    d = _pgo_data(case, seed)
    dev = torch.device("cuda")
    T, D = (torch.tensor(x, dtype=F64, device=dev) for x in (d["init"], d["D"]))
    ei, ej = (torch.tensor(x, dtype=torch.long, device=dev) for x in (d["ei"], d["ej"]))
    w = torch.ones(ei.numel(), dtype=F64, device=dev) if d["w"] is None else torch.tensor(d["w"], device=dev)
    n = d["n"]

    def inv(A):
        Rt = A[:, :3].T
        return torch.cat([Rt, -(Rt @ A[:, 3:])], 1)

    def res(xi, Ti, Tj, Dij):
        return _log_se3(_apply(inv(Dij), _apply(inv(_apply(_exp1(xi[:6]), Ti)), _apply(_exp1(xi[6:]), Tj))))

    z = torch.zeros(12, dtype=F64, device=dev)
    value = torch.func.vmap(res, in_dims=(None, 0, 0, 0))
    jac = torch.func.vmap(torch.func.jacfwd(res), in_dims=(None, 0, 0, 0))

    def cost(T):
        r = value(z, T[ei], T[ej], D)
        return 0.5 * (w * (r * r).sum(1)).sum()

    lam, F = LAM0, cost(T)
    F0 = F
    idx = torch.cat([6 * ei[:, None] + torch.arange(6, device=dev), 6 * ej[:, None] + torch.arange(6, device=dev)], 1)
    for _ in range(case["iters"]):
        J, r = jac(z, T[ei], T[ej], D), value(z, T[ei], T[ej], D)
        wJ = (w[:, None, None] * J).transpose(1, 2).contiguous()
        H = torch.zeros(6 * n, 6 * n, dtype=F64, device=dev)
        H.index_put_((idx[:, :, None].expand(-1, 12, 12), idx[:, None].expand(-1, 12, 12)), wJ @ J, accumulate=True)
        g = torch.zeros(6 * n, dtype=F64, device=dev).index_add_(0, idx.reshape(-1), (wJ @ r[..., None]).reshape(-1))
        H, g = H[6:, 6:], g[6:]
        H = H + torch.diag(lam * torch.diagonal(H).clamp_min(1e-9))
        C, info = torch.linalg.cholesky_ex(H)
        accept = False
        if int(info) == 0:
            x = -torch.cholesky_solve(g[:, None], C)[:, 0].view(-1, 6)
            Tc = torch.cat([T[:1], _apply(_exp(x), T[1:])])
            Fc = cost(Tc)
            accept = bool(Fc < F)
        if accept:
            T, F = Tc, Fc
        lam = max(lam / 10, 1e-10) if accept else min(lam * 10, 1e10)
    return {"poses": T, "cost": torch.stack([F0, F])[None], "status": None}


def _np_skew(v):
    return np.array([[0, -v[2], v[1]], [v[2], 0, -v[0]], [-v[1], v[0], 0]])


def _exact_preint(gyro, accel, dt):
    """Preintegration record of one interval at zero bias (Forster et al. 2017)."""
    R, v, p = np.eye(3), np.zeros(3), np.zeros(3)
    JR, Jvg, Jva, Jpg, Jpa, cov = (np.zeros((3, 3)) for _ in range(6))
    cov = np.zeros((9, 9))
    I3 = np.eye(3)
    for w, a in zip(gyro, accel):
        th2 = float(w @ w) * dt * dt
        b, c = 0.5, 1.0 / 6
        tb, tc = 0.5, 1.0 / 6
        for n in range(1, 10):
            tb *= -th2 / ((2 * n + 1) * (2 * n + 2))
            tc *= -th2 / ((2 * n + 2) * (2 * n + 3))
            b, c = b + tb, c + tc
        Kw = _np_skew(w * dt)
        Ek = _np_rot(w * dt)
        Jr = I3 - b * Kw + c * Kw @ Kw
        RA = R @ _np_skew(a)
        A = np.eye(9)
        A[:3, :3] = Ek.T
        A[3:6, :3] = -RA * dt
        A[6:, :3] = -0.5 * RA * dt * dt
        A[6:, 3:6] = I3 * dt
        Bg, Ba = np.zeros((9, 3)), np.zeros((9, 3))
        Bg[:3] = Jr * dt
        Ba[3:6], Ba[6:] = R * dt, 0.5 * R * dt * dt
        cov = A @ cov @ A.T + (IMU_NOISE[0] ** 2 / dt) * Bg @ Bg.T + (IMU_NOISE[1] ** 2 / dt) * Ba @ Ba.T
        Jpa = Jpa + Jva * dt - 0.5 * R * dt * dt
        Jpg = Jpg + Jvg * dt - 0.5 * RA @ JR * dt * dt
        Jva = Jva - R * dt
        Jvg = Jvg - RA @ JR * dt
        JR = Ek.T @ JR - Jr * dt
        p = p + v * dt + 0.5 * R @ a * dt * dt
        v = v + R @ a * dt
        R = R @ Ek
    dT = dt * len(gyro)
    info = np.zeros((15, 15))
    info[:9, :9] = np.linalg.inv(cov)
    info[9:12, 9:12] = I3 / (IMU_NOISE[3] ** 2 * dT)
    info[12:, 12:] = I3 / (IMU_NOISE[2] ** 2 * dT)
    rec = np.zeros(ba.VI_PREINT_DOUBLES)
    parts = [R.ravel(), v, p, [dT], JR.ravel(), Jvg.ravel(), Jva.ravel(), Jpg.ravel(), Jpa.ravel(), np.zeros(6), info.ravel()]
    rec[: sum(len(x) for x in parts)] = np.concatenate(parts)
    return rec


def _exact_vi(case, seed):
    w, x, gyro, accel, dt, grav = _vi_data(case, seed)
    n, ns = case["kf"], case["samples"]
    dev = torch.device("cuda")
    pre = torch.tensor(np.stack([_exact_preint(gyro[ns * f: ns * (f + 1)], accel[ns * f: ns * (f + 1)], dt) for f in range(n - 1)]),
                       dtype=F64, device=dev)
    g = torch.tensor(grav, dtype=F64, device=dev)
    vis, P, L = _Visual(w), w["poses"], w["points"]
    M = L.shape[0]
    info = pre[:, 67:292].view(-1, 15, 15)

    def res(z, Pi, si, Pj, sj, q):
        Pi, Pj = _apply(_exp1(z[:6]), Pi), _apply(_exp1(z[15:21]), Pj)
        si, sj = si + z[6:15], sj + z[21:]
        m = lambda a: q[a: a + 9].view(3, 3)  # noqa: E731
        bg, bA, dT = si[6:], si[3:6], q[15]
        u = m(16) @ bg
        Ku = _skew(u)
        t2 = (u * u).sum()
        a, b = 1 - t2 / 6 * (1 - t2 / 20 * (1 - t2 / 42)), 0.5 * (1 - t2 / 12 * (1 - t2 / 30 * (1 - t2 / 56)))
        dR = m(0) @ (torch.eye(3, dtype=F64, device=dev) + a * Ku + b * Ku @ Ku)
        Ri, Rj = Pi[:, :3], Pj[:, :3]
        pi, pj = -(Ri.T @ Pi[:, 3]), -(Rj.T @ Pj[:, 3])
        rv = Ri @ (sj[:3] - si[:3] - g * dT) - (q[9:12] + m(25) @ bg + m(34) @ bA)
        rp = Ri @ (pj - pi - si[:3] * dT - 0.5 * g * dT * dT) - (q[12:15] + m(43) @ bg + m(52) @ bA)
        return torch.cat([_log_rot(dR.T @ Ri @ Rj.T), rv, rp, sj[3:] - si[3:]])

    dims = (None, 0, 0, 0, 0, 0)
    value, jac = torch.func.vmap(res, in_dims=dims), torch.func.vmap(torch.func.jacfwd(res), in_dims=dims)
    z = torch.zeros(30, dtype=F64, device=dev)

    def imu(f, P, x):
        return f(z, P[:-1], x[:-1], P[1:], x[1:], pre)

    def cost(P, L, x):
        F, deep = vis.cost(P, L)
        r = imu(value, P, x)
        return F + 0.5 * (r[:, None] @ info @ r[..., None]).sum(), deep

    nS = 15 * n
    lam, F = LAM0, cost(P, L, x)[0]
    F0 = F
    at = torch.arange(n, device=dev)[:, None] * 15 + torch.arange(15, device=dev)
    idx = torch.cat([at[:-1], at[1:]], 1)
    keep = torch.arange(6, nS, device=dev)
    rows = torch.cat([at[k, :6] for k in vis.free.tolist()])
    for _ in range(case["iters"]):
        Jp, Jl, r = vis.jacobians(P, L)
        w1 = (vis.w * _rho((r * r).sum(1))[1])[:, None, None]
        wp, wl, rc = (w1 * Jp).transpose(1, 2), (w1 * Jl).transpose(1, 2), r[..., None]
        U, gp, V, gl, W = _blocks(vis, wp @ Jp, wp @ Jl, wl @ Jl, (wp @ rc)[..., 0], (wl @ rc)[..., 0], M)
        J, ri = imu(jac, P, x), imu(value, P, x)
        JI = J.transpose(1, 2).contiguous() @ info
        H = torch.zeros(nS + 3 * M, nS + 3 * M, dtype=F64, device=dev)
        H.index_put_((idx[:, :, None].expand(-1, 30, 30), idx[:, None].expand(-1, 30, 30)), JI @ J, accumulate=True)
        b = torch.zeros(nS + 3 * M, dtype=F64, device=dev).index_add_(0, idx.reshape(-1), (JI @ ri[..., None]).reshape(-1))
        H[rows[:, None], rows[None]] += torch.block_diag(*U)
        b[rows] += gp.reshape(-1)
        pt = nS + torch.arange(3 * M, device=dev)
        H[pt[:, None], rows[None]] += W.reshape(3 * M, -1)
        H[rows[:, None], pt[None]] += W.reshape(3 * M, -1).T
        ptm = pt.view(M, 3)
        H.index_put_((ptm[:, :, None].expand(-1, 3, 3), ptm[:, None].expand(-1, 3, 3)), V, accumulate=True)
        b[pt] += gl.reshape(-1)
        sel = torch.cat([keep, pt])
        Hs, bs = H[sel][:, sel], b[sel]
        Hs = Hs + torch.diag(lam * torch.diagonal(Hs).clamp_min(1e-9))
        sc = torch.rsqrt(torch.diagonal(Hs))   # the factors' information spans many orders of magnitude
        C, bad = torch.linalg.cholesky_ex(Hs * sc[:, None] * sc[None])
        accept = False
        if int(bad) == 0:
            s = torch.zeros(nS + 3 * M, dtype=F64, device=dev)
            s[sel] = -sc * torch.cholesky_solve((bs * sc)[:, None], C)[:, 0]
            xi = s[:nS].view(n, 15)
            Pc = torch.where(w["fixed"][:, None, None], P, _apply(_exp(xi[:, :6]), P))
            Lc, xc = L + s[nS:].view(M, 3), x + xi[:, 6:]
            Fc, deep = cost(Pc, Lc, xc)
            accept = deep and bool(Fc < F)
        if accept:
            P, L, x, F = Pc, Lc, xc, Fc
        lam = max(lam / 10, 1e-10) if accept else min(lam * 10, 1e10)
    return {"poses": P, "points": L, "states": x, "preint": pre, "cost": torch.stack([F0, F])[None], "status": None}


def exact(case, seed):
    return dict(window=_exact_window, pnp=_exact_pnp, tri=_exact_tri, pgo=_exact_pgo, vi=_exact_vi)[case["kind"]](case, seed)
