"""GPU parity of the batched triangulation (ba_triangulate) against the FP64
oracle (oracle/triangulate.py), through the C ABI.

FP64 mode: the oracle follows the GPU's accept/reject sequence (a flip must be a
near-tie in the oracle's own numbers); statuses are equal, and the cost of every
attempt, the final cost and the point agree to 1e-9 relative.  Mixed mode, on
the full 256-window workload in the launch the benchmark times: statuses equal
and the point within 1e-6 * max(|p|, 1 m) on sampled landmarks, every refined
cost not above its start.
"""
import math

import numpy as np
import pytest

import bagen
from oracle import triangulate as tri
from oracle.lm import LMSettings

pytestmark = pytest.mark.gpu

TOL64 = 1e-9


def _obs(b, j, obs_w=None):
    ob = tri.landmark_obs(b.intrinsics, b.extrinsics, b.poses, b.point_obs_begin, b.obs_pose, b.obs_cam,
                          b.obs_uv, b.obs_w, j)
    if obs_w is not None:
        ob.obs_w = obs_w[b.point_slice(j)]
    return ob


def _gpu(b, s, obs_w=None, obs_pose=None, with_trace=True):
    import torch
    import paper_2506_04359_amd as ba
    dev = torch.device("cuda:0")
    rig = ba.Rig(b.intrinsics, b.extrinsics.reshape(-1, 12))
    t = lambda a, dt: torch.tensor(np.ascontiguousarray(a), dtype=dt, device=dev)
    pts = torch.full((b.n_points, 3), 7.0, dtype=torch.float64, device=dev)
    tr = (torch.zeros(32 * b.n_points * max(1, s.max_iters), dtype=torch.uint8, device=dev)
          if with_trace else None)
    rep, tr = ba.triangulate(rig, s, t(b.point_obs_begin, torch.int32), t(b.poses.reshape(-1, 12), torch.float64),
                             t(b.obs_pose if obs_pose is None else obs_pose, torch.int32),
                             t(b.obs_uv, torch.float64), pts, obs_cam=t(b.obs_cam, torch.int32),
                             obs_w=None if obs_w is None else t(obs_w, torch.float64), traces=tr)
    torch.cuda.synchronize()
    out = dict(points=pts.cpu().numpy(), reports=ba.parse_reports(rep)[: b.n_points])
    if with_trace:
        out["traces"] = ba.parse_traces(tr, b.n_points, max(1, s.max_iters))
    return out


def _osettings(s):
    return LMSettings(max_iters=s.max_iters, lambda_init=s.lambda_init, huber_delta=s.huber_delta,
                      min_depth=s.min_depth)


def _check_fp64(b, s, g, obs_w=None, every=1):
    n_ok = 0
    for j in range(0, b.n_points, every):
        ob = _obs(b, j, obs_w)
        r = g["reports"][j]
        ref0 = tri.triangulate(ob, _osettings(s))
        assert r["status"] == ref0.status, (j, r, ref0.status)
        if ref0.status in (tri.STATUS_DEGENERATE, 2):
            assert np.all(np.isnan(g["points"][j]))
            continue
        if ref0.status == tri.STATUS_BEHIND:
            assert np.abs(g["points"][j] - ref0.point).max() <= TOL64 * max(1.0, np.abs(ref0.point).max())
            continue
        n_ok += 1
        tr = g["traces"][j]
        ref = tri.triangulate(ob, _osettings(s), decisions=[bool(a) for a in tr["accepted"]])
        for t, gt in zip(ref.trace, tr):
            if t["own_decision"] != bool(gt["accepted"]):
                assert abs(t["cand_cost"] - t["cost"]) <= 1e-12 * abs(t["cost"]), (j, t, gt)
            assert abs(t["cost"] - gt["cost"]) <= TOL64 * max(abs(t["cost"]), 1e-300), (j, t, gt)
        assert abs(r["final_cost"] - ref.final_cost) <= TOL64 * max(ref.final_cost, 1e-300)
        assert r["accepted"] == ref.accepted and r["chol_failures"] == ref.chol_failures
        assert np.abs(g["points"][j] - ref.point).max() <= TOL64 * max(1.0, np.abs(ref.point).max()), j
    return n_ok


@pytest.mark.parametrize("cfg,windows", [(1, 2), (2, 1), (4, 1)])
def test_fp64_landmarks_match_oracle(cfg, windows):
    """Mono (2-5 views), stereo (2 cameras, tracks up to 15 frames, outliers)
    and the 32-camera rig."""
    import paper_2506_04359_amd as ba
    b = bagen.make_tri_batch([bagen.make_window(cfg, i) for i in range(windows)])
    s = ba.Settings(max_iters=10, precision=ba.BA_FP64)
    every = 1 if b.n_points <= 500 else max(1, b.n_points // 400)
    n_ok = _check_fp64(b, s, _gpu(b, s), every=every)
    assert n_ok >= 50


def test_fp64_weights_and_least_squares():
    import paper_2506_04359_amd as ba
    b = bagen.make_tri_batch([bagen.make_window(1, 5)])
    w = np.random.default_rng(4).uniform(0.3, 2.0, b.n_obs)
    s = ba.Settings(max_iters=8, precision=ba.BA_FP64)
    _check_fp64(b, s, _gpu(b, s, obs_w=w), obs_w=w)
    s_ls = ba.Settings(max_iters=8, precision=ba.BA_FP64, huber_delta=0.0)
    _check_fp64(b, s_ls, _gpu(b, s_ls))


def test_degenerate_landmarks():
    """One view, two identical rays, a start behind the rig and an
    out-of-range pose index: statuses 3, 3, 4, 2; the other landmarks solved."""
    import paper_2506_04359_amd as ba
    K = np.array([[718.0, 718.0, 607.0, 185.0]] * 2)
    E = np.zeros((2, 3, 4))
    E[:, :, :3] = np.eye(3)
    E[1, 0, 3] = -0.54
    T = np.zeros((2, 3, 4))
    T[:, :, :3] = np.eye(3)
    T[1, 2, 3] = -1.0
    obs = [  # (pose, cam, u, v) per landmark
        [(0, 0, 700.0, 150.0), (0, 1, 687.5, 150.0)],           # fine
        [(0, 0, 600.0, 180.0)],                                 # one view
        [(0, 0, 600.0, 180.0), (0, 0, 600.0, 180.0)],           # identical rays
        [(0, 0, 600.0, 185.0), (0, 1, 620.0, 185.0)],           # diverging rays
        [(0, 0, 700.0, 150.0), (5, 1, 687.5, 150.0)],           # pose 5 does not exist
        [(0, 0, 500.0, 200.0), (1, 0, 495.0, 201.0), (1, 1, 470.0, 201.0)],
    ]
    begin = np.cumsum([0] + [len(o) for o in obs]).astype(np.int32)
    flat = [x for o in obs for x in o]
    b = bagen.TriBatch(intrinsics=K, extrinsics=E, poses=T, points_gt=np.zeros((len(obs), 3)),
                       point_obs_begin=begin, obs_pose=np.array([x[0] for x in flat], np.int32),
                       obs_cam=np.array([x[1] for x in flat], np.int32),
                       obs_uv=np.array([[x[2], x[3]] for x in flat]), obs_w=np.ones(len(flat)))
    s = ba.Settings(max_iters=6, precision=ba.BA_FP64)
    g = _gpu(b, s)
    assert list(g["reports"]["status"]) == [0, 3, 3, 4, 2, 0]
    for j in (0, 5):
        ref = tri.triangulate(_obs(b, j), _osettings(s))
        assert np.abs(g["points"][j] - ref.point).max() <= TOL64 * max(1.0, np.abs(ref.point).max())
    assert np.all(np.isnan(g["points"][[1, 2, 4]]))


def test_mixed_full_batch_sampled():
    """The 256-window workload (about 1.05 M landmarks) in the benchmark's launch."""
    import paper_2506_04359_amd as ba
    b = bagen.make_tri_batch([bagen.make_window(3, i) for i in range(256)], max_iters=10)
    s = ba.Settings(max_iters=10, precision=ba.BA_MIXED)
    g = _gpu(b, s, with_trace=False)
    r = g["reports"]
    ok = r["status"] == 0
    assert ok.mean() > 0.99
    assert np.all(r["final_cost"][ok] <= r["initial_cost"][ok])
    rng = np.random.default_rng(5)
    for j in [0, b.n_points - 1] + list(rng.integers(0, b.n_points, 60)):
        ref = tri.triangulate(_obs(b, j), _osettings(s))
        assert r["status"][j] == ref.status, j
        if ref.status == 0:
            err = np.abs(g["points"][j] - ref.point).max()
            assert err <= 1e-6 * max(1.0, np.linalg.norm(ref.point)), (j, err)


@pytest.mark.parametrize("n_kf,n_lm,weighted,bad", [(3, 1, False, False), (3, 255, True, False), (3, 257, False, True),
                                                    (10, 129, False, True), (24, 65, True, True),
                                                    (24, 130, False, False)])
def test_workgroup_edges(n_kf, n_lm, weighted, bad):
    """Counts at the edges of the workgroups (256, 128 and 64 landmarks, by the mean
    track length), with the observations staged in LDS; bad indices inside a
    staged group mark their own landmark only."""
    import paper_2506_04359_amd as ba
    b = bagen.make_tri_batch([bagen.tiny_window(seed=40 + n_lm, n_kf=n_kf, n_lm=n_lm)])
    s = ba.Settings(max_iters=6, precision=ba.BA_FP64)
    w = np.random.default_rng(n_lm).uniform(0.3, 2.0, b.n_obs) if weighted else None
    pose = b.obs_pose.copy()
    marked = [n_lm // 2, n_lm - 1] if bad else []
    for j in marked:
        pose[b.point_obs_begin[j]] = -1 if j == n_lm // 2 else b.n_poses
    g = _gpu(b, s, obs_w=w, obs_pose=pose)
    assert [int(j) for j in np.flatnonzero(g["reports"]["status"] == 2)] == marked
    if not bad:
        _check_fp64(b, s, g, obs_w=w, every=max(1, n_lm // 40))
        return
    clean = _gpu(b, s, obs_w=w)
    keep = np.setdiff1d(np.arange(n_lm), marked)
    _check_fp64(b, s, clean, obs_w=w, every=max(1, n_lm // 40))
    assert np.array_equal(clean["points"][keep], g["points"][keep])
    assert np.all(np.isnan(g["points"][marked]))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("track,weighted", [(2, False), (8, False), (8, True), (12, False), (16, False), (40, False)])
def test_landmarks_over_many_poses(track, weighted, precision):
    """Tracks over 200 poses in no order: more transforms than a workgroup keeps, in
    workgroups of 256, 128 and 64 landmarks; a bad index marks its own landmark only."""
    import paper_2506_04359_amd as ba
    rng = np.random.default_rng(100 + track)
    n_pose, n_lm = 200, 300
    poses = np.tile(np.eye(3, 4), (n_pose, 1, 1))
    poses[:, 0, 3] = np.linspace(-3, 3, n_pose)
    pts = np.stack([rng.uniform(-3, 3, n_lm), rng.uniform(-2, 2, n_lm), rng.uniform(6, 15, n_lm)], 1)
    op = rng.random((n_lm, n_pose)).argsort(1)[:, :track].ravel()
    oj = np.repeat(np.arange(n_lm), track)
    x = pts[oj] + poses[op][:, :, 3]
    uv = 458.0 * x[:, :2] / x[:, 2:] + [367.0, 248.0] + rng.normal(scale=0.4, size=(len(op), 2))
    w = rng.uniform(0.3, 2.0, len(op)) if weighted else None
    b = bagen.TriBatch(intrinsics=np.array([[458.0, 458.0, 367.0, 248.0]]), extrinsics=np.eye(3, 4)[None], poses=poses,
                       points_gt=pts, point_obs_begin=(np.arange(n_lm + 1) * track).astype(np.int32),
                       obs_pose=op.astype(np.int32), obs_cam=np.zeros(len(op), np.int32), obs_uv=uv,
                       obs_w=np.ones(len(op)))
    s = ba.Settings(max_iters=8, precision=ba.BA_FP64 if precision == "fp64" else ba.BA_MIXED)
    g = _gpu(b, s, obs_w=w)
    if precision == "fp64":
        _check_fp64(b, s, g, obs_w=w, every=7)
    else:
        for j in range(0, n_lm, 7):
            ref = tri.triangulate(_obs(b, j, w), _osettings(s))
            assert g["reports"][j]["status"] == ref.status
            if ref.status == 0:
                assert np.abs(g["points"][j] - ref.point).max() <= 1e-6 * max(1.0, np.linalg.norm(ref.point)), j
    bad = b.obs_pose.copy()
    bad[[3 * track, 290 * track + track - 1]] = [n_pose, -1]
    h = _gpu(b, s, obs_w=w, obs_pose=bad)
    keep = np.setdiff1d(np.arange(n_lm), [3, 290])
    assert np.flatnonzero(h["reports"]["status"] == 2).tolist() == [3, 290]
    assert np.array_equal(h["points"][keep], g["points"][keep], equal_nan=True)
    assert np.all(np.isnan(h["points"][[3, 290]]))
