"""Reduced systems that are not positive definite: the attempt is rejected with
status 1, counted as a factorisation failure, and the states stay as they are."""
import numpy as np
import pytest

import bagen
import oracle
from helpers import gpu_solve
from oracle import imu
from oracle import lm as olm
from test_gpu_vi import _gpu_inputs, _gpu_solve

pytestmark = pytest.mark.gpu
HUGE = np.finfo(np.float64).max


def _negative_window(n_free, slot):
    """A window whose free pose `slot` has small negative weights: its reduced block's
    first pivot is negative, the blocks before it and every landmark block are
    positive definite."""
    w = bagen.tiny_window(seed=8300 + n_free, n_kf=n_free + 2, n_lm=150 if n_free < 20 else 300, noise=0.5,
                          fixed=(0, 1))
    ow = np.ones(w.obs_pose.shape[0])
    ow[w.obs_pose == slot + 2] = -1e-4
    prob = oracle.Problem.from_window(w, obs_w=ow)
    H, _ = olm.normal_equations_dense(w.poses_init, w.points_init, prob, w.huber_delta)
    n = 6 * n_free
    for lam in (w.lambda_init, w.lambda_init * 1e4):   # first and last attempt
        Hd = H + lam * np.diag(np.maximum(np.diag(H), 1e-9))
        V = np.stack([Hd[i:i + 3, i:i + 3] for i in range(n, H.shape[0], 3)])
        assert not olm._not_pd(V)
        S = Hd[:n, :n] - Hd[:n, n:] @ np.linalg.solve(Hd[n:, n:], Hd[n:, :n])
        k = 6 * slot
        if k:
            np.linalg.cholesky(S[:k, :k])
        p = S[k, k] - (S[k, :k] @ np.linalg.solve(S[:k, :k], S[:k, k]) if k else 0.0)
        assert p < -1e-3 * abs(H[k, k]), p   # far from rounding, also in FP32
    return w, ow


# one panel wave up to 14 free poses, two to 27, three above; the failing pivot in the
# first block row, where the other waves are still on their way in, and in the last
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_free", [1, 2, 5, 14, 15, 28])
@pytest.mark.parametrize("last", [False, True])
def test_negative_pivot_rejects_every_attempt(n_free, last, precision):
    import paper_2506_04359_amd as ba
    w, ow = _negative_window(n_free, n_free - 1 if last else 0)
    s = ba.Settings(max_iters=5, precision=ba.BA_FP64 if precision == "fp64" else ba.BA_MIXED,
                    lambda_init=w.lambda_init, huber_delta=w.huber_delta)
    g = gpu_solve(w, s, obs_w=ow)
    assert [int(x) for x in g["trace"]["status"]] == [1] * 5
    assert g["report"]["chol_failures"] == 5 and g["report"]["accepted"] == 0 and g["report"]["depth_rejects"] == 0
    assert np.array_equal(g["poses"], w.poses_init) and np.array_equal(g["points"], w.points_init)


def _infinite_first_pivots(n_free):
    """A window and a damping that overflows on the first diagonal entry of reduced
    blocks (and on no other entry of any block): close landmarks, so that the pose's
    first translation axis has the largest entry, 16 times the second's."""
    w = bagen.tiny_window(seed=8400 + n_free, n_kf=n_free + 2, n_lm=150, noise=0.5, fixed=(0, 1))
    w.poses_init[:, :, 3] *= 0.05
    w.points_init *= 0.05
    w.intrinsics[:, 0] *= 4.0
    w.obs_uv[:, 0] = w.intrinsics[0, 2] + 4.0 * (w.obs_uv[:, 0] - w.intrinsics[0, 2])
    prob = oracle.Problem.from_window(w)
    H, _ = olm.normal_equations_dense(w.poses_init, w.points_init, prob, w.huber_delta)
    d, first = np.diag(H), np.zeros(H.shape[0], bool)
    first[:6 * n_free:6] = True
    lam = (1.1 / d[first].max()) * HUGE
    assert (d[~first] * (lam / HUGE) < 0.8).all()
    return w, lam


@pytest.mark.parametrize("n_free", [1, 5, 14, 15])
def test_infinite_first_pivot_rejects_every_attempt(n_free):
    import paper_2506_04359_amd as ba
    w, lam = _infinite_first_pivots(n_free)
    s = ba.Settings(max_iters=3, precision=ba.BA_FP64, lambda_init=lam, lambda_max=lam, huber_delta=w.huber_delta,
                    min_depth=1e-3)
    g = gpu_solve(w, s)
    assert [int(x) for x in g["trace"]["status"]] == [1] * 3
    assert g["report"]["chol_failures"] == 3 and g["report"]["accepted"] == 0
    assert np.array_equal(g["poses"], w.poses_init) and np.array_equal(g["points"], w.points_init)


def _vi_case(kind, n_kf, f):
    """A visual-inertial window whose factor f has an information that breaks the
    elimination of its states: negative, or so large on one velocity axis that the
    damped first entry of a state's block overflows and nothing else does."""
    vw = bagen.make_vi_window(seed=9130 + n_kf, n_kf=n_kf, n_lm=120)
    w = vw.window
    bias_bar = (vw.ba_init[0], vw.bg_init[0])
    noise = imu.ImuNoise(*vw.noise)
    vel, lam = vw.vel_init.copy(), 1e-3
    if kind == "infinite":   # at rest without gravity: the velocity rows do not couple to the rotations
        vw.gravity, vel = np.zeros(3), np.zeros_like(vel)
    factors, infos = [], []
    for i in range(n_kf - 1):
        pre = imu.preintegrate(vw.gyro[i], vw.accel[i], vw.dt, bias_bar[1], bias_bar[0], noise)
        Info = imu.imu_information(pre, noise)
        if i == f and kind == "negative":
            Info = -Info
        elif i == f:
            Info[3, 3] *= 1e6
        factors.append((i, i + 1, pre, Info))
        infos.append(Info)
    vp = imu.ViProblem(visual=oracle.Problem.from_window(w), factors=factors, gravity=vw.gravity)
    x0 = imu.ViState(poses=w.poses_init.copy(), vel=vel, ba=vw.ba_init.copy(), bg=vw.bg_init.copy(),
                     points=w.points_init.copy())
    H, _ = imu.vi_normal_equations(x0, vp, 1.0)
    _, vel_col, ns = imu.state_columns(vp)
    d = np.diag(H)
    if kind == "negative":
        V = np.stack([H[i:i + 3, i:i + 3] for i in range(ns, H.shape[0], 3)])
        assert not olm._not_pd(olm._damp(V, lam)) and d[vel_col[f]] < 0
    else:
        first = [vel_col[f], vel_col[f + 1]]
        lam = (1.1 / d[first].min()) * HUGE
        rest = np.ones(d.size, bool)
        rest[first] = False
        assert (d[rest] * (lam / HUGE) < 0.8).all()
    return vw, bias_bar, np.stack(infos), np.concatenate([vel, vw.ba_init, vw.bg_init], axis=1), lam


@pytest.mark.parametrize("kind", ["negative", "infinite"])
@pytest.mark.parametrize("n_kf,f", [(3, 0), (10, 0), (10, 8), (16, 7)])
def test_vi_elimination_failure_rejects_every_attempt(kind, n_kf, f):
    import torch
    import paper_2506_04359_amd as ba
    vw, bias_bar, infos, st0, lam = _vi_case(kind, n_kf, f)
    preint = ba.vi_preintegrate(*_gpu_inputs(vw, bias_bar)[:3], vw.dt, _gpu_inputs(vw, bias_bar)[3], vw.noise)
    preint[:, 67:67 + 225] = torch.tensor(infos.reshape(-1, 225), device=preint.device)
    s = ba.Settings(max_iters=3, precision=ba.BA_FP64, lambda_init=lam, lambda_max=max(lam, 1e10))
    g = _gpu_solve(vw, s, preint, states0=st0)
    assert [int(x) for x in g["trace"]["status"]] == [1] * 3
    assert g["report"]["chol_failures"] == 3 and g["report"]["accepted"] == 0
    assert np.array_equal(g["poses"], vw.window.poses_init) and np.array_equal(g["points"], vw.window.points_init)
    assert np.array_equal(g["states"], st0)
