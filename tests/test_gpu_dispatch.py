"""The rules that choose a kernel's variant by the window's size, at their
edges: the Schur units of windows with few free poses, and the FP64 tile and
work-item tables of a batch's size classes."""
import numpy as np
import pytest

import bagen
from helpers import check_decisions, gpu_solve, gpu_solve_batched, oracle_replay, rel_err

pytestmark = pytest.mark.gpu
TOL64 = 1e-9


def _replay_parity(w, s, g):
    prob, ref = oracle_replay(w, s, g["trace"])
    check_decisions(ref, g["trace"])
    assert abs(g["report"]["final_cost"] - ref.final_cost) <= TOL64 * ref.final_cost
    assert rel_err(g["poses"], ref.poses) <= TOL64 and rel_err(g["points"], ref.points) <= TOL64


@pytest.mark.parametrize("n_free", [1, 2, 4, 5, 7, 8, 9, 10])
def test_schur_units_of_few_free_poses(n_free):
    # off-diagonal blocks n (n - 1) / 2: a thread per entry up to 7 blocks (4 free poses),
    # per three columns up to 21 (7), per row up to 42 (9), two rows above
    import paper_2506_04359_amd as ba
    w = bagen.tiny_window(seed=8100 + n_free, n_kf=n_free + 2, n_lm=150, noise=0.5, fixed=(0, 1))
    s = ba.Settings(max_iters=6, precision=ba.BA_FP64)
    _replay_parity(w, s, gpu_solve(w, s))


@pytest.mark.parametrize("chunk_obs", [512, 2048])
def test_fp64_batch_of_every_size_class(chunk_obs):
    # up to 23 free poses 256-pair tiles, above 64-pair tiles, in one batch
    import paper_2506_04359_amd as ba
    ws = [bagen.tiny_window(seed=8200 + n, n_kf=n + 2, n_lm=300, noise=0.5, fixed=(0, 1)) for n in (6, 12, 23, 24, 28)]
    s = ba.Settings(max_iters=5, precision=ba.BA_FP64)
    for w, g in zip(ws, gpu_solve_batched(ws, s, chunk_obs=chunk_obs)):
        assert g["report"]["status"] == 0
        _replay_parity(w, s, g)


def test_launch_shape_read_and_set_back_is_the_same_shape():
    # the default work items of an FP64 batch are smaller than the mixed ones
    import paper_2506_04359_amd as ba
    ws = [bagen.tiny_window(seed=8250 + n, n_kf=n + 2, n_lm=300, noise=0.5, fixed=(0, 1)) for n in (6, 12, 24)]
    B = ba.Batch([ba.Window.from_problem(w, host_only=True) for w in ws])
    sizes = lambda: [B.workspace_size(ba.Settings(max_iters=5, precision=p)) for p in (ba.BA_FP64, ba.BA_MIXED)]
    first, cfg = sizes(), B.get_launch()
    B.set_launch_config(**cfg)
    assert sizes() == first
    B.set_launch_config(**dict(cfg, class_streams=0))
    assert sizes() == first
    B.set_launch(16384)
    one_item = sizes()
    assert one_item[0] < first[0]   # fewer partials than the default's
    B.set_launch_config(**cfg)
    assert sizes() == first and B.get_launch() == cfg


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_cached_shapes_of_the_first_fp64_grid_are_not_taken(precision, tmp_path, monkeypatch):
    # a line of the older FP64 grid would replace a default that is faster; mixed lines stand
    import torch
    import paper_2506_04359_amd as ba
    dev = torch.device("cuda:0")
    cache = tmp_path / "tune"
    monkeypatch.setenv("BA_TUNE_CACHE", str(cache))
    ws = [bagen.tiny_window(seed=8270 + n, n_kf=n + 2, n_lm=200, noise=0.5, fixed=(0, 1)) for n in (4, 8)]
    s = ba.Settings(max_iters=3, precision=ba.BA_FP64 if precision == "fp64" else ba.BA_MIXED)
    t = lambda k: torch.tensor(np.concatenate([getattr(w, k) for w in ws]), dtype=torch.float64, device=dev)
    B = ba.Batch([ba.Window.from_problem(w, host_only=True) for w in ws])
    mem = torch.empty(4 * B.workspace_size(s), dtype=torch.uint8, device=dev)
    tune = lambda: B.autotune(s, t("poses_init"), t("points_init"), t("obs_uv"), None, mem)
    tune()
    key, *shape = cache.read_text().split()
    cache.write_text(" ".join([key.replace("|0.2|", "|0|"), "65536", *shape[1:]]) + "\n")
    chosen = tune()
    if precision == "mixed":
        assert chosen == 65536 and B.get_launch()["chunk_obs"] == 65536
    else:
        assert chosen != 65536 and cache.read_text().splitlines()[1].split()[0] == key


def _many_item_window():
    w = bagen.tiny_window(seed=8601, n_kf=8, n_lm=7000, noise=0.5, fixed=(0, 1))
    assert w.obs_pose.shape[0] > 300 * 128   # more than 256 work items of 128 observations
    return w


@pytest.mark.parametrize("iters,freeze", [(4, None), (5, None), (9, "grad"), (9, "step")])
def test_windows_of_more_work_items_than_pass_a_decides_for(iters, freeze):
    # above 256 work items in any window the acceptance is a launch of its own, for
    # every window of the solve; the state's two copies end in either parity
    import math
    import oracle
    import paper_2506_04359_amd as ba
    from helpers import oracle_settings
    from oracle import lm as olm
    big = _many_item_window()
    ws = [bagen.tiny_window(seed=8602, n_kf=5, n_lm=60, noise=0.5, fixed=(0, 1)), big,
          bagen.tiny_window(seed=8603, n_kf=14, n_lm=120, noise=0.5, fixed=(0, 1))]
    s = ba.Settings(max_iters=iters, precision=ba.BA_FP64)
    prob = oracle.Problem.from_window(big)
    if freeze:   # a tolerance between two values that are far apart in the converging phase
        run = oracle.lm_solve(big.poses_init, big.points_init, prob, oracle_settings(s), backend="schur")
        v = []
        if freeze == "step":
            v = [t["step_norm"] for t in run.trace if t["accepted"]]
        else:
            P, L = big.poses_init, big.points_init
            for t in run.trace:
                sy = olm.normal_equations_blocks(P, L, prob, s.huber_delta)
                v.append(olm.reduced_gradient_norm(sy, "schur", t["lam"], prob.n_free))
                if t["accepted"]:
                    P, L = olm.apply_step(P, L, prob, olm.solve_schur(sy, t["lam"], olm._pairs_of_pairs(sy)))
        k = next(k for k in range(2, len(v)) if v[k] < 0.3 * v[k - 1])
        setattr(s, freeze + "_tol", math.sqrt(v[k] * v[k - 1]))
    g = gpu_solve_batched(ws, s, launch=dict(chunk_obs=128, tile_pairs=64))
    ref = oracle.lm_solve(big.poses_init, big.points_init, prob, oracle_settings(s), backend="schur",
                          decisions=[bool(a) for a in g[1]["trace"]["accepted"]])
    check_decisions(ref, g[1]["trace"])
    assert g[1]["report"]["iters"] == ref.iters and (freeze is None or ref.iters < iters)
    assert abs(g[1]["report"]["final_cost"] - ref.final_cost) <= TOL64 * ref.final_cost
    assert rel_err(g[1]["poses"], ref.poses) <= TOL64 and rel_err(g[1]["points"], ref.points) <= TOL64
    for i in (0, 2):
        _replay_parity(ws[i], s, g[i])
        assert np.array_equal(g[i]["poses"], gpu_solve_batched([ws[i]], s, launch=dict(chunk_obs=128, tile_pairs=64))[0]["poses"])
