"""Plans per wave and waves per workgroup follow the batch size: small batches
take few plans per wave, large ones every lane (WF_PLAN_PACK=full takes every
lane for any batch).  Both shapes against the oracle, bytewise, at ragged
batch sizes (a last group that is not full, fewer plans than a group), for
scores, schedules, ranking keys and generated candidates, in every
reclamation mode and on windows of every per-wave layout."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2609_03335_amd as pkg
from paper_2609_03335_amd import workload as W

pytestmark = pytest.mark.gpu

WINDOWS = {
    # name: (generator, its arguments)
    "small": (W.random_window, dict(n_wf=3, nodes=(2, 9), n_dev=3, n_models=4)),
    "odd": (W.random_window, dict(n_wf=6, nodes=(4, 19), n_dev=7, n_models=11)),
    "chains": (W.random_window, dict(n_wf=9, nodes=(9, 12), n_dev=5, n_models=3, p_edge=0.2,
                                     same_model_bias=0.9)),
    "wide": (W.random_window, dict(n_wf=40, nodes=(6, 16), n_dev=10, n_models=16)),
    "models": (W.random_window, dict(n_wf=20, nodes=(6, 16), n_dev=12, n_models=31, q_inel=0.0,
                                     cap_range=(20000, 90000))),
    "models64": (W.random_window, dict(n_wf=20, nodes=(6, 16), n_dev=4, n_models=64,
                                       cap_range=(20000, 90000))),
    "deep": (W.random_deep_window, dict(n_levels=(30, 40), width=(4, 12), n_dev=6, n_models=20)),
    "deep16": (W.random_deep_window, dict(n_levels=(30, 40), width=(4, 12), n_dev=16, n_models=9)),
    "late": (W.random_window, dict(n_wf=12, nodes=(6, 16), n_dev=6, n_models=10,
                                   load_range=(1 << 29, 1 << 30))),
    "checked": (W.random_window, dict(n_wf=4, nodes=(4, 8), n_dev=2, n_models=5, resident=False,
                                      lat_range=(int(1.4e7), int(7e7)),
                                      load_range=(int(1.4e8), int(4.2e8)),
                                      cap_range=(9000, 14000), w_range=(4000, 7000))),
    "devices": (W.random_window, dict(n_wf=12, nodes=(6, 16), n_dev=90, n_models=10)),
}
MODES = ("default", "caps", "paper", "batch", "paper_batch")


def make(name, mode, seed):
    gen, kw = WINDOWS[name]
    rng = np.random.default_rng([seed, len(name)])
    win = gen(rng, **kw)
    win.wf_class = rng.integers(0, 4, win.n_wf).astype(np.uint8)
    if mode == "caps":
        held = np.array([sum((int(r) >> m) & 1 for r in win.init_resident) for m in range(win.n_models)])
        win.model_replica_cap = np.maximum(np.maximum(held, 1), win.n_dev - 1).astype(np.int32)
    if mode in ("paper", "paper_batch"):
        win.victim_order = 1
    if mode in ("batch", "paper_batch"):
        win.dev_batch = rng.integers(1, 5, win.n_dev).astype(np.int32)
    return win, rng


def check(win, rng, n, tag):
    plans = W.random_plans(win, n, rng, p_bad_dev=0.002, prio_mode=("perm", "any")[n % 2])
    N, D = win.n_act, win.n_dev
    with pkg.Context(0) as ctx:
        ctx.wf_plan_upload_window(win)
        # ("late" passes 8 x 2^32 us: fp64 times; "checked" takes the two passes)
        assert ctx.wf_plan_time_bits() == (64 if tag[0] == "late" else 32)
        dev, prio, flags = pkg.device_plans(plans, "cuda:0")
        ref, sched_ref = oracle.score(win, plans, schedule=True)
        live = (ref["status"] & 1) == 0
        scores = pkg.score_batch(ctx, dev, prio, flags, n)
        sc2, sched = pkg.score_batch(ctx, dev, prio, flags, n, schedule=True, n_act=N, n_dev=D)
        keys = torch.empty((n, 32), dtype=torch.uint8, device="cuda:0")
        ctx.wf_plan_score_keys(dev, prio, flags, n, keys)
        torch.cuda.synchronize()
        assert pkg.scores_to_numpy(scores, n).tobytes() == ref.tobytes(), (tag, "scores")
        assert pkg.scores_to_numpy(sc2, n).tobytes() == ref.tobytes(), (tag, "scores with schedule")
        for a, b in zip(sched, sched_ref):
            assert np.array_equal(a.cpu().numpy()[live], b[live]), (tag, "schedule")
        kref = oracle.phi_keys(win, plans)
        assert pkg.keys_to_numpy(keys, n).tobytes() == kref.tobytes(), (tag, "keys")
        for n_mut, mode in ((3, 0), (11, 1)):
            ctx.wf_plan_search_batch(dev[0], prio[0], flags[0], 77, n_mut, 5, n, scores, mode=mode)
            ctx.wf_plan_search_keys(dev[0], prio[0], flags[0], 77, n_mut, 5, n, keys, mode=mode)
            torch.cuda.synchronize()
            cand = W.PlanBatch(*oracle.search_candidates(win, plans.dev[0], plans.prio[0],
                                                         plans.flags[0], 77, n_mut, 5, n, mode=mode))
            assert pkg.scores_to_numpy(scores, n).tobytes() == oracle.score(win, cand).tobytes(), \
                (tag, "candidates", n_mut)
            assert pkg.keys_to_numpy(keys, n).tobytes() == oracle.phi_keys(win, cand).tobytes(), \
                (tag, "candidate keys", n_mut)


@pytest.mark.parametrize("pack", ["full", "fitted"])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("name", sorted(WINDOWS))
def test_both_shapes(name, mode, pack, monkeypatch):
    if pack == "full":
        monkeypatch.setenv("WF_PLAN_PACK", "full")
    for seed, n in ((1, 45), (2, 130)):
        win, rng = make(name, mode, seed)
        check(win, rng, n, (name, mode, pack, seed))
