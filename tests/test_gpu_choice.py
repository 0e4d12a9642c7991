"""The choice between the scoring kernels: calls that the lane-per-plan kernel
serves more slowly than the kernel it would replace (mid-sized batches of
candidates, keys, windows of many narrow levels, of 17 to 32 models) and calls
that it serves faster, both timed.  Times are taken on one GPU one after the
other; a choice fails when it takes 1.4 times as long as the other kernel (the
calls that must not take the lane-per-plan kernel measured 1.6 to 2.6 times)."""
import numpy as np
import pytest
import torch

import paper_2609_03335_amd as pkg
from paper_2609_03335_amd import workload as W

pytestmark = pytest.mark.gpu

AGENTS = dict(nodes=(8, 14), p_edge=0.15, q_inel=0.1, cap_range=(20000, 60000), w_range=(4000, 40000))
WINDOWS = {
    "agents17": (W.random_window, dict(AGENTS, n_wf=2, n_dev=15, n_models=24)),
    "agents110": (W.random_window, dict(AGENTS, n_wf=10, n_dev=14, n_models=26)),
    "deep24": (W.random_deep_window, dict(n_levels=(8, 8), width=(24, 28), n_dev=15, n_models=27,
                                          cap_range=(20000, 60000), w_range=(4000, 40000))),
    "wide": (W.random_deep_window, dict(n_levels=(4, 4), width=(200, 200), n_dev=8, n_models=14, p_edge=0.01,
                                        w_range=(4000, 40000), cap_range=(40000, 190000))),
    "layered": (W.random_deep_window, dict(n_levels=(4, 4), width=(60, 64), n_dev=8, n_models=16,
                                           p_edge=0.05, w_range=(4000, 40000), cap_range=(40000, 80000))),
}
CALLS = [("agents17", True, 8, 8192), ("agents17", False, -1, 131072), ("agents110", True, 8, 8192),
         ("agents110", True, 3, 8192), ("agents110", False, -1, 65536), ("deep24", True, 8, 16384),
         ("deep24", False, 4, 16384), ("deep24", True, -1, 65536), ("wide", True, 8, 8192),
         ("wide", True, -1, 8192), ("layered", False, -1, 16384), ("layered", False, -1, 262144),
         ("layered", True, 2, 131072)]


@pytest.mark.parametrize("name,keys,n_mut,n", CALLS)
def test_the_faster_kernel_is_taken(name, keys, n_mut, n, monkeypatch):
    gen, kw = WINDOWS[name]
    rng = np.random.default_rng(len(name))
    win = gen(rng, **kw)
    few = W.random_plans(win, 1024, rng, prio_mode="perm")
    dev, prio, flags = (x.repeat((n + 1023) // 1024, 1) for x in pkg.device_plans(few, "cuda:0"))
    out = torch.empty((n, 32), dtype=torch.uint8, device="cuda:0")
    took, kernel = {}, None
    for lanes in ("on", "off", None):
        monkeypatch.delenv("WF_PLAN_LANES", raising=False)
        if lanes:
            monkeypatch.setenv("WF_PLAN_LANES", lanes)
        with pkg.Context(0) as ctx:
            ctx.wf_plan_upload_window(win)
            kernel = ctx.wf_plan_batch_kernel(n, keys, n_mut)
            if lanes is None:
                break
            assert (kernel == "score_lanes") == (lanes == "on")

            def call():
                if n_mut < 0:
                    (ctx.wf_plan_score_keys if keys else ctx.wf_plan_score_batch)(dev, prio, flags, n, out)
                else:
                    (ctx.wf_plan_search_keys if keys else ctx.wf_plan_search_batch)(
                        dev[0], prio[0], flags[0], 77, n_mut, 0, n, out)

            best = float("inf")
            for _ in range(5):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                call()
                call()
                b.record()
                torch.cuda.synchronize()
                best = min(best, a.elapsed_time(b) / 2)
            took[lanes] = best
    mine, other = (took["on"], took["off"]) if kernel == "score_lanes" else (took["off"], took["on"])
    print(f"[choice] {name} keys={keys} n_mut={n_mut} n={n}: {kernel} {mine * 1e3:.0f} us, "
          f"other {other * 1e3:.0f} us", flush=True)
    assert mine < 1.4 * other, (kernel, took)
