"""Host side of a step call: what it costs must not grow with the steps of the
schedule that the call does not take."""
import time

import pytest
import torch

from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("model", ["poisson", "radmat"])
def test_step_call_on_a_long_schedule(prec, model):
    """150 steps, one per call and all in one call, at the start of a schedule
    of 300 and of one of 30 000 (the same steps): a call does about the same
    work.  Walking the schedule to its end at every launch costs 100 times
    the steps; a factor of 3 leaves room for everything else."""
    took = {}
    for n_steps in (300, 30000):
        z_end = 1.1e6 * 2.718281828459045 ** (-2e-4 * n_steps) - 1.0
        cfg = workloads.small("c3", grid_n=16, n_side=1, n_steps=n_steps, precision=prec, box_mpc=1000.0,
                              z_begin=1.1e6 - 1.0, z_end=z_end, sort_every=20, sort_cells=3.0, model=model,
                              omega_r=1e-4 if model == "radmat" else 0.0)
        cfg["species"] = [dict(field=0, m=0.05, n=1009, n_side=1, seed=s) for s in (1, 2, 3)]
        ctx = fastdf.Context(cfg)
        for calls in ([1] * 150, [150]):
            best = 1e9
            for _ in range(4):
                fastdf.setup_workload(cfg, ctx=ctx)
                ctx.step(1)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                for n in calls:
                    ctx.step(n)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t0)
            took[n_steps, len(calls)] = best
        ctx.close()
    print("[schedule] %s %s %s" % (prec, model, took), flush=True)
    for calls in (1, 150):
        assert took[30000, calls] < 3 * took[300, calls], took
