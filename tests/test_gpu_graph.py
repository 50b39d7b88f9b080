"""Captured step sequences: a replay must do what the same call does without
the capture, on whatever the context holds by then."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu


def _job(ctx, cfg, seeds):
    """Reset, fields, species of these seeds, 12 steps: every state and weight."""
    ctx.reset()
    fields = [ctx.add_field(s) for s in cfg["fields"]]
    species = [ctx.init_species(fields[0], sp["m"], sp["n"], seed) for sp, seed in zip(cfg["species"], seeds)]
    ctx.step(12)
    return [v for s in species for v in ctx.read_state(s)] + [ctx.weights(s).cpu().numpy() for s in species]


@pytest.mark.parametrize("sort_every", [0, 5])
@pytest.mark.parametrize("prec,grid_n", [("fp64", 64), ("fp32", 128)])
def test_replay_with_other_seeds(prec, grid_n, sort_every):
    """A mesh above 4 MiB whose first interval drifts more than 3 cells: the
    untouched species is re-ordered, and sampled again, by the captured steps.
    The seeds differ in their low or in their high words."""
    cfg = workloads.small("c3", grid_n=grid_n, n_side=1, n_steps=12, precision=prec, box_mpc=6.25 * grid_n, z_begin=300.0,
                          z_end=40.0, sort_every=sort_every, sort_cells=0.0)
    cfg["species"] = [dict(field=0, m=0.05, n=20011, n_side=1), dict(field=0, m=0.02, n=3001, n_side=1)]
    plain, graph = fastdf.Context(cfg), fastdf.Context(cfg)
    graph.set_tuning(use_graph=1)
    for seeds in ((31, 1 << 60), (32, 1 << 60), (31, (1 << 60) + 1), (31 + (1 << 40), 1 << 60), (31, 1 << 60)):
        for a, b in zip(_job(graph, cfg, seeds), _job(plain, cfg, seeds)):
            assert np.array_equal(a, b), seeds
    plain.close()
    graph.close()


@pytest.mark.parametrize("tol", [0.0, 0.01])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_density_after_replayed_grid_builds(prec, tol):
    """A step that builds meshes overwrites the last density's buffers: it
    cannot be read afterwards, whether the step was enqueued, captured or
    replayed.  A step that builds none leaves it as it was."""
    cfg = workloads.small("c3", grid_n=16, n_side=9, n_steps=40, precision=prec, box_mpc=400.0, z_begin=1e5,
                          z_end=500.0, sort_every=0, sort_cells=0.0, model="radmat", omega_r=1e-4, superstep_tol=tol)
    ctx = fastdf.Context(cfg)
    ctx.set_tuning(use_graph=1)
    for _ in range(3):   # captured, then replayed
        _, _, species = fastdf.setup_workload(cfg, ctx=ctx, tuning=dict())
        ctx.step(20)
        ctx.power_spectrum(species, 4)
        ctx.read_density(0)
        ctx.step(20)
        with pytest.raises(fastdf.FastDFError):
            ctx.read_density(0)
    ctx.close()
    cfg = dict(cfg, model="poisson", omega_r=0.0, superstep_tol=0.0)
    ctx = fastdf.Context(cfg)
    ctx.set_tuning(use_graph=1)
    for _ in range(3):
        _, _, species = fastdf.setup_workload(cfg, ctx=ctx, tuning=dict())
        ctx.step(20)
        ctx.power_spectrum(species, 4)
        before = ctx.read_density(0)
        ctx.step(20)
        assert np.array_equal(ctx.read_density(0), before)
    ctx.close()


def test_workspace_replaced():
    """Captured steps belong to the workspace they were captured in."""
    cfg = workloads.small("c3", grid_n=16, n_side=9, n_steps=12, precision="fp32", box_mpc=400.0, z_begin=300.0,
                          z_end=40.0, sort_every=5, sort_cells=0.0)
    cfg["species"] = [dict(field=0, m=0.05, n=2011, n_side=1), dict(field=0, m=0.02, n=301, n_side=1)]
    ctx = fastdf.Context(cfg)
    ctx.set_tuning(use_graph=1)
    ref = _job(ctx, cfg, (5, 6))
    first = ctx.workspace                # stays allocated
    ctx.workspace = torch.empty_like(first)
    ctx._check(ctx.lib.fdf_attach_workspace(ctx.ctx, ctypes.c_void_p(ctx.workspace.data_ptr()),
                                            ctx.workspace.numel()), "fdf_attach_workspace")
    held = first.clone()
    for a, b in zip(_job(ctx, cfg, (5, 6)), ref):
        assert np.array_equal(a, b)
    assert torch.equal(first, held)
    ctx.close()
