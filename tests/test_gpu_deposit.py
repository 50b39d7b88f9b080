"""Deposit through the line table: the density of an integrated state against
the oracle's deposit of the same state (read back), at counts around a block,
on meshes where the table holds every line and where it overflows."""
import numpy as np
import pytest

from oracle import background, pipeline, stats
from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["cross", "auto"])
@pytest.mark.parametrize("n", [2, 255, 257, 1023, 1024, 1025, 6001, 131071, 131073])
@pytest.mark.parametrize("prec,grid_n", [("fp64", 8), ("fp64", 64), ("fp32", 8), ("fp32", 64)])
def test_density_matches_oracle_deposit(prec, grid_n, n, mode):
    cfg = workloads.small("c3", grid_n=grid_n, n_side=1, n_steps=6, precision=prec, box_mpc=600.0, z_begin=60.0,
                          z_end=30.0, sort_every=3, sort_cells=0.0)
    cfg["species"] = [dict(field=0, m=0.1, n=n, n_side=1, seed=41)]
    ctx, _, species = fastdf.setup_workload(cfg)
    ctx.step(6)
    k, p, nm = ctx.power_spectrum(species, 4, mode)
    x, q = ctx.read_state(species[0])
    w = ctx.weights(species[0]).cpu().numpy()
    a = pipeline.schedule(cfg)["a"][-1]
    eps, mean_eps = stats.energies(q, 0.1, a), background.mean_energy(0.1, a)
    halves = [np.arange(n)] if mode == "auto" else [np.arange(0, n, 2), np.arange(1, n, 2)]
    ref = [stats.density_contrast(x[h], w[h], eps[h], grid_n, 600.0, len(h), mean_eps) for h in halves]
    top = max(np.abs(r).max() for r in ref)
    # binary64 sums in another order, or (FP32) one rounding to binary32 per cell
    tol = 1e-12 if prec == "fp64" else 2.0 ** -23
    for h, r in enumerate(ref):
        assert np.abs(ctx.read_density(h) - r).max() <= tol * top
    ref_p = stats.binned_power(ref[0], ref[-1], 600.0, 4)
    assert np.array_equal(nm, ref_p[2])
    sel = nm > 0
    # the spectrum inherits the density's rounding (and that of a binary32 FFT)
    scale = np.abs(stats.binned_power(ref[0], ref[0], 600.0, 4)[1][sel]).max()
    assert np.abs(p - ref_p[1])[sel].max() <= (1e-10 if prec == "fp64" else 1e-4) * scale
    ctx.close()


@pytest.mark.parametrize("n", [64000, 140001])
def test_fp32_spectra_do_not_depend_on_the_order(n):
    """Particles in the order of their ids (a context without re-sorts on a
    mesh that the L2 holds): a deposit block touches more lines than its table
    holds, and part of its contributions takes the mesh atomics directly.  The
    spectra are those of sorted particles, bit for bit."""
    cfg = workloads.small("c3", grid_n=32, n_side=1, n_steps=40, box_mpc=600.0, z_begin=100.0, z_end=10.0,
                          sort_every=0, sort_cells=0.0)
    cfg["species"] = [dict(field=0, m=0.1, n=n, n_side=1, seed=41)]
    out = []
    for sort_every in (0, 3):
        ctx, _, species = fastdf.setup_workload(dict(cfg, sort_every=sort_every))
        ctx.timing()
        ctx.step(40)
        assert (ctx.read_timing("sort")[1] > 0) == (sort_every > 0)
        out.append([v for mode in ("cross", "auto") for quantity in ("density", "momentum")
                    for v in ctx.power_spectrum(species, 20, mode, quantity)])
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True)
