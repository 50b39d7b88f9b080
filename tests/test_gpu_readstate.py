"""State read back in id order on meshes of every size: through the FFT scratch
in one or several slices, through the other copy of the state, or array by
array; with and without re-sorts, whole or one half of it, at counts around a
slice; and in a time that does not grow with the square of the count."""
import ctypes
import time

import numpy as np
import pytest

from oracle import particles
from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu


def _context(prec, grid_n, n, sort_every):
    cfg = workloads.small("c3", grid_n=grid_n, n_side=1, n_steps=6, precision=prec, box_mpc=600.0, z_begin=60.0,
                          z_end=30.0, sort_every=sort_every, sort_cells=0.0)
    cfg["species"] = [dict(field=0, m=0.1, n=n, n_side=1, seed=31), dict(field=0, m=0.05, n=777, n_side=1, seed=32)]
    ctx, _, species = fastdf.setup_workload(cfg)
    return ctx, species, cfg


# ids of a slice of the scratch: FP32 16 G^3 / 24, FP64 56 G^3 / 24
@pytest.mark.parametrize("sort_every", [0, 2])
@pytest.mark.parametrize("prec,grid_n,n", [
    ("fp32", 8, 341), ("fp32", 8, 342), ("fp32", 8, 1048579), ("fp32", 16, 2731), ("fp32", 32, 21845),
    ("fp32", 32, 21847), ("fp32", 32, 65539), ("fp64", 8, 1194), ("fp64", 8, 1195), ("fp64", 8, 1048579),
    ("fp64", 16, 9558), ("fp64", 32, 152919), ("fp64", 64, 611671), ("fp32", 128, 1398103)])
def test_state_in_id_order(prec, grid_n, n, sort_every):
    ctx, species, cfg = _context(prec, grid_n, n, sort_every)
    ids = np.unique(np.concatenate([np.arange(300), np.linspace(0, n - 1, 4000).astype(np.int64),
                                    np.arange(max(0, n - 300), n)]))
    ids = ids[ids < n]
    x, q = ctx.read_state(species[0])
    assert np.array_equal(x[ids], particles.positions_f64(31, ids, cfg["box_mpc"]))
    assert np.abs(q[ids] - particles.momenta_f64(31, ids)).max() < 2e-10   # one binary32 rounding of 1e-3
    # an integrated state: the same whether its particles are re-sorted or not,
    # and as one half of it
    ctx.step(6)
    x, q = ctx.read_state(species[0])
    other, others, _ = _context(prec, max(grid_n, 8), n, 0 if sort_every else 2)
    other.step(6)
    xo, qo = other.read_state(others[0])
    assert np.array_equal(x, xo) and np.array_equal(q, qo)
    P = ctypes.POINTER(ctypes.c_double)
    h = np.zeros((n, 3))
    ctx._check(ctx.lib.fdf_read_state(ctx.ctx, species[0], h.ctypes.data_as(P), None), "fdf_read_state")
    assert np.array_equal(h, x)
    ctx._check(ctx.lib.fdf_read_state(ctx.ctx, species[0], None, h.ctypes.data_as(P)), "fdf_read_state")
    assert np.array_equal(h, q)
    # nothing of the context is disturbed
    ctx.step(-3)
    other.step(-3)
    for s, so in zip(species, others):
        for a, b in zip(ctx.read_state(s), other.read_state(so)):
            assert np.array_equal(a, b)
    ctx.close()
    other.close()


@pytest.mark.parametrize("sort_every", [0, 2])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_time_per_particle_on_a_small_mesh(prec, sort_every):
    """1 M particles on 8^3 against the same on 64^3, whose scratch takes
    hundreds of times the ids: at most 4 times as long."""
    took = {}
    for grid_n in (8, 64):
        ctx, species, _ = _context(prec, grid_n, 1 << 20, sort_every)
        ctx.step(6)
        best = 1e9
        for _ in range(4):
            t0 = time.perf_counter()
            ctx.read_state(species[0])
            best = min(best, time.perf_counter() - t0)
        took[grid_n] = best
        ctx.close()
    print("[read] %s %d %s" % (prec, sort_every, took), flush=True)
    assert took[8] < 4 * took[64], took
