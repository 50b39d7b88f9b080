"""Every launch shape of the pushes at counts where it is really taken: more
particles per thread need more than 2048 blocks of them, blocks of 1024 threads
262 144 particles and several steps.  States by id do not depend on the shape,
bit for bit."""
import numpy as np
import pytest

from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu

# constant potentials with 6 and 4 slots, super-steps with 8 and 4
FORMS = {"slots6": dict(slip_amp=0.01), "slots4": dict(slip_amp=0.0),
         "super8": dict(slip_amp=0.01, model="radmat", omega_r=1e-4, superstep_tol=0.05),
         "super4": dict(slip_amp=0.0, model="radmat", omega_r=1e-4, superstep_tol=0.05)}


def _cfg(form, prec, order, counts):
    cfg = workloads.small("c3", grid_n=64, n_side=1, n_steps=30, precision=prec, box_mpc=1000.0, z_begin=1e4,
                          z_end=3e3, sort_every=1, sort_cells=0.0, interp_order=order, **FORMS[form])
    cfg["species"] = [dict(field=0, m=0.1 / (i + 1), n=n, n_side=1, seed=70 + i) for i, n in enumerate(counts)]
    return cfg


def _run(cfg, steps, **tuning):
    ctx, _, species = fastdf.setup_workload(cfg, tuning=tuning)
    ctx.timing()
    ctx.step(steps)
    states = [v for s in species for v in ctx.read_state(s)]
    launches = [ctx.read_timing(k)[1] for k in ("push", "push_sort")]
    ctx.close()
    return states, launches


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_particles_per_thread(form, order):
    """8 per thread needs 8 x 2048 x 256 particles: one-step launches with 1,
    2, 4 and 8 per thread, plain and re-sorting, against launches of several
    steps."""
    n = 8 * 2048 * 256 + 517
    cfg = _cfg(form, "fp32", order, [n])
    ref, (plain, fused) = _run(cfg, 4, sort_every=0)
    assert plain < 4 and fused == 0
    for ppt in (1, 2, 4, 8):
        got, (plain, fused) = _run(cfg, 4, sort_every=1, sort_fused=0, particles_per_thread=ppt)
        assert plain == 4 and fused == 0    # three steps, and one with the closing kick
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), ppt
    for ppt in (1, 2, 4):
        got, (plain, fused) = _run(cfg, 4, sort_every=1, sort_push_ppt=ppt)
        assert plain == 1 and fused == 3
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), ppt
    # several steps, TSC (blocks of 256): the particles per thread asked for
    for ppt in (2, 8):
        got, _ = _run(cfg, 4, sort_every=0, particles_per_thread=ppt, push_waves=3)
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), ppt


@pytest.mark.parametrize("counts", [(262144 + 513,), (262144, 1, 1025)])
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_wide_blocks(form, prec, order, counts):
    """Launches of several steps above 262 144 particles (blocks of 1024
    threads with CIC) against one-step launches (blocks of 256), with and
    without re-sorts, in one call and in two, and walked back."""
    cfg = _cfg(form, prec, order, counts)
    one, launches = _run(cfg, 26, sort_every=1, sort_fused=0)
    assert launches == [26, 0]
    many, launches = _run(cfg, 26, sort_every=0)
    assert launches[0] < 20
    for a, b in zip(many, one):
        assert np.array_equal(a, b)
    sorting, _ = _run(cfg, 26, sort_every=9)
    for a, b in zip(sorting, one):
        assert np.array_equal(a, b)
    persistent, _ = _run(cfg, 26, sort_every=0, persistent_blocks=64)
    for a, b in zip(persistent, one):
        assert np.array_equal(a, b)
