"""Species created in spatial order: the state by id is the canonical sample
whatever the order it is kept in, at ragged counts, with and without re-sorts,
and where the temporaries do not fit and the order stays that of the ids."""
import numpy as np
import pytest

from oracle import particles
from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sort_every", [0, 5])
@pytest.mark.parametrize("prec,grid_n", [("fp64", 64), ("fp32", 128)])
@pytest.mark.parametrize("n", [1, 255, 1025, 40001, 2800003])
def test_created_state_is_the_canonical_sample(prec, grid_n, n, sort_every):
    cfg = workloads.small("c3", grid_n=grid_n, n_side=1, n_steps=8, precision=prec, box_mpc=700.0, z_begin=50.0,
                          z_end=30.0, sort_every=sort_every, sort_cells=0.0)
    cfg["species"] = [dict(field=0, m=0.1, n=n, n_side=1, seed=31), dict(field=0, m=0.05, n=513, n_side=1, seed=32)]
    ctx, _, species = fastdf.setup_workload(cfg)
    for sid, sp in zip(species, cfg["species"]):
        x, q = ctx.read_state(sid)
        ids = np.unique(np.linspace(0, sp["n"] - 1, 5000).astype(np.int64))
        assert np.array_equal(x[ids], particles.positions_f64(sp["seed"], ids, cfg["box_mpc"]))
        assert np.abs(q[ids] - particles.momenta_f64(sp["seed"], ids)).max() < 2e-10   # one binary32 rounding of 1e-3
        assert not np.any(ctx.weights(sid).cpu().numpy())
    # a second context whose steps start from another order gives the same states
    ctx.step(8)
    ref = [ctx.read_state(s) for s in species]
    ctx.close()
    cfg["sort_every"] = 3 if sort_every == 0 else 0
    ctx, _, species = fastdf.setup_workload(cfg)
    ctx.step(8)
    for (xa, qa), s in zip(ref, species):
        x, q = ctx.read_state(s)
        assert np.array_equal(x, xa) and np.array_equal(q, qa)
    ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_density_stays_readable_across_reordering(prec):
    """Re-orders in place work in the FFT scratch and leave the last density alone."""
    cfg = workloads.small("c3", grid_n=128, n_side=64, n_steps=40, precision=prec, box_mpc=500.0, z_begin=300.0,
                          z_end=20.0, sort_every=0, sort_cells=0.0)
    ctx, _, species = fastdf.setup_workload(cfg)
    ctx.step(4)
    ctx.power_spectrum(species, 8)
    before = [ctx.read_density(h) for h in (0, 1)]
    ctx.timing()
    ctx.step(36)
    assert ctx.read_timing("sort")[1] >= 2
    for h in (0, 1):
        assert np.array_equal(before[h], ctx.read_density(h))
    ctx.close()


# (precision, interpolation, particles): gathers from which a first order is made
FIRST_ORDER = {("fp32", 1, 2000003): 7, ("fp32", 2, 2000003): 3, ("fp64", 1, 2000003): 5, ("fp64", 2, 2000003): 2,
               ("fp32", 1, 270000): 12, ("fp64", 2, 270000): 3, ("fp32", 1, 3001): 24}


# one launch a call, and a launch a step
MODELS = {"poisson": {}, "radmat": dict(model="radmat", omega_r=1e-4)}


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("given", [True, False])
@pytest.mark.parametrize("prec,order,n", sorted(FIRST_ORDER))
def test_order_in_place_waits_for_a_call_that_repays_it(prec, order, n, given, model):
    """A context without re-sorts: calls too short to repay a first order in
    place, of particles given by the caller or of a species whose order at
    creation its first interval's drift outruns, leave it to the next call; the
    states are those of a context that never orders them.  A call of k steps
    makes k + 1 gathers."""
    pays = FIRST_ORDER[prec, order, n]
    calls = [([pays - 1], 1), ([pays + 1], 1), ([pays - 2], 0), ([1, 1], 1), ([1, -1], int(given or pays <= 2))]
    cfg = workloads.small("c3", grid_n=128, n_side=1, n_steps=26, precision=prec, box_mpc=2000.0, z_begin=1e4,
                          z_end=2e3, sort_every=0, sort_cells=0.0, interp_order=order, **MODELS[model])
    if not given:
        cfg.update(box_mpc=5760.0, z_begin=100.0, z_end=17.0)   # a third of a cell a step
    cfg["species"] = [dict(field=0, m=0.05, n=n, n_side=1)]
    xu, q = workloads.hand_placed(n, 2000.0)
    contexts = [fastdf.Context(dict(cfg, sort_every=sort_every)) for sort_every in (0, 1)]
    contexts[1].set_tuning(sort_every=0)
    for steps, sorts in calls:
        if 0 in steps:
            continue
        out = []
        for ctx in contexts:
            ctx.reset()
            fid = ctx.add_field(cfg["fields"][0])
            sid = ctx.set_species_state(fid, 0.05, xu, q) if given else ctx.init_species(fid, 0.05, n, 9)
            ctx.timing()
            ctx.timing_reset()
            for k in steps:
                ctx.step(k)
            out.append(ctx.read_state(sid) + (ctx.read_timing("sort")[1],))
        (xa, qa, first), (xb, qb, none) = out
        assert np.array_equal(xa, xb) and np.array_equal(qa, qb)
        assert none == 0 and min(first, 1) == sorts, steps
    for ctx in contexts:
        ctx.close()
