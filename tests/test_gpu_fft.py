"""The Fourier passes over every line length, layout of slots and precision:
potential meshes against the oracle's transforms of the same modes, a few modes
in closed form on the largest meshes, and the forward direction against the
oracle's spectrum of the density that was transformed."""
import numpy as np
import pytest

from oracle import field as ofield, pipeline, stats
from paper_2207_14256_amd import fastdf, workloads

pytestmark = pytest.mark.gpu


def close(got, ref, G, prec):
    top = np.abs(ref).max()
    if prec == "fp64":
        return np.abs(got - ref).max() <= 1e-12 * top
    # one binary32 rounding per radix-2 level and axis, and bfloat16's 8 significant bits
    return np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 3 * np.log2(G) * 2.0 ** -24 * top)


@pytest.mark.parametrize("model,slip", [("poisson", 0.0), ("poisson", 0.01), ("radmat", 0.01)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("G", [8, 16, 32, 64, 128, 256])
def test_potential_meshes(G, prec, model, slip):
    kw = dict(omega_m=0.9999, omega_r=1e-4) if model == "radmat" else {}
    cfg = workloads.small("c2", grid_n=G, n_side=1, n_steps=100, precision=prec, box_mpc=600.0, slip_amp=slip,
                          model=model, **kw)
    ctx = fastdf.Context(cfg)
    fid = ctx.add_field(cfg["fields"][0])
    ctx.build_potential_grids(fid, 1e-3)
    ref = ofield.potential_grids(ctx.read_field(fid), 600.0, 1e-3, pipeline.model_of(cfg))
    for s in range(3):
        assert close(ctx.read_grid(fid, s), ref["gpsi"][s], G, prec)
    if slip:
        for s in range(3):
            assert close(ctx.read_grid(fid, 3 + s), ref["gphi"][s], G, prec)
    if model == "radmat":
        got = ctx.read_grid(fid, 6)
        assert close(got, ref["phidot"], G, prec) if prec == "fp32" else \
            np.abs(got - ref["phidot"]).max() <= 1e-11 * np.abs(ref["phidot"]).max()
    ctx.close()


@pytest.mark.parametrize("prec,G", [("fp32", 512), ("fp64", 512), ("fp32", 1024)])
def test_plane_waves(prec, G):
    L = 600.0
    cfg = workloads.small("c2", grid_n=G, n_side=1, n_steps=100, precision=prec, box_mpc=L, slip_amp=0.0)
    modes = [((3, -5, 7), 1.0 + 0.5j), ((-G // 2 + 1, 2, G // 2 - 1), 0.25 - 2.0j), ((40, G // 2 - 2, 1), -1.5 + 1.0j)]
    dk = np.zeros((G, G, G // 2 + 1), dtype=np.complex128)
    for n, c in modes:
        dk[n] = c
    ctx = fastdf.Context(cfg)
    fid = ctx.set_field(dk)
    del dk
    ctx.build_potential_grids(fid, 1e-3)
    got = ctx.read_grid(fid, 0)
    ctx.close()
    i = np.arange(G)
    planes = [0, 1, 5, G // 2, G - 1]   # x planes
    ref = np.zeros((len(planes), G, G))
    for n, c in modes:
        k = 2 * np.pi / L * np.array(n, dtype=np.float64)
        t = ofield.potential_transfers(np.array([np.sqrt((k ** 2).sum())]), 1e-3, pipeline.model_of(cfg))[1][0]
        e = [np.exp(2j * np.pi * ((m * i) % G) / G) for m in n]
        # a mode and its complex conjugate
        ref += 2.0 * np.real(1j * k[0] * t * c * e[0][planes][:, None, None] * e[1][None, :, None] * e[2])
    assert close(got[planes], ref, G, prec)


@pytest.mark.parametrize("quantity", ["density", "momentum"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("G", [16, 32, 128, 256])
def test_spectra(G, prec, quantity):
    cfg = workloads.small("c1", grid_n=G, n_side=1, n_steps=4, precision=prec, box_mpc=600.0, z_begin=60.0, z_end=40.0)
    cfg["species"] = [dict(field=0, m=0.1, n=3001, n_side=1, seed=47)]
    ctx, _, species = fastdf.setup_workload(cfg)
    ctx.step(4)
    x, q = ctx.read_state(species[0])
    k, p, nm = ctx.power_spectrum(species, 12, "auto", quantity)
    res = dict(x=x, q=q, w=ctx.weights(species[0]).cpu().numpy())
    if quantity == "density":
        d = ctx.read_density(0)
        kr, pr, nr = stats.binned_power(d, d, 600.0, 12)
    else:
        kr, pr, nr = pipeline.momentum_spectrum(dict(cfg, pk_bins=12), 0, res, "auto", pipeline.schedule(cfg)["a"][-1])
    ctx.close()
    assert np.array_equal(nm, nr)
    sel = nm > 0
    tol = 1e-9 if prec == "fp64" else 1e-4
    assert np.abs(k - kr)[sel].max() <= 1e-12 * kr[sel].max()
    assert np.abs(p - pr)[sel].max() <= tol * np.abs(pr[sel]).max()
