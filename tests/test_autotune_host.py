"""The autotuner times only the launch parameters that a workload's launches
follow, and the saved tunings hold no others (CPU: the runs are stubbed)."""
import os
import re

import pytest

from paper_2207_14256_amd import autotune, fastdf, workloads

CSRC = os.path.join(os.path.dirname(os.path.abspath(autotune.__file__)), "csrc")


class _Context:
    def __init__(self, cfg):
        pass

    def close(self):
        pass


def _timed(cfg, monkeypatch, tmp_path):
    """Tunings that a full autotune of cfg times."""
    runs = []

    def run(ctx, cfg, tuning, steps):
        runs.append(dict(tuning))
        return dict(wall_s=1.0, push_ms=1.0, push_total_ms=1.0 + len(runs), sort_ms=0.0, sorts=0)

    monkeypatch.setattr(fastdf, "Context", _Context)
    monkeypatch.setattr(autotune, "_run", run)
    autotune.autotune(cfg, path=str(tmp_path / "cache.json"), log=lambda m: None)
    return runs


def _preset(name, **kw):
    cfg = workloads.preset(name)
    cfg.update(kw)
    return cfg


@pytest.mark.parametrize("name,kw,ppts,caps,sort_ppts", [
    # constant potentials, CIC: launches of several steps, whose shape is fixed
    ("c3", {}, {4}, {0}, {1}), ("c4", {}, {4}, {0}, {1}), ("c5", {}, {4}, {0}, {1}), ("c2", {}, {4}, {0}, {1}),
    ("c3", dict(precision="fp64"), {4}, {0}, {1}),
    ("c3", dict(model="radmat", superstep_tol=0.01), {4}, {0}, {1}),
    # meshes rebuilt at every step: launches of one step
    ("c3", dict(model="radmat"), {1, 2, 4, 8}, {0, 2, 3, 4}, {1, 2, 4}),
    ("c3", dict(model="radmat", sort_every=0), {1, 2, 4, 8}, {0, 2, 3, 4}, {1}),
    ("c2", dict(model="radmat"), {4}, {0, 2, 3, 4}, {1}),
    # TSC and the other equations of motion: blocks of 256 over several steps
    ("c3", dict(interp_order=2), {1, 2, 4, 8}, {0, 2, 3, 4}, {1}),
    ("c3", dict(eom="exact"), {4}, {0, 2, 3, 4}, {1}),
    # too few particles for blocks of 1024, or for several per thread
    ("c1", {}, {4}, {0, 2, 3, 4}, {1}),
])
def test_only_parameters_that_act_are_timed(name, kw, ppts, caps, sort_ppts, monkeypatch, tmp_path):
    runs = _timed(_preset(name, **kw), monkeypatch, tmp_path)
    assert {t["particles_per_thread"] for t in runs} == ppts
    assert {t["push_waves"] for t in runs} == caps
    assert {t["sort_push_ppt"] for t in runs} == sort_ppts


@pytest.mark.parametrize("name,kw", [("c3", {}), ("c3", dict(precision="fp64")), ("c4", {}), ("c5", {})])
def test_saved_tunings_hold_no_idle_parameter(name, kw):
    cfg = _preset(name, **kw)
    key = re.sub("^[^|]*", "gfx950", autotune.cache_key(cfg))
    tuning = autotune.load_cache()[key]
    ppts, caps, sort_ppts = autotune.launch_shapes(cfg)
    assert tuning["particles_per_thread"] in ppts and tuning["push_waves"] in caps
    assert tuning.get("sort_push_ppt", 1) in sort_ppts


def test_planning_constants():
    """launch_shapes repeats the launch planning's numbers."""
    host = open(os.path.join(CSRC, "fdf_host.cpp")).read()
    internal = open(os.path.join(CSRC, "fdf_internal.h")).read()
    assert "kMinPushBlocks = 2048;" in host and "total >= 256 * kPushWideBlock" in host
    assert "kPushBlock = 256, kPushWideBlock = 1024;" in internal
