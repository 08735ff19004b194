"""Steps that fail inside a call of many steps -- too many contacts, an overlap above
the limit -- in each route of a step: the pair search and the cells of the
one-workgroup step (up to 64 steps a launch), its two parts around gravity, staged
steps eight to a graph launch, and staged steps with gravity beside the contacts
(with and without a perturber).  The state is that at the start of the failing
step, bit for bit, and the run goes on from there like one that did not fail."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("agg_pos", "agg_vel", "agg_acc", "agg_torque", "agg_quat", "agg_spin_body")
ROUTES = {                   # spheres, G, tuning, perturber
    "pairs": (200, 0.0, {}, False),
    "pairs_most": (448, 0.0, dict(fused=1), False),
    "cells": (500, 0.0, dict(fused=1), False),
    "parts": (200, 1.0, {}, False),
    "parts_perturber": (200, 1.0, {}, True),
    "staged": (3000, 0.0, {}, False),
    "staged_large": (40000, 0.0, {}, False),
    "gravity": (3000, 1.0, {}, False),
    "gravity_perturber": (3000, 1.0, {}, True),
    "gravity_target": (3000, 1.0, dict(gravity_form=2), True),
}


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


def _sim(D, route, prec, **kw):
    """A lattice of single spheres, not yet touching, that contracts."""
    n, G, tune, pert = ROUTES[route]
    rng = np.random.default_rng(n)
    side = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)[:n]
    pos = 2.004 * (g - 0.5 * (side - 1)) + rng.uniform(-5e-4, 5e-4, (n, 3))
    prm = dict(W.CONTACT_PARAMS, dt=1e-4, G=G, soft_frac=0.5, periodic=0, box=(0.0, 0.0, 0.0))
    sim = D.Sim(prm, precision=prec, **kw)
    sim.set_tuning(**tune)
    if pert:
        sim.set_forcing(0.0, 10.0 * n, (30.0 * side, 0.0, 0.0), (0.0, 5.0, 0.0))
    return sim.add_aggregates(np.ones(n, np.int32), pos, np.ones(n), np.ones(n), -0.8 * pos,
                              rng.normal(0.0, 0.1, (n, 3)))


def _state(sim):
    st = sim.read_state(FIELDS, pairs=True)
    f = sim.get_forcing()
    return dict(st, pert_pos=f["pert_pos"], pert_vel=f["pert_vel"])


def _equal(a, b):
    for k in b:
        assert np.array_equal(a[k], b[k]), k


def _fail(D, sim, code):
    with pytest.raises(D.DemError) as ei:
        for _ in range(6):
            sim.step(37)
    assert ei.value.code == code
    assert sim.status() == code
    st = _state(sim)
    assert f"step {st['step']};" in str(ei.value)
    with pytest.raises(D.DemError):
        sim.step(1)
    _equal(_state(sim), st)
    return st


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("route", list(ROUTES))
def test_too_many_contacts(D, route, prec):
    print("[case] too many contacts", route, prec, flush=True)
    sim, ref = _sim(D, route, prec, max_contacts=1), _sim(D, route, prec, max_contacts=16)
    st = _fail(D, sim, D.DEM_ERR_CAPACITY)
    n = ROUTES[route][0]
    assert st["step"] > 0 and st["n_pairs"] <= n
    ref.step(st["step"])
    _equal(_state(ref), st)
    sim.reserve_contacts(16)
    sim.step(21)
    ref.step(21)
    got = _state(sim)
    assert got["n_pairs"] > n
    _equal(got, _state(ref))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("route", list(ROUTES))
def test_overlap_limit(D, route, prec):
    print("[case] overlap limit", route, prec, flush=True)
    sim, ref = _sim(D, route, prec, max_overlap_frac=1e-3), _sim(D, route, prec)
    st = _fail(D, sim, D.DEM_ERR_UNSTABLE)
    assert st["step"] > 0 and st["n_pairs"] > 0
    ref.step(st["step"])
    _equal(_state(ref), st)

    def deepest():
        r = ref.read_state(["sph_pos"], pairs=True)
        i, j = (r["pair_keys"] >> np.uint64(32)).astype(int), (r["pair_keys"] & np.uint64(0xffffffff)).astype(int)
        return float((2.0 - np.linalg.norm(r["sph_pos"][i] - r["sph_pos"][j], axis=1)).max())

    assert deepest() <= 1e-3
    ref.step(1)
    assert deepest() > 1e-3
