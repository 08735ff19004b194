"""The steps that the per-kernel timing covers: every step taken while it is on, the
first one after a restore among them."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


@pytest.mark.parametrize("engine", [False, True])
@pytest.mark.parametrize("graph_order", [False, True])
@pytest.mark.parametrize("gravity", [False, True])
def test_profile_covers_the_step_after_a_restore(D, gravity, graph_order, engine):
    print("[case] profile after restore", gravity, graph_order, engine, flush=True)
    if engine and graph_order:
        pytest.skip("an engine has the one-by-one timing only")
    if gravity:
        w = W.collapse_cloud(seed=3, n_agg=120, cmin=2, cmax=4, phi0=0.3)
    else:
        w = W.periodic_box(seed=3, n_agg=120, contact_seeded=True)
    ref, sim = [D.Sim(w.params) for _ in range(2)]
    for s in (ref, sim):
        s.set_tuning(fused=2)
        s.add_workload(w)
        s.step(2)
    sim.restore(sim.checkpoint())
    eng = D.Engine(1 << 32)
    if engine:
        eng.attach(sim)
    on = eng if engine else sim
    if engine:
        eng.set_profiling(True)
    else:
        sim.set_profiling(True, graph_order)
    for k, total in ((1, 1), (3, 4)):
        on.step(k)
        prof = on.profile()
        assert prof["_steps"] == total
        if not graph_order:
            assert prof["move"] > 0.0 and prof["search"] > 0.0
        if gravity:
            assert prof["gravity"] > 0.0
    ref.step(4)
    a, b = ref.read_state(pairs=True), sim.read_state(pairs=True)
    assert all(np.array_equal(a[k], b[k]) for k in a)
