"""A restored system in an engine: the step after a restore works the cells of every
member out anew, and steps it together with members of every route -- staged with
and without gravity, one workgroup with and without, each carrying its own cells --
which all go on as they do alone, bit for bit.  Large piles in one workgroup, which
take fewer steps a launch, among them."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("agg_pos", "agg_vel", "agg_acc", "agg_torque", "agg_quat", "agg_spin_body")
# spheres, G, fused: staged without gravity (the restored one first), staged with
# gravity, one workgroup by the pair search, by cells and around gravity
MEMBERS = [(3000, 0.0, 2), (5000, 0.0, 2), (2600, 1.0, 2), (97, 0.0, 0), (1500, 0.0, 1),
           (200, 1.0, 0)]


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


def _sim(D, k):
    n, G, fused = MEMBERS[k]
    rng = np.random.default_rng(100 + k)
    side = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)[:n]
    pos = 2.0 * g + rng.uniform(-2e-4, 2e-4, (n, 3))
    prm = dict(W.CONTACT_PARAMS, dt=1e-4, G=G, soft_frac=0.5, periodic=0, box=(0.0, 0.0, 0.0))
    sim = D.Sim(prm)
    sim.set_tuning(fused=fused)
    return sim.add_aggregates(np.ones(n, np.int32), pos, np.full(n, 1.0005), np.ones(n),
                              rng.normal(0.0, 2.0, (n, 3)), rng.normal(0.0, 0.2, (n, 3)))


@pytest.mark.parametrize("steps", [1, 4, 90])
@pytest.mark.parametrize("restored", [0, 2, 3, 4, 5])
def test_restored_member_beside_others(D, restored, steps):
    print("[case] engine restore", MEMBERS[restored], steps, flush=True)
    want, sims = [], []
    for k in range(len(MEMBERS)):
        a = _sim(D, k)
        a.step(10 + steps)
        want.append(a.read_state(FIELDS, pairs=True))
        a.close()
        s = _sim(D, k)
        s.step(10)
        if k == restored:
            ck = s.checkpoint()
            s.step(17)                       # another state, other cells
            s.restore(ck)
        sims.append(s)
    eng = D.Engine(1 << 33)
    for s in sims:
        eng.attach(s)
    assert eng.step(steps) == D.DEM_OK
    for k, s in enumerate(sims):
        got = s.read_state(FIELDS, pairs=True)
        assert got["step"] == 10 + steps and got["n_pairs"] > 0
        for f in FIELDS + ("pair_keys", "pair_hist"):
            assert np.array_equal(got[f], want[k][f]), (MEMBERS[k], f)
