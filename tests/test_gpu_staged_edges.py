"""Edges of the staged step's launches: gravity tiles and source segments (sizes
at which the plan, a tile or a segment changes, plain and softened, given tiles),
aggregates whose members lie in several blocks, groups of spheres with more
contacts than threads, the first step after a restore (cells worked out anew
instead of carried), and piles whose reduction ends the step or does not (64
blocks of aggregates)."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("agg_pos", "agg_vel", "agg_acc", "agg_torque", "agg_quat", "agg_spin_body", "sph_force")


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


def _params(**kw):
    return dict(W.CONTACT_PARAMS, dt=1e-4, G=0.0, soft_frac=0.5, periodic=0, box=(0.0, 0.0, 0.0), **kw)


def _grid(n, spacing, rng, noise):
    side = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)[:n]
    return spacing * g + rng.uniform(-noise, noise, (n, 3))


# -- gravity: sums over every other sphere, directly in float64 ----------------

@pytest.mark.parametrize("soft", [0.0, 0.5])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,tile", [(1, 0), (2, 0), (63, 0), (65, 0), (257, 0), (1500, 0), (1501, 0),
                                    (4500, 0), (4501, 0), (8001, 0), (24000, 0), (24001, 0),
                                    (40001, 0), (2049, -1), (9000, -1)])
def test_gravity_plan(D, n, tile, prec, soft):
    import torch
    print("[case] gravity plan", n, tile, prec, soft, flush=True)
    rng = np.random.default_rng(n)
    pos, rad = _grid(n, 2.6, rng, 0.2), rng.uniform(0.8, 1.0, n)
    mass = W.sphere_mass(rad)
    t = [torch.from_numpy(a).cuda() for a in (pos, rad, mass)]
    want = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
    for a in range(0, n, 1024):
        d = t[0][None, :, :] - t[0][a:a + 1024, None, :]
        eps = 0.5 * soft * (t[1][None, :] + t[1][a:a + 1024, None])
        r2 = (d * d).sum(2) + eps * eps
        w = torch.where((d * d).sum(2) > 0, t[2][None, :] * r2 ** -1.5, 0.0)
        want[a:a + 1024] = 0.7 * (w[:, :, None] * d).sum(1)
    want = want.cpu().numpy()
    for tl in ([0] if tile == 0 else D.gravity_tiles(prec)):
        prm = _params()
        prm.update(G=0.7, soft_frac=soft)
        sim = D.Sim(prm, precision=prec)
        sim.set_tuning(gravity_tile=int(tl), fused=2)
        sim.add_aggregates(np.ones(n, np.int32), pos, rad, mass)
        got = sim.read_state(["agg_acc"])["agg_acc"]
        sim.close()
        scale = np.abs(want).max()
        assert np.abs(got - want).max() <= (1e-12 if prec == 0 else 1e-5) * max(scale, 1e-300), tl


# -- aggregates over block edges, and many contacts per group ------------------

def _clumps(sizes, rng, radius):
    """Clumps of consecutive spheres of a lattice; neighbours of other clumps
    overlap."""
    n = int(sum(sizes))
    return (np.array(sizes, np.int32), _grid(n, 2.0, rng, 1e-4),
            np.full(n, radius) + rng.uniform(-1e-4, 1e-4, n))


@pytest.mark.parametrize("sizes,radius", [([255, 1, 256, 257], 1.001), ([300, 700, 3, 24], 1.001),
                                          ([1] * 64 + [513] + [2] * 100, 1.001),
                                          ([1] * 700, 1.45), ([2] * 130 + [1], 1.45)])
def test_staged_equals_one_workgroup(D, sizes, radius):
    print("[case] block edges", len(sizes), radius, flush=True)
    rng = np.random.default_rng(len(sizes))
    counts, pos, rad = _clumps(sizes, rng, radius)
    na = len(counts)
    vel, spin = rng.normal(0, 0.02, (na, 3)), rng.normal(0, 0.02, (na, 3))
    out = []
    for fused in (1, 2):
        for prec in (0, 1):
            sim = D.Sim(_params(), precision=prec, max_contacts=32)
            sim.set_tuning(fused=fused)
            sim.add_aggregates(counts, pos, rad, W.sphere_mass(rad), vel, spin)
            sim.step(5)
            out.append(sim.read_state(FIELDS, pairs=True))
            sim.close()
    if radius > 1.4:
        # a group of 64 spheres has more contacts than a block has threads
        assert out[0]["n_pairs"] * 2 * 64 > 256 * len(pos)
    for a, b in ((out[0], out[2]), (out[1], out[3])):
        for k in FIELDS + ("pair_keys", "pair_hist"):
            assert np.array_equal(a[k], b[k]), k


# -- carried cells, and the end of the step ------------------------------------

@pytest.mark.parametrize("n,periodic", [(300, 0), (5000, 0), (5000, 1), (16384, 0), (16385, 1)])
def test_restore_goes_on_bit_identically(D, n, periodic):
    print("[case] restore", n, periodic, flush=True)
    rng = np.random.default_rng(n)
    pos, rad = _grid(n, 2.0, rng, 2e-4) + 1.0, np.full(n, 1.0005)
    prm = _params()
    if periodic:
        prm.update(periodic=1, box=(2.0 * np.ceil(n ** (1 / 3)) + 6.0,) * 3)
    args = (np.ones(n, np.int32), pos, rad, W.sphere_mass(rad), rng.normal(0, 2.0, (n, 3)),
            rng.normal(0, 0.2, (n, 3)))
    a, b = D.Sim(prm), D.Sim(prm)
    for s in (a, b):
        s.set_tuning(fused=2)
        s.add_aggregates(*args)
    a.step(20)
    ck = a.checkpoint()
    assert ck["step"] == 20 and ck["n_pairs"] > n
    a.step(21)
    b.step(3)                            # another state, other cells
    b.restore(ck)
    b.step(1)
    b.step(20)
    x, y = a.read_state(FIELDS, pairs=True), b.read_state(FIELDS, pairs=True)
    assert x["step"] == y["step"] == 41
    for k in FIELDS + ("pair_keys", "pair_hist"):
        assert np.array_equal(x[k], y[k]), k
    a.close()
    b.close()
