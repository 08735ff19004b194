"""The search of a small pile without gravity (every pair, in one workgroup)
and its several steps per launch, against the staged step with its cells: the
same contacts, history and state bit for bit.  Sizes lie at the edges of the
threads per sphere (448 threads: 64 down to one) and of the largest pile
searched that way; a boulder has more contacts than the LDS lists keep."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("agg_pos", "agg_vel", "agg_acc", "agg_torque", "agg_quat", "agg_spin_body",
          "sph_pos", "sph_force", "sph_torque")


def _system(n, periodic):
    """Unit spheres of a jittered lattice in pairs and singles, neighbours
    overlapping; from 112 spheres on also a boulder with 30 of them on it."""
    rng = np.random.default_rng(n)
    shell = 30 if n >= 112 else 0
    m = n - shell - (1 if shell else 0)
    side = int(np.ceil(m ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)[:m]
    pos = 2.0 * g + 1.0 + rng.uniform(-2e-4, 2e-4, g.shape)
    rad = np.full(m, 1.0 + 5e-4)
    counts = []
    while sum(counts) < m:
        counts.append(min(m - sum(counts), 1 + len(counts) % 2))
    base, height = max(2.0 * side, 17.0), 2.0 * side + 20.0
    if shell:
        k = np.arange(shell) + 0.5
        z, phi = 1 - 2 * k / shell, np.pi * (1 + 5 ** 0.5) * k
        u = np.stack([np.sqrt(1 - z * z) * np.cos(phi), np.sqrt(1 - z * z) * np.sin(phi), z], 1)
        c = np.array([base / 2, base / 2, 2.0 * side + 8.5])
        pos = np.concatenate([pos, c + (7.0 - 1e-3) * u, [c]])
        rad = np.concatenate([rad, np.ones(shell), [6.0]])
        counts += [1] * (shell + 1)
    prm = dict(W.CONTACT_PARAMS, dt=1e-4, G=0.0, soft_frac=0.5, periodic=0, box=(0.0, 0.0, 0.0))
    if periodic:
        prm.update(periodic=1, box=(height,) * 3)
    else:
        prm.update(g=(0.0, 0.0, -2.0), walls=W.open_box_walls(base, base))
    na = len(counts)
    return prm, (np.array(counts, np.int32), pos, rad, W.sphere_mass(rad),
                 rng.normal(0.0, 0.05, (na, 3)), rng.normal(0.0, 0.05, (na, 3)))


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 112, 113, 224, 225, 448, 449])
def test_pairs_equal_cells(n, periodic):
    from paper_2311_11322_amd import dem
    print("[case] pairs vs cells", n, periodic, flush=True)
    prm, args = _system(n, periodic)
    got = []
    for fused in (1, 2):
        sim = dem.Sim(prm, max_contacts=64)
        sim.set_tuning(fused=fused)
        sim.add_aggregates(*args)
        out = [sim.read_state(FIELDS, pairs=True)]
        sim.step(1)
        out.append(sim.read_state(FIELDS, pairs=True))
        sim.step(66)
        out.append(sim.read_state(FIELDS, pairs=True))
        got.append(out)
        sim.close()
    assert got[0][2]["step"] == got[1][2]["step"] == 67
    j = got[0][0]["pair_keys"] & 0xffffffff
    assert n < 112 or (j == n - 1).sum() == 30
    for a, b in zip(*got):
        for k in FIELDS + ("pair_keys", "pair_hist"):
            assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("fused", [1, 2])
@pytest.mark.parametrize("n_steps", [2, 15, 16, 23, 64, 65])
def test_steps_of_one_call(fused, n_steps):
    """However many steps a call takes to a launch, the state is that of as
    many calls of one step."""
    from paper_2311_11322_amd import dem
    print("[case] steps of one call", fused, n_steps, flush=True)
    prm, args = _system(200, False)
    got = []
    for calls in ([n_steps], [1] * n_steps):
        sim = dem.Sim(prm, max_contacts=64)
        sim.set_tuning(fused=fused)
        sim.add_aggregates(*args)
        for n in calls:
            sim.step(n)
        got.append(sim.read_state(FIELDS, pairs=True))
        sim.close()
    assert got[0]["step"] == n_steps
    for k in FIELDS + ("pair_keys", "pair_hist"):
        assert np.array_equal(got[0][k], got[1][k]), k
