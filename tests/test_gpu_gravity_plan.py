"""The exact sum's pair blocks at the edges of their plan: sizes at which the tile
changes (128, 192, 256, 512, 768, 1024 slots), at which a source tile is cut into
segments or not, short last tiles (waves and segments without sources), and given
tiles of small piles (cut in halves and quarters).  Against the sum over every other
sphere in float64; and a pile in an engine of others, bit for bit as alone."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


def _pile(n):
    rng = np.random.default_rng(n)
    side = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)[:n]
    pos = 2.6 * g + rng.uniform(-0.2, 0.2, (n, 3))
    rad = rng.uniform(0.8, 1.0, n)
    return pos, rad, W.sphere_mass(rad)


def _sim(D, n, prec, tile=0, soft=0.5):
    pos, rad, mass = _pile(n)
    prm = dict(W.CONTACT_PARAMS, dt=1e-4, G=0.7, soft_frac=soft, periodic=0, box=(0.0, 0.0, 0.0))
    sim = D.Sim(prm, precision=prec)
    sim.set_tuning(gravity_tile=tile, fused=2)
    return sim.add_aggregates(np.ones(n, np.int32), pos, rad, mass)


def _exact(n, soft, idx):
    import torch
    pos, rad, mass = [torch.from_numpy(a).cuda() for a in _pile(n)]
    out = []
    for a in range(0, len(idx), 256):
        i = torch.from_numpy(idx[a:a + 256]).cuda()
        d = pos[None, :, :] - pos[i, None, :]
        d2 = (d * d).sum(2)
        eps = 0.5 * soft * (rad[None, :] + rad[i, None])
        w = torch.where(d2 > 0, mass[None, :] * (d2 + eps * eps) ** -1.5, 0.0)
        out.append(0.7 * (w[:, :, None] * d).sum(1))
    return torch.cat(out).cpu().numpy()


# tile 0: the plan's.  In FP32 12,000 and 16,000 are cut in halves as sources, 15,361 and
# 18,000 are not; in FP64 11,265 to 18,432 are cut in halves as targets (11,777: the last
# has a half); 9,700, 18,433 and 24,001 end on a tile of which some waves have no source
CASES = [(129, 0), (2500, 0), (2501, 0), (4200, 0), (4201, 0), (8000, 0), (8001, 0), (9500, 0),
         (9700, 0), (11264, 0), (11265, 0), (11777, 0), (12000, 0), (15361, 0), (16000, 0), (18000, 0),
         (18432, 0), (18433, 0), (24001, 0), (45000, 0), (45001, 0), (98304, 0), (98305, 0),
         (70, -1), (513, -1), (1025, -1), (2600, -1), (5200, -1), (11400, -1)]


@pytest.mark.parametrize("soft", [0.0, 0.5])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,tile", CASES)
def test_sum_at_the_plan_s_edges(D, n, tile, prec, soft):
    print("[case] pair blocks", n, tile, prec, soft, flush=True)
    # every slot of small piles, and a sample of the large ones
    idx = np.arange(n) if n <= 2600 else np.sort(np.random.default_rng(1).choice(n, 1500, replace=False))
    want = _exact(n, soft, idx)
    for t in ([0] if tile == 0 else D.gravity_tiles(prec)):
        sim = _sim(D, n, prec, int(t), soft)
        got = sim.read_state(["agg_acc"])["agg_acc"][idx]
        sim.close()
        # the repository's bars: 1e-12 of the largest (FP64), 1e-5 (FP32 pairs)
        assert np.abs(got - want).max() <= (1e-12 if prec == 0 else 1e-5) * np.abs(want).max(), t


@pytest.mark.parametrize("prec", [0, 1])
def test_cut_and_uncut_piles_in_one_engine(D, prec):
    print("[case] pair blocks in an engine", prec, flush=True)
    sizes = [12000, 300, 18000, 3000, 16000, 6000]
    fields = ("agg_pos", "agg_vel", "sph_force")
    alone = []
    for n in sizes:
        s = _sim(D, n, prec)
        s.step(3)
        alone.append(s.read_state(fields))
        s.close()
    eng = D.Engine(1 << 34)
    sims = [_sim(D, n, prec) for n in sizes]
    for s in sims:
        eng.attach(s)
    assert eng.step(3) == D.DEM_OK
    for s, a in zip(sims, alone):
        b = s.read_state(fields)
        assert all(np.array_equal(a[k], b[k]) for k in fields)


@pytest.mark.parametrize("n", [11265, 13001, 16000])
@pytest.mark.parametrize("prec", [0, 1])
def test_whole_and_halved_blocks_give_the_same_bits(D, prec, n):
    """A pile alone takes its tiles as targets in halves, in a launch that is full
    without in whole tiles."""
    print("[case] whole and halved blocks", prec, n, flush=True)
    fields = ("agg_pos", "agg_vel", "sph_force")
    a = _sim(D, n, prec)
    a.step(2)
    want = a.read_state(fields)
    a.close()
    eng = D.Engine(1 << 38)
    sims = [_sim(D, n if k % 3 else 20000, prec) for k in range(36)]
    for s in sims:
        eng.attach(s)
    assert eng.step(2) == D.DEM_OK
    for k in (1, 35):
        got = sims[k].read_state(fields)
        assert all(np.array_equal(want[f], got[f]) for f in fields)
    eng.detach(sims[1])
    sims[1].step(1)
    b = _sim(D, n, prec)
    b.step(3)
    x, y = b.read_state(fields), sims[1].read_state(fields)
    assert all(np.array_equal(x[f], y[f]) for f in fields)
