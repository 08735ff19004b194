"""State read-out: the fields and contacts gathered on the device.  All fields
at once (in pieces of the staging buffer, of which the orientations of single
spheres fill one exactly), each field alone, small (copied together) and large
(copied one by one), and against what the fields must satisfy."""
import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,members", [(1, 1), (2, 2), (257, 1), (1100, 3), (20000, 1), (20001, 4)])
def test_readout(n, members):
    from paper_2311_11322_amd import dem
    print("[case] read-out", n, members, flush=True)
    rng = np.random.default_rng(n)
    side = int(np.ceil(n ** (1.0 / 3.0)))
    pos = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)[:n]
    pos = 2.0 * pos + rng.uniform(-2e-4, 2e-4, pos.shape)
    rad = np.full(n, 1.0 + 5e-4)
    counts = np.full(n // members, members, np.int32)
    counts[0] += n - counts.sum()
    na = len(counts)
    prm = dict(W.CONTACT_PARAMS, dt=1e-4, G=1e-3, soft_frac=0.5, periodic=0, box=(0.0, 0.0, 0.0))
    sim = dem.Sim(prm)
    sim.add_aggregates(counts, pos, rad, W.sphere_mass(rad), rng.normal(0, 0.05, (na, 3)),
                       rng.normal(0, 0.05, (na, 3)))
    sim.step(3)
    st = sim.read_state(pairs=True)
    for k in st:
        if isinstance(st[k], np.ndarray) and not k.startswith("pair"):
            assert np.array_equal(sim.read_state([k])[k], st[k]), k
    # space-frame spins, rounded product by product
    w, x, y, z = st["agg_quat"].T
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                  2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                  2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1)
    o = st["agg_spin_body"]
    spin = np.stack([(R[:, 3 * c] * o[:, 0] + R[:, 3 * c + 1] * o[:, 1]) + R[:, 3 * c + 2] * o[:, 2]
                     for c in range(3)], 1)
    assert np.array_equal(st["agg_spin"], spin)
    # contacts in canonical order, of touching spheres of different aggregates
    keys = st["pair_keys"]
    assert len(keys) == st["n_pairs"] == len(st["pair_hist"])
    assert (np.diff(keys.astype(np.int64)) > 0).all()
    agg = np.repeat(np.arange(na), counts)
    i, j = (keys >> np.uint64(32)).astype(int), (keys & np.uint64(0xffffffff)).astype(int)
    assert (agg[i] != agg[j]).all() and (n < 257 or len(keys) > n // 2)
    d = np.linalg.norm(st["sph_pos"][i] - st["sph_pos"][j], axis=1)
    assert (d < rad[i] + rad[j] + 1e-12).all()
    # a restored copy reads the same
    ck = sim.checkpoint()
    sim.restore(ck)
    again = sim.checkpoint()
    for k in ck:
        assert np.array_equal(ck[k], again[k]), k
    sim.close()
