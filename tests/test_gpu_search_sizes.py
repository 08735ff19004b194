"""The contact search at the edges of its launches: blocks of 64 and of 256
spheres, the size from which a sphere has one lane instead of eight, and
spheres with more contacts than a run in LDS holds (18 neighbours, 16 ids),
by the allocating search, the one without allocation (after a call that fails)
and a neighbour tree on the host with the same test."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

pytestmark = pytest.mark.gpu


def _lattice(n, dense, seed):
    rng = np.random.default_rng(seed)
    side = int(np.ceil(n ** (1.0 / 3.0)))
    pos = np.stack(np.meshgrid(*3 * (np.arange(side),), indexing="ij"), -1).reshape(-1, 3)
    pos = 2.0 * pos[rng.permutation(side ** 3)[:n]] + 1.0
    pos = pos + rng.uniform(-2e-3, 2e-3, pos.shape)
    rad = np.full(n, 1.45 if dense else 1.0) + rng.uniform(-1e-3, 1e-3, n)
    return pos, rad, rng.integers(0, max(1, n // 2), n).astype(np.int32), max(6.0, 2.0 * side)


def _host(pos, rad, agg, L):
    tree = cKDTree(np.mod(pos, L) if L else pos, boxsize=L or None)
    ij = tree.query_pairs(2.0 * rad.max() * (1 + 1e-9), output_type="ndarray")
    i, j = ij.min(1), ij.max(1)
    d = pos[j] - pos[i]
    if L:
        d = np.where(d > 0.5 * L, d - L, np.where(d < -0.5 * L, d + L, d))
    S = rad[i] + rad[j]
    hit = ((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2] < S * S) & (agg[i] != agg[j])
    return np.sort((i[hit].astype(np.uint64) << np.uint64(32)) | j[hit].astype(np.uint64))


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 256, 257, 2049, 32767, 32768, 65536])
def test_search_sizes(n, periodic, dense):
    import torch
    from paper_2311_11322_amd import dem
    print("[case] search", n, periodic, dense, flush=True)
    pos, rad, agg, L = _lattice(n, dense, n)
    box = (L,) * 3 if periodic else None
    want = _host(pos, rad, agg, L if periodic else 0.0)
    dev = [torch.from_numpy(a).cuda() for a in (pos, rad, agg)]
    out = torch.full((len(want) + 8,), -1, dtype=torch.int64, device="cuda")
    bad = dev[1].clone()
    bad[n // 2] = -1.0
    with pytest.raises(dem.DemError):
        dem.find_contacts_noalloc(dev[0], bad, dev[2], box, out)
    assert bool((out == -1).all())
    assert dem.find_contacts_noalloc(*dev, box, out) == len(want)
    assert np.array_equal(out[:len(want)].cpu().numpy().view(np.uint64), want)
    assert bool((out[len(want):] == -1).all())
    assert dem.find_contacts_noalloc(*dev, box, None) == len(want)
    assert np.array_equal(dem.find_contacts(pos, rad, agg, box), want)
