"""The number of contacts that the stateless searches report when their lists are
full: the total found, as on success.  Simple cubic lattices, whose pairs within a
distance are counted offset by offset, in more blocks than the chip holds at once
(the lists are full long before the last block starts), and a boulder with more
partners than its run holds."""
import ctypes as C
import math

import numpy as np
import pytest

from paper_2311_11322_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    from paper_2311_11322_amd import dem
    dem.lib()
    return dem


def _lattice(side, seed):
    """Sites 0 .. side - 1 cubed in random order (distances are exact)."""
    g = np.stack(np.meshgrid(*3 * (np.arange(side, dtype=np.float64),), indexing="ij"), -1)
    return np.ascontiguousarray(g.reshape(-1, 3)[np.random.default_rng(seed).permutation(side ** 3)])


def _pairs_within(side, d2max):
    """Unordered pairs of sites with a squared distance below d2max."""
    r = int(math.sqrt(d2max)) + 1
    k = np.arange(-r, r + 1)
    x, y, z = np.meshgrid(k, k, k, indexing="ij")
    hit = (x * x + y * y + z * z < d2max) & ((x != 0) | (y != 0) | (z != 0))
    n = [np.maximum(0, side - np.abs(a[hit])) for a in (x, y, z)]
    return int((n[0] * n[1] * n[2]).sum()) // 2


@pytest.mark.parametrize("side", [27, 40])
def test_noalloc_total_beyond_its_lists(D, side):
    """19,683 and 64,000 spheres (eight lanes a sphere and one) with more than
    1,048,576 contacts; a search that fits follows."""
    import torch
    print("[case] noalloc total", side, flush=True)
    d2 = 16.5 if side == 27 else 5.5
    pos = _lattice(side, 1)
    n = len(pos)
    want = _pairs_within(side, d2)
    assert want > 1 << 20
    dev = (torch.from_numpy(pos).cuda(), torch.full((n,), 0.5 * math.sqrt(d2), dtype=torch.float64, device="cuda"),
           torch.arange(n, dtype=torch.int32, device="cuda"))
    out = torch.full((64,), -1, dtype=torch.int64, device="cuda")
    nout = C.c_int64(-1)
    code = D.lib().dem_find_contacts_noalloc(
        *[C.c_void_p(t.data_ptr()) for t in dev], n, None, C.c_void_p(out.data_ptr()), 64,
        C.byref(nout), D.torch_stream())
    assert code == D.DEM_ERR_CAPACITY
    assert nout.value == want
    assert bool((out == -1).all())
    rad = torch.full((n,), 0.5 * math.sqrt(1.5), dtype=torch.float64, device="cuda")
    assert D.find_contacts_noalloc(dev[0], rad, dev[2]) == _pairs_within(side, 1.5)


@pytest.mark.parametrize("side", [30, 74])
def test_search_total_beyond_its_lists(D, side):
    print("[case] search total", side, flush=True)
    d2 = 16.5
    pos = _lattice(side, 2)
    n = len(pos)
    want = _pairs_within(side, d2)
    assert want > 64 * n
    rad, agg = np.full(n, 0.5 * math.sqrt(d2)), np.arange(n, dtype=np.int32)
    keys = np.zeros(16, np.uint64)
    nout = C.c_int64(-1)
    code = D.lib().dem_find_contacts(D._p(pos), D._p(rad), D._p(agg, D._PI32), n, None,
                                     D._p(keys, D._PU64), 16, C.byref(nout))
    assert code == D.DEM_ERR_CAPACITY
    assert nout.value == want


@pytest.mark.parametrize("boulder,per_sphere,side", [(False, 16, 74), (True, 16, 30), (True, 1, 30)])
def test_contact_forces_total_beyond_its_lists(D, boulder, per_sphere, side):
    """Lists too short, a boulder's run too long (more than 2,048), and both."""
    print("[case] contact forces total", boulder, per_sphere, side, flush=True)
    d2 = 5.5 if not boulder else 1.5
    pos, rad = _lattice(side, 3), np.full(side ** 3, 0.5 * math.sqrt(d2))
    want = _pairs_within(side, d2)
    if boulder:
        centre, R = np.full(3, 0.5 * side + 0.25), 8.5
        touch = int((((pos - centre) ** 2).sum(1) < (R + rad[0]) ** 2).sum())
        assert touch > 2048
        want += touch
        pos, rad = np.concatenate([centre[None], pos]), np.append(R, rad)
    n = len(pos)
    assert boulder or want > per_sphere * n
    prm = D.make_params(dict(W.CONTACT_PARAMS, dt=1e-4, G=0.0), max_contacts=per_sphere)
    z, agg, mass = np.zeros((n, 3)), np.arange(n, dtype=np.int32), np.ones(n)
    F, T = np.zeros((n, 3)), np.zeros((n, 3))
    nout = C.c_int64(-1)
    code = D.lib().dem_contact_forces(
        C.byref(prm), n, D._p(pos), D._p(z), D._p(rad), D._p(agg, D._PI32), n, D._p(mass), D._p(z),
        0, None, None, D._p(F), D._p(T), None, None, 0, C.byref(nout))
    assert code == D.DEM_ERR_CAPACITY
    assert nout.value == want
