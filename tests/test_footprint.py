"""Device memory of systems with exact gravity: the partial sums take at most 20 rows
up to 2,500 spheres (tiles of 128), and stay near two rows per 512 spheres beyond,
whatever the pile's tiles and the segments they are cut into (an engine's budget and
the server's admission count them)."""
import math

import pytest

from paper_2311_11322_amd import dem
from paper_2311_11322_amd import workloads as W


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [100, 300, 1000, 2500, 2501, 4201, 6400, 9500, 9501, 13001, 20000, 24000,
                               32000, 45000, 45001, 98304, 98305, 124958, 131072])
def test_rows_of_partial_sums(n, prec):
    p = dict(W.CONTACT_PARAMS, dt=1e-4, G=0.0, soft_frac=0.5)
    plain = dem.footprint_bytes(p, n, n, prec)
    grav = dem.footprint_bytes(dict(p, G=1.0), n, n, prec)
    # ids in both orders, 64-byte records, the force: 96 bytes a sphere
    rows = (grav - plain - 96 * n) / (3 * (4 if prec else 8) * n)
    most = 20 if n <= 2500 else 2 * math.ceil(n / 512) + 8
    assert rows <= most + 1024 / n                           # buffers are rounded to 256 bytes
