"""The cell search at row lengths and hit counts around the sizes of its parts:
rows of three bins with fewer than 8 and more than 128 candidates, atoms with a
few and with nearly all the hits an LDS row holds (192), a row that wraps on
both sides, against the all-pairs search of the same batch (bit for bit)."""
import numpy as np
import pytest

from test_gpu_cells import build, uniform

pytestmark = pytest.mark.gpu

CASES = [   # atoms, cell, tilts, radial and angular capacity
    (1024, (60.0, 60.0, 60.0), None, 64, 32),
    (1500, (20.0, 20.0, 20.0), None, 320, 128),
    (1450, (18.4, 18.4, 24.6), None, 320, 128),
    (1300, (20.0, 21.0, 22.0), (3.0, -2.0, 1.5), 320, 128),
    (2049, (31.0, 18.3, 25.0), None, 48, 7),
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_cell_rows_equal_all_pairs(k):
    n, box, tilt, cr, ca = CASES[k]
    sts = [uniform(np.random.default_rng(90 + k), n, box, tilt)]
    print(f"[cell rows] n={n} box={box}", flush=True)
    cells, _ = build(sts, None, cr, ca)
    pairs, _ = build(sts, 100, cr, ca)
    assert cells["flags"] == pairs["flags"]
    for which in ("rad", "ang"):
        np.testing.assert_array_equal(cells[which][0], pairs[which][0])
        assert cells[which][1] == pairs[which][1]
