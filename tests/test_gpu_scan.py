"""The two-part single-image neighbor scan at the edges of its split: 8 lanes
taking ranges of 0 to 128 candidates, hits from one to more than the 192 an
atom's lane columns hold, blocks whose structures fit one 1024-atom tile or do
not, and cells on both sides of the single-image width.  Lists bit for bit
against the FP64 oracle."""
import numpy as np
import pytest

from oracle import neighbor_pairs
from paper_2507_00528_amd import synth

from test_gpu_cells import RC, RCA, build, uniform

pytestmark = pytest.mark.gpu

# (atoms, edge): ragged small ranges, whole tiles, tile straddles, dense cells
CELLS = {
    "small": [(1, 12.5), (7, 13.0), (9, 12.03), (40, 12.01), (63, 12.6), (64, 12.6), (65, 14.0)],
    "tile": [(31, 12.1), (993, 31.8), (1023, 32.0), (33, 12.2), (1024, 32.1), (255, 20.2), (257, 20.2)],
    "dense": [(330, 12.2), (520, 12.3), (700, 12.4)],
}


@pytest.mark.parametrize("tilted", [False, True])
@pytest.mark.parametrize("name", list(CELLS))
def test_two_part_scan_matches_oracle(name, tilted):
    rng = np.random.default_rng(41)
    sts = []
    for n, L in CELLS[name]:
        tilt = (0.1 * L, -0.15 * L, 0.2 * L) if tilted else None
        sts.append(uniform(rng, n, (L * (1.08 if tilted else 1.0),) * 3, tilt))
    print(f"[scan {name} tilted={tilted}] atoms {[s.n for s in sts]}", flush=True)
    cap = 640 if name == "dense" else 96
    out, (model, db, nb, ws, fl, b) = build(sts, 1, cap_rad=cap, cap_ang=cap)   # hint 1: no cell lists
    assert out["flags"] == 0
    for k, st in enumerate(sts):
        base = int(b.atom_offset[k])
        for which, rc in (("rad", RC), ("ang", RCA)):
            p = neighbor_pairs(st.pos, st.box, rc, tilt32=st.tilt)
            want = [[] for _ in range(st.n)]
            for i, j, c in p:
                want[i].append(((base + int(j)) << 5) | int(c))
            cnt, lists = out[which]
            for i in range(st.n):
                assert lists[base + i] == want[i], (k, i, which)
                assert cnt[base + i] == len(want[i])
