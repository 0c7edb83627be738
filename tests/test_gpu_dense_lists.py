"""Long angular lists: wavefronts whose atoms have so many pairs that a chunk of
64 belongs to a few of them, and wavefronts of long and short lists together,
at 32, 16 and 8 lanes an atom.  Energies, forces, virials, loss and gradient
against the FP64 oracle, as copies of one group of structures."""
import numpy as np
import pytest

from paper_2507_00528_amd import synth

from gpu_util import TOL_E, TOL_F, Case, DeviceRun, param_blocks, rel
from test_gpu_lanes import _Copies

pytestmark = pytest.mark.gpu

SIZES = {"large": synth.SIZES_LARGE, "small": synth.SIZES_SMALL, "mono": synth.SIZES_MONO, "l8": synth.SIZES_L8,
         "three_species": synth.NEPSizes(n_types=3, n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=4, l4=2, l5=1, hidden=12)}
_CASE = {}


def _cell(rng, n, density, spread):
    """n sites of a cubic grid with vacancies, displaced; with spread > 0 half
    of the cell holds most of the atoms."""
    L = (n / density) ** (1 / 3)
    m = int(np.ceil(round(n ** (1 / 3), 6))) + (2 if spread else 0)
    w = np.where(np.arange(m ** 3) // (m * m) < m // 2, 1.0, spread or 1.0)
    site = rng.choice(m ** 3, n, replace=False, p=w / w.sum())
    f = np.stack(np.unravel_index(site, (m, m, m)), -1) / m
    pos = synth.wrap32(f * L + rng.normal(0, 0.06 * L / m, (n, 3)), np.full(3, L))
    return synth.Structure(pos, np.full(3, L, np.float32), np.zeros(n, np.int32))


def _case(name, density):
    if (name, density) not in _CASE:
        rng = np.random.default_rng(47)
        sts = [_cell(rng, n, density, s) for n, s in ((63, 0.0), (65, 0.05), (57, 0.0), (71, 0.2))]
        for st in sts:
            st.types[:] = rng.integers(0, SIZES[name].n_types, st.n)
        _CASE[name, density] = Case(SIZES[name], sts)
    return _CASE[name, density]


@pytest.mark.parametrize("name,density,copies", [
    ("large", 0.12, 1), ("large", 0.12, 9), ("large", 0.12, 41), ("large", 0.25, 1), ("large", 0.25, 9),
    ("large", 0.25, 41), ("small", 0.12, 41), ("mono", 0.2, 57), ("l8", 0.12, 33), ("three_species", 0.2, 9),
    ("three_species", 0.2, 33)])
def test_calls_match_oracle(name, density, copies):
    c = _case(name, density)
    r = DeviceRun(_Copies(c, copies), cap_rad=400, cap_ang=160)
    r.neighbors()
    counts = r.nbrs.cnt_ang[:256].cpu().numpy()
    print(f"[dense {name}] N={r.N} pairs {counts.min()} to {counts.max()}, mean {counts.mean():.0f}", flush=True)
    assert counts.mean() > 24
    e_atom, _, F, W = r.efw()
    assert rel(e_atom, np.tile(np.concatenate(c.pred["Ei"]), copies)) < TOL_E
    assert rel(F, np.tile(np.concatenate(c.pred["F"], 0), (copies, 1))) < TOL_F
    assert rel(W, np.tile(c.pred["W"], (copies, 1))) < TOL_F
    loss, grad, *_ = r.loss_grad()
    assert int(r.flags.item()) == 0
    np.testing.assert_allclose(loss, c.loss, rtol=1e-4)
    for blk, sl in param_blocks(c.sizes).items():
        assert rel(grad[sl], c.grad[sl]) < TOL_F, blk


@pytest.mark.parametrize("cap_rad,cap_ang", [(60, 17), (64, 24), (90, 27), (61, 33), (120, 40)])
def test_long_lists_cut_at_their_capacity(cap_rad, cap_ang):
    """The force pass finds a pair's other entry in a cut list of more than 16
    entries, at every row alignment, or that it was cut off."""
    from test_gpu_force import cut, reference
    rng = np.random.default_rng(53)
    c = Case(synth.SIZES_LARGE, [_cell(rng, n, 0.14, s) for n, s in ((64, 0.0), (90, 0.1))], with_oracle=False)
    r = DeviceRun(c, cap_rad=cap_rad, cap_ang=cap_ang)
    r.neighbors()
    counts = r.nbrs.cnt_ang.cpu().numpy()
    print(f"[dense cut {cap_rad}/{cap_ang}] N={r.N} pairs {counts.min()} to {counts.max()}", flush=True)
    assert counts.max() > cap_ang > 16
    _, e_s, F, W = r.efw()
    ref = [reference(c.oracle, c.theta, st, (cut(p[0], cap_rad), cut(p[1], cap_ang)))
           for st, p in zip(c.structures, c.nbrs)]
    sizes = np.diff(c.batch.atom_offset)
    assert rel(e_s / sizes, np.array([q[0] for q in ref]) / sizes) < TOL_E
    assert rel(F, np.concatenate([q[1] for q in ref], 0)) < TOL_F
    assert rel(W, np.stack([q[2] for q in ref])) < TOL_F
