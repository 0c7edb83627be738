"""Lanes per atom of the forward and the adjoint (32 up to 2048 atoms, 16 up to
8192, 8 beyond): batches on both sides of each line against the FP64 oracle.
A batch is copies of one group of structures, so the loss and the gradient are
the group's and every copy has its energies, forces and virials."""
import dataclasses

import numpy as np
import pytest

from paper_2507_00528_amd import synth

from gpu_util import TOL_E, TOL_F, Case, DeviceRun, param_blocks, rel

pytestmark = pytest.mark.gpu

SIZES = {
    "large": synth.SIZES_LARGE,
    "mono": synth.SIZES_MONO,
    "l8": synth.SIZES_L8,
    "padded": dataclasses.replace(synth.SIZES_SMALL, n_types=3, n_rad=4, k_rad=7, hidden=13),
}
_CASE = {}


def _case(name):
    if name not in _CASE:
        rng = np.random.default_rng(29)
        T = SIZES[name].n_types
        sts = [synth.random_structure(rng, n, 0.031, 2.6, "amorphous") for n in (63, 65, 57, 71)]
        for st in sts:
            st.types[:] = rng.integers(0, T, st.n)
        _CASE[name] = Case(SIZES[name], sts)
    return _CASE[name]


class _Copies:
    def __init__(self, c, k):
        self.sizes, self.lam, self.theta, self.structures = c.sizes, c.lam, c.theta, c.structures * k
        self.batch = synth.Batch(self.structures)
        self.labels = dict(energy=np.tile(c.labels["energy"], k), force=np.tile(c.labels["force"], (k, 1)),
                           virial=np.tile(c.labels["virial"], (k, 1)))


@pytest.mark.parametrize("name,copies", [("large", 1), ("large", 8), ("large", 9), ("large", 32), ("large", 33),
                                         ("mono", 1), ("mono", 9), ("l8", 1), ("l8", 9), ("padded", 1),
                                         ("padded", 9)])
def test_batches_around_the_lane_counts(name, copies):
    c = _case(name)
    r = DeviceRun(_Copies(c, copies))
    print(f"[lanes {name}] N={r.N}", flush=True)
    assert r.N == 256 * copies
    r.neighbors()
    e_atom, e_s, F, W = r.efw()
    n = np.tile([st.n for st in c.structures], copies)
    assert rel(e_s / n, np.tile(c.pred["E"], copies) / n) < TOL_E
    assert rel(e_atom, np.tile(np.concatenate(c.pred["Ei"]), copies)) < TOL_E
    assert rel(F, np.tile(np.concatenate(c.pred["F"], 0), (copies, 1))) < TOL_F
    assert rel(W, np.tile(c.pred["W"], (copies, 1))) < TOL_F
    loss, grad, *_ = r.loss_grad()
    assert int(r.flags.item()) == 0
    np.testing.assert_allclose(loss, c.loss, rtol=1e-4)
    for blk, sl in param_blocks(c.sizes).items():
        assert rel(grad[sl], c.grad[sl]) < TOL_F, blk


@pytest.mark.parametrize("n", [1, 2, 5, 9])
def test_a_few_atoms(n):
    """Wavefronts with fewer atoms than slots."""
    rng = np.random.default_rng(31)
    pos = rng.uniform(4.0, 9.0, (n, 3)).astype(np.float32)
    st = synth.Structure(pos, np.full(3, 14.0, np.float32), (np.arange(n) % 2).astype(np.int32), "cluster")
    c = Case(synth.SIZES_LARGE, [st])
    r = DeviceRun(c)
    r.neighbors()
    e_atom, e_s, F, W = r.efw()
    assert rel(e_atom, np.concatenate(c.pred["Ei"])) < TOL_E
    if n > 1:
        assert rel(F, np.concatenate(c.pred["F"], 0)) < TOL_F
    loss, grad, *_ = r.loss_grad()
    assert int(r.flags.item()) == 0
    for blk, sl in param_blocks(c.sizes).items():
        assert rel(grad[sl], c.grad[sl]) < TOL_F, blk
