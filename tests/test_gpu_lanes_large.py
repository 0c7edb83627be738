"""Batches above 8192 atoms, where the forward and the adjoint run 8 lanes an
atom, for the models that the small batches of the other tests take through 16
or 32 lanes; and the one model whose adjoint takes 16 lanes at any size.
Against the FP64 oracle, as copies of one group of structures."""
import numpy as np
import pytest

from paper_2507_00528_amd import synth

from gpu_util import TOL_E, TOL_F, Case, DeviceRun, param_blocks, rel
from test_gpu_lanes import _Copies

pytestmark = pytest.mark.gpu

SIZES = {
    # four species, degrees up to 8, hidden 256: rows of 8 atoms pass the LDS
    "hidden256": synth.NEPSizes(n_types=3, n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=5, l4=0, l5=0, hidden=256),
}
_CASE = {}


def _case(name):
    if name not in _CASE:
        rng = np.random.default_rng(41)
        sts = [synth.random_structure(rng, n, 0.031, 2.6, "amorphous") for n in (63, 65, 57, 71)]
        for st in sts:
            st.types[:] = rng.integers(0, SIZES[name].n_types, st.n)
        _CASE[name] = Case(SIZES[name], sts)
    return _CASE[name]


@pytest.mark.parametrize("name,copies", [("hidden256", 1), ("hidden256", 33)])
def test_calls_match_oracle(name, copies):
    c = _case(name)
    r = DeviceRun(_Copies(c, copies))
    print(f"[lanes {name}] N={r.N}", flush=True)
    r.neighbors()
    e_atom, e_s, F, W = r.efw()
    assert rel(e_atom, np.tile(np.concatenate(c.pred["Ei"]), copies)) < TOL_E
    assert rel(F, np.tile(np.concatenate(c.pred["F"], 0), (copies, 1))) < TOL_F
    assert rel(W, np.tile(c.pred["W"], (copies, 1))) < TOL_F
    loss, grad, *_ = r.loss_grad()
    assert int(r.flags.item()) == 0
    np.testing.assert_allclose(loss, c.loss, rtol=1e-4)
    for blk, sl in param_blocks(c.sizes).items():
        assert rel(grad[sl], c.grad[sl]) < TOL_F, blk
