"""The species order's array is rounded up past its chunks (at 4096 or 12288
atoms of two species by 64 positions, at 2048 of one by 32).  The kernels of
degrees l > 4 read every position, so the ones past the chunks have to say that
they hold no atom, whatever the workspace held before: here atom 0 in every
position and 1.0 in every other word, with which a position left unwritten adds
a second share to atom 0's pair forces.  Against the FP64 oracle, as copies of
one group of structures."""
import numpy as np
import pytest

from paper_2507_00528_amd import synth

from gpu_util import TOL_E, TOL_F, Case, DeviceRun, param_blocks, rel
from test_gpu_lanes import _Copies

pytestmark = pytest.mark.gpu

SIZES = {1: synth.NEPSizes(n_types=1, n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=6, l4=2, l5=1, hidden=12),
         2: synth.SIZES_L8,
         3: synth.NEPSizes(n_types=3, n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=5, l4=0, l5=0, hidden=12)}
_CASE = {}


def _case(T):
    if T not in _CASE:
        rng = np.random.default_rng(37)
        sts = [synth.random_structure(rng, n, 0.031, 2.6, "amorphous") for n in (63, 65, 57, 71)]
        for st in sts:
            st.types[:] = rng.integers(0, T, st.n)
        _CASE[T] = Case(SIZES[T], sts)
    return _CASE[T]


@pytest.mark.parametrize("T,n_atom", [(1, 2048), (1, 10240), (2, 4096), (2, 8192), (2, 12288), (3, 2048), (3, 4096),
                                      (3, 12288)])
def test_positions_past_the_chunks_hold_no_atom(T, n_atom):
    import torch
    c = _case(T)
    k = n_atom // 256
    r = DeviceRun(_Copies(c, k))
    print(f"[order tail] T={T} N={r.N}", flush=True)
    assert r.N == n_atom
    r.ws.view(torch.float32).fill_(1.0)
    # the order is the workspace's first array: one position an atom, up to 128
    # more a chunk, and the rounding
    r.ws[:4 * (n_atom + 128 * (n_atom // 2048 + 1) + 128)].zero_()
    r.neighbors()
    e_atom, _, F, W = r.efw()
    assert rel(e_atom, np.tile(np.concatenate(c.pred["Ei"]), k)) < TOL_E
    assert rel(F, np.tile(np.concatenate(c.pred["F"], 0), (k, 1))) < TOL_F
    assert rel(W, np.tile(c.pred["W"], (k, 1))) < TOL_F
    loss, grad, *_ = r.loss_grad()
    assert int(r.flags.item()) == 0
    np.testing.assert_allclose(loss, c.loss, rtol=1e-4)
    for blk, sl in param_blocks(c.sizes).items():
        assert rel(grad[sl], c.grad[sl]) < TOL_F, blk
