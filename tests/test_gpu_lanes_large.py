"""Batches where the forward and the adjoint run 8 lanes an atom (above 8192
atoms with degrees l > 4 and in the padded classes, 14336 with at most 16
descriptors, else 10240), for the models that the small batches of the other
tests take through 16 or 32 lanes; and the model whose adjoint needs the most
LDS.  Against the FP64 oracle, as copies of one group of structures."""
import numpy as np
import pytest

from paper_2507_00528_amd import synth

from gpu_util import TOL_E, TOL_F, Case, DeviceRun, param_blocks, rel
from test_gpu_lanes import _Copies

pytestmark = pytest.mark.gpu

SIZES = {
    "large": synth.SIZES_LARGE,
    "small": synth.SIZES_SMALL,
    "mono": synth.SIZES_MONO,
    "l8": synth.SIZES_L8,
    "three_species": synth.NEPSizes(n_types=3, n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=4, l4=2, l5=1, hidden=12),
    "l6": synth.NEPSizes(n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=6, l4=2, l5=0, hidden=12),
    # four species, degrees up to 8, hidden 256: 163,328 of 163,840 bytes
    "hidden256": synth.NEPSizes(n_types=3, n_rad=4, n_ang=3, k_rad=6, k_ang=5, l3=5, l4=0, l5=0, hidden=256),
}
_CASE = {}


def _case(name, tilted=False):
    if (name, tilted) not in _CASE:
        rng = np.random.default_rng(41)
        if tilted:
            sts = [synth.triclinic_structure(rng, n, 0.031, 2.4, 0.2) for n in (63, 65, 57, 71)]
        else:
            sts = [synth.random_structure(rng, n, 0.031, 2.6, "amorphous") for n in (63, 65, 57, 71)]
        for st in sts:
            st.types[:] = rng.integers(0, SIZES[name].n_types, st.n)
        _CASE[name, tilted] = Case(SIZES[name], sts)
    return _CASE[name, tilted]


@pytest.mark.parametrize("name,tilted,copies", [
    ("hidden256", False, 1), ("hidden256", False, 33), ("large", False, 40), ("large", False, 41),
    ("small", False, 41), ("mono", False, 56), ("mono", False, 57), ("l8", False, 33), ("three_species", False, 33),
    ("l6", False, 33), ("large", True, 1), ("large", True, 9), ("large", True, 41), ("l8", True, 1), ("l8", True, 33),
    ("three_species", True, 9), ("three_species", True, 33)])
def test_calls_match_oracle(name, tilted, copies):
    c = _case(name, tilted)
    r = DeviceRun(_Copies(c, copies))
    print(f"[lanes {name}] tilted={tilted} N={r.N}", flush=True)
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


@pytest.mark.parametrize("waves", [2, 3])
@pytest.mark.parametrize("name", ["large", "small", "mono", "l8"])
def test_captured_step_at_both_occupancies(name, waves):
    """forward_waves and adjoint_waves choose between two builds of the 8-lane
    kernels."""
    import torch
    from paper_2507_00528_amd import nep
    c = _case(name)
    r = DeviceRun(_Copies(c, 57))
    print(f"[lanes {name}] waves={waves} N={r.N}", flush=True)
    P = r.params.numel()
    z = lambda n: torch.zeros(n, device="cuda")
    grad, loss, step = z(P), z(4), torch.ones(1, dtype=torch.int32, device="cuda")
    g = nep.TrainStepGraph(r.model, r.batch, r.nbrs, r.labels, c.lam, r.params, z(P), z(P), grad, loss, step, r.ws,
                           r.flags, lr_start=0.0, lr_stop=0.0, tuning={"forward_waves": waves, "adjoint_waves": waves})
    for _ in range(2):
        g.launch()
        torch.cuda.synchronize()
        assert int(r.flags.item()) == 0
        np.testing.assert_allclose(loss.cpu().numpy(), c.loss, rtol=1e-4)
        for blk, sl in param_blocks(c.sizes).items():
            assert rel(grad.cpu().numpy()[sl], c.grad[sl]) < TOL_F, blk
        grad.zero_()
        loss.zero_()
    g.close()


@pytest.mark.parametrize("name", ["small", "l8", "three_species"])
def test_one_md_call_equals_single_step_calls(name):
    """Above 8192 atoms the species order ranks by pair count, and a call of
    several steps renews it every 16: the steps between run on the order of
    other counts, with the same results bit for bit."""
    import torch
    from paper_2507_00528_amd import md, nep
    c = _case(name)
    k, n = 41, 18
    got = []
    for calls, per in ((1, n), (n, 1)):
        r = DeviceRun(_Copies(c, k))
        masses = [121.76, 127.6, 72.63][:c.sizes.n_types]
        mass = torch.tensor(masses, dtype=torch.float32, device="cuda")
        vel = torch.tensor(md.maxwell_velocities(r.case.batch.types, masses, 900.0, seed=7), device="cuda")
        e_pot, e_kin, force = (torch.zeros(m, device="cuda") for m in (r.S, r.S, 3 * r.N))
        print(f"[lanes md {name}] N={r.N} calls={calls}", flush=True)
        r.neighbors()
        counts = r.nbrs.cnt_ang.cpu().numpy()
        nep.energy_force_virial(r.model, r.batch, r.nbrs, r.params, r.ws, None, e_pot, force, None)
        for _ in range(calls):
            nep.md_step(r.model, r.batch, r.nbrs, r.params, mass, vel, force, 2.0, per, e_pot, r.ws, r.flags,
                        e_kin=e_kin)
        torch.cuda.synchronize()
        assert int(r.flags.item()) == 0
        assert not np.array_equal(counts, r.nbrs.cnt_ang.cpu().numpy())
        got.append([t.cpu().numpy() for t in (r.batch.pos, vel, force, e_pot, e_kin)])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
