"""A call of n MD steps moves the atoms inside its force passes and renews the
species order every 16 steps; n calls of one step take the separate move
launches and order every step.  Both give the same bits: neither the order nor
the launch that moves an atom enters a sum."""
import numpy as np
import pytest

from paper_2507_00528_amd import md, synth

from test_gpu_md import MASSES, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,cell,n", [("large", "ortho", 2), ("large", "ortho", 17), ("large", "tilted", 5),
                                          ("l8", "ortho", 3), ("tiny", "ortho", 35)])
def test_one_call_equals_single_step_calls(sizes, cell, n):
    import torch
    from paper_2507_00528_amd import nep
    sz = {"large": synth.SIZES_LARGE, "l8": synth.SIZES_L8, "tiny": synth.SIZES_TINY}[sizes]
    sts = synth.config_structures("c0")[:2]
    if cell == "tilted":
        t = np.array([2.0, 1.0, -1.5], np.float32)
        sts = [synth.Structure(synth.wrap_cell32(st.pos, st.box, t), st.box, st.types, "tilted", t) for st in sts]
    print(f"[md moves] {sizes} {cell} n={n}", flush=True)
    got = []
    for calls, per in ((1, n), (n, 1)):
        model, b, db, nb, ws, fl, theta = setup(sts, sz, synth.SEEDS["teacher"])
        p = torch.tensor(theta, device="cuda")
        mass = torch.tensor(MASSES, dtype=torch.float32, device="cuda")
        vel = torch.tensor(md.maxwell_velocities(b.types, MASSES, 900.0, seed=7), device="cuda")
        force = torch.zeros(3 * b.n_atom, device="cuda")
        e_pot, e_kin = torch.zeros(b.n_struct, device="cuda"), torch.zeros(b.n_struct, device="cuda")
        nep.build_neighbors(model, db, nb, ws, fl)
        nep.energy_force_virial(model, db, nb, p, ws, None, e_pot, force, None)
        for _ in range(calls):
            nep.md_step(model, db, nb, p, mass, vel, force, 2.0, per, e_pot, ws, fl, e_kin=e_kin)
        torch.cuda.synchronize()
        assert int(fl.item()) == 0
        got.append([t.cpu().numpy() for t in (db.pos, vel, force, e_pot, e_kin)])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
