"""The force pass when lists are cut at their capacity: F_i sums f_ij over the
atom's stored entries, minus f_ji where the partner's list stores the pair
too; the virial sums the stored entries.  Reference: the oracle's energy
differentiated by the vector of each stored entry.  The capacities give
partner rows of every alignment."""
import numpy as np
import pytest

from oracle.nep_oracle import shift_vectors, unpack
from paper_2507_00528_amd import synth

from gpu_util import TOL_E, TOL_F, Case, DeviceRun, rel

pytestmark = pytest.mark.gpu


def cut(pairs, cap):
    """The first cap entries of each atom's canonical list."""
    pairs = np.asarray(pairs)
    key = (pairs[:, 0].astype(np.int64) << 40) | (pairs[:, 1].astype(np.int64) << 5) | pairs[:, 2]
    pairs = pairs[np.argsort(key)]
    first = np.searchsorted(pairs[:, 0], pairs[:, 0])
    return pairs[np.arange(len(pairs)) - first < cap]


def reference(o, theta, st, lists):
    """Energies, forces and virial (xx, yy, zz, xy, yz, zx) from stored entries."""
    import torch
    x = torch.tensor(st.pos.astype(np.float64))
    HS = torch.tensor(shift_vectors(st.box, None))
    d = [((x[p[:, 1]] - x[p[:, 0]]) + HS[p[:, 2]]).requires_grad_(True) for p in lists]
    prm = unpack(o.sz, torch.tensor(theta.astype(np.float64)))
    G = o.descriptors(prm, st.types, st.n, lists[0], d[0], lists[1], d[1])
    E = o.atom_energies(prm, st.types, G)
    F, W = np.zeros((st.n, 3)), np.zeros(6)
    for p, v, f in zip(lists, d, torch.autograd.grad(E.sum(), d)):
        f, v = f.numpy(), v.detach().numpy()
        stored = {tuple(q) for q in p.tolist()}
        np.add.at(F, p[:, 0], f)
        both = np.array([(j, i, 26 - c) in stored for i, j, c in p.tolist()])
        np.add.at(F, p[both, 1], -f[both])
        for c, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (2, 0))):
            W[c] -= (f[:, a] * v[:, b]).sum()
    return E.sum().item(), F, W


@pytest.mark.parametrize("cap_rad,cap_ang", [(8, 4), (17, 5), (24, 6), (25, 8), (33, 9)])
def test_truncated_lists_match_oracle(cap_rad, cap_ang):
    c = Case(synth.SIZES_LARGE, synth.config_structures("c2", n_struct=4), with_oracle=False)
    r = DeviceRun(c, cap_rad=cap_rad, cap_ang=cap_ang)
    print(f"[truncated {cap_rad}/{cap_ang}] N={c.batch.n_atom}", flush=True)
    r.neighbors()
    e_atom, e_s, F, W = r.efw()
    ref = [reference(c.oracle, c.theta, st, (cut(p[0], cap_rad), cut(p[1], cap_ang)))
           for st, p in zip(c.structures, c.nbrs)]
    sizes = np.diff(c.batch.atom_offset)
    assert rel(e_s / sizes, np.array([q[0] for q in ref]) / sizes) < TOL_E
    assert rel(F, np.concatenate([q[1] for q in ref], 0)) < TOL_F
    assert rel(W, np.stack([q[2] for q in ref])) < TOL_F
