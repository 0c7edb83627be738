"""Batches at the edges of the species order's 2048-atom chunks: one chunk and
just over it, a last chunk of one atom, several chunks (blocks then launch by
pair count), species missing from a chunk, and one-atom structures.  Loss,
gradient, forces and virials of the captured step's calls against the FP64
oracle."""
import numpy as np
import pytest

from paper_2507_00528_amd import synth

from gpu_util import TOL_F, Case, DeviceRun, param_blocks, rel

pytestmark = pytest.mark.gpu


def structures(sizes, mono_head):
    rng = np.random.default_rng(3)
    out = []
    for k, n in enumerate(sizes):
        L = max((n / 0.031) ** (1 / 3), 6.5)
        m = int(np.ceil(round(n ** (1 / 3), 6)))
        f = np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), -1) / m
        pos = synth.wrap32(f * L + rng.normal(0, 0.2, (n, 3)), np.full(3, L))
        t = np.zeros(n, np.int32) if k < mono_head else synth.assign_types(rng, n)
        out.append(synth.Structure(pos, np.full(3, L, np.float32), t))
    return out


@pytest.mark.parametrize("name,sizes,mono_head", [
    ("one chunk", [512, 512, 512, 512], 0),
    ("one atom over", [512, 512, 512, 512, 1], 0),
    ("species missing", [700, 700, 648, 300], 3),
    ("five chunks", [900] * 9 + [141], 0),
])
def test_chunk_edges_match_oracle(name, sizes, mono_head):
    c = Case(synth.SIZES_TINY, structures(sizes, mono_head))
    r = DeviceRun(c)
    print(f"[order {name}] N={c.batch.n_atom}", flush=True)
    r.neighbors()
    loss, grad, e_s, F, W = r.loss_grad()
    assert int(r.flags.item()) == 0
    np.testing.assert_allclose(loss, c.loss, rtol=1e-4)
    assert rel(F, np.concatenate(c.pred["F"], 0)) < TOL_F
    assert rel(W, c.pred["W"]) < TOL_F
    for blk, sl in param_blocks(c.sizes).items():
        assert rel(grad[sl], c.grad[sl]) < TOL_F, blk
