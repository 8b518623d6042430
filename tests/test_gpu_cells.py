"""Neighbour lists of molecules above the all-pairs search, staged in (element,
cutoff cell) order: shapes of molecule that give one cell, a row of cells, a
layer and a block, at the smallest and largest sizes, against the FP64 oracle."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _molecule(n, box, seed):
    """n atoms at least 1 A apart in a box of the given edges (a jittered
    lattice of 1.6 A, sites taken at random)."""
    rng = np.random.default_rng(seed)
    g = [np.arange(max(int(e // 1.6), 1)) * 1.6 for e in box]
    sites = np.stack(np.meshgrid(*g, indexing="ij"), -1).reshape(-1, 3)
    assert len(sites) >= n
    pick = rng.permutation(len(sites))[:n]
    return sites[pick] + rng.uniform(-0.3, 0.3, (n, 3)), rng.integers(0, 7, n).astype(np.int32)


@pytest.mark.parametrize("n,box,cell_min", [
    (17, (5.0, 5.0, 5.0), 16),            # one cell
    (129, (9.7, 9.7, 9.7), 128),          # the first size above the default, one cell
    (200, (400.0, 1.7, 1.7), 128),        # a row: more extent than the 6 cells a side
    (300, (50.0, 40.0, 1.7), 128),        # a layer
    (1024, (32.0, 32.0, 32.0), 128),      # the largest molecule, a block of cells
])
def test_cell_lists_match_oracle(orc, hp, n, box, cell_min):
    torch = torch_cuda()
    b = synth.random_batch(3, [4, 6])     # a small molecule on either side
    pos, sp = _molecule(n, box, seed=n)
    b.coords = np.concatenate([b.coords[:4], pos, b.coords[4:]])
    b.species = np.concatenate([b.species[:4], sp, b.species[4:]])
    b.mol_offsets = np.array([0, 4, 4 + n, 10 + n], dtype=np.int32)
    w = synth.xavier_weights(1, hp["widths"], seed=9)
    h = make_handle(hp, w, 1, "fp64", b)
    h.set_knob("cell_min", cell_min)
    x, s, off = to_device(torch, b, torch.float64)
    E, F = h.energy_forces(x, s, off)
    assert h.device_status() == 0
    Eo, Fo = orc.energy_forces(hp, w, 1, b.species, b.coords, b.mol_offsets)
    np.testing.assert_allclose(E.cpu().numpy(), Eo, rtol=1e-10, atol=1e-9)
    np.testing.assert_allclose(F.cpu().numpy(), Fo, rtol=0, atol=1e-9 * np.abs(Fo).max())
    h.close()
