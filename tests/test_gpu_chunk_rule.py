"""Atoms per featuriser and force workgroup as the handle chooses them, for a
call that fills it: by the call's atoms, alike for equal and for ragged
molecules, and no launch of mostly empty workgroups."""
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("atoms,mols,apm,chunk", [
    (64, 1, 64, 4), (4096, 64, 120, 4),
    (33248, 512, 120, 8), (33248, 690, 48, 8),
    (47999, 738, 120, 8), (47999, 1000, 48, 8),          # both kinds of batch on both sides of 49,137 atoms
    (49152, 760, 64, 16), (49152, 1024, 48, 16),
    (4096, 1024, 128, 16), (4096, 512, 128, 8), (4096, 256, 128, 4),   # 32,768, 16,384 and 8,192 workgroups at 4
    (4096, 1024, 1024, 16),
])
def test_automatic_chunk(hp, atoms, mols, apm, chunk):
    torch_cuda()
    from paper_2201_08110_amd.nnp import NNP
    w = synth.xavier_weights(1, hp["widths"], seed=1)
    h = NNP(hp, w, 1, "bf16", max_atoms=atoms, max_mols=mols, max_atoms_per_mol=apm)
    assert h.get_knob("atom_chunk") == chunk
    h.set_knob("atom_chunk", 8)
    assert h.get_knob("atom_chunk") == 8
    h.close()
