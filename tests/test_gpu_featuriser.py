"""Neighbour records and bucket rows formed inside the featuriser: molecules at
the edges of a wave's one and two candidates a lane and of the step beyond
them, with the bucketing fused in and (more than 1,024 atoms) beside it,
against the FP64 oracle.  The FP64 tolerance is that of the other FP64 tests;
FP32 forces are within 1e-4 of the largest."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [1],
    [64],
    [65, 1, 63],
    [127, 2, 128],
    [129, 64, 1, 130],                 # above the records' step, smaller molecules beside
    [128] * 8,                         # 1,024 atoms: the last batch with fused bucketing
    [128] * 8 + [3],                   # the first without
])
@pytest.mark.parametrize("prec,chunk", [("fp64", 0), ("fp32", 4), ("fp32", 16)])
def test_records_and_rows_match_oracle(orc, hp, sizes, prec, chunk):
    torch = torch_cuda()
    b = synth.random_batch(7, sizes)
    w = synth.xavier_weights(1, hp["widths"], seed=9)
    h = make_handle(hp, w, 1, prec, b)
    h.set_knob("cell_min", 256)        # all molecules in the all-pairs search
    if chunk:
        h.set_knob("atom_chunk", chunk)
    x, s, off = to_device(torch, b, torch.float64 if prec == "fp64" else torch.float32)
    E, F = h.energy_forces(x, s, off)
    assert h.device_status() == 0
    Eo, Fo = orc.energy_forces(hp, w, 1, b.species, x.cpu().numpy().astype(np.float64), b.mol_offsets)
    fmax = max(np.abs(Fo).max(), 1e-3)
    tol_e, tol_f = (1e-9, 1e-9) if prec == "fp64" else (1e-4, 1e-4)
    np.testing.assert_allclose(E.cpu().numpy(), Eo, rtol=1e-10 if prec == "fp64" else 1e-5, atol=tol_e)
    np.testing.assert_allclose(F.cpu().numpy(), Fo, rtol=0, atol=tol_f * fmax)
    h.close()
