"""The same batch under other launch bounds (device-side counts) and beside other
molecules: energies, and forces summed in fixed point, are bitwise the same on
one handle, whatever tiles a call's size selects."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,M,cap,sizes", [
    ("fp32", 8, 2048, [30, 24, 60, 17] * 4),     # above and below a layer-1 backward of one workgroup a CU
    ("fp32", 8, 600, [30, 24, 60, 17] * 4),      # the same with the capacity of the K-split form
    ("fp32", 1, 8192, [10, 5]),
    ("fp64", 1, 512, [12, 20]),                  # above and below the 256 tiles of the FP64 layer-1 form
    ("fp64", 1, 64, [12, 20]),
    ("bf16", 8, 2048, [30, 24, 60, 17]),
])
def test_bits_do_not_follow_the_launch(hp, prec, M, cap, sizes):
    torch = torch_cuda()
    b = synth.random_batch(14, sizes)
    w = synth.xavier_weights(M, hp["widths"], seed=15)
    h = make_handle(hp, w, M, prec, b, max_atoms=cap, max_mols=64, max_apm=60)
    h.set_knob("force_sum", 2)
    dt = torch.float64 if prec == "fp64" else torch.float32
    x, sp, off = to_device(torch, b, dt)
    E, F = h.energy_forces(x, sp, off)
    counts = torch.tensor([b.n_mols, b.n_atoms], dtype=torch.int32, device="cuda")
    for bounds in ((b.n_mols, b.n_atoms), (64, cap)):
        out = (torch.zeros(64, dtype=torch.float64, device="cuda"), torch.zeros_like(x))
        h.energy_forces(x, sp, off, out=out, counts=counts, bounds=bounds)
        assert h.device_status() == 0
        assert torch.equal(out[0][:b.n_mols], E) and torch.equal(out[1], F), bounds
    # the first molecule alone
    n = sizes[0]
    E1, F1 = h.energy_forces(x[:n].contiguous(), sp[:n].contiguous(), off[:2].contiguous())
    assert torch.equal(E1, E[:1]) and torch.equal(F1, F[:n])
    h.close()
