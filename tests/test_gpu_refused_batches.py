"""Batches the device refuses (a molecule above the capacity, offsets that do not
end at the atom count) through the training backward: the flag is raised, no
index follows from what an earlier batch left behind, and the next batch's
results are the oracle's."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes,shift", [
    ([40, 60, 40], 0),                 # the second molecule above the capacity of 50
    ([50] * 30 + [60], 0),             # the same beyond one bucketing block
    ([40, 10, 40], -1),                # offsets that end one atom early
])
def test_coordinate_gradient_of_a_refused_batch(orc, hp, sizes, shift, prec):
    torch = torch_cuda()
    from paper_2201_08110_amd.nnp import NNP_E_CAPACITY
    dt = torch.float32 if prec == "fp32" else torch.float64
    big = synth.random_batch(5, [3] * 500)          # leaves molecule indices far above the refused batch's
    bad = synth.random_batch(6, sizes)
    w = synth.xavier_weights(1, hp["widths"], seed=7)
    h = make_handle(hp, w, 1, prec, big, max_atoms=2048, max_apm=50)
    x, sp, off = to_device(torch, big, dt)
    gE = torch.ones(big.n_mols, dtype=torch.float64, device="cuda")
    h.backward(x, sp, off, gE, None, want_coords=True)
    assert h.device_status() == 0
    xb, spb, offb = to_device(torch, bad, dt)
    offb[-1] += shift
    gEb = torch.ones(bad.n_mols, dtype=torch.float64, device="cuda")
    h.backward(xb, spb, offb, gEb, None, want_coords=True)
    torch.cuda.synchronize()
    assert h.device_status() == NNP_E_CAPACITY
    _, gx = h.backward(x, sp, off, gE, None, want_coords=True)
    assert h.device_status() == 0
    _, Fo = orc.energy_forces(hp, synth.round_to_fp32(w) if prec == "fp32" else w, 1, big.species,
                              x.double().cpu().numpy(), big.mol_offsets)
    got = gx.double().cpu().numpy()
    assert np.sqrt(np.mean((got + Fo) ** 2)) <= (1e-3 if prec == "fp32" else 1e-8)
    h.close()
