"""FP64 handles on both sides of the rule that splits layer 1's K over waves
(at most one 16 x 16 tile per CU), at two reduction lengths, against the FP64
oracle at the bounds of the other FP64 tests."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["ani2x", "ani1x"])
@pytest.mark.parametrize("sizes,M", [([1], 1), ([33], 1), ([17, 90], 1), ([100, 100], 1), ([20], 2)])
def test_fp64_layer1_split(orc, hp, model, sizes, M):
    torch = torch_cuda()
    hp = synth.ani1x_hparams() if model == "ani1x" else hp
    b = synth.random_batch(23, sizes, ratio=[1.0] * hp["n_species"])
    w = synth.xavier_weights(M, hp.get("species_widths") or hp["widths"], hp["n_species"], seed=5)
    h = make_handle(hp, w, M, "fp64", b)
    x, s, off = to_device(torch, b, torch.float64)
    E, F = h.energy_forces(x, s, off)
    torch.cuda.synchronize()
    assert h.device_status() == 0
    Eo, Fo = orc.energy_forces(hp, w, M, b.species, b.coords, b.mol_offsets)
    np.testing.assert_allclose(E.cpu().numpy(), Eo, rtol=1e-10, atol=1e-9)
    np.testing.assert_allclose(F.cpu().numpy(), Fo, rtol=0, atol=1e-9 * max(np.abs(Fo).max(), 1e-3))
    h.close()
