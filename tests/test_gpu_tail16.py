"""The fused network tail of BF16 handles with 16-row buckets (at most 256
atoms): one atom, whole and partial tiles of one and of many elements, a third
layer of 160 and of more columns, against the FP64 oracle at the bounds of the
other BF16 tests."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import (BF16_FORCE_RMS_FRAC, bf16_de_bar, errors, make_handle, oracle_inputs, to_device,
                            torch_cuda)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h3", [160, 192])
@pytest.mark.parametrize("sizes,elements", [
    ([1], 1),
    ([16], 1),
    ([17, 1], 1),
    ([40, 3, 40], 7),
    ([64, 64, 64, 64], 7),
])
def test_bf16_tail_of_16_row_tiles(orc, hp, h3, sizes, elements):
    torch = torch_cuda()
    hp = dict(hp)
    hp["widths"] = list(hp["widths"][:3]) + [h3, 1]
    M = 2
    b = synth.random_batch(17, sizes)
    b.species[:] = np.arange(len(b.species)) % elements
    w = synth.xavier_weights(M, hp["widths"], seed=3)
    h = make_handle(hp, w, M, "bf16", b)
    x, s, off = to_device(torch, b, torch.float32)
    E, F = h.energy_forces(x, s, off)
    torch.cuda.synchronize()
    assert h.device_status() == 0
    xo, wo = oracle_inputs(b, w, "bf16")
    Eo, Fo = orc.energy_forces(hp, wo, M, b.species, xo, b.mol_offsets)
    dE, rmse = errors(E.cpu().numpy(), F.double().cpu().numpy(), Eo, Fo, b.mol_offsets)[:2]
    frms = np.sqrt((Fo ** 2).mean())
    assert dE.max() <= bf16_de_bar(M)
    assert rmse.max() <= BF16_FORCE_RMS_FRAC * max(frms, 1e-6)
    h.close()
