"""FP32 handles keep FP32 accuracy: bars that operands of three bf16 parts meet and
operands of two (16 significant bits) miss.  Errors against the FP64 oracle, one
network, RMS over the batch; from an emulation of the six (and of the four
two-part) products with FP32 sums on this batch's features, without the
featuriser's own FP32 error:
  energy per atom, of the RMS atomic energy   three 1.2e-8   two 3.3e-6   bar 5e-7
  forces, of their RMS                        three 2.0e-7   two 1.3e-5   bar 3e-6
  parameter gradient of an energy loss, norm  three 1e-7     two 5e-6     bar 2e-6
The featuriser adds about 5e-8, 1e-6 and 3e-7 (FP32 terms, off by one or two
units in the last place each)."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, oracle_inputs, to_device, torch_cuda

pytestmark = pytest.mark.gpu

SIZES = [60, 50, 40, 64, 30]


@pytest.fixture(scope="module")
def reference(orc, hp):
    b = synth.random_batch(21, SIZES)
    w = synth.xavier_weights(1, hp["widths"], seed=12)
    xo, wo = oracle_inputs(b, w, "fp32")
    E, F = orc.energy_forces(hp, wo, 1, b.species, xo, b.mol_offsets)
    gE = np.random.default_rng(5).normal(size=b.n_mols)
    g = orc.param_grad(hp, wo, 1, b.species, xo, b.mol_offsets, gE, np.zeros_like(xo))
    atom = [hp["energy_scale"] * orc.atomic_nn(hp, wo, 1, 0, s, G)[0]
            for a0, a1 in zip(b.mol_offsets[:-1], b.mol_offsets[1:])
            for s, G in zip(b.species[a0:a1], orc.aev(hp, b.species[a0:a1], xo[a0:a1]))]
    return b, w, E, F, gE, g, np.sqrt(np.mean(np.square(atom)))


# 16-row buckets; 64-row ones with K split over waves in layer 1, and without
@pytest.mark.parametrize("cap", [sum(SIZES), 512, 8192])
@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("upload", ["create", "set_params"])
def test_fp32_accuracy(hp, reference, upload, path, cap):
    torch = torch_cuda()
    b, w, Eo, Fo, gE, go, e_rms = reference
    h = make_handle(hp, w if upload == "create" else 0.5 * np.asarray(w), 1, "fp32", b, max_atoms=cap)
    if upload == "set_params":
        h.set_params(torch.tensor(np.asarray(w), device="cuda"))
    h.set_knob("mlp_path", path)
    x, sp, off = to_device(torch, b, torch.float32)
    E, F = h.energy_forces(x, sp, off)
    gp, _ = h.backward(x, sp, off, torch.tensor(gE, device="cuda"), None)
    dE = np.sqrt(np.mean(((E.cpu().numpy() - Eo) / np.array(SIZES)) ** 2)) / e_rms
    dF = np.sqrt(np.mean((F.double().cpu().numpy() - Fo) ** 2) / np.mean(Fo ** 2))
    dg = np.linalg.norm(gp.double().cpu().numpy() - go) / np.linalg.norm(go)
    print(f"{upload} path {path} capacity {cap}: energy {dE:.3g} forces {dF:.3g} gradient {dg:.3g}")
    assert h.device_status() == 0
    assert dE <= 5e-7 and dF <= 3e-6 and dg <= 2e-6
    h.close()
