"""FP32 weights at the upper end of the range: the largest bf16 is 3.3895e38, so a
finite FP32 value above it must not become infinite as the first of its three
bf16 parts.  One weight of 3.4e38 in layer 1, 2 or 3, in the buckets of both
row sizes, by creation and from device memory, against the FP64 oracle: the
energy is that weight's term and relative 1e-5 of it."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, oracle_inputs, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("cap", [64, 512])
@pytest.mark.parametrize("layer", [0, 1, 2])
def test_weight_above_the_largest_bf16(orc, hp, layer, cap, path):
    torch = torch_cuda()
    b = synth.random_batch(31, [40])
    w = np.array(synth.xavier_weights(1, hp["widths"], seed=8))
    widths, at, W = hp["widths"], 0, []
    for k, n in zip(widths, widths[1:]):             # element 0's network
        W.append((w[at:at + n * k].reshape(n, k), w[at + n * k:at + n * k + n]))
        at += n * k + n
    if layer > 0:                                    # its input to the weight: CELU(0.01) for every atom
        W[layer - 1][0][0] = 0.0
        W[layer - 1][1][0] = 0.01
    W[layer][0][0, 5 if layer == 0 else 0] = 3.4e38
    x, sp, off = to_device(torch, b, torch.float32)
    xo, wo = oracle_inputs(b, w, "fp32")
    Eo, _ = orc.energy_forces(hp, wo, 1, b.species, xo, b.mol_offsets)
    assert abs(Eo[0]) > 1e30
    h = make_handle(hp, w, 1, "fp32", b, max_atoms=cap)
    h.set_knob("mlp_path", path)
    E, _ = h.energy_forces(x, sp, off)
    h.set_params(torch.tensor(w, device="cuda"))
    E2, _ = h.energy_forces(x, sp, off)
    print(layer, cap, path, Eo[0], float(E), float(E2))
    assert abs(float(E) - Eo[0]) <= 1e-5 * abs(Eo[0])
    assert float(E2) == float(E)
    h.close()


def test_infinite_weight_beside_the_end_of_k(hp):
    """FP64 layer 1 of the smallest handles splits K over waves, whose shares may
    end past K: an infinite weight in the last columns multiplies the features
    alone, as on a handle whose capacity takes the other kernel."""
    torch = torch_cuda()
    hp = synth.ani1x_hparams()                       # 384 features: 48 steps of 8 for 64 places
    b = synth.random_batch(33, [30], ratio=(30, 20, 5, 5))
    w = np.array(synth.xavier_weights(1, hp["species_widths"], n_species=4, seed=9))
    x, sp, off = to_device(torch, b, torch.float64)
    D, at, got = 384, 0, []
    big = make_handle(hp, w, 1, "fp64", b, max_atoms=1024)
    G = big.aev(x, sp, off).cpu().numpy()
    col = 376 + int(np.argmax((G[:, 376:] > 0).sum(0)))
    assert (G[:, col] > 0).any()
    for s, ws in enumerate(hp["species_widths"]):    # unit 0 of every element's first layer
        w[at + col] = -np.inf
        at += sum(n * (k + 1) for k, n in zip(ws, ws[1:]))
    for h in (make_handle(hp, w, 1, "fp64", b), make_handle(hp, w, 1, "fp64", b, max_atoms=1024)):
        E, _ = h.energy_forces(x, sp, off)
        got.append(float(E))
        h.close()
    assert abs(got[0] - got[1]) <= 1e-10 * abs(got[1])


@pytest.mark.parametrize("cap", [64, 512])
@pytest.mark.parametrize("upload", ["create", "set_weights", "set_params"])
def test_infinite_fp32_weight(hp, upload, cap):
    """-infinity in layer 1 ends where the largest negative weight does, for atoms
    with and without the feature."""
    torch = torch_cuda()
    b = synth.random_batch(31, [40])
    w0 = np.array(synth.xavier_weights(1, hp["widths"], seed=8))
    x, sp, off = to_device(torch, b, torch.float32)
    E = []
    for v in (-3.402e38, -np.inf):
        w = w0.copy()
        w[5] = v                                     # hydrogen's unit 0, a radial feature of hydrogen neighbours
        h = make_handle(hp, w if upload == "create" else w0, 1, "fp32", b, max_atoms=cap)
        if upload == "set_weights":
            h.set_weights(w)
        elif upload == "set_params":
            h.set_params(torch.tensor(w, device="cuda"))
        E.append(float(h.energy_forces(x, sp, off)[0]))
        h.close()
    assert E[0] == E[1]
