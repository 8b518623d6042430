"""Neighbour records and bucket rows formed inside the featuriser: molecules at
the edges of a wave's one and two candidates a lane and of the step beyond
them, with the bucketing fused in and (more than 4,096 atoms) beside it,
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
    [128] * 8 + [3],                   # more than one bucketing block
    [128] * 32,                        # 4,096 atoms: the last batch with fused bucketing
    [128] * 32 + [3],                  # the first without
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


def _packed(n, edge, seed, elements):
    """n atoms, 1 A lattice sites of a cube taken at random (each atom has many
    neighbours), the given elements in turn."""
    rng = np.random.default_rng(seed)
    g = np.arange(int(edge) + 1) * 1.0
    sites = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    pos = sites[rng.permutation(len(sites))[:n]] + rng.uniform(-0.05, 0.05, (n, 3))
    return pos, np.array([elements[i % len(elements)] for i in range(n)], dtype=np.int32)


@pytest.mark.parametrize("model,elements", [
    ("ani2x", [0]),                    # one block over many batches of pairs
    ("ani2x", [6, 0, 5]),              # the last elements, runs longer than one list
    ("ani2x", [0, 1, 2, 3, 4, 5, 6]),  # every block, short runs
    ("ani1x", [3, 1]),                 # four distance shifts x eight angles
])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_slot_sums_of_many_neighbours(orc, hp, model, elements, prec):
    """AEV rows where a slot's sum runs over several lists and batches; FP32
    within 1e-5 of a row's largest slot (some hundred terms of 1e-7 each)."""
    torch = torch_cuda()
    from paper_2201_08110_amd import synth
    hp = synth.ani1x_hparams() if model == "ani1x" else hp
    sizes = [3, 64, 5]
    b = synth.random_batch(11, sizes, ratio=[1.0] * hp["n_species"])
    pos, sp = _packed(64, 4, 5, elements)
    b.coords[3:67], b.species[3:67] = pos, sp
    w = synth.xavier_weights(1, hp.get("species_widths") or hp["widths"], hp["n_species"], seed=9)
    h = make_handle(hp, w, 1, prec, b)
    x, s, off = to_device(torch, b, torch.float64 if prec == "fp64" else torch.float32)
    G = h.aev(x, s, off).double().cpu().numpy()
    xo = x.double().cpu().numpy()
    o = b.mol_offsets
    Go = np.concatenate([orc.aev(hp, b.species[p:q], xo[p:q]) for p, q in zip(o[:-1], o[1:])])
    tol = 1e-11 if prec == "fp64" else 1e-5
    assert (np.abs(G - Go).max(1) <= tol * np.maximum(np.abs(Go).max(1), 1.0)).all()
    h.close()


@pytest.mark.parametrize("model,elements,chunk", [
    ("ani2x", [0], 4),                 # one block over many batches of pairs
    ("ani2x", [6, 0, 5, 1], 16),
    ("ani1x", [3, 1], 4),              # four distance shifts x eight angles
])
def test_fp32_row_tangents(orc, hp, model, elements, chunk):
    """Parameter gradients of a force term alone, which reach the parameters
    through the rows' tangents only; the bound is that of the other FP32
    parameter gradients."""
    torch = torch_cuda()
    hp = synth.ani1x_hparams() if model == "ani1x" else hp
    b = synth.random_batch(13, [3, 64, 5], ratio=[1.0] * hp["n_species"])
    b.coords[3:67], b.species[3:67] = _packed(64, 5, 6, elements)
    w = synth.xavier_weights(1, hp.get("species_widths") or hp["widths"], hp["n_species"], seed=9)
    h = make_handle(hp, w, 1, "fp32", b)
    h.set_knob("atom_chunk", chunk)
    x, s, off = to_device(torch, b, torch.float32)
    gF = np.random.default_rng(4).normal(size=(int(b.n_atoms), 3)).astype(np.float32) * 1e-2
    gE = np.zeros(b.n_mols)
    gp, _ = h.backward(x, s, off, torch.tensor(gE, device="cuda"), torch.tensor(gF, device="cuda"))
    torch.cuda.synchronize()
    assert h.device_status() == 0
    go = orc.param_grad(hp, synth.round_to_fp32(w), 1, b.species, x.double().cpu().numpy(), b.mol_offsets, gE,
                        gF.astype(np.float64))
    err = np.linalg.norm(gp.cpu().numpy() - go) / np.linalg.norm(go)
    assert err < 1e-4
    h.close()


@pytest.mark.parametrize("sizes", [
    [3] * 1023 + [2],                  # 1,024 molecules: the last FP64 batch with fused bucketing
    [3] * 1023 + [2, 4],               # the first without
    [2, 1, 0] * 1000,                  # most of them empty or one atom
    [0, 1] * 4096, [0, 1] * 4096 + [0],   # the last FP32 batch with it and the first without
])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_many_small_molecules(orc, hp, sizes, prec):
    """At most 4,096 atoms in about a thousand molecules and more."""
    test_records_and_rows_match_oracle(orc, hp, sizes, prec, 0)
