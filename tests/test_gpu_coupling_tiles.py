"""Sizes at the edges of the coupling kernel's tiles (16 MM atoms a wave, 64 NNP
atoms a pass, 16 x 16 pairs a row of lanes, 256 workgroups) against the FP64
oracle, with the bars of the full system's tests."""
import numpy as np
import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import torch_cuda

pytestmark = pytest.mark.gpu
K = synth.COULOMB_K


def _side(rng, n, lo, hi):
    q = rng.normal(0.0, 0.3, n)
    return rng.uniform(lo, hi, (n, 3)), np.stack([q, rng.uniform(2.4, 3.6, n), rng.uniform(0.02, 0.2, n)], 1)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_nnp,n_mm,cutoff", [
    (1, 15, 0.0), (16, 16, 0.0), (17, 17, 0.0), (64, 63, 9.0), (63, 65, 0.0), (128, 1023, 12.0),
    (65, 16 * 256 * 16 + 1, 0.0), (1024, 300, 0.0)])
def test_tile_edges(orc, prec, n_nnp, n_mm, cutoff):
    torch = torch_cuda()
    from paper_2201_08110_amd.nnp import Coupling
    rng = np.random.default_rng(n_nnp + n_mm)
    dt = torch.float64 if prec == "fp64" else torch.float32
    xn, pn = _side(rng, n_nnp, 0.0, 12.0)
    xm, pm = _side(rng, n_mm, 14.0, 40.0)
    if prec == "fp32":
        xn, pn, xm, pm = (synth.round_to_fp32(a) for a in (xn, pn, xm, pm))
    c = Coupling(n_nnp, n_mm, K, cutoff, prec)
    t = [torch.tensor(a, dtype=dt, device="cuda") for a in (xn, pn, xm, pm)]
    base = torch.tensor(rng.normal(size=(n_mm, 3)), dtype=dt, device="cuda")
    out = (torch.full((1,), 2.5, dtype=torch.float64, device="cuda"), torch.ones_like(t[0]), base.clone())
    E, Fn, Fm = c(*t, out=out, accumulate=True)
    E2, Fn2, Fm2 = c(*t)
    Eo, Fno, Fmo, A = orc.coupling(xn, pn, xm, pm, K, cutoff=cutoff, with_abs=True)
    scale = max(np.abs(Fno).max(), np.abs(Fmo).max(), 1.0)
    e_tol, f_tol = (1e-11, 1e-10) if prec == "fp64" else (5e-6, 1e-4)
    assert abs(float(E2) - Eo) <= e_tol * max(A, 1.0)
    for got, want in ((Fn2, Fno), (Fm2, Fmo), (Fn - 1.0, Fno), (Fm - base, Fmo)):
        assert np.abs(got.double().cpu().numpy() - want).max() <= f_tol * scale
    assert abs(float(E) - 2.5 - Eo) <= e_tol * max(A, 2.5)
    again = c(*t)
    assert all(torch.equal(a, b) for a, b in zip(again, (E2, Fn2, Fm2)))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_nnp,n_mm", [(65, 300), (130, 5000), (1024, 33), (70, 16 * 4096 + 5), (70, 8 * 16 * 4096 + 21)])
def test_accumulated_mm_forces_are_rounded_once(prec, n_nnp, n_mm):
    """An MM force is summed over all NNP atoms before it meets the caller's:
    bitwise the caller's force plus the force alone, where adding a block of
    NNP atoms at a time rounds at the caller's size once a block."""
    torch = torch_cuda()
    from paper_2201_08110_amd.nnp import Coupling
    rng = np.random.default_rng(n_nnp + n_mm)
    dt = torch.float64 if prec == "fp64" else torch.float32
    sides = (*_side(rng, n_nnp, 0.0, 12.0), *_side(rng, n_mm, 14.0, 60.0))
    t = [torch.tensor(a, dtype=dt, device="cuda") for a in sides]
    base = torch.tensor(100.0 * rng.normal(size=(n_mm, 3)), dtype=dt, device="cuda")
    c = Coupling(n_nnp, n_mm, K, 0.0, prec)
    _, _, Fm = c(*t)
    out = (torch.zeros(1, dtype=torch.float64, device="cuda"), torch.zeros_like(t[0]), base.clone())
    c(*t, out=out, accumulate=True)
    assert torch.equal(out[2], base + Fm)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_nnp,n_mm,cutoff", [
    (65, 40, 0.0),                     # two waves a group
    (300, 3000, 30.0),                 # eight, three of them without a block
    (600, 10000, 0.0),                 # four, each several blocks
    (600, 16 * 1024, 30.0), (600, 16 * 1024 + 1, 0.0),   # the last sizes with four, the first with two
    (129, 16 * 2048 + 1, 0.0),         # the first without
])
def test_blocks_shared_by_waves(orc, prec, n_nnp, n_mm, cutoff):
    """Few groups: the blocks of 64 NNP atoms are dealt out among several waves."""
    test_tile_edges(orc, prec, n_nnp, n_mm, cutoff)
