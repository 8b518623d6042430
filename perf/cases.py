"""The work this library is used for, as cases that can be timed and compared.

Each case is one pass through the public entry points of the package: energies
and forces of a batch, a training step, the NNP-MM coupling, or the whole force
step of an NNP/MM simulation.  Molecules are seeded random structures of the
element mix, density and sizes of the repository's own workloads
(paper_2201_08110_amd/synth.py); the molecule sizes of a batch follow from the
case alone, so that its work does, and the seed decides coordinates and
elements.

Energies leave the library in FP64 whatever the handle's precision.  The cases
hand them on in the handle's coordinate type, which is what an FP32 or BF16
program keeps: the sum is exact, its terms are not.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2201_08110_amd import synth
from paper_2201_08110_amd.autograd import nnp_energy_forces
from paper_2201_08110_amd.nnp import NNP, Coupling
from paper_2201_08110_amd.nnpmm import NNPMMStep

DEVICE = "cuda:0"
#: element ratio over H, C, N, O for the four-element model
RATIO_HCNO = (22, 15, 5, 6)
#: edge of a molecule's cube per cube root of its atoms (Angstrom)
EDGE = 2.2
#: learning rate of the training step: small, so that passes stay alike
LR = 1e-9
FORCE_WEIGHT = 0.1


def _case(name, kind, precision, mols, lo, hi, models=8, model="ani2x", **more):
    c = dict(kind=kind, precision=precision, mols=mols, lo=lo, hi=hi, models=models, model=model,
             replicas=False, graph=False, cap_mols=mols, mm=0, grad_x=False)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one ligand per call, the shape of a simulation step with one NNP
        # region: latency and launches count (single precision, 8 networks)
        _case("ligand64_fp32", "evaluate", "fp32", 1, 64, 64),
        # the same with the networks in BF16
        _case("ligand64_bf16", "evaluate", "bf16", 1, 64, 64),
        # one small molecule in double precision with a single network: what
        # a user checks a force field or an integrator with
        _case("molecule24_fp64", "evaluate", "fp64", 1, 24, 24, models=1),
        # a handful of ligands in one call (several replicas of a simulation,
        # one docking pose each, ...)
        _case("mols16_fp32", "evaluate", "fp32", 16, 10, 60),
        # a serving loop: batches of up to 128 molecules through one captured
        # graph, their counts on the device, this one holding 48
        _case("serve48_bf16", "evaluate", "bf16", 48, 10, 120, graph=True, cap_mols=128),
        # a large batch of molecules of many sizes, both precisions
        _case("ragged512_fp32", "evaluate", "fp32", 512, 10, 120),
        _case("ragged512_bf16", "evaluate", "bf16", 512, 10, 120),
        # many replicas of one ligand: the largest call, the benchmark's own
        _case("replicas1024_bf16", "evaluate", "bf16", 1024, 48, 48, replicas=True),
        # one big molecule: neighbour search through cutoff cells
        _case("large600_fp32", "evaluate", "fp32", 1, 600, 600),
        # a training step with a loss of energies and forces: forward, the
        # hand-written backward, the update and the new weights' upload
        _case("train64_fp32", "train", "fp32", 64, 30, 80),
        # the coupling term of a ligand in a solvated protein (47,712 atoms)
        _case("coupling64_fp32", "coupling", "fp32", 1, 64, 64, mm=47648),
        # the whole force step of that simulation: networks and coupling
        _case("nnpmm64_fp32", "nnpmm", "fp32", 1, 64, 64, mm=47648, graph=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evaluate"] * 6 + ["train"] * 2 + ["coupling", "nnpmm"])
    if kind == "coupling":
        n = rng.randint(20, 120)
        return _case(None, kind, rng.choice(["fp32", "fp64"]), 1, n, n, mm=_log(rng, 1000, 47648))
    if kind == "nnpmm":
        n = rng.randint(30, 90)
        return _case(None, kind, rng.choice(["fp32", "fp32", "bf16"]), 1, n, n, mm=_log(rng, 4000, 47648),
                     graph=True)
    model = rng.choice(["ani2x", "ani2x", "ani2x", "ani2x_elements", "ani1x"])
    if kind == "train":
        lo = rng.randint(10, 40)
        return _case(None, kind, "fp32", _log(rng, 4, 64), lo, lo + rng.randint(0, 40), model=model,
                     grad_x=rng.random() < 0.3)
    precision = rng.choice(["fp32", "fp32", "bf16", "bf16", "fp64"])
    shape = rng.choice(["one", "ragged", "ragged", "replicas"])
    if shape == "one":
        n = _log(rng, 12, 256 if precision == "fp64" else 900)
        return _case(None, kind, precision, 1, n, n, models=rng.choice([1, 8]), model=model)
    most = {"fp64": 24, "fp32": 512, "bf16": 512}[precision]
    mols = _log(rng, 4, most)
    if shape == "replicas":
        n = rng.randint(24, 64)
        return _case(None, kind, precision, mols, n, n, model=model, replicas=True)
    lo = rng.randint(5, 40)
    hi = min(120, lo + rng.randint(5, 80))
    graph = precision != "fp64" and rng.random() < 0.3
    return _case(None, kind, precision, mols, lo, hi, model=model, graph=graph,
                 cap_mols=mols * 2 if graph else mols)


# ---------------------------------------------------------------------------
# inputs


def _hparams(model):
    return {"ani2x": synth.ani2x_hparams, "ani2x_elements": synth.ani2x_heterogeneous_hparams,
            "ani1x": synth.ani1x_hparams}[model]()


def _ratio(model):
    return RATIO_HCNO if model == "ani1x" else synth.LIGAND_RATIO


@functools.lru_cache(maxsize=6)
def _weights(model, models):
    hp = _hparams(model)
    return synth.xavier_weights(models, hp.get("species_widths") or hp["widths"], hp["n_species"])


def _sizes(case):
    """Molecule sizes lo..hi in a low-discrepancy order."""
    lo, hi, n = case["lo"], case["hi"], case["mols"]
    return [lo + int((hi - lo + 1) * ((0.5 + k * 0.6180339887498949) % 1.0)) for k in range(n)]


def _place(sizes, g):
    """[A, 3] FP64 coordinates: every molecule is filled atom by atom, a
    uniform candidate in its cube accepted at least 1 Angstrom from the atoms
    before it (all molecules at once; of 64 candidates the first accepted one,
    or the farthest if none is)."""
    B, N = len(sizes), max(sizes)
    size = torch.tensor(sizes, device=DEVICE)
    edge = (size.double() ** (1.0 / 3.0) * EDGE)[:, None, None]
    pos = torch.full((B, N, 3), 1e6, dtype=torch.float64, device=DEVICE)
    cand = torch.rand((N, B, 64, 3), generator=g, dtype=torch.float64, device=DEVICE) * edge
    pos[:, 0] = cand[0, :, 0]
    for k in range(1, N):
        d2 = ((cand[k][:, :, None, :] - pos[:, None, :k, :]) ** 2).sum(-1).amin(-1)      # [B, 64]
        score = torch.where(d2 >= 1.0, 4e6 - torch.arange(64, device=DEVICE), d2)
        pos[:, k] = cand[k].gather(1, score.argmax(1)[:, None, None].expand(B, 1, 3))[:, 0]
    keep = torch.arange(N, device=DEVICE)[None, :] < size[:, None]
    return pos[keep]


def _elements(case, sizes, g):
    ratio = _ratio(case["model"])
    if case["mols"] == 1 or case["replicas"]:
        counts = synth.rounded_counts(sizes[0], ratio)
        sp = torch.repeat_interleave(torch.arange(len(ratio), device=DEVICE),
                                     torch.tensor(counts, device=DEVICE))
        sp = sp[torch.randperm(sizes[0], generator=g, device=DEVICE)]
        return sp.repeat(len(sizes)).int().contiguous()
    p = torch.tensor(ratio, dtype=torch.float32, device=DEVICE)
    return torch.multinomial(p, sum(sizes), replacement=True, generator=g).int()


def _molecules(case, seed):
    """coords [A, 3] in the handle's coordinate type, element indices, offsets."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    sizes = _sizes(case)
    if case["replicas"]:
        base = _place(sizes[:1], g)
        x = base.repeat(len(sizes), 1)
        x = x + 0.05 * torch.randn(x.shape, generator=g, dtype=torch.float64, device=DEVICE)
    else:
        x = _place(sizes, g)
    sp = _elements(case, sizes, g)
    off = torch.zeros(len(sizes) + 1, dtype=torch.int32)
    off[1:] = torch.cumsum(torch.tensor(sizes), 0).int()
    dt = torch.float64 if case["precision"] == "fp64" else torch.float32
    return x.to(dt).contiguous(), sp, off.to(DEVICE), g


def _surroundings(case, x_nnp, g):
    """MM atoms at liquid density around the ligand, at least 2.2 Angstrom
    from it, with charges and Lennard-Jones parameters for both sides."""
    n, m, dt = x_nnp.shape[0], case["mm"], x_nnp.dtype
    lig = x_nnp.double()
    edge = max((m / 0.1) ** (1.0 / 3.0), 2.0 * (float(lig.abs().max()) + 2.2) + 8.0)
    got, total = [], 0
    while total < m:
        cand = (torch.rand((2 * m, 3), generator=g, dtype=torch.float64, device=DEVICE) - 0.5) * edge
        d2 = torch.cat([((c[:, None, :] - lig[None]) ** 2).sum(-1).amin(1) for c in cand.split(16384)])
        got.append(cand[d2 >= 2.2 ** 2])
        total += got[-1].shape[0]
    x_mm = torch.cat(got)[:m]

    def parameters(k, scale):
        q = scale * torch.randn(k, generator=g, dtype=torch.float64, device=DEVICE)
        u = torch.rand((2, k), generator=g, dtype=torch.float64, device=DEVICE)
        return torch.stack([q - q.mean(), 2.4 + 1.2 * u[0], 0.02 + 0.18 * u[1]], 1).to(dt).contiguous()

    return x_mm.to(dt).contiguous(), parameters(n, 0.25), parameters(m, 0.35)


def _inputs(case, seed):
    x, sp, off, g = _molecules(case, seed)
    s = dict(case=case, x=x, sp=sp, off=off)
    if case["mm"]:
        s["x"] = x = (x - x.mean(0)).contiguous()
        s["x_mm"], s["par"], s["par_mm"] = _surroundings(case, x, g)
        s["F_engine"] = torch.randn(s["x_mm"].shape, generator=g, dtype=torch.float64, device=DEVICE).to(x.dtype)
    if case["kind"] == "train":
        s["E_ref"] = 100.0 * torch.randn(case["mols"], generator=g, dtype=torch.float64, device=DEVICE)
        s["F_ref"] = 10.0 * torch.randn(x.shape, generator=g, dtype=x.dtype, device=DEVICE)
    return s


@functools.lru_cache(maxsize=1)
def _stream():
    """The one stream a serving loop or a simulation runs on."""
    return torch.cuda.Stream()


def prepare(case, seed):
    s = _inputs(case, seed)
    x = s["x"]
    s["E"] = torch.zeros(case["mols"], dtype=torch.float64, device=DEVICE)
    s["F"] = torch.zeros_like(x)
    if case["mm"]:
        s["F_mm"] = torch.zeros_like(s["x_mm"])
        s["coupling"] = Coupling(x.shape[0], case["mm"], synth.COULOMB_K, precision="fp64"
                                 if case["precision"] == "fp64" else "fp32")
    if case["kind"] == "coupling":
        return s
    sizes = _sizes(case)
    cap = case["cap_mols"]
    atoms = sum(sizes) if cap == case["mols"] else cap * case["hi"]
    s["model"] = NNP(_hparams(case["model"]), _weights(case["model"], case["models"]), case["models"],
                     case["precision"], max_atoms=atoms, max_mols=cap, max_atoms_per_mol=max(sizes),
                     training=case["kind"] == "train")
    if case["kind"] == "train":
        s["params"] = torch.tensor(_weights(case["model"], case["models"]), dtype=torch.float32,
                                   device=DEVICE, requires_grad=True)
        if case["grad_x"]:
            x.requires_grad_(True)
    if case["graph"]:
        s["stream"] = _stream()
    if case["kind"] == "nnpmm":
        s["step"] = NNPMMStep(s["model"], s["coupling"], s["sp"], s["off"], s["par"], s["par_mm"])
    elif case["graph"]:
        s["counts"] = torch.tensor([case["mols"], sum(sizes)], dtype=torch.int32, device=DEVICE)
    return s


# ---------------------------------------------------------------------------
# one pass


def run(s):
    kind = s["case"]["kind"]
    if kind == "coupling":
        E, F, F_mm = s["coupling"](s["x"], s["par"], s["x_mm"], s["par_mm"], out=(s["E"], s["F"], s["F_mm"]))
        return {"E": E.to(F.dtype), "F": F, "F_mm": F_mm}
    if kind == "nnpmm":
        with torch.cuda.stream(s["stream"]):
            s["F_mm"].copy_(s["F_engine"])
            E, F, F_mm = s["step"](s["x"], s["x_mm"], s["E"], s["F"], s["F_mm"], s["stream"])
            return {"E": E.to(F.dtype), "F": F, "F_mm": F_mm}
    if kind == "train":
        x, params = s["x"], s["params"]
        E, F = nnp_energy_forces(s["model"], x, params, s["sp"], s["off"])
        loss = ((E - s["E_ref"]) ** 2).mean() + FORCE_WEIGHT * ((F - s["F_ref"]) ** 2).mean()
        params.grad = x.grad = None
        loss.backward()
        with torch.no_grad():
            params.sub_(params.grad, alpha=LR)
        out = {"E": E.detach().to(F.dtype), "F": F.detach(), "grad": params.grad}
        if x.grad is not None:
            out["grad_x"] = x.grad
        return out
    if s["case"]["graph"]:
        with torch.cuda.stream(s["stream"]):
            E, F = s["model"].energy_forces(s["x"], s["sp"], s["off"], out=(s["E"], s["F"]), graph=True,
                                            stream=s["stream"], counts=s["counts"])
            return {"E": E.to(F.dtype), "F": F}
    E, F = s["model"].energy_forces(s["x"], s["sp"], s["off"], out=(s["E"], s["F"]))
    return {"E": E.to(F.dtype), "F": F}


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    real = 8 if case["precision"] == "fp64" else 4
    weight = {"fp64": 8, "fp32": 4, "bf16": 2}[case["precision"]]
    atoms, mm = sum(_sizes(case)), case["mm"]
    nbytes, flops = 0.0, 0.0
    if mm:
        # 33 operations a pair; positions and parameters in, forces out
        flops += 33.0 * atoms * mm
        nbytes += real * (6 * (atoms + mm) + 3 * (atoms + mm))
    if case["kind"] == "coupling":
        return {"bytes": nbytes, "flops": flops}
    hp = _hparams(case["model"])
    per = hp.get("species_widths") or [hp["widths"]] * hp["n_species"]
    share = np.asarray(_ratio(case["model"]), dtype=float)
    share /= share.sum()
    products = [sum(a * b for a, b in zip(w, w[1:])) for w in per]
    inner = [sum(a * b for a, b in zip(w[1:], w[2:])) for w in per]
    p, q = float(share @ products), float(share @ inner)
    # forward and the backward to the features
    per_atom = 4.0 * p
    nbytes += atoms * (6 * real + 4) + 8 * case["mols"]
    if case["kind"] == "train":
        # tangents along the force cotangent, two adjoint streams below the
        # last layer, both halves of every weight gradient; weights read,
        # gradients written, weights updated
        per_atom += 2.0 * p + 4.0 * q + 4.0 * p + (2.0 * p if case["grad_x"] else 0.0)
        nbytes += 3 * 4 * case["models"] * sum(products)
    else:
        nbytes += weight * case["models"] * sum(products)
    flops += case["models"] * atoms * per_atom
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# the same results from plain torch in 64 bits


def _cutoff(r, rc):
    return 0.5 * torch.cos(math.pi * r / rc) + 0.5


def _lists(x, sizes, rc):
    """Ordered neighbour pairs (i, j) with r < rc, sorted by i, over a batch."""
    B, N = len(sizes), max(sizes)
    size = torch.tensor(sizes, device=DEVICE)
    start = torch.cumsum(size, 0) - size
    keep = torch.arange(N, device=DEVICE)[None, :] < size[:, None]
    pad = torch.full((B, N, 3), 1e6, dtype=torch.float64, device=DEVICE)
    pad[keep] = x
    d2 = torch.zeros((B, N, N), dtype=torch.float64, device=DEVICE)
    for c in range(3):
        d2 += (pad[:, :, None, c] - pad[:, None, :, c]) ** 2
    ok = (d2 < rc * rc) & keep[:, :, None] & keep[:, None, :]
    ok &= ~torch.eye(N, dtype=torch.bool, device=DEVICE)
    b, i, j = ok.nonzero(as_tuple=True)
    return start[b] + i, start[b] + j


def _features(hp, x, sp, sizes):
    """AEV rows [A, D], differentiable in x."""
    A, S = x.shape[0], hp["n_species"]
    shf_r, shf_a, shf_z = (torch.tensor(hp[k], dtype=torch.float64, device=DEVICE)
                           for k in ("shf_r", "shf_a", "shf_z"))
    nR, nAZ = len(shf_r), len(shf_a) * len(shf_z)
    xd = x.detach()
    i, j = _lists(xd, sizes, hp["rcr"])
    r = (x[j] - x[i]).norm(dim=1)
    rad = hp["radial_pref"] * torch.exp(-hp["eta_r"] * (r[:, None] - shf_r) ** 2) * _cutoff(r, hp["rcr"])[:, None]
    G_r = torch.zeros((A * S, nR), dtype=torch.float64, device=DEVICE).index_add(0, i * S + sp[j], rad)
    i, j = _lists(xd, sizes, hp["rca"])
    count = torch.bincount(i, minlength=A)
    rank = torch.arange(len(i), device=DEVICE) - (torch.cumsum(count, 0) - count)[i]
    later = count[i] - rank - 1                      # neighbours of the same atom after this one
    e1 = torch.repeat_interleave(torch.arange(len(i), device=DEVICE), later)
    e2 = e1 + 1 + torch.arange(len(e1), device=DEVICE) - (torch.cumsum(later, 0) - later)[e1]
    d = x[j] - x[i]
    r = d.norm(dim=1)
    fc = _cutoff(r, hp["rca"])
    c = hp["angle_scale"] * (d[e1] * d[e2]).sum(1) / (r[e1] * r[e2])
    cz = c[:, None] * torch.cos(shf_z) + torch.sqrt(1.0 - c * c)[:, None] * torch.sin(shf_z)
    ang = 2.0 * ((1.0 + cz) / 2.0) ** hp["zeta"]
    dist = torch.exp(-hp["eta_a"] * (0.5 * (r[e1] + r[e2])[:, None] - shf_a) ** 2) * (fc[e1] * fc[e2])[:, None]
    lo, hi = torch.minimum(sp[j[e1]], sp[j[e2]]), torch.maximum(sp[j[e1]], sp[j[e2]])
    NB = S * (S + 1) // 2
    block = lo * S - lo * (lo - 1) // 2 + (hi - lo)
    G_a = torch.zeros((A * NB, nAZ), dtype=torch.float64, device=DEVICE).index_add(
        0, i[e1] * NB + block, (dist[:, :, None] * ang[:, None, :]).flatten(1))
    return torch.cat([G_r.view(A, S * nR), G_a.view(A, NB * nAZ)], 1)


def _energies(hp, models, w, x, sp, sizes):
    """Energies [B] of the ensemble mean, differentiable in x and w."""
    S, al = hp["n_species"], hp["celu_alpha"]
    per = hp.get("species_widths") or [hp["widths"]] * S
    G = _features(hp, x, sp, sizes)
    mol = torch.repeat_interleave(torch.arange(len(sizes), device=DEVICE), torch.tensor(sizes, device=DEVICE))
    E = torch.zeros(len(sizes), dtype=torch.float64, device=DEVICE)
    rows = [(sp == s).nonzero()[:, 0] for s in range(S)]
    at = 0
    for _ in range(models):
        for s in range(S):
            a = G[rows[s]]
            for l, (n, k) in enumerate(zip(per[s][1:], per[s])):
                W, b = w[at:at + n * k].view(n, k), w[at + n * k:at + n * k + n]
                at += n * k + n
                a = a @ W.t() + b
                if l + 2 < len(per[s]):
                    a = torch.nn.functional.celu(a, al)
            E = E.index_add(0, mol[rows[s]], a[:, 0])
    return hp["energy_scale"] * E / models


def _coupling(s):
    """Energy and forces of the coupling, atom pairs in blocks."""
    x, p, xm, pm = (s[k].double() for k in ("x", "par", "x_mm", "par_mm"))
    F, F_mm, E = torch.zeros_like(x), torch.zeros_like(xm), 0.0
    for a in range(0, xm.shape[0], 8192):
        b = slice(a, a + 8192)
        d = xm[b][None, :, :] - x[:, None, :]
        r2 = (d * d).sum(-1)
        r = r2.sqrt()
        coul = synth.COULOMB_K * p[:, None, 0] * pm[b][None, :, 0] / r
        s6 = ((0.5 * (p[:, None, 1] + pm[b][None, :, 1])) ** 2 / r2) ** 3
        eps = torch.sqrt(p[:, None, 2] * pm[b][None, :, 2])
        E = E + (coul + 4.0 * eps * (s6 * s6 - s6)).sum()
        f = ((coul + 4.0 * eps * (12.0 * s6 * s6 - 6.0 * s6)) / r2)[..., None] * d     # on the MM atom
        F_mm[b] += f.sum(0)
        F -= f.sum(1)
    return E.reshape(1), F, F_mm


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "coupling":
        E, F, F_mm = _coupling(s)
        return {"E": E, "F": F, "F_mm": F_mm}
    hp, M, sizes = _hparams(case["model"]), case["models"], _sizes(case)
    train = case["kind"] == "train"
    w = torch.tensor(_weights(case["model"], M), dtype=torch.float64, device=DEVICE)
    if train:
        w = w.float().double().requires_grad_(True)
    x = s["x"].detach().double().requires_grad_(True)
    E = _energies(hp, M, w, x, s["sp"].long(), sizes)
    F = -torch.autograd.grad(E.sum(), x, create_graph=train)[0]
    if train:
        loss = ((E - s["E_ref"]) ** 2).mean() + FORCE_WEIGHT * ((F - s["F_ref"].double()) ** 2).mean()
        grads = torch.autograd.grad(loss, [w, x] if case["grad_x"] else [w])
        out = {"E": E.detach(), "F": F.detach(), "grad": grads[0]}
        if case["grad_x"]:
            out["grad_x"] = grads[1]
        return out
    out = {"E": E.detach(), "F": F.detach()}
    if case["kind"] == "nnpmm":
        E_c, F_c, F_mm = _coupling(s)
        out = {"E": out["E"] + E_c, "F": out["F"] + F_c, "F_mm": s["F_engine"].double() + F_mm}
    return out
