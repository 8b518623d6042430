"""What the autotuner tries and what it leaves open: no candidates of knobs the
handle does not read, the chunk still chosen by each call, and no choice made
among other kernels taken from a cache file."""
import json

import pytest

from paper_2201_08110_amd import synth
from tests.gpu_util import make_handle, to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _tuned(hp, prec, cap, cache):
    torch = torch_cuda()
    b = synth.random_batch(71, [70, 1, 33, 50])
    w = synth.xavier_weights(1, hp["widths"], seed=47)
    h = make_handle(hp, w, 1, prec, b, max_atoms=cap, max_mols=1000)
    x, sp, off = to_device(torch, b, torch.float32)
    return h, h.autotune(x, sp, off, reps=1, cache_path=str(cache))


@pytest.mark.parametrize("prec,cap,tried", [("fp32", 512, False), ("bf16", 154, False), ("bf16", 60000, True)])
def test_candidates(hp, prec, cap, tried, tmp_path):
    h, rep = _tuned(hp, prec, cap, tmp_path / "c")
    knobs = {k.split("=")[0] for k in rep["timings_us"]}
    assert ("gemm_stages" in knobs) == tried and ("gemm_waves" in knobs) == tried
    assert "atom_chunk" not in knobs and "force_sum" not in knobs and "force_path" in knobs
    chunk = h.get_knob("atom_chunk")                 # of a call that fills the handle
    assert chunk == (16 if cap == 60000 else 8)
    h2, rep2 = _tuned(hp, prec, cap, tmp_path / "c")
    assert rep2["cached"] and h2.get_knob("atom_chunk") == chunk
    h.set_knob("atom_chunk", 4)
    assert h.get_knob("atom_chunk") == 4


def test_choice_of_other_kernels_is_not_reused(hp, tmp_path):
    cache = tmp_path / "tune.jsonl"
    _, rep = _tuned(hp, "fp32", 512, cache)
    line = json.loads(cache.read_text())
    line["key"] = line["key"].rsplit("|", 1)[0]      # as written before the key had the kernels' revision
    cache.write_text(json.dumps(line) + "\n")
    _, rep = _tuned(hp, "fp32", 512, cache)
    assert rep["cached"] is False and len(cache.read_text().splitlines()) == 2
