"""Prefill projections at full K loops: every stage of the weight ring used several times, both columns of tile shapes, and
the row-major GEMM, against the fp32 oracle (logits, hidden state, every cached K/V row), scratch poisoned
beforehand; a second run gives the same bits."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_kv, check_logits

pytestmark = pytest.mark.gpu
# heads, head_dim, FFN width, flags (32: the projections read the caller's row-major weights).  4096 / 11000: the 7B width with
# K pieces of unequal length; 4160: K loops that end inside a stage, Q/K/V just past one round in its first shape.
MODELS = {"d8192": (64, 128, 1000, 0), "d4096": (32, 128, 11000, 0), "d4160": (65, 64, 1000, 0),
          "d4096 lean": (32, 128, 11000, 32)}


@pytest.fixture(scope="module", params=list(MODELS))
def model(request, oracle32):
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    heads, head_dim, ffn, flags = MODELS[request.param]
    cfg = wl.custom_cfg(1, heads, head_dim, ffn, 200, 720)
    w = wl.weights_astype(wl.make_weights_numpy(cfg, seed=61, gain_jitter=0.1), np.float16)
    om = oracle32.model(cfg, w)
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16), flags=flags) as s:
        yield cfg, s, om
    om.close()


@pytest.mark.parametrize("n", [50, 100, 180, 250, 300, 384, 500, 700])
def test_full_k_loops_against_the_oracle(model, n):
    cfg, s, om = model
    prompt = wl.make_tokens(n, cfg["vocab"], seed=n)
    om.reset()
    _, ref, hidden = om.prefill(prompt)
    runs = []
    for _ in range(2):
        s.ll_reset()
        s.ll_dbg_poison_scratch()
        s.ll_prefill(prompt)
        runs.append([s.ll_dbg_get_logits(), s.ll_dbg_get_hidden()] + [s.ll_dbg_get_kv(0, which, n) for which in range(2)])
    check_logits(runs[0][0], ref, "prompt %d" % n)
    check_logits(runs[0][1], hidden, "prompt %d hidden" % n, max_abs_tol=3e-2 * max(1.0, float(np.abs(hidden).max())))
    for which in range(2):
        check_kv(runs[0][2 + which], om.kv(0, which), "prompt %d %s" % (n, "KV"[which]))
    assert all(a.tobytes() == b.tobytes() for a, b in zip(*runs)), "two runs of prompt %d differ" % n
