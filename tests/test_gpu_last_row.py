"""The last layer of a prefill runs for the prompt's last row: logits and hidden state against the fp32 oracle, scratch poisoned
beforehand, where that row's kernels differ: one layer (the residual row is the embedding), more sums of squares than 16 lanes
hold at once (d_model 4160), a number of them that 16 does not divide, both head sizes, attention in 1024 threads
(max_seq above 2048) and behind an earlier chunk."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_greedy_token, check_logits

pytestmark = pytest.mark.gpu
# layers, heads, head_dim, FFN width, max_seq, prompts
MODELS = {"one layer": (1, 3, 64, 200, 80, (1, 2, 16, 17, 32, 33, 79)), "d4160": (2, 65, 64, 1000, 80, (1, 16, 17, 32, 33, 70)),
          "d2688": (2, 21, 128, 1000, 80, (1, 16, 31, 64)), "long hd64": (2, 2, 64, 136, 2100, (5, 30, 40, 1025, 1040, 2099)),
          "long hd128": (2, 2, 128, 264, 2100, (5, 30, 40, 1025, 1064, 2099))}


@pytest.fixture(scope="module", params=list(MODELS))
def model(request, oracle32):
    layers, heads, head_dim, ffn, max_seq, prompts = MODELS[request.param]
    cfg = wl.custom_cfg(layers, heads, head_dim, ffn, 200, max_seq)
    w = wl.weights_astype(wl.make_weights_numpy(cfg, seed=71, gain_jitter=0.1), np.float16)
    om = oracle32.model(cfg, w)
    refs = {}
    for n in prompts:
        om.reset()
        refs[n] = om.prefill(wl.make_tokens(n, cfg["vocab"], seed=n))
    yield cfg, w, refs
    om.close()


@pytest.mark.parametrize("flags", [0, 32], ids=["copy", "lean"])
def test_last_row_against_the_oracle(model, flags):
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    cfg, w, refs = model
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16), flags=flags) as s:
        for n, (_, ref, hidden) in refs.items():
            calls = [s.ll_prefill] + ([s.ll_prefill_static] if n <= 32 else [])
            for call in calls:
                s.ll_reset()
                s.ll_dbg_poison_scratch()
                token = call(wl.make_tokens(n, cfg["vocab"], seed=n))
                logits = s.ll_dbg_get_logits()
                check_logits(logits, ref, "prompt %d" % n)
                check_logits(s.ll_dbg_get_hidden(), hidden, "prompt %d hidden" % n,
                             max_abs_tol=3e-2 * max(1.0, float(np.abs(hidden).max())))
                check_greedy_token(token, logits, "prompt %d" % n)
