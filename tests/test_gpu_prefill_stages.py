"""Prefill projections with K loops of few ring stages, odd and even in number and ending inside one, at row counts whose tiles
keep two stages of activations in registers: two layers, so that gate/up's rows reach the second one's keys and values.
Against the fp32 oracle, scratch poisoned beforehand."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_kv, check_logits

pytestmark = pytest.mark.gpu
# heads, head_dim: 1, 3, 4.5 and 8 stages of 128
MODELS = {"d128": (2, 64), "d384": (3, 128), "d576": (9, 64), "d1024": (8, 128)}


@pytest.fixture(scope="module", params=list(MODELS))
def model(request, oracle32):
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    heads, head_dim = MODELS[request.param]
    cfg = wl.custom_cfg(2, heads, head_dim, 688, 200, 300)
    w = wl.weights_astype(wl.make_weights_numpy(cfg, seed=71, gain_jitter=0.1), np.float16)
    om = oracle32.model(cfg, w)
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16)) as s:
        yield cfg, s, om
    om.close()


@pytest.mark.parametrize("n", [25, 65, 128, 129, 180, 250])
def test_few_stages_against_the_oracle(model, n):
    cfg, s, om = model
    prompt = wl.make_tokens(n, cfg["vocab"], seed=n)
    om.reset()
    _, ref, _ = om.prefill(prompt)
    s.ll_reset()
    s.ll_dbg_poison_scratch()
    s.ll_prefill(prompt)
    check_logits(s.ll_dbg_get_logits(), ref, "prompt %d" % n)
    for layer in range(2):
        for which in range(2):
            check_kv(s.ll_dbg_get_kv(layer, which, n), om.kv(layer, which), "prompt %d layer %d %s" % (n, layer, "KV"[which]))
