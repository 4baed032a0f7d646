"""Prefill projections whose column tiles hold an odd number of 16-row weight blocks, against the fp32 oracle."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_kv, check_logits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 48, 49, 64])
def test_column_tiles_of_an_odd_number_of_weight_blocks(oracle32, n):
    """d_model 4096: Q/K/V of at most 64 rows goes out in tiles of three 16-row weight blocks, one and a half of
    the kernel's 32-column blocks."""
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    cfg = wl.custom_cfg(1, 32, 128, 688, 200, 128)
    w = wl.weights_astype(wl.make_weights_numpy(cfg, seed=52, gain_jitter=0.1), np.float16)
    prompt = wl.make_tokens(n, cfg["vocab"], seed=n)
    om = oracle32.model(cfg, w)
    _, ref, _ = om.prefill(prompt)
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16)) as s:
        s.ll_dbg_poison_scratch()
        s.ll_prefill(prompt)
        check_logits(s.ll_dbg_get_logits(), ref, "prompt %d" % n)
        for which in range(2):
            check_kv(s.ll_dbg_get_kv(0, which, n), om.kv(0, which), "prompt %d %s" % (n, "KV"[which]))
    om.close()
