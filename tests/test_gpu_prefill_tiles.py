"""Row tiles and K pieces of the prefill projections that read the fragment-major weight copy, at the edges of
their buckets: against the fp32 oracle (logits and every cached K/V row), scratch poisoned beforehand, with
an FFN width that ends inside a 32-wide K step and inside a column tile."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_kv, check_logits

pytestmark = pytest.mark.gpu
EDGES = [33, 64, 65, 128, 129, 192, 193, 256, 257, 384, 385, 512, 513, 1024]


@pytest.fixture(scope="module")
def model(oracle32):
    cfg = wl.custom_cfg(2, 2, 128, 1000, 200, 1100)
    w = wl.weights_astype(wl.make_weights_numpy(cfg, seed=51, gain_jitter=0.1), np.float16)
    return cfg, w


@pytest.fixture(scope="module")
def session(model):
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    cfg, w = model
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16)) as s:
        yield s


@pytest.mark.parametrize("n", EDGES)
def test_bucket_edges_against_the_oracle(session, model, oracle32, n):
    against_the_oracle(session, model, oracle32, n)


@pytest.mark.parametrize("n", [1025, 1056, 1057, 1099])
def test_last_chunk_behind_a_full_one_against_the_oracle(session, model, oracle32, n):
    """1024 rows in the first chunk; the rest as a short prompt (1, 32 rows) and as tiles (33, 75)."""
    against_the_oracle(session, model, oracle32, n)


def against_the_oracle(session, model, oracle32, n):
    cfg, w = model
    prompt = wl.make_tokens(n, cfg["vocab"], seed=n)
    om = oracle32.model(cfg, w)
    _, ref, _ = om.prefill(prompt)
    session.ll_reset()
    session.ll_dbg_poison_scratch()
    session.ll_prefill(prompt)
    check_logits(session.ll_dbg_get_logits(), ref, "prompt %d" % n)
    for layer in range(2):
        for which in range(2):
            check_kv(session.ll_dbg_get_kv(layer, which, n), om.kv(layer, which),
                     "prompt %d layer %d %s" % (n, layer, "KV"[which]))
    om.close()
