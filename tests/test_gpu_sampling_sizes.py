"""Stochastic selection at the vocabularies where its work split changes: fewer tokens than a wave, than the 256
candidates one wave finishes, than the 1024 threads (one token each), and just past them (two each)."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.test_gpu_sampling import _run, _session, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu
SETTINGS = [(1.0, 0, 1.0), (1.3, 0, 0.9), (0.8, 20, 0.95), (2.0, 200, 0.5), (1.0, 600, 0.9)]


@pytest.mark.parametrize("vocab", [40, 300, 1023, 1025, 2000])
def test_sampler_matches_oracle_at_small_vocabularies(torch_cuda, vocab):  # noqa: F811
    cfg = wl.custom_cfg(1, 2, 64, 136, vocab, 60)
    w = wl.make_weights_numpy(cfg, seed=57, emb_std=1.0)
    w["lm_head"] = (w["lm_head"] * 30.0).astype(w["lm_head"].dtype)     # logits a few units wide
    w = wl.weights_astype(w, np.float16)
    prompt = wl.make_tokens(6, vocab, seed=3)
    total = exact = 0
    with _session(cfg, w) as s:
        for j, (t, k, p) in enumerate(SETTINGS):
            toks, ex = _run(s, prompt, 30, t, k, p, seed=2000 + j)
            total += len(toks)
            exact += ex
    assert exact >= 0.95 * total, (exact, total)
