"""Stochastic selection at the vocabularies where its work split changes: fewer tokens than a wave, about the 256
candidates that four threads rank each, fewer than the 1024 threads (one token each), and just past them (two each)."""
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


@pytest.mark.parametrize("vocab", [1024, 32000])
def test_sampler_on_logits_that_share_a_large_offset(torch_cuda, vocab):  # noqa: F811
    """Logits around 100 within about 1: the upper half of a float's bits no longer tells the k largest from the rest, so
    the bound of the top-k cut needs its lower bits."""
    cfg = wl.custom_cfg(1, 2, 64, 136, vocab, 60)
    w = wl.make_weights_numpy(cfg, seed=58, emb_std=0.3)
    rng = np.random.default_rng(8)
    w["tok_emb"] = w["tok_emb"] + 1.0
    w["lm_head"] = 100.0 / 128 / 0.96 + rng.standard_normal(w["lm_head"].shape) * 0.5 / np.sqrt(128)
    w = wl.weights_astype(w, np.float16)
    prompt = wl.make_tokens(6, vocab, seed=3)
    total = exact = 0
    with _session(cfg, w) as s:
        for j, (t, k, p) in enumerate([(0.8, 50, 0.95), (0.8, 200, 0.95), (1.0, 700, 1.0), (1.0, 1000, 0.9)]):
            toks, ex = _run(s, prompt, 30, t, k, p, seed=3000 + j)
            total += len(toks)
            exact += ex
    assert exact >= 0.95 * total, (exact, total)


def test_equal_logits_at_a_vocabulary_that_one_wave_finishes(torch_cuda):  # noqa: F811
    """Every candidate ties at the cut (the k lowest ids stay, token = floor(u * k)) and at the nucleus threshold (half of
    the k stay, token = floor(u * k / 2))."""
    from oracle import sampling as sp
    cfg = wl.custom_cfg(1, 2, 64, 136, 40, 40)
    w = wl.make_weights_numpy(cfg, seed=59)
    w["lm_head"][:] = 0
    with _session(cfg, wl.weights_astype(w, np.float16)) as s:
        for k, p, kept in ((8, 1.0, 8), (32, 0.5, 16)):
            s.ll_reset()
            s.ll_set_sampling(1.0, k, p, 99)
            toks = [s.ll_prefill([1, 2, 3])] + [s.ll_decode_step() for _ in range(20)]
            assert toks == [int(np.float32(sp.uniform(99, i)) * np.float32(kept)) for i in range(21)]


@pytest.mark.parametrize("vocab", [960, 961, 1024, 1920, 1921, 31700])
def test_top_k_where_the_bound_and_the_ranking_change(torch_cuda, vocab):  # noqa: F811
    """The bound comes from each wave by itself up to top-k 128 where all 16 waves hold tokens (over 960 of one a thread,
    1920 of two); up to 256 and 512 candidates are ranked by four and two threads each, more have one slot per
    thread.  Either side of each line, and ~100 tokens that tie at the cut."""
    cfg = wl.custom_cfg(1, 2, 64, 136, vocab, 60)
    w = wl.make_weights_numpy(cfg, seed=61, emb_std=1.0)
    w["lm_head"] = (w["lm_head"] * 30.0).astype(w["lm_head"].dtype)     # logits a few units wide
    w["lm_head"][5::max(7, vocab // 100)] = w["lm_head"][0]
    w = wl.weights_astype(w, np.float16)
    prompt = wl.make_tokens(6, vocab, seed=3)
    total = exact = 0
    with _session(cfg, w) as s:
        for j, (k, p) in enumerate([(1, 1.0), (16, 0.9), (17, 1.0), (128, 0.95), (129, 1.0), (255, 1.0), (256, 0.95), (257, 0.5), (511, 1.0), (513, 0.95), (900, 0.9)]):
            toks, ex = _run(s, prompt, 20, 1.5, k, p, seed=4000 + j)
            total += len(toks)
            exact += ex
    assert exact >= 0.95 * total, (exact, total)
