"""Selection either side of the vocabularies that its kernels are built for (one token a thread up to 1024, eight up to 8192,
32 beyond): greedy and stochastic, alone and per slot of a batch, and greedy among equal maxima in other waves, past the
vocabularies that the stochastic path takes."""
import numpy as np
import pytest

from oracle import sampling as sp
from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_greedy_token
from tests.test_gpu_sampling import _accept, _run, _session, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu
SETTINGS = [(1.0, 0, 1.0), (1.3, 0, 0.9), (0.8, 50, 0.95), (1.0, 300, 0.9)]


def _model(vocab):
    cfg = wl.custom_cfg(1, 2, 64, 136, vocab, 60)
    w = wl.make_weights_numpy(cfg, seed=57, emb_std=1.0)
    w["lm_head"] = (w["lm_head"] * 30.0).astype(w["lm_head"].dtype)     # logits a few units wide
    return cfg, w


@pytest.mark.parametrize("vocab", [1024, 1040, 8192, 8208])
def test_draws_match_the_oracle(torch_cuda, vocab):  # noqa: F811
    cfg, w = _model(vocab)
    prompts = [wl.make_tokens(n, vocab, seed=n) for n in (6, 9, 4)]
    total = exact = 0
    with _session(cfg, w) as s:
        for j, (t, k, p) in enumerate(SETTINGS):
            toks, ex = _run(s, prompts[0], 12, t, k, p, seed=5000 + j)
            total += len(toks)
            exact += ex
        s.ll_batch_open(3, 8, 30)
        for j, (t, k, p) in enumerate(SETTINGS):
            s.ll_set_sampling(t, k, p, 6000 + j)
            slots = [s.ll_batch_add(q)[0] for q in prompts]
            for i in range(1, 8):
                toks = s.ll_batch_step()
                for slot in slots:
                    ok, same = _accept(toks[slot], s.ll_batch_dbg_get_logits(slot), t, k, p, sp.uniform(6000 + j, i))
                    assert ok, (vocab, t, k, p, i, slot)
                    total += 1
                    exact += same
            for slot in slots:
                s.ll_batch_remove(slot)
        s.ll_batch_close()
    assert exact >= 0.95 * total, (exact, total)


@pytest.mark.parametrize("vocab", [1024, 1040, 8192, 8208, 40000])
def test_greedy_takes_the_lowest_of_equal_maxima(torch_cuda, vocab):  # noqa: F811
    cfg, w = _model(vocab)
    rng = np.random.default_rng(vocab)
    for i in range(1, 8):                        # copies of a row that is often the best one, far apart
        w["lm_head"][rng.integers(0, vocab, 40)] = w["lm_head"][0] * 3
    prompts = [wl.make_tokens(n, vocab, seed=n) for n in (6, 9, 4)]
    with _session(cfg, w) as s:
        for q in prompts:
            s.ll_reset()
            token = s.ll_prefill(q)
            for _ in range(10):
                check_greedy_token(token, s.ll_dbg_get_logits(), "vocabulary %d" % vocab)
                token = s.ll_decode_step()
        s.ll_batch_open(3, 8, 30)
        slots = [s.ll_batch_add(q)[0] for q in prompts]
        for _ in range(10):
            toks = s.ll_batch_step()
            for slot in slots:
                check_greedy_token(toks[slot], s.ll_batch_dbg_get_logits(slot), "vocabulary %d slot %d" % (vocab, slot))
