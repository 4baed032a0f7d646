"""Selection either side of the vocabularies that its kernels are built for (one token a thread up to 1024, eight up to 8192,
32 beyond): greedy and stochastic, alone and per slot of a batch, and greedy among six equal maxima anywhere, past the
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


def _greedy(s, prompts, steps, check):
    """Tokens of every prompt and `steps` steps, alone; check(token, logits) for each."""
    out = []
    for q in prompts:
        s.ll_reset()
        token = s.ll_prefill(q)
        for _ in range(steps):
            check(token, s.ll_dbg_get_logits())
            out.append(token)
            token = s.ll_decode_step()
    return out


@pytest.mark.parametrize("vocab", [1024, 1040, 8192, 8208, 40000])
def test_greedy_takes_the_lowest_of_equal_maxima(torch_cuda, vocab):  # noqa: F811
    cfg, w = _model(vocab)
    prompts = [wl.make_tokens(n, vocab, seed=n) for n in (6, 9, 4)]
    with _session(cfg, w) as s:
        chosen = sorted(set(_greedy(s, prompts, 10, lambda token, logits: None)))
    # five copies of every chosen row, and of its embedding, anywhere else: the sequences stay what they are, and every choice
    # among them is a tie whose lowest index is some copy or the row itself
    used = set(chosen) | set(int(t) for q in prompts for t in q)
    free = [int(i) for i in np.random.default_rng(vocab).permutation(vocab) if int(i) not in used]
    for j, row in enumerate(chosen):
        for i in free[5 * j:5 * j + 5]:
            w["lm_head"][i] = w["lm_head"][row]
            w["tok_emb"][i] = w["tok_emb"][row]
    ties = []

    def check(token, logits, what):
        check_greedy_token(token, logits, "vocabulary %d %s" % (vocab, what))
        at = np.flatnonzero(logits == logits.max())
        ties.append(at.size)

    with _session(cfg, w) as s:
        _greedy(s, prompts, 10, lambda token, logits: check(token, logits, "alone"))
        assert min(ties) == 6, (vocab, ties)
        del ties[:]
        s.ll_batch_open(3, 8, 30)
        slots = [s.ll_batch_add(q)[0] for q in prompts]
        for _ in range(9):
            toks = s.ll_batch_step()
            for slot in slots:
                check(toks[slot], s.ll_batch_dbg_get_logits(slot), "slot %d" % slot)
        # (the batch's projections add up in another order: a step may choose a token that was not chosen alone)
        assert sum(t == 6 for t in ties) >= 20, (vocab, ties)
