"""What is left where the kernel of small models' decode steps gives up on its waits.  The give-up is asked for by the host at
a chosen token; every kernel exits as it always does."""
import contextlib

import numpy as np
import pytest

from paper_2604_23467_amd import binding as b
from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_kv, max_abs

pytestmark = pytest.mark.gpu
N, K = 20, 12


@pytest.fixture(scope="module")
def weights():
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    cfg = wl.tiny_cfg()
    w = wl.weights_astype(wl.make_weights_numpy(cfg, seed=9, gain_jitter=0.1, emb_std=0.5), np.float16)
    return wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16)


def _open(weights, sampled, flags=0, max_seq=N + K):
    s = b.Session(wl.tiny_cfg(max_seq=max_seq), weights, flags=flags)
    if sampled:
        s.ll_set_sampling(temperature=0.8, top_k=50, top_p=0.95, seed=3)
    return s


def _rows(s, n):
    return [s.ll_dbg_get_kv(layer, which, n) for layer in range(2) for which in range(2)]


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("at", [1, 2, 6, K])          # the first step, the next, one in the middle, the last
def test_steps_behind_a_give_up_are_the_kernel_chains(weights, sampled, at):
    """Up to the last position of the cache; the prompt's rows, the RoPE table and a fresh request stay what they are."""
    prompt, fresh = wl.make_tokens(N, 1024, seed=5), wl.make_tokens(N - 3, 1024, seed=6)
    out = []
    for flags in (b.LL_FLAG_MULTIKERNEL, 0):
        with _open(weights, sampled, flags) as s:
            assert s.ll_dbg_give_up_at(at) == (flags == 0)
            toks = [s.ll_prefill(prompt)]
            first = _rows(s, N)
            toks += list(s.ll_decode_n(K))
            rows = _rows(s, N + K)
            assert s.ll_position() == N + K
            for r, f in zip(rows, first):
                assert r[:N].tobytes() == f.tobytes()
            s.ll_reset()
            again = [s.ll_prefill(fresh)] + list(s.ll_decode_n(K))
            out.append((toks, rows, again, s.ll_dbg_get_logits(), _rows(s, N - 3 + K)))
            if flags == 0:
                assert not s.ll_dbg_give_up_at(-1)    # the kernel chain from there on
    (toks, rows, again, logits, rows2), (toks_s, rows_s, again_s, logits_s, rows2_s) = out
    assert toks_s == toks and again_s == again
    for r, q in zip(rows_s, rows):
        check_kv(r, q, "give-up at token %d" % at)
    assert logits_s.tobytes() == logits.tobytes()     # the same kernels on the same state
    for r, q in zip(rows2_s, rows2):
        assert r.tobytes() == q.tobytes()


@pytest.mark.parametrize("sampled", [False, True])
def test_a_launch_that_gave_up_stores_no_row(weights, sampled):
    at = 5
    with _open(weights, sampled) as s:
        s.ll_prefill(wl.make_tokens(N, 1024, seed=5))
        s.ll_decode_n(K)                              # every row of the cache holds something
        s.ll_reset()
        s.ll_prefill(wl.make_tokens(N, 1024, seed=7))
        before = _rows(s, N + K)
        assert s.ll_dbg_give_up_at(at)
        with contextlib.suppress(b.LLError):
            s.ll_dbg_time_decode(K)
        for r, q in zip(_rows(s, N + K), before):
            assert (r[N:N + at - 1] != q[N:N + at - 1]).any(-1).all()       # the steps in front of it stored theirs
            keep = list(range(N)) + list(range(N + at - 1, N + K))
            assert r[keep].tobytes() == q[keep].tobytes()


def test_steps_queued_behind_a_give_up_do_not_begin(weights):
    """A sampled call queues one launch per step.  With no poll allowed to miss, the first one gives up after its layer 0
    has stored a row; those behind it give up before."""
    with _open(weights, True) as s:
        s.ll_prefill(wl.make_tokens(N, 1024, seed=5))
        s.ll_decode_n(K)
        s.ll_reset()
        s.ll_prefill(wl.make_tokens(N, 1024, seed=7))
        before = _rows(s, N + K)
        assert s.ll_dbg_set_spin_limit(0)
        with contextlib.suppress(b.LLError):
            s.ll_dbg_time_decode(K)
        for r, q in zip(_rows(s, N + K), before):
            assert r[:N].tobytes() == q[:N].tobytes() and r[N + 1:].tobytes() == q[N + 1:].tobytes()


@pytest.mark.parametrize("sampled", [False, True])
def test_a_timed_run_that_gave_up_has_no_time(weights, sampled):
    prompt, out = wl.make_tokens(N, 1024, seed=8), []
    for flags in (b.LL_FLAG_MULTIKERNEL, 0):
        with _open(weights, sampled, flags) as s:
            s.ll_prefill(prompt)
            if flags == 0:
                assert s.ll_dbg_give_up_at(3)
                with pytest.raises(b.LLError) as e:
                    s.ll_dbg_time_decode(K)
                assert e.value.code == b.LL_E_HIP and s.ll_position() == N
                assert not s.ll_dbg_give_up_at(-1)    # the kernel chain from there on
            else:
                assert s.ll_dbg_time_decode(K) > 0
            s.ll_reset()
            out.append(([s.ll_prefill(prompt)] + list(s.ll_decode_n(K)), s.ll_dbg_get_logits().tobytes()))
    assert out[0] == out[1]


@pytest.mark.parametrize("sampled", [False, True])
def test_a_warm_up_that_gave_up_leaves_the_kernel_chain(weights, sampled):
    prompt, out = wl.make_tokens(N, 1024, seed=8), []
    for flags in (b.LL_FLAG_MULTIKERNEL, 0):
        assert b.load().ll_dbg_give_up_at(0 if flags == 0 else -1) == 0
        with _open(weights, sampled, flags) as s:
            assert not s.ll_dbg_give_up_at(-1)
            out.append(([s.ll_prefill(prompt)] + list(s.ll_decode_n(K)), s.ll_dbg_get_logits().tobytes()))
    assert out[0] == out[1]
    with _open(weights, sampled) as s:                # the next instance's warm-up is its own
        assert s.ll_dbg_give_up_at(-1)
        assert [s.ll_prefill(prompt)] + list(s.ll_decode_n(K)) == out[0][0]


def test_calls_that_take_no_give_up(weights):
    with _open(weights, False, b.LL_FLAG_EAGER) as s:
        assert not s.ll_dbg_give_up_at(3)
        s.ll_prefill(wl.make_tokens(N, 1024, seed=5))
        toks = list(s.ll_decode_n(K))
        logits = s.ll_dbg_get_logits()
    with _open(weights, False) as s:
        assert s.ll_dbg_give_up_at(2) and s.ll_dbg_give_up_at(-1)            # taken back
        s.ll_prefill(wl.make_tokens(N, 1024, seed=5))
        assert list(s.ll_decode_n(K)) == toks and max_abs(s.ll_dbg_get_logits(), logits) < 1e-4
        assert s.ll_dbg_give_up_at(-1)                # and never fell back
