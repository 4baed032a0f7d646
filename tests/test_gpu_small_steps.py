"""Decode steps of small models (one kernel on one XCD) against the oracle and against the kernel chain."""
import numpy as np
import pytest

from tests.parity_utils import check_kv, max_abs, run_teacher_forced
from paper_2604_23467_amd import binding as b
from paper_2604_23467_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    return torch


def _session(cfg, w, flags=0):
    import torch
    return b.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16), flags=flags)


def _weights(cfg, seed):
    return wl.weights_astype(wl.make_weights_numpy(cfg, seed=seed, gain_jitter=0.1, emb_std=0.5), np.float16)


# (layers, heads, head_dim, ffn, vocab): the smallest grid, odd numbers of workgroups and of vocabulary rows, both sides of
# 256 columns and of 1024 ffn columns, the largest widths, more row pairs than a wave fetches ahead
SHAPES = [(1, 1, 64, 32, 17), (1, 2, 64, 136, 301), (2, 2, 128, 344, 300), (3, 4, 64, 1024, 1030), (1, 4, 64, 1032, 64),
          (2, 5, 64, 688, 2051), (2, 3, 128, 1024, 512), (2, 8, 64, 1536, 100), (1, 4, 128, 1408, 4099)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("n_prompt", [1, 62, 250])      # 1 key up; the steps cross 64 keys; 4 waves share a head's keys
def test_small_model_steps_match_the_oracle(torch_cuda, oracle32, shape, n_prompt):
    cfg = wl.custom_cfg(*shape, 300)
    w = _weights(cfg, 5)
    prompt = wl.make_tokens(n_prompt, cfg["vocab"], seed=n_prompt)
    om = oracle32.model(cfg, w)
    with _session(cfg, w) as s:
        assert s.ll_dbg_set_spin_limit(1 << 20)            # the kernel under test is the one that runs
        run_teacher_forced(s, om, prompt, 5, "small")
        for which in range(2):
            check_kv(s.ll_dbg_get_kv(cfg["n_layers"] - 1, which, n_prompt + 5), om.kv(cfg["n_layers"] - 1, which), "small")
    om.close()


@pytest.mark.parametrize("shape", [(2, 4, 64, 688, 1024), (2, 8, 64, 1408, 600), (1, 2, 128, 136, 90)])
def test_many_steps_of_one_call_equal_single_steps_and_the_kernel_chain(torch_cuda, shape):
    cfg = wl.custom_cfg(*shape, 700)
    w = _weights(cfg, 6)
    prompt = wl.make_tokens(20, cfg["vocab"], seed=3)
    with _session(cfg, w) as s:
        one = [s.ll_prefill(prompt)] + [s.ll_decode_step() for _ in range(600)]
        l1, h1, kv1 = s.ll_dbg_get_logits(), s.ll_dbg_get_hidden(), s.ll_dbg_get_kv(0, 1, 620)
        s.ll_reset()
        many = [s.ll_prefill(prompt)] + list(s.ll_decode_n(1)) + list(s.ll_decode_n(599))
        assert many == one
        assert s.ll_dbg_get_logits().tobytes() == l1.tobytes() and s.ll_dbg_get_hidden().tobytes() == h1.tobytes()
        assert s.ll_dbg_get_kv(0, 1, 620).tobytes() == kv1.tobytes()
    with _session(cfg, w, b.LL_FLAG_MULTIKERNEL) as s:
        chain = [s.ll_prefill(prompt)] + list(s.ll_decode_n(600))
        assert chain == one
        # sums in another order: 1e-4 is what the library's other decode modes are held to among one another
        assert max_abs(s.ll_dbg_get_logits(), l1) < 1e-4 and max_abs(s.ll_dbg_get_hidden(), h1) < 1e-4


@pytest.mark.parametrize("sampled", [False, True])
def test_a_wait_that_runs_out_leaves_the_steps_to_the_kernel_chain(torch_cuda, sampled):
    cfg = wl.tiny_cfg(max_seq=96)
    w = _weights(cfg, 7)
    prompt = wl.make_tokens(12, cfg["vocab"], seed=4)
    runs = []
    for flags, limit in ((b.LL_FLAG_MULTIKERNEL, None), (0, 0)):
        with _session(cfg, w, flags) as s:
            if sampled:
                s.ll_set_sampling(temperature=0.8, top_k=50, top_p=0.95, seed=3)
            toks = [s.ll_prefill(prompt)]
            s.ll_dbg_force_next_token(7)                    # what the step feeds is not what the prefill returned
            if limit is not None:
                assert s.ll_dbg_set_spin_limit(limit)      # no poll may miss: the first step gives up
            toks += list(s.ll_decode_n(6)) + [s.ll_decode_step() for _ in range(3)]
            if limit is not None:
                assert not s.ll_dbg_set_spin_limit(1 << 20)         # the kernel is out of use from there on
            s.ll_reset()
            toks += [s.ll_prefill(prompt)] + list(s.ll_decode_n(4))
            runs.append((toks, s.ll_dbg_get_logits().tobytes(), s.ll_position()))
    assert runs[0] == runs[1]


def test_other_modes_and_wider_models_keep_the_kernel_chain(torch_cuda):
    for cfg, flags in ((wl.tiny_cfg(max_seq=64), b.LL_FLAG_EAGER), (wl.tiny_cfg(max_seq=64), b.LL_FLAG_PER_LENGTH_GRAPHS),
                       (wl.custom_cfg(1, 9, 64, 688, 64, 64), 0), (wl.custom_cfg(1, 8, 64, 1544, 64, 64), 0),
                       (wl.custom_cfg(1, 8, 64, 128, 64, 64), 0)):
        with _session(cfg, _weights(cfg, 8), flags) as s:
            assert not s.ll_dbg_set_spin_limit(1)
            s.ll_prefill(wl.make_tokens(5, 64, seed=1))
            assert len(s.ll_decode_n(3)) == 3


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("give_up", [None, 4])
def test_steps_on_both_sides_of_the_most_keys(torch_cuda, sampled, give_up):
    """A call that begins in the one kernel and ends in the chain: the same as step by step, and the chain's tokens; also
    where the kernel gives up with the chain's steps queued behind it."""
    cfg = wl.custom_cfg(1, 8, 64, 1408, 23552, 300) if not sampled else wl.custom_cfg(1, 4, 64, 688, 12800, 300)
    most = b.ll_dbg_small_plan(cfg, 0, 1)["sampled_keys" if sampled else "greedy_keys"]
    assert 20 < most < 280
    w = _weights(cfg, 10)
    prompt = wl.make_tokens(most - 7, cfg["vocab"], seed=11)
    runs = []
    for flags in (b.LL_FLAG_MULTIKERNEL, 0):
        with _session(cfg, w, flags) as s:
            if sampled:
                s.ll_set_sampling(temperature=0.8, top_k=50, top_p=0.95, seed=3)
            if flags == 0 and give_up:
                assert s.ll_dbg_give_up_at(give_up)
            many = [s.ll_prefill(prompt)] + list(s.ll_decode_n(12))
            logits = s.ll_dbg_get_logits()
            kv = [s.ll_dbg_get_kv(0, which, most + 5) for which in range(2)]
            assert s.ll_position() == most + 5
            if not give_up:
                s.ll_reset()
                assert [s.ll_prefill(prompt)] + [s.ll_decode_step() for _ in range(12)] == many
                assert s.ll_dbg_get_logits().tobytes() == logits.tobytes()
            runs.append((many, logits, kv))
    assert runs[0][0] == runs[1][0] and max_abs(runs[0][1], runs[1][1]) < 1e-4
    for a, c in zip(runs[0][2], runs[1][2]):
        check_kv(c, a, "both sides")
