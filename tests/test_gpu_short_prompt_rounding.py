"""Epilogues of prompts of at most 32 tokens to the bit: which results are rounded to fp32 on their way to fp16, and which
product of a RoPE rotation is fused.  O is zero and projections are diagonal, so that every sum in front of an epilogue is
one exact product."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.test_gpu_norm_factor_order import _embedding, _strided

pytestmark = pytest.mark.gpu
F32, F16 = np.float32, np.float16
HEADS, HD, VOCAB = 16, 128, 256
D = HEADS * HD


def _session(emb, gain, ffn, **mats):
    import torch
    from paper_2604_23467_amd import binding as b
    assert torch.cuda.is_available(), "these tests need a GPU"
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    zero = lambda r, c: torch.zeros(r, c, dtype=torch.float16, device="cuda:0")
    layer = dict(attn_norm=dev(gain), wq=zero(D, D), wk=zero(D, D), wv=zero(D, D), wo=zero(D, D), ffn_norm=dev(gain),
                 w_gate=zero(ffn, D), w_up=zero(ffn, D), w_down=zero(D, ffn))
    layer.update({k: dev(v) for k, v in mats.items()})
    cfg = wl.custom_cfg(1, HEADS, HD, ffn, VOCAB, 64)
    return b.Session(cfg, dict(tok_emb=dev(emb), lm_head=zero(VOCAB, D), final_norm=dev(gain), layers=[layer])), cfg


def _normalised(x, gain, eps, add):
    """fp32 products of the norm's operand and factor, `add` summing the squares of a row's 16-column blocks."""
    sq = np.square(x.astype(np.float64)).reshape(len(x), -1, 16).sum(-1).astype(F32)
    factor = np.array([F32(1) / np.sqrt(F32(add(s) / F32(D) + F32(eps))) for s in sq], F32)
    return (x.astype(F32) * gain.astype(F32)).astype(F16).astype(F32) * factor[:, None]


@pytest.mark.parametrize("n", [16, 32, 9, 17])
def test_key_rows_show_the_rounding_of_the_rotation(n):
    rng = np.random.default_rng(n)
    emb = _embedding(rng, VOCAB, D)
    # a sum of squares that no order changes: layer 0 takes it from the embedding kernel
    emb = (np.sign(emb) * (np.abs(emb.astype(F32)) % 1 + 1)).astype(F16)
    emb = (np.round(emb.astype(F32) * 8) / 8).astype(F16)
    gain = rng.uniform(0.5, 2.0, D).astype(F16)
    s, cfg = _session(emb, gain, 64, wk=np.eye(D, dtype=F16))
    one = two = 0
    with s:
        for r in range(16):
            p = rng.integers(0, VOCAB, n).astype(np.int32)
            s.ll_reset()
            s.ll_prefill(p)
            got = s.ll_dbg_get_kv(0, 0, n).reshape(n, HEADS, 2, HD // 2)
            k = _normalised(emb[p], gain, cfg["rms_eps"], lambda v: F32(v.astype(np.float64).sum())).reshape(n, HEADS, 2, HD // 2)
            lo, hi = k[:, :, 0], k[:, :, 1]
            phi = np.arange(n)[:, None] * float(F32(cfg["rope_theta"])) ** (-2.0 * np.arange(HD // 2) / HD)
            c, sn = np.cos(phi).astype(F32)[:, None], np.sin(phi).astype(F32)[:, None]
            first = (lo.astype(np.float64) * c - (hi * sn).astype(np.float64)).astype(F16)
            fused = hi.astype(np.float64) * c + (lo * sn).astype(np.float64)
            second = fused.astype(F32).astype(F16) if n <= 16 else fused.astype(F16)
            other = (lo.astype(np.float64) * sn + (hi * c).astype(np.float64))
            one += int((second != (fused.astype(F16) if n <= 16 else fused.astype(F32).astype(F16))).sum())
            two += int((second != (other.astype(F32).astype(F16) if n <= 16 else other.astype(F16))).sum())
            assert np.array_equal(got[:, :, 0], first.astype(F32)), int((got[:, :, 0] != first.astype(F32)).sum())
            assert np.array_equal(got[:, :, 1], second.astype(F32)), int((got[:, :, 1] != second.astype(F32)).sum())
    assert one > 0 and two > 0                # the keys tell all three forms apart


@pytest.mark.parametrize("n", [16, 32, 1, 17])
def test_hidden_state_shows_the_rounding_of_swiglu(n):
    """Gates of 20 and more, where silu(g) is g itself: the SwiGLU output is g u, rounded to fp32 and then to fp16.  Down
    is the identity, and the residual row it is added to has few enough bits for the sum to be exact."""
    rng = np.random.default_rng(100 + n)
    emb = (rng.integers(64, 128, (VOCAB, D)) / 64).astype(F16)
    gain = rng.uniform(0.5, 2.0, D).astype(F16)
    eye = np.eye(D, dtype=F16)
    s, cfg = _session(emb, gain, D, w_gate=eye * F16(128), w_up=eye, w_down=eye)
    told = 0
    with s:
        for r in range(96):
            p = rng.integers(0, VOCAB, n).astype(np.int32)
            s.ll_reset()
            s.ll_prefill(p)
            u = _normalised(emb[p[-1:]], gain, cfg["rms_eps"], _strided)[0]
            g = u * F32(128)
            assert g.min() >= 20.0 and (g.astype(np.float64) * u).max() < 2048.0
            h = (g * u).astype(F16)
            told += int((h != (g.astype(np.float64) * u).astype(F16)).sum())
            want = emb[p[-1]].astype(F32) + h.astype(F32)
            got = s.ll_dbg_get_hidden()
            assert np.array_equal(got, want), int((got != want).sum())
    assert told > 0                           # the rows tell one rounding from two
