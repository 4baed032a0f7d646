"""SwiGLU of every prefill path against its correctly rounded fp16 value, at arguments chosen next to the rounding
borders.  The model passes gate and up values through untouched (the residual stream is all ones, so the normalised operand is
exactly 1; every gate / up row has one non-zero weight; the down projection is the identity), and the hidden state shows
every element of silu(gate) * up as it was rounded to fp16."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl

pytestmark = pytest.mark.gpu
D = 1024


def _pairs(count, rng):
    """fp16 (gate, up) whose exact silu(gate) * up lies 3.6e-7 .. 6e-7 of its value from a border between two fp16 values.
    An exponential, a sum, a division and a product in fp32 are off by at most 2^-23 + 3 * 2^-24 = 3.0e-7 and cannot
    cross it; an exponential with its argument scaled by log2(e) in fp32 is off by up to 24 * log2(e) * 2^-24 * ln 2 = 1.4e-6."""
    gate, up = np.empty(0, np.float16), np.empty(0, np.float16)
    while gate.size < count:
        g = (-rng.uniform(14.0, 24.0, 1 << 20)).astype(np.float16)
        u = rng.uniform(2e4, 6e4, 1 << 20).astype(np.float16)
        v = _silu_times(g, u)
        near = v.astype(np.float16)
        other = np.where(near.astype(np.float64) < v, np.nextafter(near, np.float16(np.inf)),
                         np.nextafter(near, np.float16(0)))
        dist = np.abs(v - 0.5 * (near.astype(np.float64) + other.astype(np.float64))) / v
        keep = (dist > 3.6e-7) & (dist < 6e-7) & (np.abs(v) > 2.0 ** -6)
        gate, up = np.concatenate((gate, g[keep])), np.concatenate((up, u[keep]))
    return gate[:count], up[:count]


def _silu_times(g, u):
    g, u = g.astype(np.float64), u.astype(np.float64)
    with np.errstate(over="ignore"):
        return -(g / (1.0 + np.exp(-g)) * u)                   # the caller negates `up`: positive values


def _extremes():
    """Gates past the clamp of the exponent on both sides, zeros of both signs, and where the exponential is near 1."""
    gate = np.array([-60000, -200, -100, -89, -88.75, -87, -50, -1e-3, -0.0, 0.0, 1e-3, 0.5, 20, 88.75, 89, 200, 4000],
                    np.float16)
    up = np.where(gate > 1, -0.25, -3.0).astype(np.float16)
    return gate, up


@pytest.fixture(scope="module")
def model():
    rng = np.random.default_rng(5)
    gate, up = _pairs(D, rng)
    few = _extremes()
    gate[:few[0].size], up[:few[0].size] = few[0], -few[1]
    cfg = wl.custom_cfg(1, D // 128, 128, D, 64, 1025, rms_eps=0.0)
    z = lambda *s: np.zeros(s, np.float16)
    at = rng.permutation(D)
    layer = dict(attn_norm=np.ones(D, np.float16), ffn_norm=np.ones(D, np.float16), wq=z(D, D), wk=z(D, D), wv=z(D, D),
                 wo=z(D, D), w_gate=z(D, D), w_up=z(D, D), w_down=np.eye(D, dtype=np.float16))
    layer["w_gate"][np.arange(D), at] = gate
    layer["w_up"][np.arange(D), at[::-1]] = -up
    w = dict(tok_emb=np.ones((64, D), np.float16), final_norm=np.ones(D, np.float16), lm_head=z(64, D), layers=[layer])
    return cfg, w, np.float32(1) + _silu_times(gate, up).astype(np.float16).astype(np.float32)


@pytest.mark.parametrize("flags", [0, 32], ids=["copy", "lean"])
def test_silu_times_up_is_correctly_rounded(model, flags):
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    cfg, w, want = model
    wrong = {}
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16), flags=flags) as s:
        for n in (20, 50, 100, 180, 250, 380, 500, 1000):
            s.ll_reset()
            s.ll_prefill(wl.make_tokens(n, 64, seed=n))
            wrong[n] = int((s.ll_dbg_get_hidden() != want).sum())
    assert not any(wrong.values()), wrong
