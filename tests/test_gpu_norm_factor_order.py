"""The norm factors of prompts of at most 32 tokens, to the bit: a token's partial sums of squares are added sixteen
strided sums at a time and those as a tree, in float32.  O and down are zero here, so every norm sees the embedding row, and
V of layer 1 is the identity: a cached value row is fp16(fp16(x gain) factor) and shows the factor's last bits."""
import numpy as np
import pytest

from paper_2604_23467_amd import workloads as wl

pytestmark = pytest.mark.gpu
F32 = np.float32


def _embedding(rng, vocab, d):
    """Rows of six-bit integers, a power of two per 16 columns: the sum of the squares of a 16-column block is exact in
    float32 in any order, the sum of the blocks is not."""
    m = rng.integers(0, 32, (vocab, d)) * 2 + 1
    e = np.repeat(rng.integers(-6, 1, (vocab, d // 16)), 16, axis=1)
    return (m * rng.choice([-1, 1], (vocab, d)) * 2.0 ** e / 16).astype(np.float16)


def _tree16(v):
    q = [F32(F32(v[4 * i] + v[4 * i + 1]) + F32(v[4 * i + 2] + v[4 * i + 3])) for i in range(4)]
    return F32(F32(q[0] + q[1]) + F32(q[2] + q[3]))


def _strided(slots):
    lanes = []
    for j in range(16):
        s = F32(0)
        for v in slots[j::16]:
            s = F32(s + v)
        lanes.append(s)
    return _tree16(lanes)


def _neighbours(slots):                       # another order: four neighbours per lane, then the wave
    slots = np.concatenate([slots, np.zeros(256 - len(slots), F32)])
    lanes = [F32(F32(F32(slots[4 * i] + slots[4 * i + 1]) + slots[4 * i + 2]) + slots[4 * i + 3]) for i in range(64)]
    r = [_tree16(lanes[16 * i:16 * i + 16]) for i in range(4)]
    return F32(F32(r[0] + r[1]) + F32(r[2] + r[3]))


def _values(x, gain, add, eps):
    """Value rows of tokens with residual rows x, the blocks' sums added by `add`."""
    sq = np.square(x.astype(np.float64)).reshape(len(x), -1, 16).sum(-1).astype(F32)
    factor = np.array([F32(1) / np.sqrt(F32(add(s) / F32(x.shape[1]) + F32(eps))) for s in sq], F32)
    xg = (x.astype(F32) * gain.astype(F32)).astype(np.float16)
    return (xg.astype(F32) * factor[:, None]).astype(np.float16)


# full rows of partial sums, fewer than lanes, a number that 16 does not divide (and a width that is no power of two)
@pytest.mark.parametrize("heads,hd", [(32, 128), (4, 64), (21, 64)])
@pytest.mark.parametrize("lean", [False, True])
def test_value_rows_show_the_strided_sum(heads, hd, lean):
    import torch
    from paper_2604_23467_amd import binding as b
    assert torch.cuda.is_available(), "this test needs a GPU"
    cfg = wl.custom_cfg(2, heads, hd, 64, 256, 64)
    d, rng = cfg["d_model"], np.random.default_rng(heads)
    emb = _embedding(rng, cfg["vocab"], d)
    gain = rng.uniform(0.5, 2.0, d).astype(np.float16)
    dev = lambda a: torch.from_numpy(a).to("cuda:0")
    zero = lambda r, c: torch.zeros(r, c, dtype=torch.float16, device="cuda:0")
    layer = lambda v: dict(attn_norm=dev(gain), wq=zero(d, d), wk=zero(d, d), wv=v, wo=zero(d, d), ffn_norm=dev(gain),
                           w_gate=zero(64, d), w_up=zero(64, d), w_down=zero(d, 64))
    w = dict(tok_emb=dev(emb), lm_head=zero(cfg["vocab"], d), final_norm=dev(gain),
             layers=[layer(zero(d, d)), layer(torch.eye(d, dtype=torch.float16, device="cuda:0"))])
    told = 0
    with b.Session(cfg, w, flags=b.LL_FLAG_LEAN_WORKSPACE if lean else 0) as s:
        for n in (16, 32, 32, 32, 32, 32, 1, 31):
            p = rng.integers(0, cfg["vocab"], n).astype(np.int32)
            s.ll_reset()
            s.ll_prefill(p)
            got = s.ll_dbg_get_kv(1, 1, n)
            want = _values(emb[p], gain, _strided, cfg["rms_eps"])
            told += int((want != _values(emb[p], gain, _neighbours, cfg["rms_eps"])).sum())
            assert np.array_equal(got, want.astype(F32)), (n, int((got != want.astype(F32)).sum()))
    if heads > 16:
        assert told > 0                       # the values tell the two orders apart
