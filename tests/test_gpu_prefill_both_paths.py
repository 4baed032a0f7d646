"""O, gate/up and down of every row of a prompt at full K loops: the projections that read the weight copy against those that
read the caller's row-major weights (the last layer runs for the last row only, so a second layer's keys and values tell)."""
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.parity_utils import check_kv

pytestmark = pytest.mark.gpu
FULL = [50, 100, 180, 250, 300, 500, 700]


@pytest.fixture(scope="module", params=["d4096", "d8192"])
def both_paths(request):
    """The second layer's keys and values at every prompt length, by the projections that read the weight copy and by those that
    read the caller's row-major weights."""
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    cfg = wl.custom_cfg(2, 32, 128, 11000, 200, 720) if request.param == "d4096" else wl.custom_cfg(2, 64, 128, 1000, 200, 720)
    w = wl.make_weights_torch(cfg, seed=72, device="cuda:0")
    rows = {}
    for flags in (0, binding.LL_FLAG_LEAN_WORKSPACE):
        with binding.Session(cfg, w, flags=flags) as s:
            for n in FULL:
                s.ll_reset()
                s.ll_dbg_poison_scratch()
                s.ll_prefill(wl.make_tokens(n, cfg["vocab"], seed=n))
                rows[flags, n] = [s.ll_dbg_get_kv(1, which, n) for which in range(2)]
    return rows, binding.LL_FLAG_LEAN_WORKSPACE


@pytest.mark.parametrize("n", FULL)
def test_o_gate_up_and_down_of_every_row_at_full_k_loops(both_paths, n):
    """What a layer in front of the last one adds to every row, in the bounds that both paths keep to the oracle."""
    rows, lean = both_paths
    for which in range(2):
        check_kv(rows[0, n][which], rows[lean, n][which], "prompt %d %s" % (n, "KV"[which]))
