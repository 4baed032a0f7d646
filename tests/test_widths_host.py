"""Models wider than the kernels hold are refused by the limit they pass (no GPU)."""
import ctypes as C

import pytest

from paper_2604_23467_amd import binding as b
from paper_2604_23467_amd import workloads as wl


def _init(heads, head_dim, ffn):
    """ll_init up to its checks of the shape: they come before anything is read or the device is touched."""
    lib = b.load()
    c = b.make_config(wl.custom_cfg(1, heads, head_dim, ffn, 64, 16))
    anything = 1 << 20
    layers = (b.LLLayerWeights * 1)(b.LLLayerWeights(*([anything] * len(b.LLLayerWeights._fields_))))
    w = b.LLWeights(anything, layers, anything, anything)
    rc = lib.ll_init(C.byref(c), C.byref(w), C.c_void_p(anything), 1 << 60, None)
    return rc, b.ll_last_error()


@pytest.mark.parametrize("heads,head_dim,ffn,limit", [(129, 64, 64, "d_model = 8256, at most 8192"), (65, 128, 64, "d_model = 8320, at most 8192"),
                                                      (96, 128, 64, "d_model = 12288, at most 8192"), (2, 64, 12296, "ffn_hidden = 12296, at most 12288")])
def test_wider_models_are_refused_by_their_limit(heads, head_dim, ffn, limit):
    rc, why = _init(heads, head_dim, ffn)
    assert rc == b.LL_E_BAD_CONFIG and limit in why, (rc, why)
