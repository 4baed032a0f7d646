"""Prompts without the weight copy: the row-major GEMM with the RoPE and SwiGLU kernels behind it and slices at every
bucket, and chunks behind a full one, against the fp32 oracle."""
import pytest

from paper_2604_23467_amd import workloads as wl
from tests.test_gpu_prefill_tiles import EDGES, against_the_oracle, model  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def session(model):  # noqa: F811
    import torch
    assert torch.cuda.is_available(), "these tests need a GPU"
    from paper_2604_23467_amd import binding
    cfg, w = model
    with binding.Session(cfg, wl.weights_to_torch(w, device="cuda:0", dtype=torch.float16),
                         flags=binding.LL_FLAG_LEAN_WORKSPACE) as s:
        yield s


@pytest.mark.parametrize("n", EDGES + [1025, 1056, 1057, 1099])
def test_row_major_weights_against_the_oracle(session, model, oracle32, n):  # noqa: F811
    against_the_oracle(session, model, oracle32, n)
