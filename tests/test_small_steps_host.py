"""Host arithmetic of the small models' decode steps (no GPU)."""
import pytest

from paper_2604_23467_amd import binding as b
from paper_2604_23467_amd import workloads as wl


@pytest.mark.parametrize("max_seq", [2, 3, 64, 1024])
def test_no_launch_starts_where_its_steps_run_past_the_cache(max_seq):
    """Whatever position the device state holds, also one that another workgroup of the launch advanced."""
    cfg = wl.tiny_cfg(max_seq=max_seq)
    for steps in sorted({0, 1, 2, 3, max_seq // 2, max_seq - 1, max_seq}):
        run = max(steps, 1)
        if run > max_seq:
            continue
        for pos in sorted({0, 1, max_seq // 2, max_seq - run, max_seq - 1, max_seq, 2 * max_seq, 1 << 20}):
            first = b.ll_dbg_small_plan(cfg, pos, steps)["first_pos"]
            assert 0 <= first and first + run <= max_seq, (pos, steps, first)
            if pos + run <= max_seq:
                assert first == pos


def test_plan_of_the_one_kernel_steps():
    assert b.ll_dbg_small_plan(wl.tiny_cfg(), 5, 3) == dict(workgroups=32, first_pos=5)
    assert b.ll_dbg_small_plan(wl.tiny_cfg(), 5, 3, b.LL_FLAG_LEAN_WORKSPACE)["workgroups"] == 32
    assert b.ll_dbg_small_plan(wl.custom_cfg(1, 2, 64, 136, 64, 64), 0, 1)["workgroups"] == 17       # a gate row per wave
    for cfg, flags in ((wl.tiny_cfg(), b.LL_FLAG_EAGER), (wl.tiny_cfg(), b.LL_FLAG_MULTIKERNEL),
                       (wl.custom_cfg(1, 9, 64, 688, 64, 64), 0), (wl.custom_cfg(1, 8, 64, 1544, 64, 64), 0),
                       (wl.custom_cfg(1, 8, 64, 128, 64, 64), 0)):
        assert b.ll_dbg_small_plan(cfg, 5, 3, flags)["workgroups"] == 0
    for pos, steps in ((-1, 1), (0, -1), (0, 65)):
        with pytest.raises(b.LLError) as e:
            b.ll_dbg_small_plan(wl.tiny_cfg(max_seq=64), pos, steps)
        assert e.value.code == b.LL_E_BAD_ARG
