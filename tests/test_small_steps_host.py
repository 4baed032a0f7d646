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
    plan = b.ll_dbg_small_plan(wl.tiny_cfg(), 5, 3)
    assert plan["workgroups"] == 32 and plan["first_pos"] == 5 and plan["greedy_keys"] > plan["sampled_keys"] > 1000
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


# us per step measured in the one kernel and in the kernel chain: (layers, heads, head_dim, ffn, vocab), keys, sampled, one, chain
MEASURED = [((1, 4, 64, 688, 32000), 28, False, 37.2, 42.1), ((1, 4, 64, 688, 64000), 28, False, 62.2, 52.3),
            ((1, 8, 64, 1408, 16384), 28, False, 34.3, 38.6), ((1, 8, 64, 1408, 32000), 28, False, 50.3, 44.3),
            ((4, 8, 64, 1408, 32000), 28, False, 93.1, 103.6), ((4, 8, 64, 1408, 64000), 28, False, 125.3, 114.2),
            ((1, 1, 64, 136, 16384), 28, False, 30.8, 36.0), ((1, 1, 64, 136, 32000), 28, False, 56.7, 40.1),
            ((1, 4, 64, 688, 8192), 28, True, 42.3, 45.4), ((1, 4, 64, 688, 16384), 28, True, 51.0, 49.3),
            ((4, 8, 64, 1408, 8192), 28, True, 93.3, 105.4), ((4, 8, 64, 1408, 32000), 28, True, 125.4, 121.2),
            ((1, 4, 64, 688, 1024), 6000, False, 34.1, 38.8), ((1, 4, 64, 688, 1024), 8000, False, 41.5, 39.4),
            ((8, 4, 64, 688, 1024), 3000, False, 161.9, 188.8), ((8, 4, 64, 688, 1024), 6000, False, 247.9, 221.7),
            ((4, 8, 64, 1408, 1024), 800, False, 85.6, 96.1), ((4, 8, 64, 1408, 1024), 3000, False, 116.3, 105.6),
            ((4, 4, 128, 1536, 1024), 800, False, 88.9, 97.8), ((4, 4, 128, 1536, 1024), 3000, False, 144.5, 123.3)]


@pytest.mark.parametrize("shape,keys,sampled,one,chain", MEASURED)
def test_a_step_runs_where_it_was_measured_to_be_faster(shape, keys, sampled, one, chain):
    plan = b.ll_dbg_small_plan(wl.custom_cfg(*shape, 16384), 0, 1)
    assert (keys <= plan["sampled_keys" if sampled else "greedy_keys"]) == (one < chain), plan
