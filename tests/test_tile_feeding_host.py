"""Prefill tiles whose weights are loaded by waves of their own (no GPU): two waves per SIMD leave 256 vector registers, and
the waves that multiply, on the other side of the branch that test_tile_waits_host.py follows, load nothing into the ring and
meet the loading waves at as many barriers."""
import re

import pytest

from tests.test_kernel_resources_host import _field, metadata  # noqa: F401
from tests.test_tile_waits_host import LABEL, listing  # noqa: F401

TILE = re.compile(r"_Z14pf_tile_kernelILi(\d)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)EE")


def _fed(key):
    return key[3] * key[4] <= 9


def _pairs(key):
    return key[0] != 1 and key[2] == 2 and key[3] * key[4] == 6


def test_fed_tiles_keep_to_the_registers_of_two_waves(metadata):  # noqa: F811
    fed = 0
    for name, entry in metadata.items():
        m = TILE.match(name)
        if not m:
            continue
        key = tuple(int(x) for x in m.groups())
        assert _field(entry, "private_segment_fixed_size") == 0, name
        if _fed(key):
            fed += 1
            assert _field(entry, "vgpr_count") <= 256 and _field(entry, "max_flat_workgroup_size") == 512, name
    assert fed >= 20


def test_the_two_kinds_of_waves_meet_at_the_same_barriers(listing):  # noqa: F811
    """One barrier in front of the K loop and one in it on either side (and one more around an exchange of K halves).  The
    loop of tiles with two sets of activation registers spans two stages."""
    kernels = next(v for v in listing.values() if all(len(k) == 8 for k in v))
    for key, body in kernels.items():
        if not _fed(key):
            continue
        ends = [i for i, line in enumerate(body) if line.startswith("s_endpgm")]
        ring = [i for i, line in enumerate(body) if line.startswith("buffer_load") and line.rstrip().endswith(" lds")]
        bars = [i for i, line in enumerate(body) if line.startswith("s_barrier")]
        # the loading waves' part: from their first load to the end of the kernel behind their last
        first, last = ring[0], max(ring)
        to = min((e for e in ends if e > last), default=len(body))
        mine = [b for b in bars if first < b < to]
        others = [b for b in bars if not first < b < to]
        exchange = 1 if key[2] == 2 else 0
        assert len(mine) == 2 + exchange and len(others) == 2 + _pairs(key) + 2 * exchange, (key, len(mine), len(others))
        assert not any(LABEL.match(body[i]) is None and body[i].startswith("v_mfma") for i in range(first, to)), key
