"""Order of a batch's slots over the attention's workgroups (no GPU): every slot once, rounds from the longest sequences to
the shortest, and every second round against the first."""
import random

import pytest

from paper_2604_23467_amd import binding as b


@pytest.mark.parametrize("rows", [1, 16, 32])
@pytest.mark.parametrize("per_round", [1, 5, 8, 64])
def test_rounds_alternate(rows, per_round):
    rng = random.Random(rows * 100 + per_round)
    for _ in range(50):
        pos = [rng.choice((0, 10, 25, 500, rng.randrange(1000))) for _ in range(rows)]
        active = [int(rng.random() < 0.8) for _ in range(rows)]
        order = b.ll_dbg_batch_order(pos, active, per_round)
        assert sorted(order) == list(range(rows))
        length = [pos[s] if active[s] else -1 for s in order]
        ranked = []
        for i, first in enumerate(range(0, rows, per_round)):
            ranked += length[first:first + per_round][::-1 if i % 2 else 1]
        assert ranked == sorted(length, reverse=True)


def test_bad_arguments_are_refused():
    for pos, per_round in (([1] * 33, 8), ([], 8), ([1], 0)):
        with pytest.raises(b.LLError) as e:
            b.ll_dbg_batch_order(pos, [1] * len(pos), per_round)
        assert e.value.code == b.LL_E_BAD_ARG
