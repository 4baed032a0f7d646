"""Host logic of the prefill projections that read the weight copy (no GPU): how tiles and K pieces are dealt out, over
the model widths an instance accepts (d_model up to 8192, ffn_hidden up to 12288)."""
import pytest

from paper_2604_23467_amd import binding

ROWS = (64, 128, 192, 256, 384, 512, 1024)
QKV, RES, GATEUP = 0, 1, 2
CUS = 256
MODELS = [(256, 688), (256, 1000), (768, 2048), (2048, 5632), (3072, 8192), (4096, 11008), (4224, 12288), (5120, 12288),
          (6144, 12288), (8192, 12288)]


def _blocks(kind, n):
    """16-row blocks of the weight copy that the tiles have to cover."""
    return 3 * n // 16 if kind == QKV else n // 16 if kind == RES else -(-n // 32) * 4


def _projections(d, f):
    return [(QKV, d, d), (RES, d, d), (GATEUP, f, d), (RES, d, f)]


@pytest.mark.parametrize("rows", ROWS)
@pytest.mark.parametrize("model", MODELS, ids=lambda m: "%dx%d" % m)
def test_tiles_and_pieces_cover_the_projection(model, rows):
    for kind, n, k in _projections(*model):
        p = binding.ll_dbg_tile_plan(kind, n, k, rows)
        what = (kind, n, k, rows, p)
        blocks, steps = _blocks(kind, n), -(-k // 32)
        assert rows % p["row_tiles"] == 0 and (rows // p["row_tiles"]) % 32 == 0, what
        assert (p["col_tiles"] - 1) * p["blocks"] < blocks <= p["col_tiles"] * p["blocks"], what
        assert p["pieces"] == 1 or kind == RES, what
        runs = p["col_tiles"] * p["pieces"]
        assert p["workgroups"] == -(-runs // 8) * 8 * p["row_tiles"], what
        # no piece of the K loop is empty: stages of the ring, or eight steps of the kernel without one
        stages = -(-steps // (p["stage_steps"] or 8))
        per = -(-stages // p["pieces"])
        assert (p["pieces"] - 1) * per < stages, what


@pytest.mark.parametrize("model", MODELS, ids=lambda m: "%dx%d" % m)
def test_one_round_of_workgroups_up_to_512_rows(model):
    """A second, partly filled round costs as much as a full one, whatever the width of the model."""
    for rows in ROWS[:-1]:
        for kind, n, k in _projections(*model):
            p = binding.ll_dbg_tile_plan(kind, n, k, rows)
            assert p["row_tiles"] * p["col_tiles"] * p["pieces"] <= CUS, (kind, n, k, rows, p)


@pytest.mark.parametrize("d", [d for d, _ in MODELS if d > 4096])
def test_wide_residual_projections_cut_their_k_loop(d):
    for rows in (64, 128, 384, 512):
        p = binding.ll_dbg_tile_plan(RES, d, d, rows)
        assert p["pieces"] >= 2, (d, rows, p)


def test_plan_rejects_bad_arguments():
    for bad in ((3, 256, 256, 64), (-1, 256, 256, 64), (QKV, 0, 256, 64), (RES, 256, 0, 64), (RES, 256, 256, 100), (RES, 20, 256, 64)):
        with pytest.raises(binding.LLError) as e:
            binding.ll_dbg_tile_plan(*bad)
        assert e.value.code == binding.LL_E_BAD_ARG
