"""GPU parity where the rows that a wave copies at a time (32 keys of a thin item, 16 at head_dim 64, 8 or 16 of a full item) meet frame
borders in every way: frames shorter than the rows (several borders inside them), shorter than a tile (frames that a wave steps over),
barely longer, and the border to a chunk of strided rows."""
import pytest

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "model"])
@pytest.mark.parametrize("tpf", [7, 15, 16, 17, 31, 33, 63, 65, 100])
@pytest.mark.parametrize("D", [64, 128])
def test_rows_across_frame_borders(D, tpf, layout):
    pols = [synth.anchor_all(9), synth.anchor_topk(5, 5), synth.wave(2, 9), synth.veil(1, 3)]
    G.run_case(pols, tpf, D, [3, 3, 3], 2 * tpf + 5, seed=500 + tpf, layout=layout, check_every_append=False, label="borders")


# as many frames as it takes for the planner to choose thin items
@pytest.mark.parametrize("layout", ["packed", "model"])
@pytest.mark.parametrize("tpf,frames", [(2, 100), (3, 60), (7, 30), (15, 15), (16, 15), (17, 15), (31, 9), (32, 9), (33, 9), (63, 9), (64, 9), (65, 9)])
def test_thin_items_across_frame_borders(tpf, frames, layout):
    pols = [synth.anchor_all(frames), synth.anchor_topk(5, 5), synth.wave(2, frames), synth.veil(1, 3)]
    G.run_case(pols, tpf, 128, [frames], 41 if tpf < 33 else 2 * tpf + 5, seed=540 + tpf, layout=layout, label="thin-borders", variant=3)


@pytest.mark.parametrize("layout", ["packed", "model"])
@pytest.mark.parametrize("variant", [1, 2])
@pytest.mark.parametrize("tpf,frames,Lq", [(1, 1, 1), (2, 130, 3), (5, 40, 21), (9, 30, 300), (17, 12, 34), (63, 5, 64), (64, 3, 65), (100, 4, 259)])
def test_full_items_whose_rows_are_found_one_by_one(tpf, frames, Lq, variant, layout):
    """Full items at frames smaller than a tile and at ragged ends, where every lane finds its own row of the tile: one row in all, frames
    that divide a wave's rows and its tiles and frames that do not, and the border to a chunk of strided rows inside such a tile."""
    B.pf_set_tuning(attn_variant=variant)
    try:
        pols = [synth.anchor_all(frames), synth.wave(2, frames), synth.veil(1, 3)]
        G.run_case(pols, tpf, 128, [frames], Lq, seed=900 + tpf, layout=layout, label="rows", variant=variant)
    finally:
        B.pf_set_tuning(attn_variant=-2)
