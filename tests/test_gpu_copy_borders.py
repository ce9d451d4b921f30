"""GPU parity where the rows that a wave copies at a time (32 keys of a thin item, 16 at head_dim 64) meet frame borders in every way: frames
shorter than the rows (several borders inside them), shorter than a tile (frames that a wave steps over), barely longer, and the border
to a chunk of strided rows."""
import pytest

from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "model"])
@pytest.mark.parametrize("tpf", [7, 15, 16, 17, 31, 33, 63, 65, 100])
@pytest.mark.parametrize("D", [64, 128])
def test_rows_across_frame_borders(D, tpf, layout):
    pols = [synth.anchor_all(9), synth.anchor_topk(5, 5), synth.wave(2, 9), synth.veil(1, 3)]
    G.run_case(pols, tpf, D, [3, 3, 3], 2 * tpf + 5, seed=500 + tpf, layout=layout, check_every_append=False, label="borders")
