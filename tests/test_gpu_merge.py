"""GPU parity of the merge of a split head's partial results: every kernel, from two segments to more than the eight whose maxima are
asked for together, an odd one left over by the pairs, and query rows that end inside a block."""
import pytest

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("segments", [2, 3, 8, 9, 17])
@pytest.mark.parametrize("D,variant", [(64, -2), (128, 0), (128, 1), (128, 2)], ids=["d64", "w4x32", "pp8x32", "w4x64"])
def test_partial_results_of_many_segments(D, variant, segments):
    B.pf_set_tuning(attn_variant=variant)
    try:
        frames = segments * 16 * 64 // 256                       # segments of 16 key tiles, the last one a chunk longer or a tile short
        pols = [synth.anchor_all(frames), synth.veil(1, 3)]      # the other head stays whole
        G.run_case(pols, 256, D, [frames], 41, seed=40 + segments, seg_tiles=16, q_gain=4.0, label="merge", rows=[0, 1, 31, 32, 40])
        G.run_case(pols, 255, D, [frames], 300, seed=60 + segments, seg_tiles=16, label="merge-300", rows=[0, 31, 127, 128, 255, 256, 299])
    finally:
        B.pf_set_tuning(attn_variant=-2)
