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


@pytest.mark.parametrize("segments,frames", [(2, 14), (3, 24), (8, 68), (9, 78), (17, 152)])
def test_partial_results_of_many_thin_segments(segments, frames):
    """Thin items have a merge of their own shape (32 rows, two quads a thread).  41 and 70 rows: two and three groups of query rows, nine and
    six of them in the last one."""
    B.pf_set_tuning(attn_variant=-2)
    pols = [synth.anchor_all(frames)] * 2
    for Lq, gain in ((41, 4.0), (70, 1.0)):
        c = B.Pool(pols, 333, 128).c
        assert B.pf_plan_segments(c, frames, Lq)[2] == 2 * -(-Lq // 32) * segments
        G.run_case(pols, 333, 128, [frames], Lq, seed=80 + segments, q_gain=gain, label="thin-merge", rows=[0, 1, 31, 32, Lq - 1], variant=3)
