"""GPU: the index of pools with fewer heads than the index kernel has waves, as many, and more than one scan of 64 covers."""
import pytest

from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,tpf,Lq,seg_tiles", [(1, 70, 600, 16), (3, 400, 300, 16), (16, 70, 40, 0), (17, 300, 130, 16), (65, 2, 3, 0), (130, 40, 129, 0)])
def test_index_over_head_counts(H, tpf, Lq, seg_tiles):
    n = 9
    kinds = [synth.anchor_all(n), synth.anchor_topk(4, 4), synth.wave(2, n), synth.veil(1, 3), synth.wave(3, 16, cap=2, sink=1, recent=2)]
    G.run_case([kinds[(h * h) % 5] for h in range(H)], tpf, 64, [3, 3, 3], Lq, seed=50 + H, rows=None, check_every_append=False, seg_tiles=seg_tiles, label="heads")
