"""GPU: the append kernel for at most 64 candidates a head and 4 new frames, at its limits and against the general kernel."""
import numpy as np
import pytest
import torch

from oracle.pool import PoolOracle
from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _new(H, n, tpf, D, seed):
    """K, V and scores of n frames; scores with many ties and both infinities."""
    k, v = (synth.randn_bf16((H, n, tpf, D), 2 * seed + i) for i in (0, 1))
    sc = (synth.frame_scores(H, n, seed) * 4).floor() / 4
    sc[0, 0] = float("-inf") if seed % 2 else float("inf")
    return k, v, sc


@pytest.mark.parametrize("D,tpf", [(64, 1), (64, 33), (128, 17), (128, 130)])     # 8 units a frame; part of, exactly and just over a block
def test_append_at_the_limits_of_the_wave_plan(D, tpf):
    pols = [synth.anchor_all(70), synth.anchor_topk(5, 8, sink=1, recent=2), synth.wave(3, 40, cap=4, sink=1, recent=2), synth.veil(1, 3)]
    pool_o, pool_g = PoolOracle(pols, tpf, D), B.Pool(pols, tpf, D, device=DEV)
    B.pf_pool_reset(pool_g)
    # 57 frames in 1, 4 and 5 at a time (5: the general kernel), then 57 + 4 = 61, 61 + 3 = 64 candidates and 64 + 1 = 65
    for i, n in enumerate([1, 4, 4, 5, 4, 4, 3, 4, 4, 4, 5, 4, 4, 3, 4, 4, 3, 1, 2]):
        k, v, sc = _new(len(pols), n, tpf, D, 100 + i)
        pool_o.append(synth.bits(k), synth.bits(v), sc.numpy())
        B.pf_cache_append(pool_g, k.to(DEV), v.to(DEV), sc.to(DEV))
        G.check_pool(pool_g, pool_o)
    assert pool_g.T == 67


def test_both_append_kernels_leave_the_same_pool():
    """The same appends to a pool and to one with a further head that keeps everything (more than 64 candidates: the general
    kernel): tables and all slots of the common heads, freed ones among them, hold the same bits."""
    tpf, D = 40, 64
    pols = [synth.anchor_topk(18, 18), synth.anchor_topk(7, 12, sink=2, recent=3), synth.wave(2, 40, cap=6, recent=1), synth.veil(1, 3),
            synth.veil_merged(1, 2, 2, 3, 12)]
    H, n_common = len(pols), sum(int(p.slots) for p in pols)
    few, more = B.Pool(pols, tpf, D, device=DEV), B.Pool(pols + [synth.anchor_all(120)], tpf, D, device=DEV)
    B.pf_pool_reset(few)
    B.pf_pool_reset(more)
    for i in range(32):
        k, v, sc = (t.to(DEV) for t in _new(H + 1, 3, tpf, D, 300 + i))
        B.pf_cache_append(more, k, v, sc)
        B.pf_cache_append(few, k[:H].contiguous(), v[:H].contiguous(), sc[:H].contiguous())
    torch.cuda.synchronize()
    assert torch.equal(few.n_frames, more.n_frames[:H]) and few.T == more.T == 96
    for a, b in ((few.frame_ids, more.frame_ids), (few.frame_score.view(torch.int32), more.frame_score.view(torch.int32)),
                 (few.k_pool.view(torch.int16), more.k_pool.view(torch.int16)), (few.v_pool.view(torch.int16), more.v_pool.view(torch.int16))):
        assert np.array_equal(a.cpu().numpy(), b[:n_common].cpu().numpy())


@pytest.mark.parametrize("H,tpf", [(3, 2048), (3, 2049), (12, 4096), (12, 4097)])     # the last frame size of the small kernel, and one token more
def test_append_on_either_side_of_the_largest_frames(H, tpf):
    pols = [[synth.anchor_topk(2, 3), synth.wave(3, 8, cap=1, sink=1, recent=2), synth.veil(1, 2)][h % 3] for h in range(H)]
    pool_o, pool_g = PoolOracle(pols, tpf, 128), B.Pool(pols, tpf, 128, device=DEV)
    B.pf_pool_reset(pool_g)
    for i, n in enumerate([2, 1, 2]):
        k, v, sc = _new(H, n, tpf, 128, 500 + i)
        pool_o.append(synth.bits(k), synth.bits(v), sc.numpy())
        B.pf_cache_append(pool_g, k.to(DEV), v.to(DEV), sc.to(DEV))
        G.check_pool(pool_g, pool_o)
