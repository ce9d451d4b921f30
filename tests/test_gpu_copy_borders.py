"""GPU parity where the rows that a wave copies at a time (32 keys of a thin item, 16 at head_dim 64, 8 or 16 of a full item) meet frame
borders in every way: frames shorter than the rows (several borders inside them), shorter than a tile (frames that a wave steps over),
barely longer, and the border to a chunk of strided rows."""
import pytest
import torch

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


# bytes between token rows of the chunk: a run of tiles is cut where its 32-bit offsets would pass 2^31, here after two tiles, after one (a
# power of two, and the widest rows there may be); 2^20: not at all
@pytest.mark.parametrize("D,variant", [(64, -2), (128, -2), (128, 0), (128, 1), (128, 2)], ids=["d64", "thin", "w4x32", "pp8x32", "w4x64"])
@pytest.mark.parametrize("stride,Lq", [(1 << 20, 397), (1 << 22, 397), (1 << 23, 203), ((1 << 24) - 8, 139)])
def test_chunk_rows_far_apart(stride, Lq, D, variant):
    """The same chunk with its token rows as far apart as the layout may ask for: the packed call's bits."""
    B.pf_set_tuning(attn_variant=variant)
    try:
        H, tpf, frames, dev = 3, 150, 3, "cuda:0"
        pool = B.Pool([synth.anchor_all(frames), synth.wave(2, frames), synth.veil(1, 1)], tpf, D)
        B.pf_pool_reset(pool)
        B.pf_cache_append(pool, *(synth.randn_bf16((H, frames, tpf, D), 70 + i, device=dev) for i in (0, 1)))
        index = B.Index(pool, Lq)
        B.pf_build_index(pool, index, Lq)
        assert index.c.variant == (variant if variant >= 0 else 3 if D == 128 else 0)
        ws = torch.empty(B.pf_attn_workspace_bytes(pool, Lq), dtype=torch.uint8, device=dev)
        packed = [synth.randn_bf16((H, Lq, D), 80 + i, device=dev) for i in range(3)]
        want = torch.full_like(packed[0], float("nan"))
        B.pf_ragged_attn_fwd(pool, index, *packed, want, ws)
        # q, k, v and the output share the wide rows
        rows = torch.empty(Lq * stride, dtype=torch.bfloat16, device=dev)
        views = [torch.as_strided(rows, (H, Lq, D), (D, stride, 1), i * H * D) for i in range(4)]
        for t, view in zip(packed + [torch.full_like(want, float("nan"))], views):
            view.copy_(t)
        B.pf_ragged_attn_fwd_strided(pool, index, *views, ws)
        torch.cuda.synchronize()
        assert torch.isfinite(want.float()).all()
        assert torch.equal(views[3].contiguous().view(torch.int16), want.view(torch.int16))
        assert all(torch.equal(view.contiguous().view(torch.int16), t.view(torch.int16)) for t, view in zip(packed, views))
    finally:
        B.pf_set_tuning(attn_variant=-2)
