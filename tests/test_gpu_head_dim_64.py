"""head_dim 64: GPU parity of its attention kernel at the edges of its tiles, and the bounds its launch plans keep."""
import ctypes
import random

import pytest

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth


@pytest.mark.gpu
@pytest.mark.parametrize("tpf,chunks,Lq,layout,seg_tiles", [
    (1, [1], 1, "packed", 0),                    # two keys, one query row: three waves without rows
    (64, [1], 32, "model", 0),                   # frames and tiles coincide; one wave has rows
    (15, [3, 3, 3], 129, "model", 0),            # several frame borders inside one wave's 16 copied rows; a second query tile of one row
    (17, [3, 3, 1], 127, "packed", 0),
    (100, [3, 3, 3, 3], 128, "packed", 0),       # borders inside a copy's eight rows
    (129, [3, 2, 3], 258, "model", 16),          # heads cut into the shortest segments, merged through the workspace
    (700, [3, 3, 3], 600, "packed", 0),          # ... as the planner cuts a small launch by itself
])
def test_attention_head_dim_64(tpf, chunks, Lq, layout, seg_tiles):
    import gpu_common as G
    n = sum(chunks)
    pols = [synth.anchor_all(n), synth.anchor_topk(5, 5), synth.wave(3, n), synth.wave(2, 16, cap=3, sink=1, recent=2), synth.veil(1, 3)]
    a, r = G.run_case(pols, tpf, 64, chunks, Lq, seed=900 + tpf, layout=layout, seg_tiles=seg_tiles, label="d64")
    print("tpf %d Lq %d max-abs %.2e rel %.2e" % (tpf, Lq, a, r))


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["packed", "model"])
@pytest.mark.parametrize("tpf,frames,Lq", [
    (127, 5, 512), (128, 5, 511), (128, 5, 512), (130, 4, 520), (255, 3, 255), (255, 3, 510), (256, 3, 256), (257, 3, 70), (300, 4, 17)])
def test_attention_head_dim_64_on_both_sides_of_runs(tpf, frames, Lq, layout):
    """Frames and chunks on either side of the line from which copies follow runs of tiles: frames that are whole tiles and frames that leave
    some rows over, chunks of less than a wave's rows and of several tiles."""
    import gpu_common as G
    pols = [synth.anchor_all(frames), synth.wave(2, frames), synth.veil(1, 2)]
    G.run_case(pols, tpf, 64, [frames], Lq, seed=950 + tpf, layout=layout, label="d64-runs", rows=sorted({0, 15, 16, Lq // 2, Lq - 2, Lq - 1} & set(range(Lq))))


@pytest.mark.gpu
def test_attention_head_dim_64_rising_scores():
    """Queries 40 times as long: scores hundreds of exponent units apart, so the reference maximum moves often."""
    import gpu_common as G
    pols = [synth.anchor_all(6), synth.wave(2, 6), synth.veil(1, 3)]
    G.run_case(pols, 100, 64, [3, 3], 150, seed=77, q_gain=40.0, label="d64-rising")


def _host_pool(pols, tpf, head_dim):
    H, fake = len(pols), 1 << 12                  # the planner reads the host fields only
    hp = (B.pf_head_policy * H)(*[B.make_policy(p) for p in pols])
    c = B.pf_pool(H, head_dim, tpf, 0, sum(int(p.slots) for p in pols), fake, fake, ctypes.cast(hp, ctypes.POINTER(B.pf_head_policy)),
                  fake, fake, fake, fake, fake, fake, fake, 0, 0)
    c._keep = hp
    return c


def _rows_of(rows, seg, tiles, blocks, q_tokens):
    """Query rows per block of a plan: a multiple of eight (head, segment) teams times the query tiles.  A chunk that one block of
    either size covers does not tell them apart; then the larger."""
    teams = sum(-(-t // s) for t, s in zip(tiles, seg))
    return max(r for r in rows if -(-teams // 8) * 8 * -(-q_tokens // r) == blocks)


@pytest.mark.parametrize("head_dim,rows", [(64, (128,)), (128, (32, 256))])
def test_plans_stay_inside_their_workspace_and_unsplit_launches_stay_unsplit(head_dim, rows):
    """Over random pools: a plan's partial results fit pf_attn_workspace_bytes, and a launch whose heads are at most 48 key tiles
    long, which one segment covers, needs no workspace at all."""
    rng = random.Random(5)
    B.pf_set_tuning(attn_variant=-2, seg_tiles=0)
    unsplit = short = 0
    planned = set()
    for _ in range(150):
        T, H, n = rng.randint(0, 40), rng.randint(1, 24), rng.randint(1, 3)
        tpf = rng.choice([1, 16, 77, 200, 333, 700, 1560])
        pols = [p._replace(slots=max(1, B.slots_needed(p, max(T, 1)))) for p in synth.drawn_policies(H, rng.randint(0, 999), max(T, 1))]
        c = _host_pool(pols, tpf, head_dim)
        seg, blocks, partials = B.pf_plan_segments(c, T, n * tpf)
        ws = int(B.lib().pf_attn_workspace_bytes(ctypes.byref(c), n * tpf))
        tiles = [-(-(B.pf_selected_count(p, T) + n) * tpf // 64) for p in pols]
        per_block = _rows_of(rows, seg, tiles, blocks, n * tpf)
        planned.add(per_block)
        assert partials * per_block * (head_dim + 2) * 4 <= ws
        if max(tiles) <= 48:
            unsplit += 1
            assert partials == 0
        if head_dim == 64:
            short += min(seg) < 48
            assert min(seg) >= 48 or blocks <= 640 + 7 * -(-n * tpf // 128)
    assert unsplit > 10 and (head_dim == 128 or short > 10) and planned == set(rows)


@pytest.mark.parametrize("heads,policy,T,chunk,tpf,limit", [
    (24, "veil", 6, 2, 700, 0), (64, "veil", 23, 3, 1560, 0), (40, "all", 57, 3, 1560, 0), (80, "all", 28, 1, 700, 0), (16, "veil", 124, 2, 1560, 0),
    (64, "all", 235, 2, 700, 160 << 20), (64, "skewed", 39, 3, 1000, 160 << 20), (80, "skewed", 48, 2, 1560, 160 << 20),
    (64, "wave", 85, 1, 1560, 160 << 20),
])
def test_launches_that_need_no_workspace_or_fit_the_library_array_keep_to_that(heads, policy, T, chunk, tpf, limit):
    """Launches that can be made without a workspace, or through pf_ragged_attn_fwd_static (160 MiB), however much sooner more and
    shorter segments would let them finish."""
    n_all = {"veil": 0, "all": heads, "skewed": heads // 4 + 1, "wave": 0}[policy]
    pols = [synth.anchor_all(T)] * n_all + [synth.wave(2, T) if policy == "wave" else synth.veil(1, 3)] * (heads - n_all)
    c = _host_pool([p._replace(slots=max(1, B.slots_needed(p, T))) for p in pols], tpf, 64)
    B.pf_set_tuning(attn_variant=-2, seg_tiles=0)
    _, _, partials = B.pf_plan_segments(c, T, chunk * tpf)
    assert partials * 128 * (64 + 2) * 4 <= limit


@pytest.mark.gpu
def test_a_whole_launch_runs_without_a_workspace():
    import torch
    H, T, tpf, Lq = 24, 4, 200, 2400                 # 19 query tiles; 3200 keys a head: 50 tiles, more than the shortest planned segment
    pool = B.Pool([synth.anchor_all(T)] * H, tpf, 64)
    B.pf_pool_reset(pool)
    k, v = (synth.randn_bf16((H, T, tpf, 64), i, device="cuda:0") for i in (1, 2))
    B.pf_cache_append(pool, k, v)
    q, k_cur, v_cur = (synth.randn_bf16((H, Lq, 64), 3 + i, device="cuda:0") for i in range(3))
    index = B.Index(pool, Lq)
    B.pf_build_index(pool, index, Lq)
    out = torch.full_like(q, float("nan"))
    B.pf_ragged_attn_fwd(pool, index, q, k_cur, v_cur, out, None)
    want = torch.nn.functional.scaled_dot_product_attention(*(t.float() for t in (q, torch.cat([k.flatten(1, 2), k_cur], 1), torch.cat([v.flatten(1, 2), v_cur], 1))))
    assert (out.float() - want).abs().max() < 2e-2   # the oracle's bound
