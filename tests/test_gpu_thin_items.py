"""GPU parity of the attention launches that the planner builds from thin work items (32 query rows, the keys split over a
workgroup's eight waves): small launches, where the library's own choice is left in place."""
import pytest
import torch

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu

THIN_VARIANT = 3


@pytest.fixture(autouse=True)
def own_choice():
    B.pf_set_tuning(attn_variant=-2)
    yield
    B.pf_set_tuning(attn_variant=-2)


def _pols(n):
    return [synth.anchor_all(n), synth.anchor_topk(5, 5), synth.wave(3, n), synth.wave(2, 16, cap=3, sink=1, recent=2), synth.veil(1, 3)]


@pytest.mark.parametrize("tpf,chunks,Lq,layout,variant", [
    (1, [1], 1, "packed", 1),                    # too short for thin items: heads of at most three key tiles take full ones
    (32, [3], 32, "packed", 1),
    (1, [1], 300, "packed", THIN_VARIANT),       # one key of history, ten steps: some waves with one, some with two
    (32, [3, 3], 64, "packed", THIN_VARIANT),    # frames and steps coincide
    (16, [3, 3, 3, 1], 48, "model", THIN_VARIANT),   # heads of 96 to 208 keys: waves without keys
    (33, [3, 3], 33, "model", THIN_VARIANT),     # every step crosses a border, one row in the last query group
    (40, [1, 3, 2, 5, 1, 1, 4, 3, 3], 100, "model", THIN_VARIANT),
    (90, [3, 3, 3, 3], 187, "packed", THIN_VARIANT),   # borders inside a copy's four rows
    (333, [3, 3, 3], 666, "packed", THIN_VARIANT),     # long heads: segments of several waves, merged through the workspace
])
def test_small_launches_of_thin_items(tpf, chunks, Lq, layout, variant):
    a, r = G.run_case(_pols(sum(chunks)), tpf, 128, chunks, Lq, seed=700 + tpf, layout=layout, label="thin", variant=variant)
    print("tpf %d Lq %d max-abs %.2e rel %.2e" % (tpf, Lq, a, r))


@pytest.mark.parametrize("gain,scale", [(8.0, 0.0), (64.0, 0.0), (1.0, 0.37), (1.0, 1.5)])
@pytest.mark.parametrize("tpf,chunks,Lq", [(90, [3, 3, 3, 3], 187), (333, [3, 3, 3], 666)])       # whole heads; heads cut and merged
def test_thin_items_with_scores_far_apart(tpf, chunks, Lq, gain, scale):
    """Longer queries and explicit scales: a wave's reference maximum moves in the middle of its keys, and the waves (and
    segments) that are merged have maxima hundreds of exponent units apart."""
    a, r = G.run_case(_pols(sum(chunks)), tpf, 128, chunks, Lq, seed=760 + tpf, q_gain=gain, scale=scale, check_every_append=False,
                      label="thin-far", variant=THIN_VARIANT)
    print("tpf %d gain %.0f scale %.2f max-abs %.2e rel %.2e" % (tpf, gain, scale, a, r))


def test_thin_items_replay_from_a_hip_graph():
    """Index and attention of a launch of thin items whose heads are cut and merged, captured into a graph: every replay gives the
    eager launch's bits, also after other work in between."""
    dev, tpf, Lq, n = "cuda:0", 333, 666, 9
    pols = _pols(n)
    pool = B.Pool(pols, tpf, 128)
    B.pf_pool_reset(pool)
    for ci in range(3):
        k, v = (synth.randn_bf16((len(pols), 3, tpf, 128), 900 + 2 * ci + i, device=dev) for i in (0, 1))
        B.pf_cache_append(pool, k, v, synth.frame_scores(len(pols), 3, 930 + ci, device=dev))
    index = B.Index(pool, Lq)
    q, k_cur, v_cur = (synth.randn_bf16((len(pols), Lq, 128), 940 + i, device=dev) for i in range(3))
    out = torch.zeros_like(q)
    ws = torch.empty(B.pf_attn_workspace_bytes(pool, Lq), dtype=torch.uint8, device=dev)

    def run():
        B.pf_build_index(pool, index, Lq)
        B.pf_ragged_attn_fwd(pool, index, q, k_cur, v_cur, out, ws)

    run()
    torch.cuda.synchronize()
    assert index.c.variant == THIN_VARIANT and index.c.n_partials > 0
    eager = out.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            run()
    torch.cuda.synchronize()
    for rep in range(3):
        out.fill_(float("nan"))
        ws.fill_(0xff)                               # partial results of an earlier launch must not matter
        (q * 2).sum().item()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), eager.view(torch.int16)), "replay %d differs" % rep


def test_the_planner_takes_thin_items_where_they_fill_the_chip():
    pools = {}
    for Lq, tpf, n_frames in [(666, 333, 9), (4680, 1560, 18)]:
        pool = B.Pool([synth.anchor_all(n_frames)] * 5 if Lq == 666 else [synth.anchor_all(n_frames)] * 12, tpf, 128)
        B.pf_pool_reset(pool)
        for _ in range(n_frames // 3):
            k = synth.randn_bf16((pool.n_heads, 3, tpf, 128), 1, device="cuda:0")
            B.pf_cache_append(pool, k, k)
        index = B.Index(pool, Lq)
        B.pf_build_index(pool, index, Lq)
        assert B.pf_index_status(index) == 0
        pools[Lq] = index.c.variant
    assert pools[666] == THIN_VARIANT and pools[4680] == 1
