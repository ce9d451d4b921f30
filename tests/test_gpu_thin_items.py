"""GPU parity of the attention launches that the planner builds from thin work items (32 query rows, the keys split over a
workgroup's eight waves): small launches, where the library's own choice is left in place."""
import pytest

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu

THIN_VARIANT = 3


@pytest.fixture(autouse=True)
def own_choice():
    B.pf_set_tuning(attn_variant=-2)
    yield
    B.pf_set_tuning(attn_variant=1)


@pytest.mark.parametrize("tpf,chunks,Lq,layout", [
    (1, [1], 1, "packed"),                       # one key of history, one query token: seven waves without keys
    (32, [3], 32, "packed"),                     # frames and steps coincide
    (33, [3, 3], 33, "model"),                   # every step crosses a border, one row in the last query group
    (40, [1, 3, 2, 5, 1, 1, 4, 3, 3], 100, "model"),
    (90, [3, 3, 3, 3], 187, "packed"),           # borders inside a copy's four rows
    (333, [3, 3, 3], 666, "packed"),             # long heads: segments of several waves, merged through the workspace
])
def test_small_launches_of_thin_items(tpf, chunks, Lq, layout):
    n = sum(chunks)
    pols = [synth.anchor_all(n), synth.anchor_topk(5, 5), synth.wave(3, n), synth.wave(2, 16, cap=3, sink=1, recent=2), synth.veil(1, 3)]
    a, r = G.run_case(pols, tpf, 128, chunks, Lq, seed=700 + tpf, layout=layout, label="thin")
    print("tpf %d Lq %d max-abs %.2e rel %.2e" % (tpf, Lq, a, r))


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
