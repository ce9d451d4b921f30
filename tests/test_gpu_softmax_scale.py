"""GPU parity of the attention kernels at softmax scales a caller with pre-scaled queries passes, where a wave's first keys are
the ragged end of a sequence: the first reference maximum is not known yet when the masked keys' weights are formed."""
import pytest

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth
import gpu_common as G

pytestmark = pytest.mark.gpu

CASES = [                                       # ..., the kernel that the library chooses
    (64, 16, [], 48, "packed", 0),              # one ragged tile is all there is: every lane holds masked keys
    (64, 16, [], 59, "model", 0),               # ... the most keys with which that is so; one more, and some lanes hold none
    (64, 16, [], 60, "packed", 0),
    (64, 300, [3, 3, 3], 330, "model", 0),      # long heads, cut and merged
    (128, 16, [], 48, "model", 1),
    (128, 1, [1], 1, "packed", 1),
    (128, 16, [3, 3, 3, 1], 48, "packed", 3),   # thin items; head 0: 208 keys in seven steps of 32, the last wave's only one holds 16
    (128, 61, [3], 48, "model", 3),             # ... 231 keys, seven of them in the last wave's step
    (128, 52, [2, 2], 48, "packed", 3),         # ... 256 keys, a full step per wave
    (128, 300, [3, 3, 3], 330, "model", 3),
]


# the library's own choice of kernel and the three that can be asked for (head_dim 64 has one kernel)
@pytest.mark.parametrize("variant,case", [(v, c) for v in (-2, 0, 1, 2) for c in CASES if c[0] == 128 or v == -2],
                         ids=lambda x: "v%d" % x if isinstance(x, int) else "D%d-tpf%d-T%d-Lq%d" % (x[0], x[1], sum(x[2]), x[3]))
@pytest.mark.parametrize("scale", [0.78, 1.0, 4.0])     # the start value -3e38 times scale * log2(e) is finite up to 0.786
def test_explicit_scales(variant, case, scale):
    D, tpf, chunks, Lq, layout, chosen = case
    n = max(sum(chunks), 1)
    B.pf_set_tuning(attn_variant=variant)
    try:
        a, r = G.run_case([synth.anchor_all(n), synth.veil(1, 3), synth.wave(2, n)], tpf, D, chunks, Lq, seed=1200 + tpf + Lq,
                          layout=layout, scale=scale, label="scale", variant=chosen if variant == -2 else variant)
    finally:
        B.pf_set_tuning(attn_variant=-2)
    print("D %d scale %.2f max-abs %.2e rel %.2e" % (D, scale, a, r))
