"""GPU: the classification kernels give the same types and periods, bit for bit, on either side of the lines between them."""
import numpy as np
import pytest
import torch

from oracle import classify as OC
from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hist", [81, 100, 256])
def test_few_long_sequences_agree_with_many(hist):
    logits, _ = synth.head_logits(64, 12, hist, 5)               # 768 sequences: batches of 16
    logits = logits.to("cuda:0")
    _, types, periods = B.pf_classify_heads(logits)
    _, t, p = B.pf_classify_heads(logits[:63].contiguous())      # 756: a workgroup each
    torch.cuda.synchronize()
    assert torch.equal(t, types[:63]) and torch.equal(p.view(torch.int64), periods[:63].view(torch.int64))


@pytest.mark.parametrize("hist", [3, 4, 7, 10, 11, 24, 69, 70, 71, 72, 73, 80, 200])
def test_kernels_agree_on_either_side_of_the_lines_between_them(hist):
    """4800 sequences: in LDS up to 72 frames, else by rounds; 4607 and 768: by rounds up to 10 and from 71 frames on; 767: a workgroup each."""
    logits, _ = synth.head_logits(200, 24, hist, 6)
    flat = logits.to("cuda:0").view(1, 4800, hist)
    _, types, periods = B.pf_classify_heads(flat)
    for n in (4608, 4607, 768, 767):
        _, t, p = B.pf_classify_heads(flat[:, :n].contiguous())
        assert torch.equal(t, types[:, :n]) and torch.equal(p.view(torch.int64), periods[:, :n].view(torch.int64)), n


# shortest and longest of the kernel that keeps sequences in LDS, its neighbour; bins left over beside the groups of 16: 0, 1, 2, 3, 4, 5
# (N/2 = 16, 17, 18, 35, 20, 21) and a group of its own; even lengths whose rows start in few banks.  Once over (920 sequences) those of
# 4 to 6 and of 71 and 72 frames go by rounds
@pytest.mark.parametrize("times", [1, 6])
@pytest.mark.parametrize("hist", [4, 5, 6, 33, 35, 38, 42, 44, 64, 69, 71, 72, 73])
@pytest.mark.parametrize("skip", [0, 1])
def test_short_sequences_in_lds(hist, skip, times):
    logits, _ = synth.head_logits(40, 23, hist, 11)
    flat = torch.empty(times * logits.numel() + skip, device="cuda:0")   # skip = 1: no 16-byte border at the start
    flat[skip:] = logits.flatten().to("cuda:0").repeat(times)
    view = flat[skip:].view(times * 40, 23, hist)
    head, types, periods = B.pf_classify_heads(view)
    want_head, want_types, want_periods = OC.classify_heads(logits.numpy())
    assert (head.cpu().numpy() == want_head).all() and (types.cpu().numpy() == np.tile(want_types, (times, 1))).all()
    assert (periods.cpu().numpy() == np.tile(want_periods, (times, 1))).all()


@pytest.mark.parametrize("hist", [73, 100, 200])
def test_rounds_whose_row_buffer_is_emptied_and_filled_again(hist):
    """40 000 sequences that are hardly settled by their signs: 64 for a workgroup, whose buffer holds 48, 32 and 16 rows."""
    logits, _ = synth.head_logits(4, 250, hist, 8)
    logits = (logits - logits.mean(dim=2, keepdim=True)).view(1, 1000, hist)
    _, want_types, want_periods = OC.classify_heads(logits.numpy())
    _, types, periods = B.pf_classify_heads(logits.to("cuda:0").repeat(40, 1, 1))
    assert (types.cpu().numpy() == np.tile(want_types, (40, 1))).all() and (periods.cpu().numpy() == np.tile(want_periods, (40, 1))).all()


def test_more_sequences_per_workgroup_than_lds_holds():
    logits, _ = synth.head_logits(16, 360, 72, 3)
    logits = logits.to("cuda:0").repeat(21, 1, 1)                # 120 960 sequences: two rounds of each workgroup
    _, types, periods = B.pf_classify_heads(logits)
    _, t, p = B.pf_classify_heads(logits[:16].contiguous())
    assert torch.equal(types, t.repeat(21, 1)) and torch.equal(periods, p.repeat(21, 1))


@pytest.mark.parametrize("prompts", [1, 2, 15, 16, 17, 32, 33, 112, 113, 127, 128, 129, 144, 145, 257])
@pytest.mark.parametrize("heads", [3, 64, 65])
def test_votes_of_any_number_of_prompts(prompts, heads):
    """On either side of what one wave counts (every 16th prompt), of its eight loads in flight and of their next turn."""
    logits, _ = synth.head_logits(prompts, heads, 12, 40 + prompts)
    head, types, _ = B.pf_classify_heads(logits.to("cuda:0"))
    want, want_types, _ = OC.classify_heads(logits.numpy())
    assert (types.cpu().numpy() == want_types).all() and (head.cpu().numpy() == want).all()


def _hand_made(n):
    t = np.arange(n)
    n_pos = -(-8 * n // 10)                                      # the fewest positive values that settle a sequence
    share = lambda k: np.where((t * 7) % n < k, 1.0, -1.0) if n % 7 else np.where((t * 5) % n < k, 1.0, -1.0)   # k of n positive, spread out
    rows = [share(n_pos), share(n_pos - 1), share(n - n_pos), share(n - n_pos + 1), np.ones(n), np.zeros(n),
            t - 0.5 * (n - 1), 0.5 * (n - 1) - t, t - 0.5 * (n - 1) + 0.25,        # every difference the same: no spectrum; the mean decides
            np.where(t % 2 == 0, 1.0, -1.0), np.sin(2 * np.pi * t / 6.0), np.sin(2 * np.pi * t / 20.0) - 0.05,
            np.sin(2 * np.pi * t / 12.0) + 0.7 * np.sin(2 * np.pi * t / 6.0 + 1.1), np.sin(2 * np.pi * t / 10.0) + np.sin(2 * np.pi * t / 5.0)]
    if n % 4 == 3:
        # two jumps half the transform apart, equally far from its ends: all odd bins alike, so the lowest of those with a third harmonic
        up = (n - 3) // 4
        rows.append(np.where((t > up) & (t <= n - 2 - up), 0.5, -0.5))
    wave = np.sin(2 * np.pi * t / 6.0)
    for bad in (np.nan, np.inf, -np.inf):                        # at an end, in the middle
        for at in (0, n // 2, n - 1):
            rows.append(np.where(t == at, bad, wave))
    return np.stack(rows).astype(np.float32)


# some 46 sequences: a workgroup each; 920: by rounds or in LDS; 4700: in LDS up to 72 frames
@pytest.mark.parametrize("times", [1, 20, 102])
@pytest.mark.parametrize("n", [6, 15, 23, 24, 25, 27, 39, 40, 65, 69, 70, 71, 72, 73, 75, 79, 80, 83, 100])
@pytest.mark.parametrize("first", [0, 5])
def test_hand_made_sequences(n, first, times):
    """Sign rates on and beside their thresholds, flat and empty spectra, tied peaks, infinities and NaN, which must not reach the sequences
    that are transformed with theirs.  Two prompts: the second one's rows in another order."""
    rows = np.roll(_hand_made(n), first, axis=0)
    logits = np.stack([rows, rows[::-1]])
    with np.errstate(invalid="ignore"):
        want = [np.tile(w, times) for w in OC.classify_heads(logits)]
    got = [g.cpu().numpy() for g in B.pf_classify_heads(torch.from_numpy(np.tile(logits, (1, times, 1))).to("cuda:0"))]
    for g, w in zip(got, want):                                  # heads, types, periods
        assert g.shape == w.shape and (g == w).all(), np.argwhere(g != w)
