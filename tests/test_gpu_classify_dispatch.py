"""GPU: both classification kernels give the same types and periods, bit for bit, on either side of the line between them."""
import pytest
import torch

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
