"""GPU checks of the LM-head pass on rows and tokens that are not finite: they
stay out of the other rows' and tokens' results, whatever tile they meet."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import check_candidates

pytestmark = pytest.mark.gpu

brisk = pytest.importorskip("paper_2609_33390_amd")
DEV = "cuda"


def _propose(H, W, K):
    cl, ci = brisk.propose_block(H.to(DEV), W.to(DEV), K)
    torch.cuda.synchronize()
    return cl.cpu(), ci.cpu()


@pytest.mark.parametrize("rows,K", [(20, 16), (40, 8), (40, 16), (100, 12), (300, 8), (300, 16), (40, 24)])
def test_nan_tokens_leave_the_finite_ones_their_places(rows, K):
    """The first tile holds every row's best tokens, and every ninth token of
    the vocabulary is NaN: the K best finite ones come out."""
    d, V = 64, 256 * 600
    g = torch.Generator().manual_seed(rows + K)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    W = torch.randn(V, d, generator=g) * 0.01
    W[:256] *= 100
    W[4::9] = float("nan")
    W = W.to(torch.bfloat16)
    cl, ci = _propose(H, W, K)
    ol = oracle.lm_logits(oracle.bf16_to_f64(synth.bf16_bits(H)), synth.bf16_bits(W))
    check_candidates(cl.numpy(), ci.numpy(), np.where(np.isnan(ol), -1e30, ol))
