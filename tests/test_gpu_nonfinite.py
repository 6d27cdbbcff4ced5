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


# the last tile of a share holds 240 or 224 of 256 tokens (126464 in 256 or
# 128 equal shares), or 240 of the last whole-tile run
PARTIAL = [(20, 126464, 8), (33, 126464, 8), (64, 126464, 16), (100, 126464, 8), (128, 126464, 16),
           (200, 256 * 600 - 16, 8), (300, 256 * 600 - 16, 16), (1000, 256 * 600 - 16, 8), (40, 126464, 24)]


@pytest.mark.parametrize("rows,V,K", PARTIAL)
def test_a_nan_row_has_no_candidates(rows, V, K):
    """No token of a row of NaNs enters its lists, and no place past the end
    of a share does: every id is -1, and the verifier's token too."""
    d = 256
    g = torch.Generator().manual_seed(rows)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    W = (torch.randn(V, d, generator=g) * 0.1).to(torch.bfloat16)
    ref = _propose(H, W, K)
    bad = rows // 2
    H[bad] = float("nan")
    cl, ci = _propose(H, W, K)
    assert (ci[bad] == -1).all() and cl[bad].isnan().all()
    keep = torch.arange(rows) != bad
    assert torch.equal(cl[keep], ref[0][keep]) and torch.equal(ci[keep], ref[1][keep])
    _, _, tok = brisk.propose_verify(H.to(DEV), W.to(DEV), 1, K)
    assert int(tok[bad - 1]) == -1


@pytest.mark.parametrize("rows,V,K", PARTIAL)
def test_minus_infinite_logits_come_before_places_without_a_token(rows, V, K):
    """Rows with an infinite element: a few tokens have a logit of -inf, all
    others NaN.  Those few come out in id order, then empty places."""
    d = 256
    g = torch.Generator().manual_seed(rows + 1)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    W = (torch.randn(V, d, generator=g) * 0.1).to(torch.bfloat16)
    H[::7, 0] = float("inf")
    W[:, 0] = 0
    few = torch.randperm(V, generator=g)[:K - 3].sort().values
    W[few, 0] = -1
    cl, ci = _propose(H, W, K)
    want = torch.cat([few, torch.full((3,), -1)]).to(torch.int32)
    assert torch.equal(ci[::7], want.expand(ci[::7].shape))
    assert (cl[::7, :K - 3] == -float("inf")).all() and cl[::7, K - 3:].isnan().all()


@pytest.mark.parametrize("d", [72, 200, 1000])
@pytest.mark.parametrize("rows,K", [(20, 8), (20, 64), (60, 16), (60, 24), (100, 8), (200, 8), (300, 16), (300, 24)])
def test_an_infinite_row_leaves_its_neighbours_alone(rows, K, d):
    """A ragged d: the last slice of a row's copy runs into the next row, whose
    infinities and NaNs must not reach the products."""
    V = 256 * 300 + 9
    g = torch.Generator().manual_seed(rows + d)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16).to(DEV)
    W = (torch.randn(V, d, generator=g) * 0.1).to(torch.bfloat16).to(DEV)
    ref = brisk.propose_block(H, W, K)
    bad = torch.zeros(rows, dtype=torch.bool, device=DEV)
    bad[1::5] = True
    H[1::10, :] = float("inf")
    H[6::10, :] = float("nan")
    out = brisk.propose_block(H, W, K)
    for a, b in zip(out, ref):
        assert torch.equal(a[~bad], b[~bad])


@pytest.mark.parametrize("rows", [20, 60, 300])
def test_an_infinite_verifier_row_leaves_its_neighbours_alone(rows):
    d, V, K = 72, 256 * 300 + 9, 8
    g = torch.Generator().manual_seed(rows)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16).to(DEV)
    W = (torch.randn(V, d, generator=g) * 0.1).to(torch.bfloat16).to(DEV)
    ids = torch.rand(rows, 1000, generator=g).argsort(1)[:, :K].to(torch.int32).to(DEV)
    prob = torch.full((rows, K), 1.0 / K, device=DEV)
    u = torch.rand(rows, generator=g).to(DEV)
    run = lambda: brisk.spec_verify(H, W, ids[:, :1].contiguous(), ids, prob, u, 5)  # noqa: E731
    ref = run()
    H[1::5] = float("inf")
    out = run()
    keep = torch.ones(rows, dtype=torch.bool, device=DEV)
    keep[1::5] = False
    for k in ("row_accept", "row_resample"):
        assert torch.equal(out[k].view(-1)[keep], ref[k].view(-1)[keep])
