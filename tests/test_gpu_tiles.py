"""GPU parity of the LM-head pass at the edges of its row tiles and shares.

Row counts sit on either side of each row tile (32, 64, 128, 192, 256 and the
combinations above); vocabularies give every workgroup one whole tile and a
partial one, or whole tiles only; d covers whole 64-wide slices, a ragged last
slice and a single slice.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import check_candidates
from plan import plan

pytestmark = pytest.mark.gpu

brisk = pytest.importorskip("paper_2609_33390_amd")
DEV = "cuda"


@pytest.mark.parametrize("rows,d,V,K", [
    (33, 128, 256 * 270, 8), (64, 136, 256 * 330 + 5, 16), (65, 64, 256 * 300, 4), (128, 200, 256 * 400 + 1, 8),
    (129, 72, 256 * 300 + 77, 16), (192, 128, 256 * 460, 8), (193, 136, 256 * 290, 8), (256, 64, 256 * 350 + 3, 16),
    (300, 128, 128 * 300, 8), (320, 200, 128 * 600 + 9, 10), (512, 72, 128 * 390, 16), (546, 128, 85 * 300, 10),
    (600, 192, 51 * 700 + 11, 8), (1024, 64, 64 * 600 + 1, 12), (100, 64, 700, 33), (260, 136, 20011, 40),
])
def test_row_tiles_and_partial_shares(rows, d, V, K):
    g = torch.Generator().manual_seed(rows * 7919 + V)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    W = (torch.randn(V, d, generator=g) * 0.1).to(torch.bfloat16)
    # the last token of the vocabulary, in the last place of the last share, is
    # the top one of the rows at the tiles' edges and of every 40th or so
    ends = [r for t in (64, 128, 192, 256) for r in range(t - 1, rows, t)]
    rs = np.array(sorted({0, rows - 1, *range(0, rows, max(1, rows // 40)), *ends}))
    u = torch.randn(d, generator=g)
    u /= u.norm()
    H[rs] = (H[rs].float() + 8 * u).to(torch.bfloat16)
    W[V - 1] = (4 * u).to(torch.bfloat16)
    print(f"rows {rows} d {d} V {V} K {K}", flush=True)
    cl, ci = brisk.propose_block(H.to(DEV), W.to(DEV), K)
    torch.cuda.synchronize()
    ol = oracle.lm_logits(oracle.bf16_to_f64(synth.bf16_bits(H[rs])), synth.bf16_bits(W))
    assert (ol.argmax(1) == V - 1).all()
    check_candidates(cl.cpu().numpy()[rs], ci.cpu().numpy()[rs], ol)


@pytest.mark.parametrize("rows,V,left", [(40, 256 * 300, 0), (128, 256 * 300 + 5, 0), (200, 256 * 301 - 7, 249), (512, 64 * 600 + 9, 9)])
def test_partial_tiles_keep_exact_ties_in_id_order(rows, V, left):
    """Equal LM-head rows in the partial tiles of different shares, and in whole
    ones, have equal logits and come in id order.  Up to 128 rows these sizes
    make 256 equal shares of a whole and a partial tile; above, the last tile
    of the vocabulary holds `left` tokens."""
    d, K = 192, 16
    g = torch.Generator().manual_seed(5)
    if left:
        assert V % 256 == left
        ids = torch.cat([torch.arange(V - left, V)[:8], torch.randperm(V - 300, generator=g)[:K - 8]])
    else:
        assert plan(rows, d, V, K)[1] == 256
        start = [(s * V // 256) & ~15 for s in range(256)] + [V]
        shares = torch.randperm(255, generator=g)[:K - 3].tolist() + [255]
        ids = torch.tensor([start[s] + 256 + (7 * s) % (start[s + 1] - start[s] - 256) for s in shares] + [0, 300])
    ids = ids.unique()
    assert len(ids) == K
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    W = (torch.randn(V, d, generator=g) * 0.01).to(torch.bfloat16)
    W[ids] = (H[:200].float().mean(0) * 2).to(torch.bfloat16)
    cl, ci = brisk.propose_block(H.to(DEV), W.to(DEV), K)
    cl, ci = cl.cpu(), ci.cpu()
    # other logits have a standard deviation of 0.01 |H| ~ 0.14: the largest of
    # V is near 0.6, and 1.2 is out of their reach
    top = H.float() @ W[ids[0]].float() > 1.2
    assert int(top.sum()) > 5
    assert torch.equal(ci[top], ids.to(torch.int32).expand(int(top.sum()), K))
    assert torch.equal(cl[top], cl[top][:, :1].expand(-1, K))


@pytest.mark.parametrize("left", [1, 17, 100, 255])
@pytest.mark.parametrize("rows,K", [(40, 8), (64, 16), (100, 4), (128, 16), (200, 8), (250, 16), (520, 8)])
def test_a_last_share_shorter_than_a_tile(rows, K, left):
    """The last share has `left` tokens, and its tile starts among the share
    before: the best tokens lie on both sides of the border, each comes once."""
    d, V = 128, 156 * 256 + left
    g = torch.Generator().manual_seed(rows + left)
    H = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    W = torch.randn(V, d, generator=g) * 0.05
    W[-300:] *= 4
    W = W.to(torch.bfloat16)
    cl, ci = brisk.propose_block(H.to(DEV), W.to(DEV), K)
    ol = oracle.lm_logits(oracle.bf16_to_f64(synth.bf16_bits(H)), synth.bf16_bits(W))
    check_candidates(cl.cpu().numpy(), ci.cpu().numpy(), ol)
