"""GPU parity of the rerank on either side of every rule that decides how the
scan gets its step inputs: gathered from the tables, copied beside the
projections, copied in a pass, or turned into u = a u + b by the gate pass."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle_io import oracle_inputs
from parity import check_rerank, rerank_pick_ok

pytestmark = pytest.mark.gpu

brisk = pytest.importorskip("paper_2609_33390_amd")


@pytest.mark.parametrize("B,L,K,r,tables", [
    (1, 5, 8, 32, True), (5, 34, 8, 64, True), (6, 34, 8, 64, True), (46, 6, 8, 32, True), (47, 6, 8, 32, True),
    (64, 3, 8, 32, True), (2, 9, 9, 256, True), (56, 4, 16, 32, True), (57, 4, 16, 32, True), (3, 70, 16, 40, True),
    (3, 12, 24, 96, True), (3, 12, 24, 96, False), (2, 33, 64, 32, True), (4, 7, 6, 320, True), (4, 7, 6, 320, False),
    (5, 20, 16, 72, False), (2, 5, 4, 8, True), (1, 1, 12, 256, True),
    (1, 24, 9, 32, True), (1, 25, 9, 32, True), (43, 4, 16, 32, True), (44, 4, 16, 32, True),
    (3, 5, 8, 257, True), (3, 5, 8, 257, False), (8, 24, 8, 257, True), (8, 24, 8, 320, True), (64, 3, 8, 320, True),
    (64, 3, 8, 257, True), (16, 6, 16, 512, True), (20, 5, 16, 512, True), (3, 6, 16, 512, False),
    (256, 2, 63, 256, False), (256, 2, 64, 256, False), (256, 2, 64, 256, True), (128, 2, 64, 511, False),
    (128, 2, 64, 512, False),
])
def test_rerank_at_the_edges_of_its_input_rules(B, L, K, r, tables):
    wl = synth.Workload("scanin", B=B, L=L, d=72, V=300, K=K, r=r, sigma=0.3, flat_frac=0.5, seed=B + L + K)
    blk = synth.make_block(wl, "cuda", psi_std=0.1)
    io = oracle_inputs(blk)
    cl, ci = brisk.propose_block(blk.H, blk.W, K)
    # neighbours share candidates, so features 2 and 3 are met
    ci[1::2, 1] = torch.where((ci[1::2] == ci[0::2][:ci[1::2].shape[0], :1]).any(1), ci[1::2, 1], ci[0::2][:ci[1::2].shape[0], 0])
    corr = brisk.Corrector(blk.psi, blk.alpha, blk.b_g)
    if tables:
        corr.prepare(blk.W, blk.E)
    rr = brisk.rerank_verify(corr, blk.H, blk.h_c, blk.x0, blk.W, blk.E, cl, ci, blk.verifier, B, L, want_scores=True)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in rr.items()}
    g.update(cand_logit=cl.cpu().numpy(), cand_id=ci.cpu().numpy())
    orc = oracle.rerank(io["psi"], io["alpha"], io["b_g"], io["H"], io["h_c"], io["x0"], io["W_bits"], io["E_bits"],
                        g["cand_logit"], g["cand_id"], B, L, prefix=g["selected"])
    check_rerank(g, orc)
    rerank_pick_ok(g["selected"], orc, g["cand_id"])
    acc, _ = oracle.verify_accept(g["selected"], io["verifier"])
    assert np.array_equal(acc, g["accept_len"])
