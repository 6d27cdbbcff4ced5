"""GPU parity of the corrector's training loss (brisk_corrector_loss) against
the CPU oracle, on the decoding path's own candidates, refined logits and
accept lengths."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

brisk = pytest.importorskip("paper_2609_33390_amd")


def _run(wl, psi_std=0.02, sigma=0.3):
    blk = synth.make_block(wl, "cuda", psi_std=psi_std)
    cl, ci = brisk.propose_block(blk.H, blk.W, wl.K)
    corr = brisk.Corrector(blk.psi, blk.alpha, blk.b_g)
    rr = brisk.rerank(corr, blk.H, blk.h_c, blk.x0, blk.W, blk.E, cl, ci, wl.B, wl.L, want_scores=True)
    acc, _ = brisk.verify_accept(rr["selected"], blk.verifier)
    g = torch.Generator(device="cuda").manual_seed(3)
    Hv = (blk.H.float() + sigma * torch.randn(blk.H.shape, generator=g, device="cuda")).to(torch.bfloat16)
    out = brisk.corrector_loss(Hv, blk.W, ci, cl, rr["refined"], acc, wl.B, wl.L)
    torch.cuda.synchronize()
    g_out = {k: v.cpu().numpy() for k, v in out.items()}
    o = oracle.corrector_loss(oracle.bf16_to_f64(synth.bf16_bits(Hv)), synth.bf16_bits(blk.W),
                              ci.cpu().numpy(), cl.cpu().numpy().astype(np.float64),
                              rr["refined"].cpu().numpy().astype(np.float64), acc.cpu().numpy(), wl.L)
    return g_out, o


def _check(g, o):
    assert np.all(g["loss_pos"][~o["mask"]] == 0.0)   # unreached positions contribute nothing
    np.testing.assert_allclose(g["loss_pos"], o["loss_pos"], rtol=1e-3, atol=2e-3)
    np.testing.assert_allclose(g["ce"][o["mask"]], o["ce"][o["mask"]], rtol=1e-3, atol=2e-3)
    np.testing.assert_allclose(g["kl"][o["mask"]], o["kl"][o["mask"]], rtol=1e-3, atol=2e-3)
    assert int(g["loss_mean"][1]) == o["count"]
    assert g["loss_mean"][0] == pytest.approx(o["mean"], rel=1e-3, abs=1e-3)


@pytest.mark.parametrize("name", ["tiny-d64-v512", "llada8b-b1-l32",
                                  pytest.param("llada8b-b64-l32", marks=pytest.mark.slow),
                                  pytest.param("dream7b-b16-l32", marks=pytest.mark.slow),
                                  pytest.param("llada8b-b256-l16", marks=pytest.mark.slow)])
def test_loss_matches_oracle(name):
    g, o = _run(synth.WORKLOADS[name])
    print(f"[loss] {name}: {o['count']} of {len(o['mask'])} positions reached", flush=True)
    _check(g, o)


@pytest.mark.parametrize("B,L,K,d,V", [(5, 7, 16, 136, 900), (33, 4, 5, 64, 300), (2, 40, 64, 72, 700)])
def test_loss_ragged_and_scaled_corrector(B, L, K, d, V):
    wl = synth.Workload("lossr", B=B, L=L, d=d, V=V, K=K, r=32, sigma=0.3, flat_frac=0.5, seed=B + L + K)
    g, o = _run(wl, psi_std=0.2)
    _check(g, o)
    assert 0 < o["count"] <= B * L


@pytest.mark.parametrize("B,L,K,d,V", [(3, 5, 4, 4096, 500), (3, 5, 5, 4104, 500), (2, 6, 9, 520, 300),
                                       (1100, 1, 8, 64, 300), (41, 100, 1, 8, 300)])
def test_loss_at_the_edges_of_its_batches(B, L, K, d, V):
    """Candidates either side of a pair and of a round of pairs, d either side
    of one round of loads and of a chunk, rows either side of the mean's batch."""
    g = torch.Generator().manual_seed(B + d)
    rows = B * L
    Hv, W = (torch.randn(n, d, generator=g).to(torch.bfloat16) for n in (rows, V))
    W = (W.float() * d ** -0.5).to(torch.bfloat16)
    ci = torch.rand(rows, V, generator=g).argsort(1)[:, :K].to(torch.int32).contiguous()
    cl, ref = (torch.randn(rows, K, generator=g) for _ in range(2))
    acc = torch.randint(0, L + 1, (B,), generator=g).to(torch.int32)
    out = brisk.corrector_loss(*(t.cuda() for t in (Hv, W, ci, cl, ref, acc)), B, L)
    torch.cuda.synchronize()
    o = oracle.corrector_loss(oracle.bf16_to_f64(synth.bf16_bits(Hv)), synth.bf16_bits(W), ci.numpy(),
                              cl.double().numpy(), ref.double().numpy(), acc.numpy(), L)
    _check({k: v.cpu().numpy() for k, v in out.items()}, o)
