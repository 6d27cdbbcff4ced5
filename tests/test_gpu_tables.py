"""GPU parity of the per-token tables (brisk_corrector_prepare) with their
definition in float64, at the edges of the kernels that build them: token
counts either side of a share's 16-token cut and of a 256-token tile, widths
that are not multiples of 8 or 4, one to eight 32-wide steps, a ragged d,
vocabularies on both sides of the kernels' rules."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

brisk = pytest.importorskip("paper_2609_33390_amd")
DEV = "cuda"


@pytest.mark.parametrize("V,d,ds,dh,dt,rank", [
    (5, 8, 4, 3, 1, 1), (16, 64, 32, 16, 16, 16), (777, 200, 96, 48, 48, 48), (2049, 136, 250, 30, 31, 33),
    (4096, 192, 256, 128, 128, 128), (33000, 72, 64, 32, 64, 65), (700, 128, 320, 100, 130, 200),
    (1000, 264, 512, 256, 256, 256), (501, 64, 257, 64, 2, 129), (32768 + 17, 128, 16, 8, 96, 100),
    (9999, 72, 40, 8, 24, 100), (10000, 72, 40, 8, 24, 100), (15999, 200, 64, 32, 64, 64), (16000, 200, 64, 32, 64, 64),
    (15999, 64, 320, 160, 160, 176), (16000, 64, 320, 160, 160, 176), (16001, 128, 512, 256, 256, 240),
    (16016, 64, 250, 30, 193, 192), (70000, 1024, 32, 16, 16, 16), (70000, 1032, 32, 16, 16, 65),
    (16005, 8, 4, 3, 1, 1), (16005, 136, 250, 30, 31, 33), (16384, 64, 32, 16, 16, 16), (32768, 192, 96, 48, 48, 48),
    (16005, 128, 320, 100, 130, 200), (16005, 72, 257, 64, 2, 129), (40000, 64, 256, 128, 128, 128),
])
def test_tables_match_their_definition(V, d, ds, dh, dt, rank):
    g = torch.Generator().manual_seed(V + d)
    dims = dict(d_state=ds, d_hproj=dh, d_tproj=dt, d_pos=3, d_feat=5, rank=rank, max_L=4)
    psi = {n: (torch.randn(s, generator=g) * 0.1).to(torch.bfloat16) for n, s in synth.psi_shapes(dims, d).items()}
    W, E = (torch.randn(V, d, generator=g).to(torch.bfloat16) for _ in range(2))
    corr = brisk.Corrector({n: t.to(DEV) for n, t in psi.items()}, 0.1, 0.2)
    tab = corr.prepare(W.to(DEV), E.to(DEV)).cpu()
    p = {n: t.double() for n, t in psi.items()}
    e = E.double() @ p["P_e"].T
    want = [(W.double() @ p["W_c"].T) @ p["W_s"], e @ p["W_z"][:, dh:dh + dt].T, e @ p["W_h"][:, dh:dh + dt].T]
    assert torch.all(tab[:, :, ds:] == 0)
    for k in range(3):
        # two chained 32-bit sums: a few 2^-24 of the largest value
        err = (tab[k, :, :ds].double() - want[k]).abs().max() / want[k].abs().max()
        assert err < 2e-6, (k, float(err))


@pytest.mark.parametrize("V", [600, 16400])
def test_table_padding_is_zero_beside_infinite_inputs(V):
    """Weights and embeddings with infinities stay in their own tokens and
    outputs; the padding past d_state stays zero."""
    d, ds = 72, 40
    g = torch.Generator().manual_seed(3)
    dims = dict(d_state=ds, d_hproj=8, d_tproj=24, d_pos=3, d_feat=5, rank=24, max_L=4)
    psi = {n: (torch.randn(s, generator=g) * 0.1).to(torch.bfloat16) for n, s in synth.psi_shapes(dims, d).items()}
    W, E = (torch.randn(V, d, generator=g).to(torch.bfloat16) for _ in range(2))
    ref = brisk.Corrector({n: t.to(DEV) for n, t in psi.items()}, 0.1, 0.2).prepare(W.to(DEV), E.to(DEV)).cpu()
    E[7, 0] = W[300, 0] = float("inf")
    psi["W_c"][23, 0] = float("inf")     # the row after the last but one: its first element follows row 22's end
    tab = brisk.Corrector({n: t.to(DEV) for n, t in psi.items()}, 0.1, 0.2).prepare(W.to(DEV), E.to(DEV)).cpu()
    assert torch.all(tab[:, :, ds:] == 0)
    others = torch.arange(V) != 7
    assert torch.equal(tab[1:, others], ref[1:, others]) and not torch.isfinite(tab[1:, 7, :ds]).any()
    assert not torch.isfinite(tab[0, :, :ds]).any()      # every token's last rank component is infinite
