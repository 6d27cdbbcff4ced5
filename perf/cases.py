"""Workloads for timing the decoding hot path through its public entry points.

Every case is one call, or one short chain of calls, that a decoding server or
a training run of the corrector makes in earnest.  The vocabulary and width
pairs (4096, 126464) and (3584, 152064) are the full-size ones of ``synth`` and
``bench.py``; the other sizes are generic.  A case is a dict:

  op        which calls (one of ``OPS``)
  B, L      blocks and positions of a block; rows = B * L
  d, V, K   hidden width, vocabulary, candidates of a position
  r         corrector state width (0 where no corrector takes part)

``prepare`` draws the inputs on the GPU, ``run`` makes one pass, ``exact``
gives the floating outputs of that pass in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2609_33390_amd as brisk

DEV = "cuda"
OPS = ("step", "propose", "rerank", "rerank_direct", "tables", "selfverify", "spec", "loss", "profile")
ACCEPT = 0.85          # chance that a position's proposal and verifier agree
FLAT = 0.25            # share of rows without a clear winner among the tokens


def listed():
    return [
        # one request decoding alone: the whole step, bound by the read of the LM head and by launches
        dict(name="step-b1-l32", op="step", B=1, L=32, d=4096, V=126464, K=8, r=256),
        # batched serving: the whole step, bound by the matrix cores
        dict(name="step-b64-l32", op="step", B=64, L=32, d=4096, V=126464, K=8, r=256),
        # a few requests at a time, between the latency and the throughput regime
        dict(name="propose-b3-l32", op="propose", B=3, L=32, d=4096, V=126464, K=8, r=0),
        # the wide vocabulary with 16 candidates
        dict(name="propose-b16-l32-k16", op="propose", B=16, L=32, d=3584, V=152064, K=16, r=0),
        # the largest batch: the benchmark's headline shape
        dict(name="propose-b256-l16", op="propose", B=256, L=16, d=4096, V=126464, K=8, r=0),
        # the corrector with its per-token tables, 16 candidates, as serving calls it
        dict(name="rerank-b16-l32-k16", op="rerank", B=16, L=32, d=3584, V=152064, K=16, r=256),
        # the corrector without tables, with its scores: a training run, whose
        # weights change from call to call; the paper's 128-wide state
        dict(name="rerank-direct-b64-l16-r128", op="rerank_direct", B=64, L=16, d=4096, V=126464, K=8, r=128),
        # the per-token tables of a newly loaded or newly trained corrector
        dict(name="tables-r256", op="tables", B=1, L=32, d=4096, V=126464, K=8, r=256),
        # self-verifying decoding (proposal and verifier rows in one pass, then the
        # commit), with a ragged batch, block length, vocabulary and list length
        dict(name="selfverify-b13-l21", op="selfverify", B=13, L=21, d=2560, V=100277, K=10, r=0),
        # stochastic verification of a sampled batch
        dict(name="spec-b64-l16", op="spec", B=64, L=16, d=4096, V=126464, K=8, r=0),
        # the corrector's training loss on a large batch of verified blocks
        dict(name="loss-b256-l16", op="loss", B=256, L=16, d=4096, V=126464, K=8, r=0),
        # acceptance statistics over a long run's blocks: the smallest call
        dict(name="profile-n1m-m32", op="profile", B=1 << 20, L=32, d=0, V=0, K=0, r=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(OPS)
    if op == "profile":
        return dict(op=op, B=_log_int(rng, 1 << 10, 1 << 20), L=_log_int(rng, 4, 256), d=0, V=0, K=0, r=0)
    if op == "tables":
        return dict(op=op, B=1, L=32, d=8 * rng.randint(128, 512), V=rng.randint(20000, 152064), K=8,
                    r=8 * rng.randint(8, 32))
    most = 4096 * 4096 * 126464 // (2 if op in ("selfverify", "spec") else 1)
    while True:
        L = rng.randint(4, 64)
        B = _log_int(rng, 1, 256)
        d = rng.choice((4096, 3584, 8 * rng.randint(96, 512)))
        V = rng.choice((126464, 152064, rng.randint(20000, 152064)))
        K = rng.choice((4, 8, 8, 16, rng.randint(4, 32)))
        r = rng.choice((128, 256, 8 * rng.randint(4, 32))) if op in ("step", "rerank", "rerank_direct") else 0
        if B * L * d * V <= most and B * L <= 4096:
            return dict(op=op, B=B, L=L, d=d, V=V, K=K, r=r)


# ------------------------------------------------------------------- inputs
def _gen(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (seed + 1) + OPS.index(case["op"]))
    return g


def _dims(r, L):
    """Corrector widths in the ratios of the paper's head."""
    return dict(ds=r, dh=r // 2, dt=r // 2, dp=r // 8, df=r // 8, rank=r // 2, max_L=L)


def _corrector(case, g):
    """Weights at the scale of a trained head: every map keeps its input's
    scale, and the residual is as large as the gaps between candidates."""
    m, d = _dims(case["r"], case["L"]), case["d"]
    d_in = m["dh"] + m["dt"] + m["dp"] + m["df"]
    shapes = {"A_h": (m["ds"], d), "A_e": (m["ds"], d), "P_h": (m["dh"], d), "P_e": (m["dt"], d),
              "pos_emb": (m["max_L"], m["dp"]), "P_phi": (m["df"], 5), "W_z": (m["ds"], d_in),
              "W_h": (m["ds"], d_in), "W_s": (m["rank"], m["ds"]), "W_c": (m["rank"], d), "w_g": (m["ds"] + 5,)}
    t = {}
    for n, s in shapes.items():
        std = 0.1 if n == "W_c" else s[-1] ** -0.5
        t[n] = (std * torch.randn(s, generator=g, device=DEV)).to(torch.bfloat16)
    return t, 0.5, 0.125


def _matrix(n, d, g, std):
    return torch.randn(n, d, generator=g, device=DEV).mul_(std).to(torch.bfloat16)


def _head(case, g, H):
    """An LM head in which most rows of H have a token that stands out by a few logits."""
    V, d = case["V"], case["d"]
    W = torch.randn(V, d, generator=g, device=DEV).mul_(0.02)
    rows = H.shape[0]
    target = torch.randperm(V, generator=g, device=DEV)[:rows]     # distinct: one row adds to a token
    Hf = H.float()
    boost = Hf * (0.12 * (4096 / d) ** 0.5 / Hf.norm(dim=1, keepdim=True))
    boost[torch.rand(rows, generator=g, device=DEV) < FLAT] = 0
    W.index_add_(0, target, boost)
    return W.to(torch.bfloat16), target


def _candidates(case, g):
    """K distinct ids of each row in random order, some rows from a short
    range so that neighbours share tokens, and logits that fall from the first."""
    rows, V, K = case["B"] * case["L"], case["V"], case["K"]
    wide = torch.where(torch.rand(rows, 1, generator=g, device=DEV) < 0.25, 2 * K, V - K + 1).double()
    ids = (torch.rand(rows, K, generator=g, device=DEV, dtype=torch.float64) * wide).long().sort(dim=1).values
    ids = ids + torch.arange(K, device=DEV)
    ids = ids.gather(1, torch.rand(rows, K, generator=g, device=DEV).argsort(dim=1))
    gaps = torch.empty(rows, K, device=DEV).exponential_(2.0, generator=g)
    return (8.0 - gaps.cumsum(dim=1)).contiguous(), ids.to(torch.int32).contiguous()


def _agree(case, g, token):
    """Verifier tokens that agree with ``token`` [rows] with the chance ACCEPT."""
    rows = token.numel()
    other = torch.randint(0, case["V"], (rows,), generator=g, device=DEV)
    keep = torch.rand(rows, generator=g, device=DEV) < ACCEPT
    return torch.where(keep, token.long(), other).to(torch.int32).view(case["B"], case["L"])


def _accept_lens(B, L, g):
    miss = torch.rand(B, L, generator=g, device=DEV) >= ACCEPT
    first = torch.where(miss, torch.arange(L, device=DEV), L).min(dim=1).values
    return first.to(torch.int32)


def _inputs(case, seed):
    op, g = case["op"], _gen(case, seed)
    s = {"case": case}
    if op == "profile":
        s["accept_len"] = _accept_lens(case["B"], case["L"], g)
        return s
    B, L, d, V = case["B"], case["L"], case["d"], case["V"]
    rows = B * L
    if case["r"]:
        s["psi"], s["alpha"], s["b_g"] = _corrector(case, g)
        s["E"] = _matrix(V, d, g, 0.02)
    if op == "tables":
        s["W"] = _matrix(V, d, g, 0.02)
        return s
    s["H"] = _matrix(rows, d, g, 1.0)
    if op == "selfverify":
        noise = 0.3 * torch.randn(rows, d, generator=g, device=DEV)
        s["H2"] = torch.cat([s["H"], (s["H"].float() + noise).to(torch.bfloat16)])
    s["W"], s["target"] = _head(case, g, s["H"])
    if op in ("step", "rerank", "rerank_direct"):
        s["h_c"] = _matrix(B, d, g, 1.0)
        s["x0"] = torch.randint(0, V, (B,), generator=g, device=DEV).to(torch.int32)
    if op == "step":
        s["verifier"] = _agree(case, g, s["target"])
    if op == "selfverify":
        # the block under verification: proposed by the pass before
        s["proposal"] = _agree(case, g, s["target"])
    if op in ("rerank", "rerank_direct", "spec", "loss"):
        s["cand_logit"], s["cand_id"] = _candidates(case, g)
    if op == "rerank":
        s["verifier"] = _agree(case, g, s["cand_id"][:, 0])
    if op == "spec":
        prob = torch.softmax(s["cand_logit"], dim=1)
        pick = torch.multinomial(prob, 1, generator=g)
        s["cand_prob"] = prob.contiguous()
        s["proposal"] = s["cand_id"].gather(1, pick).view(B, L).contiguous()
        s["u"] = torch.rand(rows, generator=g, device=DEV)
        s["seed"] = seed
    if op == "loss":
        s["refined"] = s["cand_logit"] + 0.5 * torch.randn(rows, case["K"], generator=g, device=DEV)
        s["accept_len"] = _accept_lens(B, L, g)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["r"]:
        s["corr"] = brisk.Corrector(s["psi"], s["alpha"], s["b_g"])
        if case["op"] in ("step", "rerank"):
            s["corr"].prepare(s["W"], s["E"])
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    op, B, L, K = case["op"], case["B"], case["L"], case["K"]
    if op == "profile":
        return brisk.accept_profile(s["accept_len"], L)
    if op == "tables":
        return s["corr"].prepare(s["W"], s["E"])
    if op == "propose":
        return brisk.propose_block(s["H"], s["W"], K)
    if op == "step":
        cl, ci = brisk.propose_block(s["H"], s["W"], K)
        out = brisk.rerank_verify(s["corr"], s["H"], s["h_c"], s["x0"], s["W"], s["E"], cl, ci, s["verifier"], B, L)
        return dict(out, cand_logit=cl, cand_id=ci)
    if op == "rerank":
        return brisk.rerank_verify(s["corr"], s["H"], s["h_c"], s["x0"], s["W"], s["E"], s["cand_logit"],
                                   s["cand_id"], s["verifier"], B, L, want_scores=True)
    if op == "rerank_direct":
        return brisk.rerank(s["corr"], s["H"], s["h_c"], s["x0"], s["W"], s["E"], s["cand_logit"], s["cand_id"],
                            B, L, want_scores=True)
    if op == "selfverify":
        cl, ci, tok = brisk.propose_verify(s["H2"], s["W"], B * L, K)
        acc, committed, n = brisk.verify_commit(s["proposal"], tok.view(B, L))
        return dict(cand_logit=cl, cand_id=ci, ver_token=tok, accept_len=acc, committed=committed, n_committed=n)
    if op == "spec":
        return brisk.spec_verify(s["H"], s["W"], s["proposal"], s["cand_id"], s["cand_prob"], s["u"], s["seed"])
    return brisk.corrector_loss(s["H"], s["W"], s["cand_id"], s["cand_logit"], s["refined"], s["accept_len"], B, L)


# ------------------------------------------------------ what a pass has to do
def _distinct(n, V):
    """Distinct tokens expected among n uniform draws."""
    return V * (1.0 - (1.0 - 1.0 / V) ** n)


def _corrector_work(case, tables):
    B, L, d, V, K, r = (case[k] for k in ("B", "L", "d", "V", "K", "r"))
    rows, m = B * L, _dims(case["r"], case["L"])
    ds, dh, dt, rank = m["ds"], m["dh"], m["dt"], m["rank"]
    d_in = dh + dt + m["dp"] + m["df"]
    maps = d * (2 * ds + dh + (0 if tables else dt + rank)) + 2 * ds * d_in + (0 if tables else rank * ds)
    by = 2 * maps + 2 * d * (rows + 2 * B) + rows * K * 8 + 4 * B
    # the previous token's LM-head row, and the candidates' residual directions
    by += 2 * d * _distinct(rows, V)
    fl = 2 * d * (2 * ds * B + dh * rows + rows) + rows * (4 * ds * d_in + 2 * ds * K)
    if tables:
        by += 4 * ds * (rows * K + 2 * rows)
    else:
        by += 2 * d * (_distinct(rows * K, V) + _distinct(rows, V))
        fl += 2 * d * rows * (rank * K + dt) + 2 * rank * ds * rows
    return by, fl


def work(case):
    op, B, L, d, V, K = (case[k] for k in ("op", "B", "L", "d", "V", "K"))
    rows = B * L
    if op == "profile":
        return dict(bytes=4.0 * B + 8 * (3 * L + 2), flops=0.0)
    if op == "tables":
        m = _dims(case["r"], case["L"])
        ds, dt, rank = m["ds"], m["dt"], m["rank"]
        return dict(bytes=4.0 * V * d + 2 * d * (dt + rank) + 12.0 * V * max(256, ds),
                    flops=2.0 * V * d * (dt + rank) + 2.0 * V * ds * (2 * dt + rank))
    if op == "loss":
        reached = sum(ACCEPT ** j for j in range(L)) * B
        return dict(bytes=2.0 * d * (_distinct(reached * K, V) + reached) + 12.0 * reached * K + 12.0 * rows,
                    flops=2.0 * reached * K * d)
    if op in ("rerank", "rerank_direct"):
        by, fl = _corrector_work(case, op == "rerank")
        return dict(bytes=by + 4.0 * rows * (2 + 2 * K) + 8.0 * B, flops=fl)
    n = 2 * rows if op == "selfverify" else rows
    by, fl = 2.0 * V * d + 2.0 * n * d + 8.0 * rows * K, 2.0 * n * d * V
    if op == "selfverify":
        by += 4.0 * (2 * rows + B * (L + 3))
    if op == "spec":
        by += 16.0 * rows + 8.0 * B
    if op == "step":
        cby, cfl = _corrector_work(case, True)
        by, fl = by + cby - 2 * d * rows - 8 * rows * K + 4.0 * (2 * rows + 2 * B), fl + cfl
        by -= 2 * d * _distinct(rows, V)     # LM-head rows: the pass has read them
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """About four times what the 32-bit sums show against 64 bits."""
    op = case["op"]
    if op == "profile":
        return {"rel": 1e-12, "max": 1e-11}
    if op == "spec":
        return {"rel": 0.0, "differ": 2e-3}
    if op == "loss":
        return {"rel": 4e-6, "max": 2e-4}      # KL: differences of nearly equal logs
    # whole numbers change where two logits are closer than their rounding
    return {"rel": 2e-6, "max": 1e-4, "differ": 2e-3}


# ------------------------------------------------------------ in 64 bits
def _topk64(H, W, K):
    H = H.double()
    best = None
    for v in range(0, W.shape[0], 8192):
        x = H @ W[v:v + 8192].double().T
        if best is not None:
            x = torch.cat([best, x], dim=1)
        best = x.topk(K, dim=1).values
    return best


def _rerank64(s):
    """The corrector position by position, on the candidates in ``s``."""
    case = s["case"]
    B, L, K = case["B"], case["L"], case["K"]
    p = {n: t.double() for n, t in s["psi"].items()}
    sig = torch.sigmoid
    H = s["H"].double().view(B, L, -1)
    ids, base = s["cand_id"].long().view(B, L, K), s["cand_logit"].double().view(B, L, K)
    prev = s["x0"].long()
    u = torch.tanh(s["h_c"].double() @ p["A_h"].T + s["E"][prev].double() @ p["A_e"].T)
    sig_a = 1.0 / (1.0 + math.exp(-s["alpha"]))
    refined, gamma, resid = [], [], []
    for i in range(L):
        m, c, b = H[:, i], ids[:, i], base[:, i]
        pl = (s["W"][prev].double() * m).sum(1)
        phi = torch.stack([b[:, 0] - b[:, 1], b[:, 0] - b[:, 3], (c[:, 0] == prev).double(),
                           (c[:, :4] == prev[:, None]).any(1).double(), b[:, 0] - pl], dim=1)
        x = torch.cat([m @ p["P_h"].T, s["E"][prev].double() @ p["P_e"].T, p["pos_emb"][i].expand(B, -1),
                       phi @ p["P_phi"].T], dim=1)
        z = sig(x @ p["W_z"].T)
        u = (1 - z) * u + z * (x @ p["W_h"].T)
        g = sig_a * sig(torch.cat([u, phi], dim=1) @ p["w_g"] + s["b_g"])
        e = (s["W"][c].double().view(B * K, -1) @ p["W_c"].T).view(B, K, -1)
        res = (e * (u @ p["W_s"].T)[:, None]).sum(-1)
        lt = b + g[:, None] * res
        prev = c.gather(1, lt.argmax(1, keepdim=True)).squeeze(1)
        refined.append(lt), gamma.append(g), resid.append(res)
    flat = lambda v: torch.stack(v, dim=1).reshape(B * L, *v[0].shape[1:])  # noqa: E731
    return dict(refined=flat(refined), gamma=flat(gamma), resid=flat(resid))


def _profile64(s):
    M = s["case"]["L"]
    n = torch.bincount(s["accept_len"].long(), minlength=M + 1).double()
    reached = n.flip(0).cumsum(0).flip(0)[:M]           # blocks whose prefix is at least i - 1 long
    a = 1 - n[:M] / reached.clamp(min=1)
    A = a.cumprod(0)
    S = torch.cat([A[:M - 1].flip(0).cumsum(0).flip(0), A.new_zeros(1)])
    num, den = 2 + S[0], 2 - A[M - 1]
    w_raw = (1 - a) * (A[M - 1] * num + den * S) / num ** 2
    return dict(a=a, w_raw=w_raw, w=M * w_raw / w_raw.sum(), tpf_fpt=torch.stack([num / den, den / num]))


def _loss64(s):
    case = s["case"]
    B, L, K = case["B"], case["L"], case["K"]
    lv = torch.empty(B * L, K, dtype=torch.float64, device=DEV)
    for i in range(0, B * L, 1024):
        lv[i:i + 1024] = (s["W"][s["cand_id"][i:i + 1024].long()].double() * s["H"][i:i + 1024, None].double()).sum(-1)
    lp, lq, lr = (torch.log_softmax(x.double(), dim=1) for x in (lv, s["cand_logit"], s["refined"]))
    on = (torch.arange(L, device=DEV)[None] <= s["accept_len"][:, None]).reshape(-1).double()
    ce = -(lp.exp() * lr).sum(1) * on
    kl = (lq.exp() * (lq - lr)).sum(1) * on
    pos = ce + 0.01 * kl
    return dict(loss_pos=pos, ce=ce, kl=kl, loss_mean=torch.stack([pos.sum() / on.sum(), on.sum()]))


def exact(case, seed):
    s = _inputs(case, seed)
    op, K = case["op"], case["K"]
    if op == "profile":
        return _profile64(s)
    if op == "tables":
        p = {n: t.double() for n, t in s["psi"].items()}
        m = _dims(case["r"], case["L"])
        t = slice(m["dh"], m["dh"] + m["dt"])
        out = torch.zeros(3, case["V"], max(256, m["ds"]), dtype=torch.float64, device=DEV)
        for v in range(0, case["V"], 8192):
            e = s["E"][v:v + 8192].double() @ p["P_e"].T
            out[0, v:v + 8192, :m["ds"]] = (s["W"][v:v + 8192].double() @ p["W_c"].T) @ p["W_s"]
            out[1, v:v + 8192, :m["ds"]] = e @ p["W_z"][:, t].T
            out[2, v:v + 8192, :m["ds"]] = e @ p["W_h"][:, t].T
        return out
    if op == "propose":
        return _topk64(s["H"], s["W"], K), None
    if op in ("step", "selfverify"):
        return dict(cand_logit=_topk64(s["H"], s["W"], K))
    if op in ("rerank", "rerank_direct"):
        return _rerank64(s)
    if op == "loss":
        return _loss64(s)
    return None            # whole numbers only
