"""Timed cases: the calls that a user of this package makes, at the sizes its
tests and benchmark configurations name.

A case is one call (or the short chain a user makes of it) on one alignment or
a small batch: objective and gradient, the autograd path, reweighting, the
fits, the mean-field start and the scores.  Alignments are drawn on the GPU
from the seed: column profiles with planted correlated pairs and gaps, most
rows diverse and a share of them close copies, so that pairwise identities lie
on both sides of the reweighting threshold.
"""
from __future__ import annotations

import math

import torch

import paper_1401_4832_amd as plm

Q = 21
GAP = 20
# 16 alignments with N in [60, 300] and B in [2000, 30000] are the ragged
# configuration; five of that range make a batch of ordinary families
RAGGED = "61x2003,97x5200,120x9000,151x4100,203x12007"


def listed():
    return [
        # the smallest configuration, all sites: latency and launches count
        dict(name="objgrad_n40_b500", kind="objgrad", N=40, B=500, path=0),
        # the differentiable objective inside a training loop, forward and backward
        dict(name="autograd_n150_b8000", kind="autograd", N=150, B=8000),
        # the largest configuration, one all-sites evaluation on the path its fit takes
        dict(name="objgrad_n500_b50000", kind="objgrad", N=500, B=50000, path=6),
        # sequence weights of an ordinary family and of the largest one
        dict(name="reweight_n120_b5000", kind="reweight", N=120, B=5000, theta=0.8),
        dict(name="reweight_n500_b50000", kind="reweight", N=500, B=50000, theta=0.8),
        # a converged fit of the smallest family with the default options
        dict(name="fit_n40_b500", kind="fit", N=40, B=500, path=0, max_iter=300),
        # the first twenty iterations of the largest fit, on the path the tuner picks
        dict(name="fit_n500_b50000_20it", kind="fit", N=500, B=50000, path=6, max_iter=20, refine=-1),
        # several families of different sizes fitted together
        dict(name="fit_batch_ragged", kind="batch", sizes=RAGGED, path=6, max_iter=300),
        # the symmetric variant, with its refinement on the precise path
        dict(name="symmetric_n120_b5000", kind="symmetric", N=120, B=5000, path=5, max_iter=300),
        # the mean-field start of a large family
        dict(name="mf_init_n300_b30000", kind="mf", N=300, B=30000),
        # pair scores: the default of the largest fit, and a variant with its frequencies
        dict(name="score_n500", kind="score", N=500, B=0, variant="default"),
        dict(name="score_burkoff_n200", kind="score", N=200, B=10000, variant="burkoff"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["objgrad", "objgrad", "autograd", "reweight", "reweight", "fit", "batch", "symmetric", "mf",
                       "score"])
    if kind == "objgrad":
        return dict(kind=kind, N=_log_int(rng, 20, 500), B=_log_int(rng, 200, 50000), path=rng.choice([0, 0, 4, 5, 6]))
    if kind == "autograd":
        return dict(kind=kind, N=_log_int(rng, 20, 300), B=_log_int(rng, 200, 20000))
    if kind == "reweight":
        return dict(kind=kind, N=_log_int(rng, 30, 500), B=_log_int(rng, 200, 50000), theta=rng.choice([0.7, 0.8, 0.9]))
    if kind == "fit":
        # the fixed-point path needs enough sequences for its rounding to stay below the tolerance
        path = rng.choice([0, 6])
        return dict(kind=kind, N=_log_int(rng, 20, 160), B=_log_int(rng, 3000 if path else 200, 8000), path=path,
                    max_iter=300)
    if kind == "batch":
        sizes = ",".join("%dx%d" % (rng.randint(60, 200), _log_int(rng, 2000, 10000)) for _ in range(rng.randint(2, 5)))
        return dict(kind=kind, sizes=sizes, path=6, max_iter=300)
    if kind == "symmetric":
        return dict(kind=kind, N=_log_int(rng, 20, 120), B=_log_int(rng, 1000, 5000), path=5, max_iter=300)
    if kind == "mf":
        return dict(kind=kind, N=_log_int(rng, 20, 300), B=_log_int(rng, 500, 30000))
    variant = rng.choice(["default", "burkoff", "min_lp"])
    return dict(kind=kind, N=_log_int(rng, 20, 500), B=_log_int(rng, 500, 10000) if variant == "burkoff" else 0,
                variant=variant)


# ---- inputs ---------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1009 + stream) % (1 << 31))
    return g


def _msa(seed, N, B):
    """uint8 [B, N]: rows are noisy copies of ancestors drawn from column profiles."""
    g = _gen(seed, 1)
    dev = "cuda"
    cum = torch.softmax(1.2 * torch.randn(N, Q, generator=g, device=dev), 1).cumsum(1)

    def profile(rows):
        u = torch.rand(rows, N, generator=g, device=dev)
        out = torch.zeros(rows, N, dtype=torch.uint8, device=dev)
        for k in range(Q - 1):
            out += u > cum[:, k]
        return out

    n_anc = max(2, B // 25)
    anc = profile(n_anc)
    pick = torch.randint(n_anc, (B,), generator=g, device=dev)
    # families share their gaps
    anc[torch.rand(n_anc, N, generator=g, device=dev) < 0.1] = GAP
    # a fifth of the rows are close copies, the others diverse
    rate = 0.35 + 0.6 * torch.rand(B, 1, generator=g, device=dev)
    close = torch.rand(B, 1, generator=g, device=dev) < 0.2
    rate = torch.where(close, 0.15 * torch.rand(B, 1, generator=g, device=dev), rate)
    msa = torch.where(torch.rand(B, N, generator=g, device=dev) < rate, profile(B), anc[pick])
    # N/2 planted pairs: the second column follows the first through a permutation
    order = torch.randperm(N, generator=g, device=dev).tolist()
    for a, b in zip(order[0::2], order[1::2]):
        perm = torch.randperm(Q, generator=g, device=dev).to(torch.uint8)
        tie = torch.rand(B, generator=g, device=dev) < torch.where(close[:, 0], 0.02, 0.35)
        msa[:, b] = torch.where(tie, perm[msa[:, a].long()], msa[:, b])
    msa[torch.rand(B, N, generator=g, device=dev) < 0.02] = GAP
    return msa.contiguous()


def _params(seed, N, sd_h, sd_J):
    g = _gen(seed, 2)
    h = sd_h * torch.randn(N, Q, generator=g, device="cuda")
    J = sd_J * torch.randn(N, N, Q, Q, generator=g, device="cuda")
    i = torch.arange(N, device="cuda")
    J[i, i] = 0.0
    return h, J


def _sd_J(N):
    return 0.05 if N > 200 else 0.1


def _weighted(seed, N, B, uniform=False):
    msa = _msa(seed, N, B)
    _, w, beff = plm.reweight(msa, theta=0.8, uniform=uniform)
    return msa, w, beff


def _sizes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["sizes"].split(",")]


def _options(case):
    kw = dict(path=case["path"], max_iter=case["max_iter"], tol=1e-6)
    if case["kind"] == "symmetric":
        # the first fit stops above its rounding floor, the precise path finishes
        N, B = case["N"], case["B"]
        params = N * Q + N * (N - 1) // 2 * Q * Q
        kw.update(tol=max(1e-6, 8 * 2.0 ** -23 * math.sqrt(params * B / 3.0) / B), refine_tol=1e-6)
    elif case["path"] == 6:
        kw.update(refine_tol=7e-7, refine=case.get("refine", 0))
    return plm.FitOptions(**kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "reweight":
        return dict(kind=kind, msa=_msa(seed, case["N"], case["B"]), theta=case["theta"])
    if kind in ("objgrad", "autograd"):
        N, B = case["N"], case["B"]
        msa, w, beff = _weighted(seed, N, B)
        h, J = _params(seed, N, 0.3, _sd_J(N))
        if kind == "autograd":
            h.requires_grad_(True)
            J.requires_grad_(True)
        return dict(kind=kind, msa=msa, w=w, beff=beff, h=h, J=J, path=case.get("path", 0))
    if kind == "fit":
        # the smallest alignments are fitted with uniform weights, as their configuration asks
        msa, w, beff = _weighted(seed, case["N"], case["B"], uniform=case["B"] <= 1000)
        return dict(kind=kind, msa=msa, w=w, beff=beff, opts=_options(case))
    if kind == "symmetric":
        msa, w, beff = _weighted(seed, case["N"], case["B"])
        return dict(kind=kind, msa=msa, w=w, beff=beff, opts=_options(case))
    if kind == "batch":
        items = [_weighted(seed * 31 + k, N, B) for k, (N, B) in enumerate(_sizes(case))]
        return dict(kind=kind, items=items, opts=_options(case))
    if kind == "mf":
        msa, w, beff = _weighted(seed, case["N"], case["B"])
        return dict(kind=kind, msa=msa, w=w, beff=beff)
    h, J = _params(seed, case["N"], 0.3, 0.1)
    state = dict(kind=kind, J=J, variant=case["variant"])
    if case["variant"] == "burkoff":
        state["msa"], state["w"], state["beff"] = _weighted(seed, case["N"], case["B"])
    return state


# ---- one pass -------------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "objgrad":
        return plm.objgrad(state["msa"], state["w"], state["beff"], state["h"], state["J"], path=state["path"])
    if kind == "autograd":
        h, J = state["h"], state["J"]
        h.grad = J.grad = None
        f = plm.plm_objective(h, J, state["msa"], state["w"], state["beff"])
        f.sum().backward()
        return f.detach(), h.grad, J.grad
    if kind == "reweight":
        return plm.reweight(state["msa"], theta=state["theta"])
    if kind == "fit":
        r = plm.fit(state["msa"], state["w"], state["beff"], state["opts"])
        return r.h, r.J
    if kind == "symmetric":
        r = plm.fit_symmetric(state["msa"], state["w"], state["beff"], state["opts"])
        return r.h, r.J
    if kind == "batch":
        return [(r.h, r.J) for r in plm.fit_batch(state["items"], state["opts"])]
    if kind == "mf":
        return plm.mf_init(state["msa"], state["w"], state["beff"])
    if state["variant"] == "burkoff":
        freq = plm.frequencies(state["msa"], state["w"], state["beff"])
        return (freq,) + plm.score(state["J"], norm="burkoff", freq=freq)
    if state["variant"] == "min_lp":
        return plm.score(state["J"], combine="min", norm="lp", p=1.5, exclude_gap=True, correction="asc")
    return plm.score(state["J"])


# ---- what a pass cannot do without ------------------------------------------------

def _eval_work(N, B):
    """One all-sites objective and gradient: an add per (site, row, column, state) in each direction."""
    return dict(bytes=B * N + 8 * B + 8 * (N * Q + N * N * Q * Q) + 8 * N, flops=2.0 * B * N * N * Q)


def _fit_work(N, B, evals):
    one = _eval_work(N, B)
    return dict(bytes=one["bytes"], flops=evals * one["flops"])


def work(case):
    kind = case["kind"]
    if kind == "reweight":
        N, B = case["N"], case["B"]
        return dict(bytes=B * N + 20 * B + 8, flops=0.5 * B * B * N)
    if kind in ("objgrad", "autograd"):
        return _eval_work(case["N"], case["B"])
    if kind == "fit":
        return _fit_work(case["N"], case["B"], min(case["max_iter"], 100))
    if kind == "symmetric":
        return _fit_work(case["N"], case["B"], min(case["max_iter"], 100))
    if kind == "batch":
        parts = [_fit_work(N, B, min(case["max_iter"], 100)) for N, B in _sizes(case)]
        return dict(bytes=sum(p["bytes"] for p in parts), flops=sum(p["flops"] for p in parts))
    if kind == "mf":
        N, B = case["N"], case["B"]
        n = N * (Q - 1)
        # pair histograms of the weights, and a symmetric inverse
        return dict(bytes=B * N + 8 * B + 4 * N * N * Q * Q, flops=0.5 * B * N * N + float(n) ** 3)
    N, B = case["N"], case["B"]
    return dict(bytes=4 * N * N * Q * Q + 16 * N * N + B * (N + 8), flops=8.0 * N * N * Q * Q)


# ---- 64-bit values of the same outputs ------------------------------------------------

def _weights64(msa, theta=0.8):
    B, N = msa.shape
    hot = torch.nn.functional.one_hot(msa.long(), Q).reshape(B, N * Q).to(torch.float16)
    need = next((t for t in range(N + 1) if t / N >= theta), N + 1)
    m = torch.zeros(B, dtype=torch.int32, device=msa.device)
    for a in range(0, B, 4096):
        # counts up to N are whole numbers that FP16 holds
        m[a:a + 4096] = ((hot[a:a + 4096] @ hot.t().contiguous()) >= need - 0.5).sum(1).to(torch.int32)
    w = 1.0 / m.double()
    return m, w, w.cumsum(0)[-1:].clone()


def _objgrad64(msa, w, beff, h, J, lam_h=0.01, lam_J=0.01):
    B, N = msa.shape
    hot = torch.nn.functional.one_hot(msa.long(), Q).reshape(B, N * Q).double()
    h, J = h.detach().double(), J.detach().double()
    W = J.permute(1, 2, 0, 3).reshape(N * Q, N * Q).contiguous()  # rows (i, k), columns (r, s)
    E = (hot @ W + h.reshape(1, -1)).reshape(B, N, Q)
    at = msa.long().unsqueeze(2)
    lse = torch.logsumexp(E, 2)
    data = (w[:, None] * (lse - E.gather(2, at).squeeze(2))).sum(0)
    P = torch.softmax(E, 2)
    del E
    P.scatter_add_(2, at, torch.full_like(at, -1, dtype=torch.float64))
    R = (P * w[:, None, None]).reshape(B, N * Q)
    del P
    gW = hot.t().contiguous() @ R
    gJ = gW.reshape(N, Q, N, Q).permute(2, 0, 1, 3).contiguous()
    i = torch.arange(N, device=msa.device)
    gJ[i, i] = 0.0
    gJ += beff * 2 * (0.5 * lam_J) * J
    gh = R.sum(0).reshape(N, Q) + beff * 2 * lam_h * h
    f = data + beff * (lam_h * h.square().sum(1) + 0.5 * lam_J * J.square().sum((1, 2, 3)))
    return f, gh, gJ


def _mf64(msa, w, beff, pc=0.5):
    B, N = msa.shape
    hot = torch.nn.functional.one_hot(msa.long(), Q).reshape(B, N * Q).double()
    F = (hot.t().contiguous() @ (hot * w[:, None])) / beff
    del hot
    fi = (1 - pc) * F.diagonal().reshape(N, Q) + pc / Q
    F = (1 - pc) * F + pc / (Q * Q)
    F = F.reshape(N, Q, N, Q)
    i = torch.arange(N, device=msa.device)
    F[i, :, i, :] = torch.diag_embed(fi)
    r = Q - 1
    fr = fi[:, :r].reshape(-1)
    C = F[:, :r, :, :r].reshape(N * r, N * r) - fr[:, None] * fr[None, :]
    X = torch.linalg.inv(C.cpu()).to(C.device).reshape(N, r, N, r)
    Jr = -X.permute(0, 2, 3, 1)  # [a][i][k][s]
    Jr = Jr.clone()
    Jr[i, i] = 0.0
    J = torch.zeros(N, N, Q, Q, dtype=torch.float64, device=msa.device)
    J[:, :, :r, :r] = Jr
    h = torch.zeros(N, Q, dtype=torch.float64, device=msa.device)
    h[:, :r] = torch.log(fi[:, :r] / fi[:, r:]) - (Jr * fi[None, :, :r, None]).sum((1, 2))
    return h, J


def _ising64(J):
    """Both estimates of every pair in the Ising gauge, indexed (state of i, state of j)."""
    A = J.double().permute(0, 1, 3, 2)

    def gauge(x):
        return x - x.mean(2, keepdim=True) - x.mean(3, keepdim=True) + x.mean((2, 3), keepdim=True)

    return gauge(A), gauge(A.permute(1, 0, 3, 2))


def _score64(J, variant, freq=None):
    N = J.shape[0]
    A, B = _ising64(J)
    if variant == "min_lp":
        X = torch.minimum(A, B)[:, :, :Q - 1, :Q - 1]
        raw = X.abs().pow(1.5).sum((2, 3)).pow(1 / 1.5)
    elif variant == "burkoff":
        X = 0.5 * (A + B)
        T = torch.log(freq)[:, None, :, None] + torch.log(freq)[None, :, None, :] + X
        P = torch.softmax(T.reshape(N, N, -1), 2)
        raw = (P * X.reshape(N, N, -1)).sum(2) - torch.logsumexp(T.reshape(N, N, -1), 2)
    else:
        raw = (0.5 * (A + B)).square().sum((2, 3)).sqrt()
    up = torch.triu(raw, 1)
    raw = up + up.t()
    rows, total = raw.mean(1), raw.mean()
    if variant == "min_lp":
        cor = raw - rows[:, None] - rows[None, :] + total
    else:
        cor = raw - rows[:, None] * rows[None, :] / total
    cor.fill_diagonal_(0.0)
    return raw, cor


def exact(case, seed):
    kind = case["kind"]
    if kind in ("fit", "batch", "symmetric"):
        # a fit ends where its tolerance or iteration cap stops it: no closed value
        return None
    if kind == "reweight":
        return _weights64(_msa(seed, case["N"], case["B"]), case["theta"])
    if kind in ("objgrad", "autograd"):
        msa = _msa(seed, case["N"], case["B"])
        _, w, beff = _weights64(msa)
        return _objgrad64(msa, w, beff, *_params(seed, case["N"], 0.3, _sd_J(case["N"])))
    if kind == "mf":
        msa = _msa(seed, case["N"], case["B"])
        _, w, beff = _weights64(msa)
        return _mf64(msa, w, beff)
    _, J = _params(seed, case["N"], 0.3, 0.1)
    if case["variant"] != "burkoff":
        return _score64(J, case["variant"])
    msa = _msa(seed, case["N"], case["B"])
    _, w, beff = _weights64(msa)
    hot = torch.nn.functional.one_hot(msa.long(), Q).double()
    freq = (hot * w[:, None, None]).sum(0) / beff
    return (freq,) + _score64(J, "burkoff", freq)
