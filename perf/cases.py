"""Performance cases: the calls a program makes on this framework, over the
sizes it makes them at.

A case is a dict of plain values; `prepare` makes its inputs on the GPU from a
seed, `run` is one pass through the public entry points, `exact` the same
results in FP64 with plain torch. Haplotypes are mosaics of a few founders
(the recipe of lsinputs, drawn on the device), which gives the columns the
block-structured similarity real samples have.

Kinds of calls:
  point      both tables moved to one variant and combined there (posteriors
             and half distances of one locus)
  decode     backward and forward sweep over all variants with posteriors and
             half distances at several targets
  distances  full N x N distance matrices at several targets
  fit        one optimisation step: the PAC log-likelihood and its gradient
             with respect to every rho_l and mu, through autograd
  mapfit     the same with respect to the recombination map's parameters and
             a mutation probability per variant
  linkage    half distances symmetrised and clustered (average linkage)
"""

from __future__ import annotations

import math

import torch

import paper_2212_11403_amd as ls

EPS = 2.0 ** -52
HAPLOTYPES = dict(K=100, switch=1e-3, flip=1e-4, mu=1e-4, d=1e-3)


def listed():
    return [
        # one locus of a small panel: latency, launches and short columns
        dict(name="point_small", kind="point", N=300, L=200, t=90, prec="fp32", **HAPLOTYPES),
        # the small FP64 workload of the tests and the paper's example data size
        dict(name="decode_small_fp64", kind="decode", N=200, L=2000, T=10, prec="fp64",
             R=0, vec=False, prior=False, K=20, switch=1e-2, flip=1e-3, mu=1e-3, d=1e-2),
        # a few query haplotypes against a large panel: one group per compute
        # unit, a serial chain of variants
        dict(name="decode_few_recipients", kind="decode", N=10_000, L=2000, T=5, prec="fp32",
             R=8, vec=False, prior=False, **HAPLOTYPES),
        # the benchmark's workload (N = 10,000, all recipients), fewer variants
        dict(name="distances_10k", kind="distances", N=10_000, L=1024, T=4, window=0,
             prec="fp32", **HAPLOTYPES),
        # a panel whose size fits no vector or word, in recipient windows
        dict(name="distances_ragged", kind="distances", N=4_999, L=1500, T=7, window=2_000,
             prec="fp32", **HAPLOTYPES),
        # double precision at the benchmark's panel size
        dict(name="decode_10k_fp64", kind="decode", N=10_000, L=1024, T=2, prec="fp64",
             R=2_500, vec=False, prior=False, **HAPLOTYPES),
        # half-stored tables at the precision study's panel size
        dict(name="decode_50k_f16", kind="decode", N=50_000, L=400, T=2, prec="f16",
             R=512, vec=False, prior=False, **HAPLOTYPES),
        # a recipient window of the largest panel
        dict(name="decode_100k_window", kind="decode", N=100_000, L=300, T=1, prec="fp32",
             R=1024, vec=False, prior=False, **HAPLOTYPES),
        # the model's options: a prior copying matrix and a mu per variant
        dict(name="decode_prior_mu_vector", kind="decode", N=3_001, L=600, T=3, prec="fp32",
             R=0, vec=True, prior=True, **HAPLOTYPES),
        # parameter estimation at the gradient workload's panel size
        dict(name="fit_fp32", kind="fit", N=2_000, L=5_000, prec="fp32", **HAPLOTYPES),
        # estimation of a recombination map and per-variant mutation in FP64
        dict(name="mapfit_fp64", kind="mapfit", N=500, L=2_000, prec="fp64", **HAPLOTYPES),
        # clustering of the distance matrices of several targets
        dict(name="linkage_3k", kind="linkage", N=3_000, T=6, prec="fp32", K=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["point", "decode", "decode", "distances", "fit", "mapfit", "linkage"])
    c = dict(kind=kind)
    if kind == "linkage":
        c.update(N=_log_int(rng, 64, 2_500), T=rng.randint(1, 6), prec=rng.choice(["fp32", "fp64"]),
                 K=rng.randint(10, 200))
        return c
    c.update(K=rng.randint(20, 200), switch=rng.choice([1e-2, 1e-3, 5e-4]),
             flip=rng.choice([1e-3, 1e-4]), mu=rng.choice([1e-3, 1e-4]),
             d=rng.choice([1e-2, 1e-3]))
    if kind == "point":
        c.update(N=_log_int(rng, 64, 3_000), L=rng.randint(100, 800),
                 prec=rng.choice(["fp32", "fp64", "f16"]))
        c.update(t=rng.randrange(20, c["L"] - 20))
    elif kind == "decode":
        prec = rng.choice(["fp32", "fp32", "fp64", "f16"])
        prior = rng.random() < 0.25
        N = _log_int(rng, 100, 8_000 if prior else (40_000 if prec == "fp64" else 100_000))
        R = 0 if N <= 3_000 else _log_int(rng, 4, 1.5e7 / N)
        L = min(2_500, int(4e10 / (N * (R or N))) + 50)
        c.update(N=N, L=rng.randint(min(200, L), L), T=rng.randint(1, 4), prec=prec, R=R,
                 vec=rng.random() < 0.25, prior=prior)
    elif kind == "distances":
        N = _log_int(rng, 150, 8_000)
        L = min(2_500, int(4e10 / (N * N)) + 50)
        c.update(N=N, L=rng.randint(min(200, L), L), T=rng.randint(1, 4),
                 window=rng.choice([0, 0, N // 2 + 1]), prec=rng.choice(["fp32", "fp64"]))
    elif kind == "fit":
        N = _log_int(rng, 64, 3_000)
        L = min(4_000, int(8e9 / (N * N)) + 50)
        c.update(N=N, L=rng.randint(min(200, L), L), prec=rng.choice(["fp32", "fp32", "fp64"]))
    else:
        c.update(N=_log_int(rng, 64, 800), L=_log_int(rng, 200, 2_000),
                 prec=rng.choice(["fp32", "fp64"]))
    return c


# ---- inputs -----------------------------------------------------------------

def _haplotypes(case, g):
    """0/1 alleles [L][N] (uint8): a mosaic of K founders with switches and
    flips; founder allele frequencies Beta(1/2, 1/2)."""
    N, L, K = case["N"], case["L"], case["K"]
    dev = "cuda"
    p = torch.sin(torch.rand(L, generator=g, device=dev) * (math.pi / 2)) ** 2
    F = (torch.rand((L, K), generator=g, device=dev) < p[:, None]).to(torch.uint8)
    h = torch.empty((L, N), dtype=torch.uint8, device=dev)
    rows = torch.arange(L, dtype=torch.int32, device=dev)[:, None]
    for j0 in range(0, N, 1 << 14):
        n = min(N, j0 + (1 << 14)) - j0
        sw = torch.rand((L, n), generator=g, device=dev) < case["switch"]
        sw[0] = True
        at = torch.cummax(torch.where(sw, rows, 0), dim=0).values
        fo = torch.randint(K, (L, n), generator=g, device=dev)
        f = torch.gather(F, 1, torch.gather(fo, 0, at.long()))
        flip = torch.rand((L, n), generator=g, device=dev) < case["flip"]
        h[:, j0:j0 + n] = f ^ flip.to(torch.uint8)
    return h


def _pack(h):
    """[L][stride] 32-bit words: haplotype j is bit j % 32 of word j / 32,
    rows padded to 32 bytes."""
    L, N = h.shape
    stride = ((N + 31) // 32 + 7) // 8 * 8
    out = torch.empty((L, stride), dtype=torch.int32, device=h.device)
    bit = torch.arange(32, device=h.device)
    for a in range(0, L, 256):
        b = min(L, a + 256)
        w = torch.zeros((b - a, stride * 32), dtype=torch.int64, device=h.device)
        w[:, :N] = h[a:b]
        v = (w.view(b - a, stride, 32) << bit).sum(-1)
        out[a:b] = torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32)
    return out


def _targets(case):
    L, T = case["L"], case["T"]
    return [((2 * k + 1) * L) // (2 * T) for k in range(T)]


def _inputs(case, seed):
    """Alleles and parameters of a case (everything but the linkage's)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    N, L = case["N"], case["L"]
    h = _haplotypes(case, g)
    x = dict(h=h)
    gaps = -torch.log1p(-torch.rand(L - 1, generator=g, device="cuda", dtype=torch.float64))
    x["rho"] = -torch.expm1(-case["d"] * gaps)
    x["cM"] = 100.0 * case["d"] * gaps
    if case.get("vec") or case["kind"] == "mapfit":
        x["mu"] = case["mu"] * torch.exp(0.5 * torch.randn(L, generator=g, device="cuda",
                                                           dtype=torch.float64))
    else:
        x["mu"] = case["mu"]
    x["prior"] = None
    if case.get("prior"):
        w = torch.rand((N, N), generator=g, device="cuda", dtype=torch.float64) ** 2
        w.fill_diagonal_(0.0)
        x["prior"] = w / w.sum(0, keepdim=True)
    R = case.get("R", 0)
    x["rec"] = torch.arange(N, dtype=torch.int32, device="cuda") if not R or R >= N else \
        torch.randperm(N, generator=g, device="cuda")[:R].sort().values.to(torch.int32)
    return x


def _half_distances(case, seed):
    """E [T][N][N] as a decode leaves it: donors on the recipient's founder
    share most of the posterior, the others the jump mass."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    N, T, K = case["N"], case["T"], case["K"]
    E = torch.empty((T, N, N), dtype=torch.float64, device="cuda")
    for k in range(T):
        f = torch.randint(K, (N,), generator=g, device="cuda")
        p = torch.rand((N, N), generator=g, device="cuda", dtype=torch.float64) ** 3
        p = torch.where(f[:, None] == f[None, :], p + 0.1, 1e-5 * p + 1e-12)
        p.fill_diagonal_(0.0)
        p = p / p.sum(1, keepdim=True)
        E[k] = -0.5 * torch.log(p.clamp_min(EPS))
        E[k].fill_diagonal_(0.0)
    return E.to(torch.float64 if case["prec"] == "fp64" else torch.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "linkage":
        E = _half_distances(case, seed)
        return dict(case=case, E=E, D=torch.empty_like(E))
    x = _inputs(case, seed)
    s = dict(case=case, rec=x["rec"])
    H = _pack(x["h"])
    if kind == "fit":
        # parameters as an optimiser holds them, in the sweep's precision
        dt = torch.float64 if case["prec"] == "fp64" else torch.float32
        s.update(H=H, rho=x["rho"].to(dt).requires_grad_(),
                 mu=torch.tensor(case["mu"], dtype=dt, device="cuda", requires_grad=True))
        return s
    if kind == "mapfit":
        dt = torch.float64 if case["prec"] == "fp64" else torch.float32
        s.update(H=H, cM=x["cM"], mu=x["mu"].to(dt).detach().requires_grad_(),
                 s=torch.tensor(0.9, dtype=dt, device="cuda", requires_grad=True),
                 gamma=torch.tensor(1.0625, dtype=dt, device="cuda", requires_grad=True))
        return s
    s["model"] = ls.Model(H, case["N"], x["rho"], x["mu"], prior=x["prior"])
    if kind == "point":
        s["fwd"] = ls.Table(s["model"], 0, case["prec"], x["rec"])
        s["bck"] = ls.Table(s["model"], 1, case["prec"], x["rec"])
        shape = (len(x["rec"]), case["N"])
        s["P"] = torch.empty(shape, dtype=ls.io_dtype(case["prec"]), device="cuda")
        s["E"] = torch.empty_like(s["P"])
    return s


# ---- one pass ---------------------------------------------------------------

def run(s):
    case = s["case"]
    kind, prec = case["kind"], case["prec"]
    if kind == "point":
        m, fwd, bck = s["model"], s["fwd"], s["bck"]
        fwd.reset(m, s["rec"])
        bck.reset(m, s["rec"])
        ls.forward(fwd, m, case["t"])
        ls.backward(bck, m, case["t"])
        ls.posterior_distance(fwd, bck, m, s["P"], s["E"])
        return dict(P=s["P"], E=s["E"], fwd=fwd.state, bck=bck.state)
    if kind == "decode":
        out = ls.decode(s["model"], _targets(case), prec, recipients=s["rec"], want=("P", "E"))
        # log-likelihoods kept in the type of the other results
        return dict(P=out["P"], E=out["E"], fwd=out["fwd"].state, bck=out["bck"].state,
                    loglik=out["fwd"].log_scale.to(out["P"].dtype))
    if kind == "distances":
        out = ls.distance_matrices(s["model"], _targets(case), prec, window=case["window"])
        return dict(D=out["D"], loglik=out["loglik"].to(out["D"].dtype))
    if kind == "fit":
        rho, mu = s["rho"], s["mu"]
        pac = ls.PACLoglik.apply(rho.double(), mu.double(), s["H"], case["N"], prec)
        g = torch.autograd.grad(pac, (rho, mu))
        return dict(pac=pac.detach().to(rho.dtype), rho=g[0], mu=g[1])
    if kind == "mapfit":
        rho = ls.RhoMap.apply(s["cM"], s["s"].double(), s["gamma"].double())
        pac = ls.PACLoglik.apply(rho, s["mu"].double(), s["H"], case["N"], prec)
        g = torch.autograd.grad(pac, (s["s"], s["gamma"], s["mu"]))
        return dict(pac=pac.detach().to(s["mu"].dtype), s=g[0], gamma=g[1], mu=g[2])
    D = ls.distance_symmetrise(s["E"], s["D"], prec)
    Z, order = ls.average_linkage(D)
    return dict(Z=Z, order=order)


def work(case):
    """Inputs read once, outputs written once; 4 flops per cell and sweep
    (multiply-add, emission, column sum), 4 more per cell for the gradient's
    two products. Linkage: the merged rows' updates."""
    N, kind = case["N"], case["kind"]
    e = 8 if case["prec"] == "fp64" else 4
    if kind == "linkage":
        T = case["T"]
        return dict(bytes=T * (e * N * N + 36 * N), flops=2.5 * T * N * N)
    L = case["L"]
    R = case.get("R", 0) or N
    rows = L * N / 8
    if kind == "point":
        st = 2 if case["prec"] == "f16" else e
        return dict(bytes=rows + 2 * R * N * (e + st), flops=4.0 * R * N * L)
    if kind == "decode":
        st = 2 if case["prec"] == "f16" else e
        b = rows + 2 * R * N * (case["T"] * e + st) + (8.0 * R * N if case["prior"] else 0)
        return dict(bytes=b, flops=8.0 * R * N * L)
    if kind == "distances":
        return dict(bytes=rows + case["T"] * N * N * e, flops=8.0 * N * N * L)
    return dict(bytes=rows + 32.0 * L, flops=12.0 * N * N * L)


# ---- the same results in 64 bits ----------------------------------------------

class _Exact:
    """The scaled recursions for a set of recipients, FP64, step by step."""

    def __init__(self, x, rec, rho, mu):
        self.h = x["h"].bool()
        self.N, self.L = self.h.shape[1], self.h.shape[0]
        self.rec = rec.long()
        self.rho = rho.double().tolist()
        if not (torch.is_tensor(mu) and mu.dim()):
            mu = torch.full((self.L,), float(mu), dtype=torch.float64)
        self.mu_l = mu.detach().double().cuda()
        self.match_l = (1.0 - 2.0 * self.mu_l) + self.mu_l
        self.mu = self.mu_l.tolist()
        r = torch.arange(len(self.rec), device="cuda")
        self.self_at = (r, self.rec)
        if x["prior"] is not None:
            self.pi = x["prior"].t()[self.rec].contiguous()
        else:
            self.pi = torch.full((len(self.rec), self.N), 1.0 / (self.N - 1),
                                 dtype=torch.float64, device="cuda")
        self.pi[self.self_at] = 0.0

    def mismatch(self, l):
        return self.h[l][None, :] ^ self.h[l][self.rec][:, None]

    def theta(self, l):
        return torch.where(self.mismatch(l), self.mu_l[l], self.match_l[l])

    def first(self):
        a = self.theta(0) * self.pi
        return a, a.sum(1, keepdim=True)

    def forward(self, a, S, l):
        """alpha^l and its sum from alpha^{l-1} and its sum."""
        r = self.rho[l - 1]
        a = torch.addcmul(r * self.pi, a, (1.0 - r) / S).mul_(self.theta(l))
        return a, a.sum(1, keepdim=True)

    def last(self):
        b = torch.ones_like(self.pi)
        b[self.self_at] = 0.0
        return b

    def backward(self, y, W, l):
        """beta^l from y = theta^{l+1} beta^{l+1} and W = sum Pi y."""
        b = (y * ((1.0 - self.rho[l]) / W)).add_(self.rho[l])
        b[self.self_at] = 0.0
        return b

    def decode(self, targets, t_fwd, t_bck):
        """(alpha, beta) at the targets, the tables at t_fwd and t_bck and
        log P as far as the forward table went."""
        A, B = {}, {}
        a, S = self.first()
        ll = torch.log(S)
        for l in range(t_fwd + 1):
            if l:
                a, S = self.forward(a, S, l)
                ll += torch.log(S)
            if l in targets:
                A[l] = a
        b = self.last()
        for l in range(self.L - 1, t_bck - 1, -1):
            if l < self.L - 1:
                y = self.theta(l + 1).mul_(b)
                b = self.backward(y, (self.pi * y).sum(1, keepdim=True), l)
            if l in targets:
                B[l] = b
        return A, B, a, b, ll[:, 0]

    def posterior(self, A, B):
        q = A * B
        P = q / q.sum(1, keepdim=True)
        E = -0.5 * torch.log(P.clamp_min(EPS))
        E[self.self_at] = 0.0
        return P, E

    def gradient(self):
        """log P [R], d PAC / d rho [L-1] and d PAC / d mu^l [L]."""
        L, R = self.L, len(self.rec)
        A = torch.empty((L, R, self.N), dtype=torch.float64, device="cuda")
        a, S = self.first()
        ll = torch.log(S)
        A[0] = a
        for l in range(1, L):
            a, S = self.forward(a, S, l)
            ll += torch.log(S)
            A[l] = a
        grho, gmu = [], []
        b = self.last()
        for l in range(L - 1, -1, -1):
            if l < L - 1:
                y = self.theta(l + 1).mul_(b)
                W = (self.pi * y).sum(1, keepdim=True)
                d = (A[l] * y).sum(1)
                n = A[l].sum(1) * W[:, 0]
                r = self.rho[l]
                grho.append(((n - d) / ((1.0 - r) * d + r * n)).sum())
                b = self.backward(y, W, l)
            q = A[l] * b
            M = (q * self.mismatch(l)).sum(1) / q.sum(1)
            gmu.append((M / self.mu[l] - (1.0 - M) / (1.0 - self.mu[l])).sum())
        return ll[:, 0], torch.stack(grho[::-1]), torch.stack(gmu[::-1])


def _exact_gradient(case, x, rho, mu):
    N, L = case["N"], case["L"]
    step = max(1, min(N, int(6e10 / (8.0 * N * L))))
    pac, grho, gmu = 0.0, 0.0, 0.0
    for r0 in range(0, N, step):
        rec = torch.arange(r0, min(N, r0 + step), device="cuda")
        ll, gr, gm = _Exact(x, rec, rho, mu).gradient()
        pac, grho, gmu = pac + ll.sum(), grho + gr, gmu + gm
        del ll, gr, gm
    return pac, grho, gmu


def exact(case, seed):
    kind = case["kind"]
    if kind == "linkage":
        return None  # a chain of decisions on the given type's values
    x = _inputs(case, seed)
    if kind in ("fit", "mapfit"):
        dt = torch.float64 if case["prec"] == "fp64" else torch.float32
        if kind == "fit":
            pac, gr, gm = _exact_gradient(case, x, x["rho"].to(dt),
                                          torch.tensor(case["mu"], dtype=dt))
            return dict(pac=pac, rho=gr, mu=gm.sum())
        s, gamma = (torch.tensor(v, dtype=dt).double().item() for v in (0.9, 1.0625))
        m = x["cM"] / 100.0
        mg = m ** gamma
        pac, gr, gm = _exact_gradient(case, x, -torch.expm1(-s * mg), x["mu"].to(dt))
        e = gr * mg * torch.exp(-s * mg)
        return dict(pac=pac, s=e.sum(),
                    gamma=torch.where(m > 0, s * e * torch.log(m), 0.0).sum(), mu=gm)
    ex = _Exact(x, x["rec"], x["rho"], x["mu"])
    f16 = case["prec"] == "f16"  # half tables hold scaled vectors
    if kind == "point":
        t = case["t"]
        A, B, a, b, _ = ex.decode([t], t, t)
        P, E = ex.posterior(A[t], B[t])
        return dict(P=P, E=E, fwd=None if f16 else a, bck=None if f16 else b)
    targets = _targets(case)
    A, B, a, b, ll = ex.decode(targets, case["L"] - 1, 0)
    P, E = zip(*(ex.posterior(A[t], B[t]) for t in targets))
    if kind == "distances":
        D = torch.stack([e + e.t() for e in E])
        return dict(D=D, loglik=ll)
    return dict(P=torch.stack(P), E=torch.stack(E), fwd=None if f16 else a,
                bck=None if f16 else b, loglik=ll)
