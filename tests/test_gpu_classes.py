"""Sweeps carried per haplotype class (long moves over haplotypes that repeat
within blocks of 16, 32 or 64 variants) against the FP64 oracle and against
the plain sweep, through the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from lsinputs import MosaicSpec, mosaic_haplotypes, rho_from_spacings, spacings

from _gpu import (F32_POST_ATOL, F64_ATOL_LOG, F64_ATOL_PROB, check_reduced, f64_rtol,
                  forced_shape, need_gpu, rel_close)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


def _np(t):
    return t.double().cpu().numpy()


def _case(N, L, K, seed, switch=2e-3, vec=False):
    H, _ = mosaic_haplotypes(MosaicSpec(N, L, K, switch, 1e-4, seed))
    rho = rho_from_spacings(spacings(L - 1, 1e-3, seed + 1))
    rng = np.random.default_rng(seed)
    rho[rng.random(L - 1) < 0.05] = 0.0     # variants at one map position
    rho[rng.random(L - 1) < 0.01] = 0.85    # and hot spots
    mu = 10.0 ** rng.uniform(-5, -1, L) if vec else 1e-3
    return H, rho, mu


def _model(ls, H, N, rho, mu):
    m = ls.Model(H, N, rho, mu)
    assert m.c.reserved != 0, "the case does not take the class sweep"
    return m


# N: the smallest with classes, the edges of donor words and id words, one
# more wave than 160 donor words, and a group of several waves; L: one block,
# one variant more, ragged last blocks, more than one launch of the sweep;
# targets at the first and last variants of blocks and of the sequence; many
# classes: groups of seven waves, and FP64 on four waves and on the plain sweep
@pytest.mark.parametrize("N,L,K,vec,switch", [
    (512, 65, 4, False, 2e-3), (513, 128, 4, True, 2e-3), (640, 200, 5, False, 2e-3),
    (703, 129, 6, False, 2e-3), (1000, 2200, 12, True, 2e-3), (2049, 333, 20, False, 2e-3),
    (4160, 97, 60, False, 2e-3), (10241, 150, 100, False, 2e-3), (21000, 80, 100, True, 2e-3),
    (9900, 100, 100, False, 1e-3), (50000, 70, 300, False, 1e-4), (5000, 100, 700, False, 2e-3)])
def test_class_sweep_vs_oracle(ls, N, L, K, vec, switch):
    H, rho, mu = _case(N, L, K, seed=N + L, switch=switch, vec=vec)
    rec = np.unique([0, 63, 64, N // 2, N - 65, N - 2, N - 1]).astype(np.int32)
    targets = sorted({0, 15, 16, 31, 32, 63, L - 2, L - 1})
    m = _model(ls, H, N, rho, mu)
    ref = oracle.run_pass(H, N, L, rho, mu, rec, targets, want=("A", "B", "P", "E"))
    for prec in ("fp64", "fp32"):
        r = ls.decode(m, targets, prec, recipients=rec, want=("P", "E"))
        if prec == "fp64":
            tol = f64_rtol(N)
            rel_close(_np(r["P"]), ref["P"], tol, F64_ATOL_PROB)
            rel_close(_np(r["bsnap"]), ref["B"], tol, F64_ATOL_PROB)
            rel_close(_np(r["fwd"].state), ref["A"][-1], tol, F64_ATOL_PROB)
            rel_close(_np(r["bck"].state), ref["B"][0], tol, F64_ATOL_PROB)
            rel_close(_np(r["E"]), ref["E"], tol, max(F64_ATOL_LOG, tol))
            rel_close(_np(r["fwd"].log_scale), ref["llf"], tol, F64_ATOL_LOG)
        else:
            check_reduced(prec, _np(r["P"]), ref["P"], "prob")
            check_reduced(prec, _np(r["fwd"].log_scale), ref["llf"], "log")
            for got, want in ((r["fwd"].state, ref["A"][-1]), (r["bck"].state, ref["B"][0])):
                err = np.abs(_np(got) - want).max(axis=1) / want.sum(axis=1)
                assert err.max() <= F32_POST_ATOL, err.max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_class_sweep_equals_plain_sweep(ls, prec):
    """Tables and log scales of long moves, whole and cut inside blocks, with
    and without classes (a forced shape is a plain sweep): within the
    precision's bound of each other."""
    N, L = 1500, 700
    H, rho, mu = _case(N, L, 10, seed=9)
    m = _model(ls, H, N, rho, mu)
    rec = np.array([0, 700, 1499], np.int32)

    def moved(cuts):
        out = []
        for d, stops in ((0, cuts), (1, [L - 1 - c for c in cuts])):
            t = ls.Table(m, d, prec, rec)
            for s in stops:
                (ls.forward if d == 0 else ls.backward)(t, m, s)
            out += [_np(t.state), _np(t.log_scale)]
        return out

    whole, cut = moved([L - 1]), moved([69, 70, 333, 420, L - 1])
    with forced_shape(*ls.kernel_shape(N, prec)):
        plain = moved([L - 1])
    for other in (cut, plain):
        for a, b in zip(whole, other):
            if prec == "fp64":
                rel_close(a, b, 1e-12, 1e-300)
            elif a.ndim == 2:
                assert (np.abs(a - b).max(axis=1) / b.sum(axis=1)).max() <= F32_POST_ATOL
            else:
                check_reduced(prec, a, b, "log")


def test_fp64_with_many_classes_is_plain(ls):
    """Sixteen class words: FP32 takes the class sweep, FP64 the plain one (the
    bits of a forced shape)."""
    N, L = 5000, 100
    H, rho, mu = _case(N, L, 700, seed=N + L)
    m = _model(ls, H, N, rho, mu)
    assert m.c.reserved >> 8 == 16
    rec = np.array([0, 4999], np.int32)

    def moved(prec):
        t = ls.Table(m, 0, prec, rec)
        ls.forward(t, m, L - 1)
        return _np(t.state)

    for prec, same in (("fp64", True), ("fp32", False)):
        own = moved(prec)
        with forced_shape(*ls.kernel_shape(N, prec)):
            assert np.array_equal(own, moved(prec)) == same


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_class_sweep_is_deterministic(ls, prec):
    """The same bits run after run, for a subset of the recipients, in
    recipient windows, in launches of another length, and for log P with and
    without the gradient."""
    import torch
    N, L = 1300, 300
    H, rho, mu = _case(N, L, 10, seed=3)
    m = _model(ls, H, N, rho, mu)
    targets = np.array([40, 64, 250], np.int32)
    a = ls.decode(m, targets, prec, want=("P",))
    b = ls.decode(m, targets, prec, want=("P",))
    assert torch.equal(a["P"], b["P"]) and torch.equal(a["fwd"].log_scale, b["fwd"].log_scale)
    sub = np.array([1299, 5, 640], np.int32)
    c = ls.decode(m, targets, prec, recipients=sub, want=("P",))
    assert torch.equal(a["P"][:, torch.as_tensor(sub).long().cuda()], c["P"])
    d = ls.distance_matrices(m, targets, prec, window=500)
    e = ls.distance_matrices(m, targets, prec, window=0)
    assert torch.equal(d["D"], e["D"]) and torch.equal(d["loglik"], e["loglik"])
    g = ls.loglik_grad(m, None, prec, grad=True)
    p = ls.loglik_grad(m, None, prec, grad=False)
    assert torch.equal(g["loglik"], p["loglik"]) and torch.equal(g["pac"], p["pac"])


def test_class_sweep_range(ls):
    """Recipients that match no donor for many variants in a row: the column
    sum falls by mu at each, far below FP32's range over the run."""
    N, L = 600, 256
    H, _ = mosaic_haplotypes(MosaicSpec(N, L, 4, 1e-3, 0.0, 5))
    h = np.unpackbits(H.view(np.uint8).reshape(L, -1), axis=1, bitorder="little")[:, :N].copy()
    h[100:140, :] = 0
    h[100:140, 7] = 1  # recipient 7 is alone over 40 variants
    from lsinputs import pack_haplotypes
    H = pack_haplotypes(h)
    rho = rho_from_spacings(spacings(L - 1, 1e-3, 8))
    mu = 1e-6
    m = _model(ls, H, N, rho, mu)
    rec = np.array([7, 8], np.int32)
    targets = [99, 110, 127, 128, 139, 200]
    ref = oracle.run_pass(H, N, L, rho, mu, rec, targets, want=("P",))
    for prec in ("fp64", "fp32"):
        r = ls.decode(m, targets, prec, recipients=rec, want=("P",))
        if prec == "fp64":
            rel_close(_np(r["P"]), ref["P"], f64_rtol(N), F64_ATOL_PROB)
            rel_close(_np(r["fwd"].log_scale), ref["llf"], f64_rtol(N), F64_ATOL_LOG)
        else:
            check_reduced(prec, _np(r["P"]), ref["P"], "prob")
            check_reduced(prec, _np(r["fwd"].log_scale), ref["llf"], "log")


@pytest.mark.parametrize("what", ["rho", "mu_low", "mu_high", "distinct", "prior"])
def test_models_without_classes(ls, what):
    """Parameters outside the class sweep's range, haplotypes that do not
    repeat and models with a prior matrix run the plain sweep."""
    N, L = 600, 100
    H, rho, mu = _case(N, L, 4, seed=1)
    prior = None
    if what == "rho":
        rho[7] = 1.0
    elif what == "mu_low":
        mu = 0.0
    elif what == "mu_high":
        mu = 0.6
    elif what == "prior":
        prior = np.full((N, N), 1.0 / (N - 1))
        np.fill_diagonal(prior, 0.0)
    else:
        H = np.random.default_rng(0).integers(0, 2 ** 32, H.shape, dtype=np.uint32)
    m = ls.Model(H, N, rho, mu, prior=prior)
    assert m.c.reserved == 0
