"""Models whose recombination (nearly) stops over runs of variants: a donor's
share of a column then falls by mu at every mismatch with no jump to hold it
up, and a class that had all but vanished can become the best one again.
Against the FP64 oracle, through the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from lsinputs import pack_haplotypes, rho_from_spacings, spacings

from _gpu import F64_ATOL_LOG, F64_ATOL_PROB, check_reduced, f64_rtol, need_gpu, rel_close

pytestmark = pytest.mark.gpu

N, L = 601, 192
SELF = 600


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


def _np(t):
    return t.double().cpu().numpy()


def _haplotypes(spans):
    """Recipient 600 carries 0 everywhere; `spans` lists (half, first variant,
    mismatches): the donors of half 0 (0 .. 299) or 1 (300 .. 599) carry 1 at
    that many variants from the first, every second one where a block of 64
    has room for it. One variant splits both halves."""
    h = np.zeros((L, N), np.uint8)
    for half, l0, n in spans:
        step = 2 if n < 32 else 1
        h[l0:l0 + step * n:step, 300 * half:300 * half + 300] = 1
    h[190, :150] = h[190, 300:450] = 1
    return pack_haplotypes(h)


def _rho(kind):
    rho = rho_from_spacings(spacings(L - 1, 1e-3, 3))
    if kind == "zero":
        rho[:] = 0.0
    elif kind == "run":         # one map position over most of the sequence
        rho[2:180] = 0.0
    elif kind == "tiny":        # a share still falls no lower than 2^-76 at mu = 1e-4
        rho[:] = 2.0 ** -52
    elif kind == "least":       # the same at mu = 0.11 (and too little at 1e-4)
        rho[:] = 2.0 ** -72
    elif kind == "tiniest":
        rho[:] = 1e-300
    return rho


def _takes_classes(ls, H):
    m = ls.Model(H, N, rho_from_spacings(spacings(L - 1, 1e-3, 3)), 1e-4)
    return m.c.reserved != 0


# half 0 mismatches in block 0, half 1 in block 1 (blocks of 64): by 2^-106 to
# 2^-150 in FP32's range cases, by 2^-957 and more in FP64's
@pytest.mark.parametrize("kind", ["zero", "run", "tiny", "tiniest"])
@pytest.mark.parametrize("mu,a,b", [(1e-8, 4, 5), (1e-8, 4, 4), (1e-9, 4, 4), (1e-4, 8, 9),
                                    (2.0 ** -29, 33, 34), (1e-3, 2, 1)])
def test_sweeps(ls, kind, mu, a, b):
    H, rho = _haplotypes([(0, 1, a), (1, 65, b)]), _rho(kind)
    assert _takes_classes(ls, H)
    rec = np.array([SELF, 0, 599], np.int32)
    targets = [0, 63, 64, 127, 130, 191]  # (the tables end at the outer ones)
    ref = oracle.run_pass(H, N, L, rho, mu, rec, targets, want=("A", "B", "P"))
    m = ls.Model(H, N, rho, mu)
    # (33 mismatches of 2^-29 leave FP32's range, in every sweep)
    for prec in ("fp64", "fp32") if a < 33 or kind == "tiny" else ("fp64",):
        r = ls.decode(m, targets, prec, recipients=rec, want=("P",))
        if prec == "fp64":
            tol = f64_rtol(N)
            rel_close(_np(r["P"]), ref["P"], tol, F64_ATOL_PROB)
            rel_close(_np(r["fwd"].state), ref["A"][-1], tol, F64_ATOL_PROB)
            rel_close(_np(r["bck"].state), ref["B"][0], tol, F64_ATOL_PROB)
            rel_close(_np(r["fwd"].log_scale), ref["llf"], tol, F64_ATOL_LOG)
        else:
            check_reduced(prec, _np(r["P"]), ref["P"], "prob")
            # log P is near 0 here, so the bound is absolute: a column sum passes
            # through at most 16 FP32 additions and products a variant
            err = np.abs(_np(r["fwd"].log_scale) - ref["llf"]).max()
            assert err <= 16 * L * 2.0 ** -24, err


# half 0 falls up to both ends of a block in which half 1 falls further: both
# vectors of half 0 are small at that block's ends and their product smaller
@pytest.mark.parametrize("kind", ["zero", "run", "tiny", "least", "tiniest"])
@pytest.mark.parametrize("mu,a,b", [(1e-4, 6, 13), (1e-3, 2, 5), (1e-6, 3, 7), (0.11, 22, 63)])
def test_gradient(ls, kind, mu, a, b):
    H, rho = _haplotypes([(0, 65 - 2 * a, a), (1, 65, b), (0, 128, a)]), _rho(kind)
    assert _takes_classes(ls, H)
    rec = np.array([SELF, 0], np.int32)
    ref = oracle.run_gradient(H, N, L, rho, mu, rec)
    m = ls.Model(H, N, rho, mu)
    for prec in ("fp64", "fp32"):
        # a term's FP32 error: the mismatch ratio is rounded once (2^-25) and
        # every product with it once more (2^-24), in both vectors, over at most
        # 2a + b factors in the numerator and the denominator each
        tol = 1e-10 if prec == "fp64" else 3 * (2 * a + b) * 2.0 ** -24
        g = ls.loglik_grad(m, rec, prec)
        ll = ref["loglik"].sum()
        lim = 1e-12 * max(abs(ll), 1.0) if prec == "fp64" else 2 * 16 * L * 2.0 ** -24
        assert abs(g["pac"].item() - ll) <= lim
        want = ref["grad_rho"].sum(axis=0)
        err = np.abs(_np(g["grad_rho"]) - want) / np.maximum(np.abs(ref["grad_rho"]).sum(axis=0), 1.0)
        err_mu = abs(g["grad_mu"].item() - ref["grad_mu"].sum()) / max(np.abs(ref["grad_mu"]).sum(), 1.0)
        print(f"{kind} mu={mu} {prec}: rho {err.max():.2e}, mu {err_mu:.2e}")
        assert err.max() <= tol and err_mu <= tol
