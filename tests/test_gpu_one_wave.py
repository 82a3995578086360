"""Single-wave groups (panels of at most 2,048 haplotypes, the gradient and
models with a prior matrix of at most 512) at the edges of their slot counts,
against the FP64 oracle through the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from lsinputs import pack_haplotypes, rho_from_spacings

from _gpu import (F32_LOGLIK_RTOL, F64_ATOL_LOG, F64_ATOL_PROB, F64_RTOL, check_reduced, need_gpu,
                  rel_close)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


def _np(t):
    return t.double().cpu().numpy()


def _case(N, L, seed):
    rng = np.random.default_rng(seed)
    h = (rng.random((L, N)) < 0.3).astype(np.uint8)
    return pack_haplotypes(h), rho_from_spacings(rng.exponential(0.05, L - 1)), rng


SIZES = [64, 65, 128, 129, 192, 193, 256, 257, 512, 513, 768, 1024, 1025, 1281, 1536, 1793, 2047,
         2048, 2049]


@pytest.mark.parametrize("N", SIZES)
def test_decode(ls, N):
    L = 24
    H, rho, _ = _case(N, L, N)
    nw = ls.kernel_shape(N, "fp32")[1]
    assert (nw == 1) == (N <= 2048)
    rec = np.unique([0, N // 2, N - 1]).astype(np.int32)
    targets = [0, 11, L - 1]
    m = ls.Model(H, N, rho, 0.01)
    ref = oracle.run_pass(H, N, L, rho, 0.01, rec, targets, want=("P",))
    for prec in ("fp64", "fp32", "f16"):
        r = ls.decode(m, targets, prec, recipients=rec, want=("P",))
        if prec == "fp64":
            rel_close(_np(r["P"]), ref["P"], F64_RTOL, F64_ATOL_PROB)
            rel_close(_np(r["fwd"].log_scale), ref["llf"], F64_RTOL, F64_ATOL_LOG)
        else:
            check_reduced(prec, _np(r["P"]), ref["P"], "prob")
            check_reduced(prec, _np(r["fwd"].log_scale), ref["llf"], "log")


@pytest.mark.parametrize("vec", [False, True])
@pytest.mark.parametrize("N", [64, 129, 256, 512, 513])
def test_prior_and_gradient(ls, N, vec):
    L = 20
    H, rho, rng = _case(N, L, N + 7)
    mu = 10.0 ** rng.uniform(-3, -1, L) if vec else 0.01
    Pi = rng.random((N, N)) + 0.05
    np.fill_diagonal(Pi, 0.0)
    Pi /= Pi.sum(axis=0, keepdims=True)
    rec = np.unique([0, N // 3, N - 1]).astype(np.int32)
    for prior in (None, Pi):
        m = ls.Model(H, N, rho, mu, prior=prior)
        ref = oracle.run_gradient(H, N, L, rho, mu, rec, prior=prior)
        dec = oracle.run_pass(H, N, L, rho, mu, rec, [9], want=("P",), prior=prior)
        gmu = (ref["grad_mu_l"] if vec else ref["grad_mu"][:, None]).sum(axis=0)
        smu = np.abs(ref["grad_mu_l"] if vec else ref["grad_mu"]).sum()
        for prec, tol, tol_ll in (("fp64", 1e-10, 1e-12), ("fp32", 1e-6, F32_LOGLIK_RTOL)):
            P = _np(ls.decode(m, [9], prec, recipients=rec, want=("P",))["P"])
            if prec == "fp64":
                rel_close(P, dec["P"], F64_RTOL, F64_ATOL_PROB)
            else:
                check_reduced(prec, P, dec["P"], "prob")
            g = ls.loglik_grad(m, rec, prec, grad=True)
            ll = ref["loglik"].sum()
            assert abs(g["pac"].item() - ll) <= tol_ll * abs(ll)
            err = np.abs(_np(g["grad_rho"]) - ref["grad_rho"].sum(axis=0)).max()
            assert err <= tol * max(np.abs(ref["grad_rho"]).sum(axis=0).max(), 1.0)
            assert np.abs(_np(g["grad_mu"]) - gmu).max() <= tol * max(smu, 1.0)
