"""The gradient carried per haplotype class against the FP64 oracle's score,
through the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from lsinputs import (MosaicSpec, mosaic_haplotypes, pack_haplotypes, rho_from_spacings,
                      spacings)

from _gpu import F32_LOGLIK_RTOL, forced_shape, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


def _case(N, L, K, seed, vec=False):
    H, _ = mosaic_haplotypes(MosaicSpec(N, L, K, 2e-3, 1e-4, seed))
    rho = rho_from_spacings(spacings(L - 1, 1e-3, seed + 1))
    rng = np.random.default_rng(seed)
    rho[rng.random(L - 1) < 0.02] = 0.8
    mu = 10.0 ** rng.uniform(-4, -1, L) if vec else 1e-3
    return H, rho, mu


def _check(ls, H, N, L, rho, mu, rec, precs=("fp64", "fp32")):
    """Errors relative to the summed magnitudes of the recipients' terms, as
    for the other gradient passes."""
    m = ls.Model(H, N, rho, mu)
    assert m.c.reserved != 0, "the case does not take the class gradient"
    ref = oracle.run_gradient(H, N, L, rho, mu, rec)
    vec = np.ndim(mu) == 1
    gmu = (ref["grad_mu_l"] if vec else ref["grad_mu"][:, None]).sum(axis=0)
    smu = np.abs(ref["grad_mu_l"] if vec else ref["grad_mu"]).sum()
    ll = ref["loglik"].sum()
    for prec in precs:
        tol, tol_ll = (1e-10, 1e-12) if prec == "fp64" else (1e-6, F32_LOGLIK_RTOL)
        g = ls.loglik_grad(m, rec, prec, grad=True)
        assert abs(g["pac"].item() - ll) <= tol_ll * abs(ll)
        err = np.abs(g["grad_rho"].cpu().numpy() - ref["grad_rho"].sum(axis=0)).max()
        lim = tol * max(np.abs(ref["grad_rho"]).sum(axis=0).max(), 1.0)
        err_mu = np.abs(g["grad_mu"].cpu().numpy() - gmu).max()
        print(f"N={N} L={L} {prec}: rho {err / lim * tol:.2e}, mu {err_mu / max(smu, 1.0):.2e}")
        assert err <= lim and err_mu <= tol * max(smu, 1.0)


# one block of variants, a last block of one variant, ragged groups of eight
# variants; all block ends kept, and groups of blocks (long L, few vectors);
# one and several waves
@pytest.mark.parametrize("N,L,K,vec", [
    (512, 65, 4, False), (600, 64, 4, True), (703, 129, 6, False), (1000, 999, 8, True),
    (1000, 5000, 8, False), (2049, 200, 20, False), (5200, 150, 40, True)])
def test_class_gradient_vs_oracle(ls, N, L, K, vec):
    H, rho, mu = _case(N, L, K, seed=N + L, vec=vec)
    rec = np.unique([0, 63, 64, N // 2, N - 1]).astype(np.int32)
    _check(ls, H, N, L, rho, mu, rec)


def test_class_gradient_range(ls):
    """A recipient alone with its alleles over 40 variants: both vectors'
    sums fall by mu at each, and its class keeps no member but itself."""
    N, L = 600, 256
    H, _ = mosaic_haplotypes(MosaicSpec(N, L, 4, 1e-3, 0.0, 5))
    h = np.unpackbits(H.view(np.uint8).reshape(L, -1), axis=1, bitorder="little")[:, :N].copy()
    h[100:140, :] = 0
    h[100:140, 7] = 1
    from lsinputs import pack_haplotypes
    rho = rho_from_spacings(spacings(L - 1, 1e-3, 8))
    _check(ls, pack_haplotypes(h), N, L, rho, 1e-6, np.array([7, 8], np.int32))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_class_gradient_repeats_and_agrees(ls, prec):
    """The same bits run after run and in two calls (checkpoints, then the
    adjoint); the plain passes' gradient within the precision's bound."""
    import torch
    from paper_2212_11403_amd import api
    N, L = 900, 700
    H, rho, mu = _case(N, L, 8, seed=2)
    m = ls.Model(H, N, rho, mu)
    a = ls.loglik_grad(m, None, prec, grad=True)
    b = ls.loglik_grad(m, None, prec, grad=True)
    g_rho, g_mu = api.Checkpoints(m, None, prec).gradient()
    assert torch.equal(a["grad_rho"], b["grad_rho"]) and torch.equal(a["grad_mu"], b["grad_mu"])
    assert torch.equal(a["grad_rho"], g_rho) and torch.equal(a["grad_mu"], g_mu)
    with forced_shape(16, 1):
        c = ls.loglik_grad(m, None, prec, grad=True)
    tol = 1e-10 if prec == "fp64" else 1e-6
    # every recipient's term is at most 1 / rho and the sum has N of them; the
    # largest component bounds the scale from below
    assert (a["grad_rho"] - c["grad_rho"]).abs().max() <= tol * c["grad_rho"].abs().max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_class_gradient_of_private_alleles(ls, prec):
    """A recipient that mismatches every donor at a variant has mismatch mass
    1 there: d log P / d mu^l = 1/mu to FP64's rounding, in FP32 too (its
    matching classes add exactly 0)."""
    N, L, mu = 700, 300, 1e-4
    H, rho, _ = _case(N, L, 6, seed=4)
    h = np.unpackbits(H.view(np.uint8).reshape(L, -1), axis=1, bitorder="little")[:, :N].copy()
    at = np.array([0, 5, 63, 64, 130, 255, 256, 299])
    h[at, :] = 0
    h[at, 17] = 1
    m = ls.Model(pack_haplotypes(h), N, rho, np.full(L, mu))
    assert m.c.reserved != 0
    g = ls.loglik_grad(m, recipients=np.array([17], np.int32), prec=prec)["grad_mu"].cpu().numpy()
    assert np.abs(g[at] * mu - 1.0).max() <= 1e-14
