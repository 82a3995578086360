"""The gradient per class where the workspace holds fewer checkpoints than there
are block ends (groups of blocks, formed again from one checkpoint each), where
a block has more class words than the adjoint is built for (class checkpoints,
plain adjoint), and models whose workspace has no room for classes; through the
C ABI (libls.so)."""

from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle
from _gpu import F32_LOGLIK_RTOL
from test_gpu_grad_classes import _case, ls  # noqa: F401

pytestmark = pytest.mark.gpu


def _groups(m):
    """Block ends to keep, and vectors the workspace has room for: checkpoints
    every ceil(sqrt(L)) variants and every second vector of a segment."""
    L, B = m.L, 1 << (m.c.reserved & 7)
    seg = int(np.ceil(np.sqrt(L)))
    return -(-L // B) - 1, -(-L // seg) + max(1, (seg - 1) // 2)


def _check(ls, m, H, N, L, rho, mu, rec, precs):  # noqa: F811
    ref = oracle.run_gradient(H, N, L, rho, mu, rec)
    vec = np.ndim(mu) == 1
    gmu = (ref["grad_mu_l"] if vec else ref["grad_mu"][:, None]).sum(axis=0)
    smu = np.abs(ref["grad_mu_l"] if vec else ref["grad_mu"]).sum()
    ll = ref["loglik"].sum()
    out = {}
    for prec in precs:
        tol, tol_ll = (1e-10, 1e-12) if prec == "fp64" else (1e-6, F32_LOGLIK_RTOL)
        g = out[prec] = ls.loglik_grad(m, rec, prec, grad=True)
        assert abs(g["pac"].item() - ll) <= tol_ll * abs(ll)
        err = np.abs(g["grad_rho"].cpu().numpy() - ref["grad_rho"].sum(axis=0)).max()
        assert err <= tol * max(np.abs(ref["grad_rho"]).sum(axis=0).max(), 1.0)
        assert np.abs(g["grad_mu"].cpu().numpy() - gmu).max() <= tol * max(smu, 1.0)
        # the log-likelihood alone: the same bits
        p = ls.loglik_grad(m, rec, prec, grad=False)
        import torch
        assert torch.equal(g["loglik"], p["loglik"])
    return out


# the last group whole, of one block, of one variant; groups of two and of more
@pytest.mark.parametrize("vec", [False, True])
@pytest.mark.parametrize("L", [12_000, 12_033, 36_000])
def test_groups_of_blocks(ls, L, vec):  # noqa: F811
    N = 520
    H, rho, mu = _case(N, L, 4, seed=L, vec=vec)
    rec = np.array([0, 300, N - 1], np.int32)
    m = ls.Model(H, N, rho, mu)
    assert m.c.reserved != 0
    ends, room = _groups(m)
    assert ends > room
    got = _check(ls, m, H, N, L, rho, mu, rec, ("fp64", "fp32"))
    # the two halves of the gradient as separate calls: the same bits
    import torch
    from paper_2212_11403_amd import api
    for prec, g in got.items():
        g_rho, g_mu = api.Checkpoints(m, rec, prec).gradient()
        assert torch.equal(g["grad_rho"], g_rho) and torch.equal(g["grad_mu"], g_mu)


# 10, 12 and 16 class words
@pytest.mark.parametrize("N,K,words,vec", [(3000, 400, 10, False), (5000, 450, 12, True),
                                           (5000, 700, 16, False)])
def test_many_classes(ls, N, K, words, vec):  # noqa: F811
    L = 100
    H, rho, mu = _case(N, L, K, seed=N + L, vec=vec)
    m = ls.Model(H, N, rho, mu)
    assert m.c.reserved >> 8 == words
    _check(ls, m, H, N, L, rho, mu, np.array([0, 64, N - 1], np.int32), ("fp64", "fp32"))


def test_workspace_without_classes(ls):  # noqa: F811
    """A workspace that ends before the class section: accepted, and the sweeps
    are the plain ones, bit for bit."""
    import torch
    from paper_2212_11403_amd import _lib
    N, L = 600, 300
    H, rho, mu = _case(N, L, 4, seed=6)
    m = ls.Model(H, N, rho, mu)
    assert m.c.reserved != 0
    rows = L * (-(-(2 * (N // 64) + 1) // 8) * 8) * 8
    need = -(-rows // 256) * 256 + 40 * L + 32 * L + 8 + 16 * N
    full = _lib.load().ls_model_workspace_bytes(N, L)
    assert need < full
    small = ls.Model(H, N, rho, mu)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    init = lambda nbytes: _lib.load().ls_model_init(  # noqa: E731
        ctypes.byref(small.c), ctypes.c_void_p(ws.data_ptr()), nbytes, st)
    assert init(need - 1) != 0
    assert init(need) == 0
    assert small.c.reserved == 0
    m.c.reserved = 0  # the same model without its classes
    for prec in ("fp64", "fp32"):
        a = ls.decode(m, [100, 250], prec, want=("P",))
        b = ls.decode(small, [100, 250], prec, want=("P",))
        assert torch.equal(a["P"], b["P"]) and torch.equal(a["fwd"].log_scale, b["fwd"].log_scale)
        g, k = (ls.loglik_grad(x, None, prec) for x in (m, small))
        assert torch.equal(g["grad_rho"], k["grad_rho"]) and torch.equal(g["grad_mu"], k["grad_mu"])


def test_long_launches(ls, monkeypatch):  # noqa: F811
    """Launches meant to be longer than one launch's checkpoints: log P of the
    gradient is still that of the log-likelihood alone, bit for bit."""
    import torch
    N, L = 520, 60_000
    H, rho, mu = _case(N, L, 4, seed=1)
    m = ls.Model(H, N, rho, mu)
    ends, room = _groups(m)
    assert ends > 2 * 256 and room > 256  # more than 256 checkpoints kept
    rec = np.array([0, 300, N - 1], np.int32)
    monkeypatch.setenv("LS_SWEEP_CHUNK", "1000000")
    for prec in ("fp64", "fp32"):
        g, p = (ls.loglik_grad(m, rec, prec, grad=grad) for grad in (True, False))
        assert torch.equal(g["loglik"], p["loglik"])
