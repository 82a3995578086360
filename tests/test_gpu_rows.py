"""Posterior rows and symmetrised matrices at the edges of their kernels: rows
read 16 bytes or one element at a time, the longest rows held in registers and
the first that are not, full and ragged tiles; against numpy in FP64."""

from __future__ import annotations

import numpy as np
import pytest

from _gpu import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("N", [7, 1023, 1025, 8191, 8193, 16383, 16384, 16385, 32768, 32772])
def test_posterior_rows(ls, N, prec):
    """Two tables with chosen vectors at variant 0 of a one-variant model."""
    import torch
    L = 1
    H = np.zeros((L, ((N + 31) // 32 + 7) // 8 * 8), np.uint32)
    m = ls.Model(H, N, np.zeros(0), 0.01)
    rec = np.array([0, N // 2, N - 1], np.int32)
    f, b = ls.Table(m, 0, prec, rec), ls.Table(m, 1, prec, rec)
    ls.forward(f, m, 0)
    ls.backward(b, m, 0)
    g = torch.Generator(device="cuda").manual_seed(N)
    for t in (f, b):
        t.state.copy_(torch.rand(t.state.shape, generator=g, device="cuda", dtype=t.state.dtype) ** 8)
        t.state[torch.arange(3), torch.as_tensor(rec).long()] = 0.0
    f.state[1, : N // 3] = 0.0  # posteriors below eps
    P, E = torch.empty_like(f.state), torch.empty_like(f.state)
    ls.posterior_distance(f, b, m, P, E)
    q = f.state.double().cpu().numpy() * b.state.double().cpu().numpy()
    ref = q / q.sum(axis=1, keepdims=True)
    eps = 2.0 ** -52
    e = -0.5 * np.log(np.maximum(ref, eps))
    e[np.arange(3), rec] = 0.0
    # a product, a sum of N terms in a tree of chains of at most 33, a quotient
    u = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    rel = 64 * u
    assert np.abs(P.double().cpu().numpy() - ref).max() <= rel * ref.max()
    assert np.abs(E.double().cpu().numpy() - e).max() <= rel + 4 * u * np.abs(e).max()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("N", [1, 63, 64, 65, 127, 129, 193])
def test_symmetrise(ls, N, prec):
    import torch
    dt = torch.float64 if prec == "fp64" else torch.float32
    E = torch.rand((3, N, N), generator=torch.Generator(device="cuda").manual_seed(N), device="cuda",
                   dtype=dt)
    want = E + E.transpose(1, 2)
    want[:, torch.arange(N), torch.arange(N)] = 0.0
    D = torch.empty_like(E)
    ls.distance_symmetrise(E, D, prec)
    assert torch.equal(D, want)
    ls.distance_symmetrise(E, E, prec)
    assert torch.equal(E, want)
