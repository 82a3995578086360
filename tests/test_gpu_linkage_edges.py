"""Average linkage at the edges of the merge kernel's loops: one slot a thread,
one more, its unrolled loops with and without a remainder, the last sizes
whose state fits local memory and the first that does not; with negative
distances, both zeros, infinities and NaN rows. Bit for bit against the
oracle."""

from __future__ import annotations

import numpy as np
import pytest

import oracle

from _gpu import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


def _matrix(N, seed, dtype):
    """Signed distances with ties, both zeros, an infinite pair and a NaN row."""
    rng = np.random.default_rng(seed)
    A = np.triu(rng.integers(-40, 400, size=(N, N)) / 8.0, 1)
    A = (A + A.T).astype(dtype)
    A[A == 1.0] = -0.0
    if N > 4:
        A[0, N - 1] = A[N - 1, 0] = np.inf
        A[2, :] = A[:, 2] = np.nan
    np.fill_diagonal(A, 0.0)
    return A


def _check(ls, mats):
    import torch
    Z, order = ls.average_linkage(torch.from_numpy(np.stack(mats)).cuda())
    torch.cuda.synchronize()
    for t, D in enumerate(mats):
        Zr, orr = oracle.average_linkage(D)
        assert np.array_equal(Z[t].cpu().numpy(), Zr, equal_nan=True), t
        assert np.array_equal(order[t].cpu().numpy(), orr), t


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("N", [2, 3, 5, 64, 65, 1023, 1024, 1025, 4096, 4099])
def test_merge_loops(ls, N, dtype):
    _check(ls, [_matrix(N, N + 1, dtype)])


def test_state_at_the_local_memory_limit(ls):
    """FP32 keeps 8 bytes per slot: N = 20,000 fits 160 KB beside the
    reductions' entries, N = 20,500 does not."""
    for N in (20_000, 20_500):
        rng = np.random.default_rng(N)
        x = rng.random((N, 2)).astype(np.float32)
        D = np.abs(x[:, :1] - x[:, :1].T) + np.abs(x[:, 1:] - x[:, 1:].T)
        _check(ls, [D])
