"""Two threads with streams of their own that launch the same kernels with
different amounts of local memory, through the C ABI (libls.so)."""

from __future__ import annotations

import threading

import numpy as np
import pytest

from _gpu import need_gpu
from lsinputs import MosaicSpec, mosaic_haplotypes, rho_from_spacings, spacings

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


def _together(works):
    """Runs the works four times each at once; their results of every run."""
    import torch
    out = [[] for _ in works]
    errors = []

    def body(k, work):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    out[k].append(work())
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=body, args=(k, w)) for k, w in enumerate(works)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    return out


def test_linkage(ls):
    """Matrices of N = 8,300 and 8,800 (67 and 71 KB of local memory)."""
    import torch
    D = []
    for N in (8300, 8800):
        d = torch.rand((N, N), device="cuda", generator=torch.Generator(device="cuda").manual_seed(N))
        D.append(d + d.t())
    want = [ls.average_linkage(d.clone()) for d in D]
    torch.cuda.synchronize()
    got = _together([lambda d=d: ls.average_linkage(d.clone()) for d in D])
    for (Z, order), runs in zip(want, got):
        for z, o in runs:
            assert torch.equal(Z, z) and torch.equal(order, o)


def test_class_sweeps(ls):
    """Class sweeps of N = 50,000 and 57,000 with 16 class words (groups of
    seven and eight waves of 112 donor words: 70 and 78 KB)."""
    import torch
    works, want = [], []
    for N in (50_000, 57_000):
        L = 70
        H, _ = mosaic_haplotypes(MosaicSpec(N, L, 850, 1e-4, 0.0, N))
        m = ls.Model(H, N, rho_from_spacings(spacings(L - 1, 1e-3, 1)), 1e-3)
        assert (m.c.reserved >> 8) == 16
        rec = np.arange(64, dtype=np.int32)
        works.append(lambda m=m, rec=rec: ls.decode(m, [40], "fp32", recipients=rec, want=("P",))["P"])
        want.append(works[-1]())
    torch.cuda.synchronize()
    for w, runs in zip(want, _together(works)):
        for p in runs:
            assert torch.equal(w, p)
