"""Single-wave groups with a target at every variant, at runs of variants and at
the ends of launches, against the FP64 oracle through the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from lsinputs import pack_haplotypes, rho_from_spacings

from _gpu import F64_ATOL_PROB, F64_RTOL, check_reduced, need_gpu, rel_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


# 1 to 20 slots: with and without what is read ahead kept over a target
@pytest.mark.parametrize("chunk", [0, 7])
@pytest.mark.parametrize("vec", [False, True])
@pytest.mark.parametrize("N", [64, 65, 130, 257, 300, 512, 700, 1000, 1200])
def test_dense_targets(ls, monkeypatch, N, vec, chunk):
    if chunk:
        monkeypatch.setenv("LS_SWEEP_CHUNK", str(chunk))
    L = 40
    rng = np.random.default_rng(N)
    H = pack_haplotypes((rng.random((L, N)) < 0.3).astype(np.uint8))
    rho = rho_from_spacings(rng.exponential(0.05, L - 1))
    mu = 10.0 ** rng.uniform(-3, -1, L) if vec else 0.01
    m = ls.Model(H, N, rho, mu)
    rec = np.unique([0, N // 2, N - 1]).astype(np.int32)
    for targets in (list(range(L)), [0, 1, 2, 14, 15, 20, 21, 22, L - 2, L - 1], [L - 1], [0]):
        ref = oracle.run_pass(H, N, L, rho, mu, rec, targets, want=("B", "P"))
        for prec in ("fp64", "fp32", "f16"):
            r = ls.decode(m, targets, prec, recipients=rec, want=("P",))
            P, B = (r[k].double().cpu().numpy() for k in ("P", "bsnap"))
            assert not B[:, np.arange(len(rec)), rec].any()
            if prec == "fp64":
                rel_close(P, ref["P"], F64_RTOL, F64_ATOL_PROB)
                rel_close(B, ref["B"], F64_RTOL, F64_ATOL_PROB)
            else:
                check_reduced(prec, P, ref["P"], "prob")
