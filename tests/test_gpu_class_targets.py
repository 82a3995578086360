"""Moves with many targets on a model that has classes: at most one target per
eight variants takes the class sweep, more the plain one, bit for bit; through
the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
import test_gpu_classes
from _gpu import F64_ATOL_PROB, check_reduced, f64_rtol, rel_close
from test_gpu_classes import ls  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("T,plain", [(1, False), (25, False), (26, True), (200, True)])
def test_targets(ls, T, plain, prec):  # noqa: F811
    import torch
    N, L = 900, 201  # moves of 200 variants
    H, rho, mu = test_gpu_classes._case(N, L, 6, seed=2)
    m = test_gpu_classes._model(ls, H, N, rho, mu)
    rec = np.array([0, 64, N - 1], np.int32)
    targets = np.sort(np.random.default_rng(T).choice(L, T, replace=False)).astype(np.int32)
    r = ls.decode(m, targets, prec, recipients=rec, want=("P",))
    ref = oracle.run_pass(H, N, L, rho, mu, rec, targets, want=("P",))
    got = r["P"].double().cpu().numpy()
    if prec == "fp64":
        rel_close(got, ref["P"], f64_rtol(N), F64_ATOL_PROB)
    else:
        check_reduced(prec, got, ref["P"], "prob")
    m.c.reserved = 0  # the same model without its classes
    p = ls.decode(m, targets, prec, recipients=rec, want=("P",))
    for k in ("fwd", "bck"):
        assert torch.equal(r[k].state, p[k].state) == plain
