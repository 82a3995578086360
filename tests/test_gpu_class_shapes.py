"""Class sweeps over the donor words per wave and the class words that the
choice of a shape takes, and cut into launches that do not end with blocks;
through the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
import test_gpu_classes
from _gpu import check_reduced
from test_gpu_classes import ls  # noqa: F401

pytestmark = pytest.mark.gpu


# FP32 donor words x waves 24 .. 144 x 1, 96 and 128 x 2, 112 x 5, FP64 24 .. 80 x 1 .. 7;
# few founders and many (2 to 12 class words)
@pytest.mark.parametrize("N,K,vec", [
    (1500, 4, False), (1500, 250, True), (2000, 4, True), (2000, 300, False), (3000, 4, False),
    (3000, 500, True), (4000, 4, False), (4000, 500, False), (5200, 700, False), (6500, 4, True),
    (7300, 4, False), (7300, 400, True), (8300, 4, True), (8300, 250, False), (12000, 100, False),
    (16000, 4, False), (16000, 250, True), (33000, 4, True)])
def test_shapes(ls, N, K, vec):  # noqa: F811
    test_gpu_classes.test_class_sweep_vs_oracle(ls, N, 66, K, vec, 1e-4)


@pytest.mark.parametrize("N", [56_000, 81_920])
def test_largest_fp32(ls, N):  # noqa: F811
    """Past FP64's largest panel: seven waves of 128 donor words, eight of 160 (the
    largest with classes)."""
    L = 66
    H, rho, mu = test_gpu_classes._case(N, L, 4, seed=N, switch=1e-4)
    m = test_gpu_classes._model(ls, H, N, rho, mu)
    rec = np.array([0, N // 2, N - 1], np.int32)
    ref = oracle.run_pass(H, N, L, rho, mu, rec, [31, 64], want=("P",))
    r = ls.decode(m, [31, 64], "fp32", recipients=rec, want=("P",))
    check_reduced("fp32", r["P"].double().cpu().numpy(), ref["P"], "prob")
    check_reduced("fp32", r["fwd"].log_scale.double().cpu().numpy(), ref["llf"], "log")


def test_past_the_largest_panel(ls):  # noqa: F811
    """No classes and no room for them one donor further."""
    from paper_2212_11403_amd import _lib
    N, L = 81_921, 66
    rows = L * (-(-(2 * (N // 64) + 1) // 8) * 8) * 8
    need = -(-rows // 256) * 256 + 40 * L + 32 * L + 8 + 16 * N
    assert _lib.load().ls_model_workspace_bytes(N, L) == need
    H, rho, mu = test_gpu_classes._case(N, L, 4, seed=N, switch=1e-4)
    assert ls.Model(H, N, rho, mu).c.reserved == 0


@pytest.mark.parametrize("chunk", [33, 100])
def test_launches_that_cut_blocks(ls, monkeypatch, chunk):  # noqa: F811
    """Launches of 33 and 100 variants: shorter than a block, and ending inside
    one in the backward direction."""
    monkeypatch.setenv("LS_SWEEP_CHUNK", str(chunk))
    test_gpu_classes.test_class_sweep_vs_oracle(ls, 1000, 700, 12, True, 2e-3)
