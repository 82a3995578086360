"""Posterior rows read one element at a time at the edges of their forms: two
passes over short rows, then 4, 8 or 16 values held per thread."""

from __future__ import annotations

import pytest

import test_gpu_rows
from test_gpu_rows import ls  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("N", [1021, 1025, 4095, 4097])
def test_short_rows(ls, N, prec):  # noqa: F811
    test_gpu_rows.test_posterior_rows(ls, N, prec)
