"""Average linkage in FP64 on either side of the last size whose state fits
local memory (12 bytes per slot), bit for bit against the oracle."""

from __future__ import annotations

import numpy as np
import pytest

from test_gpu_linkage_edges import _check, ls  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [13_200, 13_400])
def test_state_at_the_local_memory_limit(ls, N):  # noqa: F811
    rng = np.random.default_rng(N)
    x = rng.random((N, 2))
    _check(ls, [np.abs(x[:, :1] - x[:, :1].T) + np.abs(x[:, 1:] - x[:, 1:].T)])
