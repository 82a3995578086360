"""Single waves of 513 to 2,048 haplotypes (row words held, of every slot count):
a call over few recipients gives the bits of the call over all of them, through
the C ABI (libls.so)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from lsinputs import pack_haplotypes, rho_from_spacings

from _gpu import check_reduced, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ls():
    need_gpu()
    import paper_2212_11403_amd as m
    m.load()
    return m


# every slot count (12 to 32), its fewest and most words, full and ragged last
# words, few recipients and more than the card's compute units
@pytest.mark.parametrize("vec", [False, True])
@pytest.mark.parametrize("N", [513, 575, 768, 769, 1024, 1025, 1088, 1280, 1281, 1536, 1537, 1601,
                               1792, 1793, 2047, 2048])
def test_few_and_all_recipients(ls, N, vec):
    import torch
    L = 30
    rng = np.random.default_rng(N)
    H = pack_haplotypes((rng.random((L, N)) < 0.3).astype(np.uint8))
    rho = rho_from_spacings(rng.exponential(0.05, L - 1))
    mu = 10.0 ** rng.uniform(-3, -1, L) if vec else 0.01
    m = ls.Model(H, N, rho, mu)
    few = np.unique([0, 63, 64, N // 2, N - 65, N - 1]).astype(np.int32)
    targets = [0, 13, L - 1]
    ref = oracle.run_pass(H, N, L, rho, mu, few, targets, want=("P",))
    at = torch.as_tensor(few).long().cuda()
    for prec in ("fp32", "f16"):
        a = ls.decode(m, targets, prec, want=("P",))
        for rec in (few, np.concatenate([few, np.arange(512 - len(few))]).astype(np.int32)):
            b = ls.decode(m, targets, prec, recipients=rec, want=("P",))
            k = len(few)
            assert torch.equal(a["P"][:, at], b["P"][:, :k])
            for t in ("fwd", "bck"):
                assert torch.equal(a[t].state[at], b[t].state[:k])
                assert torch.equal(a[t].log_scale[at], b[t].log_scale[:k])
            # moved in steps
            c = ls.Table(m, 0, prec, rec[:k])
            for stop in (5, 6, 20, L - 1):
                ls.forward(c, m, stop)
            assert torch.equal(c.state, b["fwd"].state[:k])
        check_reduced(prec, b["P"][:, :k].double().cpu().numpy(), ref["P"], "prob")
