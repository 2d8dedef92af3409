"""GPU: weights whose powers are all 1 or 2 (kernels that multiply instead of
calling pow()) and weights just outside that rule (kernels with pow()),
against the oracle: right-hand sides at the bar of the other right-hand-side
tests (1e-11 of the component scale), on both sides of every edge of the rule
(p, q and, with L = 0, p q), for each order and direction."""
import numpy as np
import pytest

import oracle as orc
from paper_2603_26272_amd import workloads as W

from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (L, p, q): powers 1 and 2 only, then one power beyond
SQUARE = [(1.0, 2.0, 1.0), (1.0, 1.0, 2.0), (0.5, 2.0, 2.0), (0.0, 2.0, 1.0), (0.0, 1.0, 2.0)]
BEYOND = [(1.0, 1.5, 1.0), (0.5, 1.0, 3.0), (0.0, 2.0, 2.0)]


@pytest.mark.parametrize("L,p,q", SQUARE + BEYOND)
@pytest.mark.parametrize("r", [2, 3, 5])
def test_rhs_against_oracle(L, p, q, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_26272_amd.za import Context
    for dim, data in ((1, W.riemann_1d(5, 129)), (2, W.quadrants_2d(7, 65, 33))):
        P, q0 = data
        # a ripple rules out exactly tied indicators (r = 2)
        x = np.arange(P.nx)[None, :] + 0.37 * np.arange(P.ny)[:, None]
        q0 = q0.copy()
        q0[0] *= 1 + 1e-3 * np.sin(x)
        P = P.with_(order=r, weight_L=L, p=p, weight_q=q)
        with Context(P) as ctx:
            got = ctx.rhs(torch.from_numpy(q0).cuda()).cpu().numpy()
        ref, st = orc.rhs(P, q0)
        assert st == 0
        assert_close(got, ref, 1e-11, f"dim={dim} r={r} L={L} p={p} q={q}")
