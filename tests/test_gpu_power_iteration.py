"""The constant step's norm by kernels over the uploaded FP64 values (the
automatic preparation of small LPs) against the host's power iteration, bit
for bit: sizes at the ends of a group of 8 lanes, of a workgroup's 32 rows and
of the 256 workgroups, rows of 0 to 600 entries, an LP without entries, and
limits of one round."""

import numpy as np
import pytest

from oracle import pdhg as OP
from lpgen import random_lp
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_17650_amd as P
    P.load()
    return P


def _eta(P, lp, **kw):
    with P.Session(lp, P.opdhg_vanilla_params(1e-2, tol=0.0, **kw)) as s:
        eta = s.state()[4].eta
        s.run(5)
        x, y, _, _, st = s.state()
    assert st.eta == eta
    return eta, x, y


@pytest.mark.parametrize("m,n", [(1, 1), (7, 8), (9, 31), (40, 32), (33, 33), (300, 257),
                                 (130, 8193), (2000, 700)])
@pytest.mark.parametrize("rounds", [200, 1])
def test_device_norm_equals_host(P, m, n, rounds):
    lp = random_lp((m, n), m, n, degree=("powerlaw", 1.5, 1, 600), eq_frac=0.5)
    dev = _eta(P, lp, power_iters=rounds)
    host = _eta(P, lp, power_iters=rounds, prep=P.OPDHG_PREP_HOST)
    assert dev[0] == host[0]
    assert np.array_equal(dev[1], host[1]) and np.array_equal(dev[2], host[2])
    p = P.opdhg_vanilla_params(1e-2, power_iters=rounds)
    assert dev[0] == p.step_scale / P.opdhg_spectral_norm(lp, p)
    if m * n < 1000:
        slp = oracle.rescale(lp, p.ruiz_iters, p.pc_beta, True)
        assert dev[0] == p.step_scale / OP.spectral_norm_estimate(slp, rounds, p.power_tol)


def test_no_entries(P):
    lp = random_lp(1, 4, 9, degree=("fixed", 1))
    lp.row_ptr = np.zeros_like(lp.row_ptr)
    lp.col_idx, lp.val = lp.col_idx[:0], lp.val[:0]
    dev, host = _eta(P, lp), _eta(P, lp, prep=P.OPDHG_PREP_HOST)
    assert dev[0] == host[0] == P.opdhg_vanilla_params(0.0).step_scale
    assert np.array_equal(dev[1], host[1])
