"""What the constant step's norm costs at session creation: not much more
than on the host, whichever side the automatic preparation takes, and the same
bits. Best of several creations; the bounds are a few milliseconds where
launches for nothing would take ten."""

import time

import numpy as np
import pytest

from lpgen import random_lp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_17650_amd as P
    P.load()
    return P


def _permutation_lp(n):
    lp = random_lp(2, n, n, degree=("fixed", 1))
    lp.row_ptr = np.arange(n + 1, dtype=np.int64)
    lp.col_idx = np.random.default_rng(2).permutation(n).astype(np.int32)
    lp.val = np.ones(n)
    return lp


def _create(P, lp, **kw):
    """Shortest creation of eight, in milliseconds, and the step size."""
    p = P.opdhg_vanilla_params(0.0, power_iters=1000, **kw)
    best, eta = np.inf, None
    for _ in range(8):
        t = time.perf_counter()
        with P.Session(lp, p) as s:
            best = min(best, time.perf_counter() - t)
            eta = s.state()[4].eta
    return best * 1e3, eta


def test_rounds_end_where_the_norm_has_converged(P):
    # a scaled permutation: converged after two rounds of a thousand
    lp = _permutation_lp(13000)
    dev, host = _create(P, lp), _create(P, lp, prep=P.OPDHG_PREP_HOST)
    assert dev[1] == host[1]
    assert dev[0] < host[0] + 4.0, (dev, host)
