"""What the constant step's norm costs at session creation: not much more
than on the host, whichever side the automatic preparation takes, and the same
bits. Best of several creations; the bounds are a few milliseconds where
launches for nothing would take ten, and 0.7 where they would take 1.3. And
the same bits from the fewest entries that the device takes (2560) on, in one
row, in one column and at the ends of a group of 8 lanes and of a workgroup's
32 rows, with limits around the rounds after which it looks for the end, in
sessions, packed sets and the allocation-free solve."""

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


def test_small_lps_cost_no_more_than_on_the_host(P):
    for m, n in ((20, 45), (200, 300)):
        lp = random_lp((m, n), m, n, degree=("uniform", 3, 8), eq_frac=0.5)
        dev, host = _create(P, lp), _create(P, lp, prep=P.OPDHG_PREP_HOST)
        assert dev[1] == host[1]
        assert dev[0] < host[0] + 0.7, (m, n, dev, host)


@pytest.mark.parametrize("m,n,degree", [(1, 2560, 1), (7, 861, 3), (8, 857, 3), (9, 650, 4),
                                        (500, 8, 320), (5000, 1, 2600), (200, 33, 78), (31, 257, 10),
                                        (31, 257, 12), (600, 1100, 6)])
def test_device_norm_from_its_fewest_entries_on(P, m, n, degree):
    lp = random_lp((m, n), m, n, degree=("fixed", degree), eq_frac=0.5)
    assert lp.val.size >= 2560
    for rounds in (1, 8, 9, 24, 25, 200):
        got = []
        for prep in (P.OPDHG_PREP_AUTO, P.OPDHG_PREP_HOST):
            with P.Session(lp, P.opdhg_vanilla_params(0.0, power_iters=rounds, prep=prep)) as s:
                got.append(s.state()[4].eta)
        assert got[0] == got[1], rounds


def test_packed_and_allocation_free_solves(P):
    # the allocation-free solve has no pinned memory to see the end in
    lps = [random_lp((3, k), 300, 500, degree=("uniform", 3, 8), eq_frac=0.5) for k in range(3)]
    lps += [_permutation_lp(2000)]
    for rounds in (1, 8, 9, 24, 25, 56, 57, 1000):
        p = P.opdhg_vanilla_params(1e-2, tol=0.0, max_iter=20, power_iters=rounds)
        solo = [P.opdhg_solve(lp, P.opdhg_vanilla_params(1e-2, tol=0.0, max_iter=20, power_iters=rounds,
                                                         prep=P.OPDHG_PREP_HOST)) for lp in lps]
        for got in (P.opdhg_solve_batch(lps, p), [P.opdhg_solve_noalloc(lp, p) for lp in lps]):
            for a, b in zip(got, solo):
                assert a[2].eta == b[2].eta, rounds
                assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
