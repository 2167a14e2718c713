"""Where a session's reads through pinned staging put each coordinate, against
reads that do not go through it: the result of a solve equals the packed
solve's of the same LP (which reads one vector at a time), and an LP with its
rows and columns in another order, whose rows have other places on the
device, gives the same x, y, T and Sigma in that order (FP64 sums do not
depend on the order), bit for bit."""

import copy

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


def _lp(m, n):
    return random_lp((6, m), m, n, degree=("powerlaw", 2.2, 1, 400), bounds=("box", 0.0, 10.0))


def _staged(m, n, bytes_):
    """x, y, T and Sigma take 16 MiB or more: they are read in pieces."""
    return 2 * bytes_ * (m + n) >= 16 << 20


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_results_equal_the_packed_solve(P, prec):
    m, n = (500007, 580003) if prec == "fp64" else (700001, 1400007)
    assert _staged(m, n, 8 if prec == "fp64" else 4)
    lp = _lp(m, n)
    p = P.opdhg_default_params(precision=P.OPDHG_FP32 if prec == "fp32" else P.OPDHG_FP64,
                               tol=0.0, max_iter=3, lr=1e-2, phi=1)
    x, y, res = P.opdhg_solve(lp, p)
    want = P.opdhg_solve_batch([lp], p)[0]
    assert res.iterations == want[2].iterations == 3 and np.any(x != 0) and np.any(y != 0)
    assert np.array_equal(x, want[0]) and np.array_equal(y, want[1])


def test_another_order_of_rows_and_columns(P):
    m, n = 500007, 580003
    assert _staged(m, n, 8)
    lp = _lp(m, n)
    r = np.random.default_rng(3)
    rows, cols = r.permutation(m), r.permutation(n)  # new row i is old row rows[i]
    other = copy.copy(lp)
    lens = np.diff(lp.row_ptr)[rows]
    other.row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    at = np.repeat(lp.row_ptr[rows] - other.row_ptr[:-1], lens) + np.arange(lp.val.size)
    place = np.empty(n, np.int64)
    place[cols] = np.arange(n)
    other.col_idx, other.val = place[lp.col_idx[at]].astype(np.int32), lp.val[at]
    other.b, other.sense = lp.b[rows], lp.sense[rows]
    other.c, other.l, other.u = lp.c[cols], lp.l[cols], lp.u[cols]
    p = P.opdhg_default_params(tol=0.0, lr=1e-2, phi=1)
    got = []
    for one in (lp, other):
        with P.Session(one, p) as s:
            s.run(3)
            got.append(s.state())
    assert np.any(got[0][2] != 1.0) and np.any(got[0][3] != 1.0)
    for a, b, order in zip(got[0][:4], got[1][:4], (cols, rows, cols, rows)):
        assert np.array_equal(a[order], b)
