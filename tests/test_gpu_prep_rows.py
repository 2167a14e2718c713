"""The device preparation's row statistics, eight lanes a row and a wave for
rows above 256 entries, against the host's, bit for bit: rows of 0 to 600
entries on either side, sizes at the ends of a lane group, of a workgroup's 32
rows, and an LP of one row or column."""

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


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("l2,beta", [(0, 1.0), (1, 0.5), (1, -1.0)])
@pytest.mark.parametrize("m,n,degree", [
    (1, 1, ("fixed", 1)), (1, 700, ("fixed", 1)), (700, 1, ("fixed", 650)),
    (31, 33, ("powerlaw", 1.2, 1, 31)), (700, 257, ("powerlaw", 0.8, 1, 600)),
    (40, 3000, ("uniform", 1, 17)), (900, 2049, ("uniform", 7, 9))])
def test_row_statistics(P, m, n, degree, l2, beta, precision):
    lp = random_lp((m, n, 5), m, n, degree=degree, eq_frac=0.5)
    if m > 30:  # rows without entries
        keep = np.ones(lp.col_idx.size, bool)
        counts = np.diff(lp.row_ptr)
        for i in (0, m // 2, m - 1):
            keep[lp.row_ptr[i]:lp.row_ptr[i + 1]] = False
            counts[i] = 0
        lp.row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        lp.col_idx, lp.val = lp.col_idx[keep], lp.val[keep]
    got = []
    for prep in (P.OPDHG_PREP_DEVICE, P.OPDHG_PREP_HOST):
        p = P.opdhg_default_params(prep=prep, l2_rescale=l2, pc_beta=beta, tol=0.0, lr=1e-3,
                                   windows=P.OPDHG_WINDOWS_OFF,
                                   precision=P.OPDHG_FP32 if precision == "fp32" else P.OPDHG_FP64)
        with P.Session(lp, p) as s:
            start = s.state()
            s.run(20)
            got.append((start, s.state()))
    if beta == 0.5:  # pow on the two sides may differ in the last bits: the first step only
        a, b = got[0][0][4], got[1][0][4]
        assert abs(a.eta - b.eta) <= 1e-13 * b.eta and abs(a.omega - b.omega) <= 1e-13 * b.omega
        return
    for a, b in zip(got[0], got[1]):
        assert a[4].eta == b[4].eta and a[4].omega == b[4].omega
        for u, v in zip(a[:4], b[:4]):
            assert np.array_equal(u, v)
