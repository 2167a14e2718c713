"""Session reads on both sides of the size where they go through pinned
staging in pieces, with row classes that move rows (so the caller's order is
not the device's): x, y, T and Sigma equal the vectors read one at a time,
and the unscaled x and y equal the scaled ones times the diagonals, bit for
bit. At 1e-30 tolerance the sessions are paused, not finished."""

import ctypes

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


# bytes of x, y, T and Sigma: 16 MiB - 16 (no staging), 16 MiB, ragged 16.8 and
# 17.3 MB (the last piece of each vector short)
@pytest.mark.parametrize("m,n,prec", [(524287, 524288, "fp64"), (524288, 524288, "fp64"),
                                      (700001, 1400007, "fp32"), (500007, 580003, "fp64")])
def test_reads_in_pieces(P, m, n, prec):
    lp = random_lp((5, m), m, n, degree=("powerlaw", 2.2, 1, 400), bounds=("box", 0.0, 10.0))
    p = P.opdhg_default_params(precision=P.OPDHG_FP32 if prec == "fp32" else P.OPDHG_FP64,
                               tol=1e-30, lr=1e-2, phi=1, prep=P.OPDHG_PREP_HOST)
    _, dr, dc = P.opdhg_rescale(lp, p)
    with P.Session(lp, p) as s:
        s.run(3)
        x, y, T, S, st = s.state()
        assert st.k == 3 and np.any(x != 0) and np.any(T != 1.0)
        lib = P.load()
        for k, v in enumerate((x, y, T, S)):  # one vector at a time
            one = np.full(v.size, np.nan)
            args = [None] * 4
            args[k] = one.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
            assert lib.opdhg_session_state(s._h, *args, None) == 0
            assert np.array_equal(one, v)
        xr, yr, res = s.result()
        assert res.iterations == 3
        assert np.array_equal(xr, x * dc) and np.array_equal(yr, y * dr)
    # the same LP stepped again reads the same bits
    with P.Session(lp, p) as s:
        s.run(3)
        again = s.state()
        assert all(np.array_equal(a, b) for a, b in zip(again[:4], (x, y, T, S)))
