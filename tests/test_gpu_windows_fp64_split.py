"""FP64 windows beside rows above 16384 entries, which are split in pieces with
a partial slot each, against the tiles, bit for bit: chunks as small as fit
the slots and smaller (the side then stays in tiles), default lanes."""

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


def _split_lp(seed, longs, shorts, k, n):
    """`longs` rows of 20000 entries before `shorts` rows of k."""
    r = np.random.default_rng(seed)
    rows = [np.sort(r.choice(n, 20000, replace=False)) for _ in range(longs)]
    rows += [np.sort(r.choice(n, k, replace=False)) for _ in range(shorts)]
    lp = random_lp(seed, len(rows), n, degree=("fixed", 1))
    lp.row_ptr = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int64)
    lp.col_idx = np.concatenate(rows).astype(np.int32)
    lp.val = r.standard_normal(lp.col_idx.size)
    return lp


# sides: those in windows
@pytest.mark.parametrize("longs,shorts,k,n,rows,sides", [
    (10, 2000, 4, 20000, 64, ""), (10, 2000, 4, 20000, 256, "TA"), (1, 3000, 18, 20011, 55, ""),
    (1, 3000, 18, 20011, 64, "A"), (2, 9000, 18, 30001, 0, "TA")])
def test_windows_equal_tiles(P, longs, shorts, k, n, rows, sides):
    lp = _split_lp((longs, rows), longs, shorts, k, n)
    kw = dict(prep=P.OPDHG_PREP_DEVICE, tol=0.0, lr=1e-2, phi=3)
    got = []
    for extra in (dict(windows=P.OPDHG_WINDOWS_ALWAYS, window_rows=rows),
                  dict(windows=P.OPDHG_WINDOWS_OFF)):
        with P.Session(lp, P.opdhg_default_params(**kw, **extra)) as s:
            if not got:
                r = s.route()
                assert ("T" in sides) == (r.chunks_t > 0) and ("A" in sides) == (r.chunks_a > 0)
            s.run(150)
            got.append(s.state())
    for a, b in zip(got[0][:4], got[1][:4]):
        assert np.array_equal(a, b)
    assert got[0][4].eta == got[1][4].eta and got[0][4].attempts == got[1][4].attempts
