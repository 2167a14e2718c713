"""FP64 windows against the tiles, bit for bit (double-double sums do not
depend on the order): chunks of one slice of 64 rows up to several, a last
chunk and a last slice that are not full, one to eight passes, a last bucket
that ends early (odd and even widths, a single column of it), sides without
short rows, rows without entries, long and medium rows beside the windows:
as segments, or in tiles where their columns do not ascend (blocks with
columns of two classes); a band, where rows may be cut anywhere."""

import numpy as np
import pytest

from lpgen import block_angular_lp, random_lp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_17650_amd as P
    P.load()
    return P


def _empty_rows(lp, rows):
    keep = np.ones(lp.col_idx.size, bool)
    for i in rows:
        keep[lp.row_ptr[i]:lp.row_ptr[i + 1]] = False
    counts = np.diff(lp.row_ptr)
    counts[rows] = 0
    lp.row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    lp.col_idx, lp.val = lp.col_idx[keep], lp.val[keep]
    return lp


def _from_rows(seed, n, rows):
    """A random LP's data around rows of the given columns."""
    r = np.random.default_rng(seed)
    lp = random_lp(seed, len(rows), n, degree=("fixed", 1))
    lp.row_ptr = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int64)
    lp.col_idx = np.concatenate(rows).astype(np.int32)
    lp.val = r.standard_normal(lp.col_idx.size)
    return lp


def _two_classes():
    r = np.random.default_rng(11)
    rows = [[] for _ in range(4 * 700)]
    for j in range(4 * 1500):
        b = j // 1500
        for i in r.choice(700, 40 if j % 30 == 0 else 5, replace=False):
            rows[b * 700 + i].append(j)
    rows += [np.sort(r.choice(6000, 420, replace=False)) for _ in range(6)]
    return _from_rows(11, 6000, rows)


LPS = {
    "two_classes": _two_classes,
    "band": lambda: _from_rows(12, 9005, [np.arange(2 * i, 2 * i + 1 + i % 14) for i in range(4490)]),
    "block": lambda: block_angular_lp(3, blocks=9, block_rows=411, block_cols=1097, col_degree=6,
                                      link_rows=20, link_nnz_per_row=500),
    "block_3": lambda: block_angular_lp(9, blocks=3, block_rows=1200, block_cols=3001, col_degree=5,
                                        link_rows=14, link_nnz_per_row=600),
    "odd": lambda: random_lp(4, 3001, 9729, degree=("uniform", 3, 8), eq_frac=0.5),
    "one_over": lambda: random_lp(5, 4097, 9217, degree=("uniform", 1, 4), eq_frac=0.5),
    "even": lambda: random_lp(6, 5000, 7170, degree=("powerlaw", 1.6, 1, 600), eq_frac=0.5),
    "dense": lambda: random_lp(7, 600, 9000, degree=("fixed", 40), eq_frac=0.5),
    "empty": lambda: _empty_rows(random_lp(8, 3000, 8001, degree=("fixed", 5)),
                                 np.r_[0:200, 1500:1503, 2990:3000]),
}


@pytest.mark.parametrize("rows,buckets", [(0, 0), (64, 0), (1000, 2), (8192, 1), (320, 2)])
@pytest.mark.parametrize("name", list(LPS))
def test_windows_equal_tiles(P, name, rows, buckets):
    lp = LPS[name]()
    kw = dict(prep=P.OPDHG_PREP_DEVICE, lanes=64, tol=0.0, lr=1e-2, phi=3)
    got = []
    for extra in (dict(windows=P.OPDHG_WINDOWS_ALWAYS, window_rows=rows, window_buckets=buckets),
                  dict(windows=P.OPDHG_WINDOWS_OFF)):
        with P.Session(lp, P.opdhg_default_params(**kw, **extra)) as s:
            s.run(150)
            got.append(s.state())
    for a, b in zip(got[0][:4], got[1][:4]):
        assert np.array_equal(a, b)
    assert got[0][4].eta == got[1][4].eta and got[0][4].attempts == got[1][4].attempts


def test_direct_mode_and_preconditioned_norms(P):
    lp = LPS["block"]()
    kw = dict(prep=P.OPDHG_PREP_DEVICE, lanes=64, max_iter=200, tol=0.0, lr=1e-3,
              step_norm=P.OPDHG_STEP_NORM_PRECOND)
    on = P.opdhg_default_params(windows=P.OPDHG_WINDOWS_ALWAYS, window_rows=192, **kw)
    off = P.opdhg_default_params(windows=P.OPDHG_WINDOWS_OFF, **kw)
    a, b, c = P.opdhg_solve(lp, on), P.opdhg_solve(lp, off), P.opdhg_solve_noalloc(lp, on)
    for o in (b, c):
        assert np.array_equal(a[0], o[0]) and np.array_equal(a[1], o[1])
        assert a[2].rel_kkt == o[2].rel_kkt
