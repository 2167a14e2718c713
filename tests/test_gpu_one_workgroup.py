"""Small FP64 LPs whose attempts run in one workgroup (k_one), against the
step kernels (windows off: every row in tiles) bit for bit and against the
oracle: rows of every class on both sides, empty rows and columns, no rows at
all, one row or column, sizes at the ends of a slice of 64 rows, rejected
attempts, every schedule, the weighted and the constant step, packed sets,
workspaces without room for the packed entries, and pauses inside a launch
sequence."""

import numpy as np
import pytest

import oracle
from oracle.params import default_params, vanilla_params
from lpgen import block_angular_lp, config_lp, random_lp
from gpu_common import check_final_fp64, lib_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_17650_amd as P
    P.load()
    return P


def _mixed(m=520, n=260):
    """Columns of 1 to 285 entries (long, medium and short rows of A^T), 23
    empty rows of A."""
    return random_lp((3, m), m, n, degree=("powerlaw", 1.8, 1, 300), eq_frac=0.3,
                     bounds=("mix", 0.5, 0.3, 0.2, 1.0, 100.0))


def _linked(rows, nnz):
    """Linking rows: long or medium rows of A."""
    return block_angular_lp((4, rows), blocks=4, block_rows=60, block_cols=100, col_degree=2,
                            link_rows=rows, link_nnz_per_row=nnz)


LPS = {
    "cfg0": lambda: config_lp("cfg0", seed=2),
    "mixed": _mixed,
    "long rows": lambda: _linked(3, 300),
    "medium rows": lambda: _linked(7, 50),
    "one row": lambda: random_lp(5, 1, 40, degree=("fixed", 1)),
    "one column": lambda: random_lp(6, 7, 1, degree=("fixed", 3)),
    "64 x 128": lambda: random_lp(7, 64, 128, degree=("uniform", 1, 9)),
    "65 x 129": lambda: random_lp(8, 65, 129, degree=("uniform", 1, 9)),
    "1025 x 700": lambda: random_lp(9, 1025, 700, degree=("uniform", 2, 6)),
}
OPS = {
    "plain": dict(max_iter=700),
    "learner": dict(max_iter=700, lr=1e-2, phi=1),
    "norm schedule": dict(max_iter=300, lr=1e-2, phi=3, schedule=1),
    "constant rate": dict(max_iter=300, lr=1e-3, phi=2, schedule=2, normalize=False),
    "weighted": dict(max_iter=300, lr=1e-2, phi=4, step_norm=1),
    "eval 7": dict(max_iter=200, eval_every=7, lr=1e-2),
}


def _both(P, lp, op):
    one = P.opdhg_solve(lp, lib_params(P, op))
    off = P.opdhg_solve(lp, lib_params(P, op, windows=P.OPDHG_WINDOWS_OFF))
    return one, off


def _same(a, b):
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    for f in ("status", "which", "iterations", "attempts", "restarts", "rel_kkt", "eta", "omega"):
        x, y = getattr(a[2], f), getattr(b[2], f)
        assert x == y, (f, x, y)


def _packed(P, lp):
    """The workspace holds packed entries: the LP's attempts run in k_one."""
    return (P.opdhg_workspace_bytes(lp, P.opdhg_default_params()) >
            P.opdhg_workspace_bytes(lp, P.opdhg_default_params(windows=P.OPDHG_WINDOWS_OFF)))


@pytest.mark.parametrize("name", list(LPS))
@pytest.mark.parametrize("opn", list(OPS))
def test_equals_step_kernels(P, name, opn):
    lp, op = LPS[name](), default_params(**OPS[opn])
    assert _packed(P, lp)
    one, off = _both(P, lp, op)
    _same(one, off)
    if name in ("cfg0", "mixed"):
        check_final_fp64(one, oracle.solve(lp, op), label=f"{name} {opn}")


def test_constant_step_and_rejections(P):
    lp = _mixed(140, 150)
    assert _packed(P, lp)
    op = vanilla_params(lr=1e-1, max_iter=400)
    one, off = _both(P, lp, op)
    _same(one, off)
    check_final_fp64(one, oracle.solve(lp, op), label="vanilla")
    lp = config_lp("cfg1", scale=0.006)  # badly scaled rows: rejected attempts
    op = default_params(max_iter=1000, lr=1e-2)
    assert _packed(P, lp)
    one, off = _both(P, lp, op)
    assert one[2].attempts > one[2].iterations
    _same(one, off)


def test_no_rows(P):
    lp = random_lp(4, 3, 30, degree=("fixed", 1), bounds=("box", -1.0, 2.0))
    lp.m, lp.row_ptr = 0, np.zeros(1, dtype=np.int64)
    lp.col_idx, lp.val = lp.col_idx[:0], lp.val[:0]
    lp.b, lp.sense = lp.b[:0], lp.sense[:0]
    _same(*_both(P, lp, default_params(max_iter=300)))


def test_set_of_different_sizes_and_small_workspace(P):
    lps = [f() for f in LPS.values()]
    p = lib_params(P, default_params(max_iter=300, lr=1e-2))
    solo = [P.opdhg_solve(lp, p) for lp in lps]
    for got, ref in zip(P.opdhg_solve_batch(lps, p), solo):
        _same(got, ref)
    # workspaces sized for the step kernels alone are still accepted
    off = lib_params(P, default_params(max_iter=300, lr=1e-2), windows=P.OPDHG_WINDOWS_OFF)
    ws = P.capi.device_workspace(P.opdhg_workspace_bytes(lps[1], off))
    _same(P.opdhg_solve(lps[1], p, workspace=ws), solo[1])
    ws = P.capi.device_workspace(P.opdhg_batch_workspace_bytes(lps, off))
    for got, ref in zip(P.opdhg_solve_batch(lps, p, workspace=ws), solo):
        _same(got, ref)
    with pytest.raises(P.capi.OpdhgError):
        P.opdhg_solve(lps[1], p, workspace=ws[: P.opdhg_workspace_bytes(lps[1], off) - 4096])


@pytest.mark.parametrize("name", ["cfg0", "mixed"])
def test_pauses_inside_a_sequence(P, name):
    lp, op = LPS[name](), default_params(tol=0.0, max_iter=10**6, lr=1e-2, phi=5)
    ks = (1, 2, 63, 64, 65, 130, 200)
    with P.Session(lp, lib_params(P, op)) as a, \
            P.Session(lp, lib_params(P, op, windows=P.OPDHG_WINDOWS_OFF)) as b:
        for k in ks:
            a.run(k)
            b.run(k)
            sa, sb = a.state(), b.state()
            assert sa[4].k == sb[4].k == k and sa[4].attempts == sb[4].attempts
            assert sa[4].need_eval == sb[4].need_eval and sa[4].eta == sb[4].eta
            for u, v in zip(sa[:4], sb[:4]):
                assert np.array_equal(u, v)
        # a replay of the step kernels leaves slots idle before a guarded
        # evaluation, k_one's does not: compared at the same iteration
        a.replay(2)
        b.replay(2)
        a.run(512)
        b.run(512)
        sa, sb = a.state(), b.state()
        assert sa[4].attempts == sb[4].attempts and np.array_equal(sa[0], sb[0])
