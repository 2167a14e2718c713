"""FP64 partial sums per workgroup and LP, at the chunkings where they can go
wrong: chunks of more than one window of 32 work items, several LPs in one
chunk, an LP spread over several chunks, and one tile per chunk.

Every FP64 sum is a double-double rounded once, so the chunking changes no
bit of a result: solves and packed sets are compared with the one-LP solve
of the default chunking bit for bit, and that solve with the oracle.
"""

import numpy as np
import pytest

import oracle
from oracle.params import default_params
from lpgen import config_lp
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


OP = dict(max_iter=1500, lr=1e-2, phi=5)


@pytest.fixture(scope="module")
def solved(P):
    lps = [config_lp("cfg0", seed=0), config_lp("cfg3", index=0, scale=0.1),
           config_lp("cfg1", scale=0.02), config_lp("cfg0", seed=1)]
    op = default_params(**OP)
    got = [P.opdhg_solve(lp, lib_params(P, op)) for lp in lps]
    for i, lp in enumerate(lps):
        check_final_fp64(got[i], oracle.solve(lp, op), label=f"LP {i}")
    return lps, got


def _same(a, b):
    assert a[2].status == b[2].status and a[2].attempts == b[2].attempts
    assert a[2].rel_kkt == b[2].rel_kkt and a[2].eta == b[2].eta
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("tile,wg", [(64, 1), (64, 3), (64, 40), (256, 8), (16, 2), (0, 2048)])
def test_chunking_changes_no_bit(P, solved, tile, wg):
    lps, ref = solved
    p = lib_params(P, default_params(**OP), tile_nnz=tile, workgroups=wg,
                   windows=P.OPDHG_WINDOWS_OFF)
    for lp, r in zip(lps, ref):
        _same(P.opdhg_solve(lp, p), r)
    for got, r in zip(P.opdhg_solve_batch(lps, p), ref):
        _same(got, r)
