"""Which kernels run a session's attempts (opdhg_session_route), so that
comparisons of windows with tiles compare what they say: which sides of the
FP64 window tests' LPs are in windows, in several passes and with segments,
and which are meant to stay in tiles (too few partial slots beside the tiles'
or too little room for the plan, more than eight passes, no short rows). With
default lanes the windows are compared with the tiles here, bit for bit."""

import numpy as np
import pytest

from lpgen import block_angular_lp, config_lp
from test_gpu_windows_fp64 import LPS

pytestmark = pytest.mark.gpu

SETTINGS = [(0, 0), (64, 0), (1000, 2), (8192, 1), (320, 2)]  # window_rows, window_buckets
# sides in tiles, by lanes and LP: every setting's, or those of these window_rows
TILES = {
    64: {"two_classes": ("", [], [64]), "band": ("", [64], [8192]), "block": ("", [], [8192]),
         "block_3": ("", [], [64, 8192]), "odd": ("", [], [64, 8192]),
         "one_over": ("", [64], [64, 8192]), "even": ("", [], []), "dense": ("TA", [], []),
         "empty": ("", [64], [])},
    0: {"two_classes": ("T", [], [64]), "band": ("", [64, 320], [64, 8192]),
        "block": ("", [64], [64, 8192]), "block_3": ("", [64], [64, 8192]),
        "odd": ("", [64], [8192]), "one_over": ("", [64], [64, 8192]), "even": ("T", [], []),
        "dense": ("TA", [], []), "empty": ("", [64], [64])},
}


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_17650_amd as P
    P.load()
    return P


def _params(P, lanes, rows, buckets, windows):
    return P.opdhg_default_params(prep=P.OPDHG_PREP_DEVICE, lanes=lanes, tol=0.0, lr=1e-2, phi=3,
                                  window_rows=rows, window_buckets=buckets, windows=windows)


@pytest.mark.parametrize("name", list(LPS))
@pytest.mark.parametrize("lanes", [64, 0])
def test_windows_run_where_they_are_meant_to(P, name, lanes):
    lp = LPS[name]()
    whole, rows_t, rows_a = TILES[lanes][name]
    if lanes == 0:
        with P.Session(lp, _params(P, 0, 0, 0, P.OPDHG_WINDOWS_OFF)) as s:
            s.run(100)
            off = s.state()
    most = [0, 0]
    for rows, buckets in SETTINGS:
        with P.Session(lp, _params(P, lanes, rows, buckets, P.OPDHG_WINDOWS_ALWAYS)) as s:
            r = s.route()
            if lanes == 0 and (r.chunks_t or r.chunks_a):
                s.run(100)
                for a, b in zip(s.state()[:4], off[:4]):
                    assert np.array_equal(a, b), (rows, buckets)
        assert not r.one_workgroup
        assert (r.chunks_t == 0) == ("T" in whole or rows in rows_t), (rows, buckets)
        assert (r.chunks_a == 0) == ("A" in whole or rows in rows_a), (rows, buckets)
        if buckets:
            most = [max(most[0], r.passes_t), max(most[1], r.passes_a)]
        else:  # the whole LDS holds what these chunks gather from
            assert r.passes_t <= 1 and r.passes_a <= 1
        # long and medium rows: in segments, but where their columns do not ascend
        if r.chunks_a:
            assert (r.segments_a > 0) == (name in ("block", "block_3", "odd", "even"))
        if r.chunks_t:
            assert (r.segments_t > 0) == (name == "two_classes")
    if "T" not in whole:
        assert most[0] > 1
    if "A" not in whole and name != "band":
        assert most[1] > 1


def test_small_lps_and_fp32(P):
    small = config_lp("cfg0", seed=0)
    for windows, one in ((P.OPDHG_WINDOWS_AUTO, 1), (P.OPDHG_WINDOWS_ALWAYS, 1),
                         (P.OPDHG_WINDOWS_OFF, 0)):
        with P.Session(small, P.opdhg_default_params(windows=windows)) as s:
            r = s.route()
            assert r.one_workgroup == one and r.chunks_t == r.chunks_a == 0
    lp = block_angular_lp(7, blocks=6, block_rows=3000, block_cols=8000, col_degree=6,
                          link_rows=40, link_nnz_per_row=600)
    for windows, on in ((P.OPDHG_WINDOWS_ALWAYS, True), (P.OPDHG_WINDOWS_OFF, False)):
        with P.Session(lp, P.opdhg_default_params(precision=P.OPDHG_FP32, windows=windows)) as s:
            r = s.route()
            assert (r.chunks_a > 0) == (r.passes_a > 0) == on
            assert not r.one_workgroup
