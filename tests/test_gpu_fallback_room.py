"""The FP64 fallback of a small request takes what room the arena has: with a
request that never ends beside it and space for its slot, but not for the
packed entries that let it run in one workgroup, it runs at once (in tiles)
instead of waiting for memory that does not come free. With more room, and
with none beside it, the results are the same."""

import numpy as np
import pytest

from lpgen import config_lp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_17650_amd as P
    P.load()
    return P


@pytest.mark.parametrize("extra", [0, 1 << 20])
def test_fallback_runs_beside_a_full_arena(P, extra):
    def params(**kw):
        return P.opdhg_default_params(lr=1e-3, **kw)

    big, small = config_lp("cfg3", index=1, scale=0.05), config_lp("cfg0", seed=3)
    endless = params(precision=P.OPDHG_FP32, tol=0.0, max_iter=10**9, time_limit_s=1e9)
    short = params(precision=P.OPDHG_FP32, tol=0.0, max_iter=30)
    least = P.opdhg_workspace_bytes(small, params(windows=P.OPDHG_WINDOWS_OFF))
    need = P.opdhg_workspace_bytes(small, params())
    endless.windows = P.OPDHG_WINDOWS_OFF
    room = P.opdhg_workspace_bytes(big, endless) + 1024 + least
    assert room + 4096 < P.opdhg_workspace_bytes(big, endless) + need
    with P.Server(64 << 20, precision=P.OPDHG_FP32, fallback=P.OPDHG_FALLBACK_FP64,
                  budget_bytes=room + 1024 + extra) as srv:
        t_big = srv.submit(big, endless)
        t = srv.submit(small, short)
        x, y, r = srv.wait(t, 20.0)
        assert srv.precision(t) == P.OPDHG_FP64 and srv.stats().fallbacks == 1
        srv.cancel(t_big)
        with pytest.raises(P.OpdhgError) as e:
            srv.wait(t_big, 20.0)
        assert e.value.code == P.capi.OPDHG_ERR_CANCELLED
    want = P.opdhg_solve(small, params(tol=0.0, max_iter=30))
    assert np.array_equal(x, want[0]) and np.array_equal(y, want[1])
    assert r.rel_kkt == want[2].rel_kkt and r.iterations == 30
