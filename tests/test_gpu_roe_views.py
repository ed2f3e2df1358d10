"""The Roe average of two near views of one state (a grid's faces) loads
otherwise than that of unrelated sides: both against the oracle and against
each other, over shifts either way, tile remainders, points per thread and
batch tasks; padding is left alone."""
import pytest
import torch

import oracle
from gpu_common import DTYPES, GAMMA, host, require_gpu, states
from metrics import TOL, group_error, roe_error, state_groups
from paper_1809_09851_amd import batch as B
from paper_1809_09851_amd import fdbb as F

pytestmark = pytest.mark.gpu

GUARD = -3.0
SAME = {"f64": 1e-14, "f32": 1.2e-7}  # contractions may differ between the two paths


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("ppt", (1, 2, 4))
@pytest.mark.parametrize("dim,dt", [(d, t) for d in (1, 2, 3) for t in ("f64", "f32")])
def test_near_views(dim, dt, ppt):
    K = dim + 2
    Uo, U = states(dim, 3000, 11, dt)
    op, code = F.OPS["roe_average"], F.dtype_code(DTYPES[dt])
    block, p0, cap, nt = F.fdbb_get_launch_config(op, dim, code)
    small = F.fdbb_get_small_launch_config(op, dim, code)
    F.fdbb_set_launch_config(op, dim, code, 128, ppt)
    F.fdbb_set_small_launch_config(op, dim, code, 0)
    try:
        for n, l, r in ((1, 0, 1), (64, 5, 4), (129, 0, 0), (1025, 3, 0), (2047, 0, 953), (2049, 300, 0), (1500, 0, 1500)):
            UL, UR = U[:, l:l + n], U[:, r:r + n]
            Uh = F.empty_fields(K, n, DTYPES[dt])
            Uh._base.fill_(GUARD)
            F.fdbb_roe_average(dim, GAMMA, UL, UR, Uh)
            assert bool((Uh._base[:, n:] == GUARD).all())
            apart = F.roe_average(F.to_fields(UL.clone()), F.to_fields(UR.clone()), GAMMA)
            batched = F.empty_fields(K, n, DTYPES[dt])
            B.run_noalloc([B.roe_task(UL, UR, batched, GAMMA)], block=64, ppt=ppt)
            want = oracle.roe_average(dim, GAMMA, Uo[:, l:l + n], Uo[:, r:r + n])
            for got in (Uh, apart, batched):
                assert roe_error(host(got), want, Uo[:, l:l + n], Uo[:, r:r + n]) <= TOL[dt]
                assert group_error(host(got), host(Uh), state_groups(dim)) <= SAME[dt]
    finally:
        F.fdbb_set_launch_config(op, dim, code, block, p0, cap, nt)
        if small[0]:
            F.fdbb_set_small_launch_config(op, dim, code, *small)
