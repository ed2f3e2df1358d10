"""Output rows that start inside cache lines change the launch of large
pointwise calls: both sides of the bound, packed and offset rows, against the
same call on padded rows (whose results the other tests hold against the
oracle); what lies around the output is left alone."""
import pytest
import torch

from gpu_common import DTYPES, GAMMA, require_gpu, states
from paper_1809_09851_amd import fdbb as F

pytestmark = pytest.mark.gpu

BOUND = 1 << 19
GUARD = -3.0
SAME = {"f64": 1e-14, "f32": 1.2e-7}  # contractions may differ between store variants


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def calls(dim, U, W, X):
    """(rows written, call) of every op whose launch can change."""
    K = dim + 2
    G, gradT = X[:dim * dim], X[:dim]
    yield K * dim, lambda o: F.fdbb_flux(dim, GAMMA, U, o)
    yield K, lambda o: F.fdbb_flux_direction(dim, dim - 1, GAMMA, U, o)
    yield 2 * dim + 1, lambda o: F.fdbb_riemann_invariants(dim, GAMMA, U, o)
    yield K, lambda o: F.fdbb_flux_adjoint(dim, -1, GAMMA, U, X, o)
    yield K, lambda o: F.fdbb_char_apply(dim, 0, 0, GAMMA, U, W, o)
    yield K, lambda o: F.fdbb_roe_average(dim, GAMMA, U, U.flip(1).contiguous(), o)
    yield K * dim, lambda o: F.fdbb_viscous_flux(dim, 0.1, 0.2, U, G, gradT, o)
    yield K, lambda o: F.fdbb_cons2char(dim, 0, GAMMA, U, o)
    yield K, lambda o: F.fdbb_char2cons(dim, 0, GAMMA, W, o)


@pytest.mark.parametrize("n", (BOUND - 1, BOUND, BOUND + 3))
@pytest.mark.parametrize("dim,dt", [(d, t) for d in (1, 2, 3) for t in ("f64", "f32")])
def test_ragged_rows(dim, dt, n):
    K, dtype = dim + 2, DTYPES[dt]
    _, U = states(dim, n, 3, dt)
    W = F.cons2char(U, 0, GAMMA)
    X = F.to_fields(torch.linspace(-1.0, 1.0, K * dim * n, dtype=torch.float64, device="cuda").view(K * dim, n).to(dtype))
    for rows, call in calls(dim, U, W, X):
        want = F.empty_fields(rows, n, dtype)
        call(want)
        for ld in (n, n + 7, F.padded_ld(n)):
            for start in (0, 5) if ld > n else (3,):
                base = torch.full((rows * ld + start + 64,), GUARD, dtype=dtype, device="cuda")
                got = torch.as_strided(base, (rows, n), (ld, 1), start)
                call(got)
                err = ((got.double() - want.double()).abs().amax(0) / want.double().abs().amax(0)).max()
                assert float(err) <= SAME[dt]
                got.fill_(GUARD)
                assert bool((base == GUARD).all())
