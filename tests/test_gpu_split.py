"""Calls whose K x K blocks do not fit in the last-level cache deal the parts
of a 3D tile to different workgroups; smaller calls give a tile to one.  Both
sides of that bound, ragged, for every combination of outputs, against the
oracle (a stretch at the start, one across two spans of tiles and the tail)
and against the same points evaluated by smaller calls; padding is left
alone."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import DTYPES, GAMMA, host, require_gpu, states
from metrics import TOL, blocks_error, flux_groups, group_error, riemann_groups
from paper_1809_09851_amd import fdbb as F

pytestmark = pytest.mark.gpu

BOUND = 256 << 20
SPAN = 131072
GUARD = -3.0


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def guarded(t):
    t._base.fill_(GUARD)
    return t


def padding_intact(t, n):
    base = t._base
    return bool((base[:, n:] == GUARD).all())


def stretches(n):
    return [slice(0, 700), slice(SPAN - 300, SPAN + 300), slice(n - 1031, n)]


@pytest.mark.parametrize("past", (False, True))
@pytest.mark.parametrize("dt", ("f64", "f32"))
def test_fused_parts(dt, past):
    es = 8 if dt == "f64" else 4
    n = BOUND // (75 * es) + (1 if past else 0)
    Uo, U = states(3, n, 5, dt)
    m = n // 3 + 1
    Fp, Ap, Rp = zip(*[F.euler_fused(U[:, a:a + m], GAMMA) for a in range(0, n, m)])
    pieces = torch.cat(Fp, 1), torch.cat(Ap, 1), torch.cat(Rp, 1)
    for want in ((1, 1, 1), (1, 1, 0), (0, 1, 1), (0, 1, 0), (1, 0, 1)):
        Fg = guarded(F.empty_fields(15, n, DTYPES[dt])) if want[0] else None
        A = guarded(F.empty_blocks(3, n, DTYPES[dt])) if want[1] else None
        R = guarded(F.empty_fields(7, n, DTYPES[dt])) if want[2] else None
        F.fdbb_euler_fused(3, GAMMA, U, Fg, A, R)
        for got, whole in zip((Fg, A, R), pieces):
            if got is None:
                continue
            assert padding_intact(got, n)
            # the order of contracted operations may differ between the two
            scale = whole.abs().amax().item()
            assert float((got.double() - whole.double()).abs().amax()) <= TOL[dt] * scale
        for s in stretches(n):
            Fo, Ao, Ro = oracle.fused(3, GAMMA, np.ascontiguousarray(Uo[:, s]))
            if Fg is not None:
                assert group_error(host(Fg[:, s]), Fo, flux_groups(3)) <= TOL[dt]
            if A is not None:
                assert blocks_error(host(A[:, s]), Ao) <= TOL[dt]
            if R is not None:
                assert group_error(host(R[:, s]), Ro, riemann_groups(3)) <= TOL[dt]
    A = guarded(F.empty_blocks(3, n, DTYPES[dt]))
    F.fdbb_flux_jacobian(3, GAMMA, U, A)
    assert padding_intact(A, n)
    for s in stretches(n):
        assert blocks_error(host(A[:, s]), oracle.flux_jacobian(3, GAMMA, np.ascontiguousarray(Uo[:, s]))) <= TOL[dt]


@pytest.mark.parametrize("past", (False, True))
@pytest.mark.parametrize("dt", ("f64", "f32"))
def test_eigenvector_parts(dt, past):
    es = 8 if dt == "f64" else 4
    n = BOUND // (150 * es) + (1 if past else 0)
    Uo, U = states(3, n, 6, dt)
    for left, right in ((1, 1), (1, 0), (0, 1)):
        L = guarded(F.empty_blocks(3, n, DTYPES[dt])) if left else None
        R = guarded(F.empty_blocks(3, n, DTYPES[dt])) if right else None
        F.fdbb_eigenvectors(3, GAMMA, U, L, R)
        for s in stretches(n):
            Lo, Ro = oracle.eigenvectors(3, GAMMA, np.ascontiguousarray(Uo[:, s]))
            if L is not None:
                assert blocks_error(host(L[:, s]), Lo) <= TOL[dt]
            if R is not None:
                assert blocks_error(host(R[:, s]), Ro) <= TOL[dt]
        for t in (L, R):
            assert t is None or padding_intact(t, n)
