"""3D FP32 calls and lists on both sides of 512 MiB of blocks, where tiles
dealt apart give way to whole tiles with few waves resident: stretches of the
outputs against the oracle, padding left alone."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import GAMMA, host, require_gpu, states
from metrics import TOL, blocks_error, flux_groups, group_error, riemann_groups
from paper_1809_09851_amd import batch as B
from paper_1809_09851_amd import fdbb as F
from test_gpu_split import guarded, padding_intact, stretches

pytestmark = pytest.mark.gpu

AT = (512 << 20) // (75 * 4)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def outputs(n):
    f32 = torch.float32
    return guarded(F.empty_fields(15, n, f32)), guarded(F.empty_blocks(3, n, f32)), guarded(F.empty_fields(7, n, f32))


def check(Uo, n, out):
    for o in out:
        assert padding_intact(o, n)
    Fg, A, R = out
    for s in stretches(n):
        Fo, Ao, Ro = oracle.fused(3, GAMMA, np.ascontiguousarray(Uo[:, s]))
        assert group_error(host(Fg[:, s]), Fo, flux_groups(3)) <= TOL["f32"]
        assert blocks_error(host(A[:, s]), Ao) <= TOL["f32"]
        assert group_error(host(R[:, s]), Ro, riemann_groups(3)) <= TOL["f32"]


@pytest.mark.parametrize("n", (AT, AT + 1))
def test_single_calls(n):
    Uo, U = states(3, n, 8, "f32")
    out = outputs(n)
    F.fdbb_euler_fused(3, GAMMA, U, *out)
    check(Uo, n, out)
    A = guarded(F.empty_blocks(3, n, torch.float32))
    F.fdbb_flux_jacobian(3, GAMMA, U, A)
    assert padding_intact(A, n)
    for s in stretches(n):
        assert blocks_error(host(A[:, s]), oracle.flux_jacobian(3, GAMMA, np.ascontiguousarray(Uo[:, s]))) <= TOL["f32"]


@pytest.mark.parametrize("extra", (0, 1))
def test_lists(extra):
    sizes = [AT // 3 + 7, AT // 3 - 7]
    sizes.append(AT - sum(sizes) + extra)
    blocks = []
    for i, n in enumerate(sizes):
        Uo, U = states(3, n, 9 + i, "f32")
        out = outputs(n)
        blocks.append((Uo, n, out, B.fused_task(U, *out, gamma=GAMMA), U))
    plan = B.Plan([b[3] for b in blocks])
    for graph in (True, False):
        for b in blocks:
            for o in b[2]:
                guarded(o)
        plan.run(graph=graph)
        torch.cuda.synchronize()
        for b in blocks:
            check(*b[:3])
    plan.close()
