"""Batch lists whose tasks all write K x K blocks of one dim and storage type
have a kernel of their own; other lists take the general one.  Both against
the oracle, over tile edges, empty and one-point tasks, output combinations,
shapes and store modes, and as a plan's list changes from one kind to the
other between launches, replays and captures; padding is left alone."""
import pytest
import torch

import oracle
from gpu_common import DTYPES, GAMMA, host, require_gpu, states
from metrics import TOL, blocks_error, flux_groups, group_error, riemann_groups
from paper_1809_09851_amd import batch as B
from paper_1809_09851_amd import fdbb as F

pytestmark = pytest.mark.gpu

GUARD = -3.0
EDGES = (1, 255, 0, 256, 257, 511, 64, 1025, 63, 2049)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


class Block:
    """One task's input, outputs and expected values; `want` as (F, A, R)."""

    def __init__(self, dim, dt, n, seed, want, jacobian=False):
        K = dim + 2
        self.dim, self.dt, self.n, self.want = dim, dt, n, want
        if n:
            self.Uo, U = states(dim, n, seed, dt)
        else:
            U = torch.zeros(K, 0, dtype=DTYPES[dt], device="cuda")
        self.U = U
        make = (lambda: F.empty_fields(K * dim, n, DTYPES[dt]), lambda: F.empty_blocks(dim, n, DTYPES[dt]),
                lambda: F.empty_fields(2 * dim + 1, n, DTYPES[dt]))
        self.out = [m() if w else None for m, w in zip(make, want)]
        self.clear()
        if jacobian:
            self.task = B.jacobian_task(U, self.out[1], GAMMA)
        elif not want[1] and not want[2]:
            self.task = B.flux_task(U, self.out[0], GAMMA)
        else:
            self.task = B.fused_task(U, *self.out, gamma=GAMMA)

    def clear(self):
        for o in self.out:
            if o is not None and self.n:
                o._base.fill_(GUARD)

    def check(self):
        if not self.n:
            return
        Fo, Ao, Ro = oracle.fused(self.dim, GAMMA, self.Uo)
        got = self.out
        for o in got:
            assert o is None or bool((o._base[:, self.n:] == GUARD).all())
        if got[0] is not None:
            assert group_error(host(got[0]), Fo, flux_groups(self.dim)) <= TOL[self.dt]
        if got[1] is not None:
            assert blocks_error(host(got[1]), Ao) <= TOL[self.dt]
        if got[2] is not None:
            assert group_error(host(got[2]), Ro, riemann_groups(self.dim)) <= TOL[self.dt]


WANTS = ((1, 1, 1), (0, 1, 0), (1, 1, 0), (0, 1, 1))


def uniform(dim, dt, sizes=EDGES, seed=0):
    return [Block(dim, dt, n, seed + i, WANTS[i % 4], jacobian=WANTS[i % 4] == (0, 1, 0) and i % 8 == 1)
            for i, n in enumerate(sizes)]


def mixed(dim, dt, sizes=EDGES, seed=50):
    return [Block(dim, dt, n, seed + i, (1, 0, 0) if i % 2 else (1, 1, 1)) for i, n in enumerate(sizes)]


def tasks(blocks):
    return [b.task for b in blocks]


def checked(blocks, run):
    for b in blocks:
        b.clear()
    run()
    torch.cuda.synchronize()
    for b in blocks:
        b.check()


@pytest.mark.parametrize("dim,dt", [(d, t) for d in (1, 2, 3) for t in ("f64", "f32")])
def test_shapes(dim, dt):
    blocks = uniform(dim, dt)
    shapes = [(0, 1, 0, 1)] + [(64, 1, 3, 0), (128, 2, 0, 1), (256, 1, 7, 2)] + ([(64, 4, 0, 2)] if dim < 3 else [])
    for block, ppt, grid, nt in shapes:
        plan = B.Plan(tasks(blocks), block=block, ppt=ppt, grid=grid, nontemporal=nt)
        checked(blocks, lambda: plan.run(graph=True))
        checked(blocks, lambda: plan.run(graph=False))
        plan.close()
    checked(blocks, lambda: B.run_noalloc(tasks(blocks)))


@pytest.mark.parametrize("dt", ("f64", "f32"))
def test_parts_apart(dt):
    """Past the last-level cache a 3D tile's parts are units of their own;
    more than 64 tasks, so that the owner of a unit is found in two steps."""
    es = 8 if dt == "f64" else 4
    sizes = [200 + 37 * i for i in range(67)] + [(256 << 20) // (75 * es)]
    blocks = uniform(3, dt, sizes)
    plan = B.Plan(tasks(blocks))
    checked(blocks, lambda: plan.run(graph=True))
    plan.close()


@pytest.mark.parametrize("dt", ("f64", "f32"))
def test_list_changes(dt):
    lists = uniform(3, dt), mixed(3, dt), uniform(2, dt, seed=20), uniform(3, dt, EDGES[::-1], 30)
    for first in (lists[0], None):
        plan = B.Plan(tasks(first) if first else [], capacity=len(EDGES))
        for blocks in (*lists, lists[1], lists[0]):
            plan.update(tasks(blocks))
            for graph in (True, False, True):
                checked(blocks, lambda: plan.run(graph=graph))
        plan.close()


def test_captured_launch_follows_later_lists():
    lists = uniform(3, "f64"), mixed(3, "f64"), uniform(2, "f64", seed=20)
    plan = B.Plan(tasks(lists[0]))
    checked(lists[0], plan.run)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.run(graph=False)
    for blocks in (*lists, *lists):
        plan.update(tasks(blocks))
        checked(blocks, graph.replay)
        checked(blocks, lambda: plan.run(graph=False))
    del graph
    plan.close()
