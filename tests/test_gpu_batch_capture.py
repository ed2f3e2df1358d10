"""Launches of a batch plan recorded into a graph of the caller's, over a list
that stages nothing or an empty one, replayed over later lists that stage
blocks in LDS; and lists uploaded by a graph of the caller's."""
import pytest
import torch

from gpu_common import require_gpu
from paper_1809_09851_amd import batch as B
from test_gpu_batch_fused import Block, checked, mixed, tasks, uniform

pytestmark = pytest.mark.gpu

SIZES = (257, 1, 0, 1025)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def flux_only(seed=70):
    return [Block(3, "f64", n, seed + i, (1, 0, 0)) for i, n in enumerate(SIZES)]


@pytest.mark.parametrize("created", ("empty", "with blocks"))
@pytest.mark.parametrize("at_capture", ("flux", "empty"))
@pytest.mark.parametrize("graph", (False, True))
def test_captured_over_a_list_that_stages_nothing(created, at_capture, graph):
    lists = uniform(3, "f64", SIZES), mixed(3, "f64", SIZES), flux_only()
    plan = B.Plan(tasks(lists[0]) if created == "with blocks" else [], capacity=len(SIZES))
    plan.update(tasks(flux_only()) if at_capture == "flux" else [])
    recorded = torch.cuda.CUDAGraph()
    with torch.cuda.graph(recorded):
        plan.run(graph=graph)
    for blocks in (*lists, *lists):
        plan.update(tasks(blocks))
        checked(blocks, recorded.replay)
        checked(blocks, lambda: plan.run(graph=graph))
    del recorded
    plan.close()


def test_uploaded_by_a_graph():
    """The captured upload brings the list that was current at its capture;
    until it runs, launches still find the one before."""
    first, later = mixed(3, "f64", SIZES), flux_only()
    plan = B.Plan(tasks(first), capacity=len(SIZES))
    recorded = torch.cuda.CUDAGraph()
    with torch.cuda.graph(recorded):
        plan.update(tasks(later))
        plan.run(graph=False)
    checked(first, lambda: plan.run(graph=False))
    for _ in range(3):
        checked(later, recorded.replay)
        checked(later, lambda: plan.run(graph=False))
    del recorded
    plan.close()
