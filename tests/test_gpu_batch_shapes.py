"""Batch plans in other shapes of the installed configuration: the kernel of
block-writing lists at 1, 2 and 4 points per thread, with persistent grids
and grids that leave the units to the hardware, and the general kernel."""
import pytest
import torch

from gpu_common import require_gpu
from paper_1809_09851_amd import batch as B
from paper_1809_09851_amd import fdbb as F
from test_gpu_batch_fused import checked, mixed, tasks, uniform

pytestmark = pytest.mark.gpu

SHAPES = ((64, 1, 64, 1), (256, 1, 2, 0), (128, 2, 64, 2), (64, 2, 1, 1), (64, 4, 64, 0), (64, 8, 4, 1))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.fixture
def installed():
    saved = {dt: F.fdbb_get_batch_config(dt) for dt in (F.F64, F.F32)}
    yield
    for dt, cfg in saved.items():
        F.fdbb_set_batch_config(dt, *cfg)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dim,dt", [(d, t) for d in (1, 2, 3) for t in ("f64", "f32")])
def test_installed_shapes(dim, dt, shape, installed):
    try:
        F.fdbb_set_batch_config(F.F64 if dt == "f64" else F.F32, *shape)
    except F.FdbbError:
        pytest.skip("3D FP64 blocks of this shape do not fit in LDS")
    for blocks in (uniform(dim, dt), mixed(dim, dt)):
        plan = B.Plan(tasks(blocks))
        checked(blocks, lambda: plan.run(graph=True))
        checked(blocks, lambda: plan.run(graph=False))
        plan.close()


@pytest.mark.parametrize("shape", ((256, 1, 2, 1), (128, 1, 64, 1)))
@pytest.mark.parametrize("dt", ("f64", "f32"))
def test_past_the_last_level_cache(dt, shape, installed):
    """Dealt apart only where the grid leaves the units to the hardware."""
    F.fdbb_set_batch_config(F.F64 if dt == "f64" else F.F32, *shape)
    blocks = uniform(3, dt, [200 + 37 * i for i in range(67)] + [(256 << 20) // (75 * (8 if dt == "f64" else 4))])
    plan = B.Plan(tasks(blocks))
    checked(blocks, lambda: plan.run(graph=True))
    plan.close()
    torch.cuda.empty_cache()
