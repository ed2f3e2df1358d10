"""Other threads run while the native helpers allocate: where the caching
allocator has to give blocks back to the driver first, the allocation waits
for the work that is queued on the device."""
import threading
import time

import pytest
import torch

from gpu_common import require_gpu
from paper_1809_09851_amd import fdbb as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def longest_pause(call):
    """(duration of call(), longest time that another thread stood still)."""
    stamps, stop = [], threading.Event()

    def spin():
        while not stop.is_set():
            stamps.append(time.perf_counter())

    other = threading.Thread(target=spin)
    other.start()
    time.sleep(0.05)
    t0 = time.perf_counter()
    call()
    t1 = time.perf_counter()
    time.sleep(0.02)
    stop.set()
    other.join()
    return t1 - t0, max(b - a for a, b in zip(stamps, stamps[1:]) if b >= t0 and a <= t1)


GiB = 1 << 30


@pytest.mark.parametrize("helper,args,points", ((F._fields_like, (15,), 32 << 20), (F._blocks_like, (3,), 7 << 20)))
def test_allocation_lets_other_threads_run(helper, args, points):
    F.library()
    U = torch.empty(5, points, dtype=torch.float64, device="cuda")
    x = torch.randn(8192, 8192, device="cuda") / 100.0
    y = torch.empty_like(x)
    torch.mm(x, x, out=y)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    cached = [torch.empty(2 * GiB, dtype=torch.uint8, device="cuda") for _ in range(2)]
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + GiB) / total)
    try:
        del cached
        for _ in range(20):
            torch.mm(x, x, out=y)
        took, pause = longest_pause(lambda: helper(*args, U))
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
    print(f"{helper.__name__}: {took * 1e3:.1f} ms, longest pause {pause * 1e3:.1f} ms")
    assert took > 0.05, "the allocation did not wait for the device: nothing to see"
    assert pause < took / 2
