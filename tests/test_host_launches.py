"""What the library's host code launches, copies and refuses, checked without
a device (see hip_host.py)."""
import pytest

import hip_host

STAGED_3D_F64 = 256 * 25 * 8  # LDS of 3D FP64 blocks at 256 threads, one point each


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    stand_ins = hip_host.build(tmp_path_factory.mktemp("hip"))
    return lambda script: hip_host.run(stand_ins, script)


@pytest.mark.parametrize("first", ("[]", "[task(FUSED, 3, 1000)]"))
@pytest.mark.parametrize("at_capture", ("[task(FLUX, 3, 100)]", "[]"))
def test_captured_launch_has_room_for_every_later_list(run, first, at_capture):
    """A launch recorded over a list without block-writing tasks, or over an
    empty one, is replayed over lists that stage 3D FP64 blocks in LDS."""
    run(f"""
s = h.stream()
plan = h.plan({first}, block=256)
assert h.update(plan, {at_capture}, s) == 0
graph = h.capture(s, lambda: h.run(plan, s, 0))
assert h.update(plan, [task(FUSED, 3, 1000), task(CONS2PRIM, 2, 50)], s) == 0
h.replay(graph, s)
(l,) = h.launches()
assert l.replay and l.units == 5 and l.lds >= {STAGED_3D_F64}, l
""")


def test_launch_between_a_captured_upload_and_its_replay(run):
    """The table on the device is still the list before: the launch has the
    LDS which that one stages."""
    run(f"""
s = h.stream()
plan = h.plan([task(FUSED, 3, 1000), task(CONS2PRIM, 2, 50)], block=256)
for later in ([task(FLUX, 3, 100)], []):
    graph = h.capture(s, lambda: h.update(plan, later, s))
    h.run(plan, s, 0)
    (l,) = h.launches()
    assert l.units == 5 and l.lds >= {STAGED_3D_F64}, l
""")


@pytest.mark.parametrize("listed", ("[task(FUSED, 3, 1000)]", "[task(FLUX, 3, 100)]", "[]"))
def test_graph_launch_is_recorded_by_a_capture(run, listed):
    """The runtime runs a graph launch on a capturing stream at once and
    records nothing: run(graph=True) under capture has to be a launch."""
    run(f"""
s = h.stream()
plan = h.plan({listed})
graph = h.capture(s, lambda: h.run(plan, s, 1))
assert not h.launches()
for _ in range(2):
    h.replay(graph, s)
    assert len(h.launches()) == 1
""")


LISTS = ("[task(FUSED, 3, 1000)]", "[task(FUSED, 3, 1000), task(FLUX, 2, 70)]", "[task(FLUX, 1, 500)]",
         "[task(JACOBIAN, 2, 300, F32), task(FUSED, 2, 9, F32)]")


@pytest.mark.parametrize("block,ppt", ((0, 1), (256, 1), (64, 2), (64, 8)))
@pytest.mark.parametrize("listed", LISTS)
def test_graph_holds_the_first_lists_launch(run, listed, block, ppt):
    """run(graph=True) replays a graph for every kind of list that a plan is
    created with, and for a later list that wants the same launch."""
    run(f"""
s = h.stream()
tasks = {listed}
plan = h.plan(tasks, block={block}, ppt={ppt})
h.run(plan, s, 1)
h.run(plan, s, 0)
replayed, direct = h.launches()
assert replayed.replay and not direct.replay
assert str(replayed).split()[:-1] == str(direct).split()[:-1]
assert h.update(plan, {listed}, s) == 0
h.run(plan, s, 1)
(l,) = h.launches()
assert l.replay
assert h.update(plan, tasks + [task(FLUX, 1, 40000)], s) == 0
h.run(plan, s, 1)
(l,) = h.launches()
assert not l.replay and l.units > replayed.units
""")


def test_a_failed_capture_query_leaves_the_plan_alone(run):
    """The query fails on the default stream while another thread captures:
    that is no capture of this stream.  Neither it nor an upload that fails
    under a capture takes the list's own launch from the plan for good."""
    run("""
s = h.stream()
tasks = [task(FUSED, 3, 1000)]
plan = h.plan(tasks)
h.run(plan, s, 0)
(own,) = h.launches()
assert "k_batch_fused" in own.kernel
h.fail("hipStreamIsCapturing")
assert h.update(plan, tasks, s) == 0
h.fail("hipStreamIsCapturing", False)
h.run(plan, s, 0)
assert str(h.launches()[0]) == str(own)
h.fail("hipMemcpyAsync")
h.capture(s, lambda: h.update(plan, tasks, s))
h.fail("hipMemcpyAsync", False)
h.run(plan, s, 0)
assert str(h.launches()[0]) == str(own)
""")


def test_a_failed_upload_leaves_the_list_that_was(run):
    """The table on the device is unchanged, so the launch still is the one
    that reads it, and what the plan reports too."""
    run("""
s = h.stream()
plan = h.plan([task(FUSED, 3, 1000), task(FLUX, 2, 70)])
h.run(plan, s, 0)
(own,) = h.launches()
for failing in ("hipMemcpyAsync", "hipEventRecord"):
    h.fail(failing)
    assert h.update(plan, [task(FUSED, 3, 5000)], s) == EHIP
    h.fail(failing, False)
    h.run(plan, s, 0)
    (l,) = h.launches()
    points, tiles = ctypes.c_int64(), ctypes.c_int64()
    h.lib.fdbb_batch_plan_info(plan, ctypes.byref(points), ctypes.byref(tiles))
    if failing == "hipMemcpyAsync":
        assert str(l) == str(own) and (points.value, tiles.value) == (1070, 5), l
    else:  # the table has arrived
        assert "k_batch_fused" in l.kernel and (points.value, tiles.value) == (5000, 20), l
""")


def test_a_callers_configuration_is_launched_as_it_is(run):
    """Rows that start inside cache lines change the library's own choice of
    shape and store mode, not the one a caller set."""
    run("""
n = (1 << 20) + 1
U, F = address(5, n), address(15, n)
def launch():
    assert h.lib.fdbb_flux(3, ctypes.c_double(1.4), F64, ctypes.c_void_p(U), ctypes.c_int64(n), ctypes.c_void_p(F),
                           ctypes.c_int64(n), ctypes.c_int64(n), None) == 0
    (l,) = h.launches()
    return l.block, "Li0EEEv" in l.kernel  # regular stores
small = lambda *a: h.lib.fdbb_set_small_launch_config(FLUX, 3, F64, ctypes.c_int64(1 << 21), *a)
install = lambda level, bound, *a: h.lib.fdbb_install_launch_config(FLUX, 3, F64, level, ctypes.c_int64(bound), *a)
assert install(2, 0, 256, 1, 0, 1) == 0
assert launch() == (512, True)
assert h.lib.fdbb_set_launch_config(FLUX, 3, F64, 128, 1, 0, 1) == 0
assert launch() == (128, False)
assert install(1, 1 << 21, 64, 1, 0, 1) == 0
assert launch() == (512, True)
assert small(128, 1, 0, 1) == 0
assert launch() == (128, False)
assert small(64, 1, 0, 1) == 0   # the library's own again
assert launch() == (512, True)
assert h.lib.fdbb_set_small_launch_config(FLUX, 3, F64, ctypes.c_int64(0), 0, 0, 0, 0) == 0
assert launch() == (128, False)
assert h.lib.fdbb_set_launch_config(FLUX, 3, F64, 256, 1, 0, 1) == 0
assert launch() == (512, True)
assert install(1, 1 << 21, 100, 1, 0, 1) == EINVAL
""")


CALLS = """
def fused(dtype, n, dim=3):
    t = task(FUSED, dim, n, dtype)
    assert h.lib.fdbb_task_run(ctypes.byref(t), None) == 0
    (l,) = h.launches()
    return l
def flux(dtype, n, dim=3):
    t = task(FLUX, dim, n, dtype)
    assert h.lib.fdbb_task_run(ctypes.byref(t), None) == 0
    (l,) = h.launches()
    return l
def shape(op, dim, dtype, *cfg):
    assert h.lib.fdbb_set_launch_config(op, dim, dtype, *cfg) == 0
    h.lib.fdbb_set_small_launch_config(op, dim, dtype, ctypes.c_int64(0), 0, 0, 0, 0)
"""


@pytest.mark.parametrize("dtype,es", (("F64", 8), ("F32", 4)))
def test_only_one_point_per_thread_is_bounded_or_dealt_apart(run, dtype, es):
    """Reserved LDS and parts of a tile in workgroups of their own are for
    uncapped launches of one point per thread; other shapes lose by them."""
    run(CALLS + f"""
n = 1 << 20
for block, ppt, cap in ((128, 2, 0), (64, 4, 0), (128, 1, 2048), (128, 1, 0)):
    shape(FLUX, 3, {dtype}, block, ppt, cap, 1)
    shape(FUSED, 3, {dtype}, block, ppt, cap, 1)
    plain = (ppt, cap) != (1, 0)
    l = flux({dtype}, 8 * n)
    assert (l.lds == 0) == plain, l
    l = fused({dtype}, n)
    tiles = n // (block * ppt)
    assert l.grid == (min(tiles, cap or tiles) if plain else tiles * (3 if {es} == 8 else 4)), l
    assert (l.lds == block * ppt * 25 * {es}) == plain, l
""")


@pytest.mark.parametrize("dim,dtype,es", ((3, "F64", 8), (3, "F32", 4), (2, "F64", 8)))
@pytest.mark.parametrize("mib,ragged", ((192, 0), (48, 1)))
def test_rows_are_bounded_past_the_cache_only(run, dim, dtype, es, mib, ragged):
    """A pointwise call reserves LDS where it writes 192 MiB or more, 48 MiB
    where its rows start inside cache lines."""
    run(CALLS + f"""
per = {(dim + 2) * dim} * {es}
at = max(-(-({mib} << 20) // per), 1 << 19)  # rows below 2^19 points count as whole lines
shape(FLUX, {dim}, {dtype}, 128, 1, 0, 1)
if {ragged}:
    below, above = (at - 1) | 1, at | 1
    below -= 2 * (below >= at)
else:
    below, above = at // 32 * 32 - 32, at + -at % 32
assert flux({dtype}, below, {dim}).lds == 0
assert flux({dtype}, above, {dim}).lds > 0
""")


@pytest.mark.parametrize("listed", ("[task(FUSED, 3, 1 << 20)]", "[task(JACOBIAN, 2, 300, F32), task(FUSED, 2, 9, F32)]",
                                    "[task(FUSED, 3, 1000), task(FLUX, 2, 70)]"))
@pytest.mark.parametrize("block,ppt,grid,nt", ((256, 1, 0, 1), (64, 4, 0, 2), (128, 1, 1024, 0), (64, 8, 5, 1)))
def test_a_plan_of_explicit_shape_launches_in_it(run, listed, block, ppt, grid, nt):
    """The kernels and bounds of installed configurations are for these."""
    run(f"""
s = h.stream()
tasks = {listed}
plan = h.plan(tasks, block={block}, ppt={ppt}, grid={grid}, nt={nt})
h.run(plan, s, 0)
(l,) = h.launches()
assert "7k_batchILi{ppt}ELi{nt}E" in l.kernel and l.block == {block}, l
assert l.grid == min({grid} or 256 * (2048 // {block}), l.units)
staged = max({block} * {ppt} * (t.dim + 2) ** 2 * (4 if t.dtype == F32 else 8) for t in tasks if t.op != FLUX)
assert l.lds == (max(staged, 163840 * {block} // 512) if {ppt} == 1 else staged)
""")


def test_rows_inside_cache_lines_take_long_runs(run):
    """Whatever shape the library would take for whole lines: one point per
    thread, 512 threads, regular stores for the flux; the characteristic
    transforms at several points per thread and small outputs stay."""
    run("""
def shape(op, dim, n, dtype):
    t = task(op, dim, n, dtype)
    assert h.lib.fdbb_task_run(ctypes.byref(t), None) == 0
    (l,) = h.launches()
    return l.block, l.kernel
def same(l, block, ppt, nt=None):
    assert l[0] == block and f"Li{ppt}ELi" in l[1], l
    assert nt is None or f"Li{nt}EEEv" in l[1], l
same(shape(FLUX, 3, 1 << 20, F64), 256, 2)
same(shape(FLUX, 3, (1 << 20) + 1, F64), 512, 1, 0)
same(shape(FLUX, 3, (1 << 20) + 1, F32), 512, 1, 0)
same(shape(FLUX, 3, (1 << 19) - 1, F64), 256, 2)
same(shape(FLUX, 1, (1 << 20) + 1, F32), 256, 4)
same(shape(FLUX_DIR, 3, 1000003, F32), 256, 4)
same(shape(FLUX_DIR, 3, 2500009, F32), 512, 1, 0)
same(shape(CONS2CHAR, 1, 2500009, F64), 256, 2)
""")


def test_own_choice_by_size(run):
    """The library's own entries for fewer and for more points apply beside
    its own other two, and not where a caller set one of those."""
    run("""
I64 = ctypes.c_int64
install = lambda level, bound, *a: h.lib.fdbb_install_launch_config(FLUX, 2, F64, level, I64(bound), *a)
def at(n):
    v = [ctypes.c_int() for _ in range(4)]
    assert h.lib.fdbb_launch_config_for(FLUX, 2, F64, I64(n), *map(ctypes.byref, v)) == 0
    return tuple(x.value for x in v)
cfg = [(64, 1, 0, 1), (128, 1, 0, 1), (256, 2, 0, 1), (512, 4, 0, 0)]
bound = [1000, 5000, 0, 20000]
for level in range(4):
    assert install(level, bound[level], *cfg[level]) == 0
sizes = (0, 1000, 1001, 5000, 5001, 19999, 20000, 1 << 30)
assert [cfg.index(at(n)) for n in sizes] == [0, 0, 1, 1, 2, 2, 3, 3]
h.lib.fdbb_set_small_launch_config(FLUX, 2, F64, I64(5000), 64, 2, 0, 1)
assert at(1) == at(1001) == (64, 2, 0, 1) and at(20000) == cfg[3]
h.lib.fdbb_set_launch_config(FLUX, 2, F64, 64, 4, 0, 1)
assert at(5001) == at(20000) == (64, 4, 0, 1)
h.lib.fdbb_set_small_launch_config(FLUX, 2, F64, I64(5000), *cfg[1])
h.lib.fdbb_set_launch_config(FLUX, 2, F64, *cfg[2])
assert [cfg.index(at(n)) for n in sizes] == [0, 0, 1, 1, 2, 2, 3, 3]
assert install(0, 0, 0, 0, 0, 0) == 0 and install(3, 0, 0, 0, 0, 0) == 0
assert [cfg.index(at(n)) for n in sizes] == [1, 1, 1, 1, 2, 2, 2, 2]
assert install(0, 10, 100, 1, 0, 1) == install(4, 10, 64, 1, 0, 1) == install(3, -1, 64, 1, 0, 1) == EINVAL
assert h.lib.fdbb_install_launch_config(FUSED, 2, F64, 0, I64(10), 512, 1, 0, 1) == EINVAL
""")


@pytest.mark.parametrize("op,mib,blocks,parts", (("FUSED", 512, 3, 4), ("JACOBIAN", 512, 3, 3), ("EIGEN", 6144, 6, 6)))
def test_fp32_parts_apart_up_to_a_bound(run, op, mib, blocks, parts):
    """3D FP32 tiles are dealt apart past the last-level cache and up to this
    much of blocks."""
    run(CALLS + f"""
per = {blocks} * 25 * 4
shape({op}, 3, F32, 256, 1, 0, 1)
for bound, expected in ((256 << 20, (1, {parts})), ({mib} << 20, ({parts}, 1))):
    for n, sets in zip((bound // per, bound // per + 1), expected):
        t = task({op}, 3, n, F32)
        assert h.lib.fdbb_task_run(ctypes.byref(t), None) == 0
        (l,) = h.launches()
        assert l.grid == -(-n // 256) * sets, (n, l)
""")


@pytest.mark.parametrize("mode", (0, 1))
def test_a_server_bounds_waves_on_its_one_stream_only(run, mode):
    """Slots with streams of their own share the chip: a request that runs
    alone in one reserves no LDS; the one-stream mode has the chip to itself."""
    run(CALLS + f"""
import time
shape(FLUX, 3, F64, 128, 1, 0, 1)
server = ctypes.c_void_p()
assert h.lib.fdbb_server_create(ctypes.c_int64(1 << 30), 2, 8, ctypes.c_double(1e6), {mode}, ctypes.byref(server)) == 0
h.launches()
t = task(FLUX, 3, 1 << 21)
assert h.lib.fdbb_server_submit(server, ctypes.byref(t), ctypes.c_uint64(1)) == 0
done, count = (ctypes.c_char * 4096)(), ctypes.c_int()
for _ in range(2000):
    assert h.lib.fdbb_server_poll(server, done, 8, ctypes.byref(count)) == 0
    if count.value:
        break
    time.sleep(0.002)
assert count.value == 1
(l,) = h.launches()
assert (l.lds > 0) == bool({mode}), l
h.lib.fdbb_server_destroy(server)
""")
