"""Launch-configuration autotuner.

Searches workgroup size x points per thread x grid cap x store mode for an
(op, dim, dtype) and installs the winner.  Results are kept in a JSON table
keyed by device architecture, HIP runtime version and (op, dim, dtype); the
binding applies the table shipped next to the library when it loads it.

    python -m paper_1809_09851_amd.tune --ops fused,flux_jacobian --dims 1,2,3 \\
        --dtypes f64,f32 --write paper_1809_09851_amd/tuned_gfx950.json

Calls fall into four classes by size (``CLASSES``: up to 3 * 2^17 points, up
to 2^21, beyond, and from 3 * 2^23 on), each with an entry of its own where one
pays.  Each shape is timed at every size of the class, odd ones and powers of
two, in captured graphs over rotating sets of arrays of 1.2 GB in all and over
one set; ``rank`` says which is taken, given the one in the table.  ``--n N``
tunes the plain entry at N points alone instead, by the median of single
launches.

The op ``batch`` tunes the batch kernels (block x points per thread x
workgroups per compute unit x store mode) on three lists of the batched
workload and stores the result as ``batch/3/<dtype>``; plans created without
an explicit configuration use it.

The op ``serve`` tunes the request server's batch configuration on
batches packed from the serving request mix (``serve_batch/0/mix``).

``--small N`` tunes the small-launch class at N points alone: a winner more
than 2 % faster than the large configuration at that size is stored with
max_n = 2N (``fdbb_set_small_launch_config``).
"""
from __future__ import annotations

import argparse
import itertools
import json
import math
import os
import statistics
import sys

import torch

from . import fdbb as F

GAMMA = 1.4
BLOCKS = (64, 128, 256, 512, 1024)
PPTS = (1, 2, 4)
GRID_CAPS = (0, 2048, 4096, 8192)
STORE_MODES = (1, 0)
# the batch kernels: block x points per thread x workgroups per
# compute unit x store mode (0 regular, 1 nt, 2 nt + sc1)
BATCH_BLOCKS = (64, 128, 256)
BATCH_PPTS = (1, 2, 4, 8)
BATCH_GRID_PER_CU = (1, 2, 4, 8, 16, 64, 256, 1024)
BATCH_STORE_MODES = (1, 2, 0)
DEFAULT_TABLE = os.environ.get(
    "FDBB_TUNED_TABLE", os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuned_gfx950.json"))
DT = {"f64": (F.F64, torch.float64), "f32": (F.F32, torch.float32)}


def arch_key() -> str:
    props = torch.cuda.get_device_properties(torch.cuda.current_device())
    arch = getattr(props, "gcnArchName", "unknown").split(":")[0]
    return f"{arch}/hip{torch.version.hip}"


def _state(dim, n, dtype, seed=1234):
    """A valid conservative state built on the device (no host data needed)."""
    V = F.empty_fields(dim + 2, n, dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    V[0].uniform_(0.5, 2.0, generator=g)
    for k in range(dim):
        V[1 + k].normal_(0.0, 0.5, generator=g)
    V[dim + 1].uniform_(0.5, 2.0, generator=g)
    U = F.empty_fields(dim + 2, n, dtype)
    F.fdbb_prim2cons(dim, GAMMA, V, U)
    return U


def workload(op: str, dim: int, dtype, n: int):
    """Inputs and outputs resident on the device; returns one launch as a
    closure."""
    K = dim + 2
    U = _state(dim, n, dtype)
    if op == "fused":
        Fo, A, R = (F.empty_fields(K * dim, n, dtype), F.empty_blocks(dim, n, dtype),
                    F.empty_fields(2 * dim + 1, n, dtype))
        return lambda: F.fdbb_euler_fused(dim, GAMMA, U, Fo, A, R)
    if op == "flux_jacobian":
        A = F.empty_blocks(dim, n, dtype)
        return lambda: F.fdbb_flux_jacobian(dim, GAMMA, U, A)
    if op == "flux":
        Fo = F.empty_fields(K * dim, n, dtype)
        return lambda: F.fdbb_flux(dim, GAMMA, U, Fo)
    if op == "flux_dir":
        Fd = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_flux_direction(dim, dim - 1, GAMMA, U, Fd)
    if op == "cons2prim":
        V = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_cons2prim(dim, GAMMA, U, V)
    if op == "prim2cons":
        V = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_prim2cons(dim, GAMMA, U, V)
    if op == "v_mag2":
        y = torch.empty(n, dtype=dtype, device="cuda")
        return lambda: F.fdbb_velocity_magnitude2(dim, U, y)
    if op == "eos":
        p = torch.empty(n, dtype=dtype, device="cuda")
        c = torch.empty(n, dtype=dtype, device="cuda")
        return lambda: F.fdbb_eos(dim, GAMMA, U, p, c)
    if op == "riemann_invariants":
        R = F.empty_fields(2 * dim + 1, n, dtype)
        return lambda: F.fdbb_riemann_invariants(dim, GAMMA, U, R)
    if op == "cons2char":
        W = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_cons2char(dim, 0, GAMMA, U, W)
    if op == "char2cons":
        W = F.empty_fields(K, n, dtype)
        F.fdbb_cons2char(dim, 0, GAMMA, U, W)
        return lambda: F.fdbb_char2cons(dim, 0, GAMMA, W, U)
    if op == "eigenvectors":
        L, R = F.empty_blocks(dim, n, dtype), F.empty_blocks(dim, n, dtype)
        return lambda: F.fdbb_eigenvectors(dim, GAMMA, U, L, R)
    if op == "char_apply":
        X = F.empty_fields(K, n, dtype).normal_()
        Y = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_char_apply(dim, 0, 0, GAMMA, U, X, Y)
    if op == "viscous_flux":
        G = F.empty_fields(dim * dim, n, dtype).normal_()
        gT = F.empty_fields(dim, n, dtype).normal_()
        Fv = F.empty_fields(K * dim, n, dtype)
        return lambda: F.fdbb_viscous_flux(dim, 1e-3, 2e-3, U, G, gT, Fv)
    if op == "eos_pvt":
        p, c, T = (torch.empty(n, dtype=dtype, device="cuda") for _ in range(3))
        return lambda: F.fdbb_eos_pvt(dim, 1, (4.4, 0.1, 2.5), U, p, c, T)
    if op == "roe_average":
        UR = _state(dim, n, dtype, seed=4321)
        Uh = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_roe_average(dim, GAMMA, U, UR, Uh)
    if op == "adjoint":
        Fb = F.empty_fields(K * dim, n, dtype).normal_()
        Ub = F.empty_fields(K, n, dtype)
        return lambda: F.fdbb_flux_adjoint(dim, -1, GAMMA, U, Fb, Ub)
    raise ValueError(op)


def bytes_per_point(op: str, dim: int, elem: int) -> int:
    """Algorithmic HBM bytes per point of one launch of `op`."""
    K = dim + 2
    per = {"cons2prim": 2 * K, "prim2cons": 2 * K, "cons2char": 2 * K, "char2cons": 2 * K,
           "eos": K + 2, "v_mag2": dim + 2, "flux": K + K * dim, "flux_dir": 2 * K, "flux_jacobian": K + dim * K * K,
           "riemann_invariants": K + 2 * dim + 1, "fused": K + K * dim + dim * K * K + 2 * dim + 1,
           "adjoint": K * K, "eigenvectors": K + 2 * dim * K * K, "char_apply": 3 * K,
           "roe_average": 3 * K, "eos_pvt": K + 3, "viscous_flux": K + dim * dim + dim + K * dim}[op]
    return per * elem


def auto_size(op: str, dim: int, elem: int, target_bytes: float = 2e9) -> int:
    """A size whose working set (about 2 GB) is far larger than the 256 MB
    last-level cache, so that the search sees HBM behaviour."""
    n = target_bytes / bytes_per_point(op, dim, elem)
    e = min(27, max(22, int(round(math.log2(n)))))
    return 1 << e


def time_launch(fn, reps: int = 7, warmup: int = 2) -> float:
    """Median milliseconds of one launch, HIP events on the current stream."""
    for _ in range(warmup):
        fn()
    stream = torch.cuda.current_stream()
    times = []
    for _ in range(reps):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record(stream)
        fn()
        b.record(stream)
        b.synchronize()
        times.append(a.elapsed_time(b))
    return statistics.median(times)


def time_queued(fns, launches: int = 256, rounds: int = 2) -> float:
    """Milliseconds per launch of `launches` back-to-back launches cycling
    over `fns` (one event pair around all of them; best of `rounds`)."""
    for f in fns:
        f()
    stream = torch.cuda.current_stream()
    best = float("inf")
    for _ in range(rounds):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record(stream)
        for k in range(launches):
            fns[k % len(fns)]()
        b.record(stream)
        b.synchronize()
        best = min(best, a.elapsed_time(b) / launches)
    return best


# The classes of calls by size, with the level of fdbb_install_launch_config, its
# bound and the sizes to time.  Each may have an entry: tiny/ and small/ with
# max_n, the plain name, huge/ with min_n.
CLASSES = {
    "large": (2, 0, (3000017, 1 << 22, 8000009, 12000017, 1 << 24)),
    "huge": (3, 3 << 23, (33554467, 1 << 26, 100000007)),
    "small": (1, 1 << 21, (600011, 1000003, 1 << 20, 1500001, 1900013)),
    "tiny": (0, 3 << 17, (1009, 4099, 20011, 130003, 300007)),
}
BESIDE = {"tiny": "small", "huge": "large"}  # whose shape a class without an entry takes
KEEP_MARGIN = 0.03  # a shape in force stays unless another is this much faster
MAX_BYTES = 12e9       # moved by one launch
ROTATED_BYTES = 1.2e9  # in the sets of arrays that launches go through in turn
SCREEN_MARGIN = 1.10


def time_graph(fns, launches: int, rounds: int = 4) -> float:
    """Microseconds per launch of `launches` launches cycling over `fns`,
    captured in one graph (best of `rounds` replays)."""
    for f in fns:
        f()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for k in range(launches):
            fns[k % len(fns)]()
    g.replay()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / launches * 1e3)
    return best


def rank(times: dict, in_force=None) -> list:
    """[(mean, worst, shape)] of {shape: [time at each size]}, the one to take
    first: `mean` is the geometric mean, `worst` the maximum, over the sizes
    of the time over the best shape's at that size.  The shape `in_force` stays
    if its mean is within KEEP_MARGIN of the lowest: what kernels of other ops
    leave in the caches moves a shape's time by as much.  Otherwise, of the
    shapes whose mean is within 0.5 % of the lowest, the one with the lowest
    worst case leads."""
    best = [min(t) for t in zip(*times.values())]
    rows = []
    for cfg, t in times.items():
        r = [x / b for x, b in zip(t, best)]
        rows.append((math.exp(sum(map(math.log, r)) / len(r)), max(r), cfg))
    rows.sort()
    kept = [r for r in rows if r[2] == in_force and r[0] <= rows[0][0] * (1 + KEEP_MARGIN)]
    near = kept or [r for r in rows if r[0] <= rows[0][0] * 1.005]
    lead = min(near, key=lambda r: (r[1], r[0]))
    return [lead] + [r for r in rows if r is not lead]


def search_range(op: str, dim: int, dt: str, cls: str, in_force=None):
    """Times every shape over the sizes of a class, over rotating sets of arrays
    and over one set, part of which stays in the last-level cache as in a step
    that reads its state again; returns ({shape: [us at each size, rotating,
    then at each size, one set]}, sizes).  Shapes without a grid cap are tried,
    since a cap keeps a launch from being dealt in parts or fitted to its rows,
    and the one in force.  Shapes that are more than SCREEN_MARGIN off the best in all four timings at the class's second and
    last size are not timed at the others."""
    code, dtype = DT[dt]
    bpp = bytes_per_point(op, dim, 8 if dt == "f64" else 4)
    sizes = [n for n in CLASSES[cls][2] if n * bpp <= MAX_BYTES]
    if not sizes:
        return {}, []
    one_entry(op, dim, code)
    old = F.fdbb_get_small_launch_config(op, dim, code)
    shapes = [c for c in itertools.product(BLOCKS, PPTS, (0,), STORE_MODES)
              if F.fdbb_kernel_info(op, dim, code, c[1], c[3])[1] == 0]
    if in_force and in_force not in shapes:
        shapes.append(in_force)
    times = {}
    screens = {sizes[min(1, len(sizes) - 1)], sizes[-1]}
    seen = [(m, w) for m in screens for w in (0, 1)]
    try:
        for n in sorted(sizes, key=lambda n: n not in screens):
            if n not in screens and seen:
                best = {k: min(t[k] for t in times.values()) for k in seen}
                shapes = [c for c in shapes if c in times and
                          (c == in_force or any(times[c][k] <= SCREEN_MARGIN * best[k] for k in seen))]
                seen = []
            sets = max(2, min(64, math.ceil(ROTATED_BYTES / (bpp * n))))
            fns = [workload(op, dim, dtype, n) for _ in range(sets)]
            launches = max(sets, min(256, int(1e10 / (bpp * n))))
            for c in shapes:
                try:
                    F.fdbb_set_small_launch_config(op, dim, code, 1 << 30, *c)
                    t = times.setdefault(c, {})
                    t[n, 0], t[n, 1] = time_graph(fns, launches), time_graph(fns[:1], launches)
                except F.FdbbError:
                    times.pop(c, None)  # a configuration this kernel cannot take (block size, LDS)
            del fns
            torch.cuda.empty_cache()
    finally:
        F.fdbb_set_small_launch_config(op, dim, code, *old)
    keys = [(n, w) for w in (0, 1) for n in sizes]
    return {c: [t[k] for k in keys] for c, t in times.items() if len(t) == len(keys)}, sizes


def one_entry(op, dim, code):
    """Lifts the entries beside the small and the large one, so that a shape
    set for all sizes is what every call takes."""
    for level in (0, 3):
        F.fdbb_install_launch_config(op, dim, code, level, 0)


def shape_of(entry: dict | None):
    return tuple(entry[k] for k in ("block", "ppt", "grid_cap", "nt")) if entry else None


def range_entry(times: dict, sizes: list, cls: str, in_force=None) -> dict:
    """The table's entry of a search_range."""
    rows = rank(times, in_force)
    block, ppt, cap, nt = rows[0][2]
    e = {"block": block, "ppt": ppt, "grid_cap": cap, "nt": nt, "sizes": list(sizes),
         "us": [round(t, 2) for t in times[rows[0][2]]],
         "top5": [[round(m, 4), round(w, 4), list(c)] for m, w, c in rows[:5]]}
    level, bound = CLASSES[cls][:2]
    if level != 2:
        e["min_n" if level == 3 else "max_n"] = bound
    return e


def tune_range(op: str, dim: int, dt: str, entries: dict) -> None:
    """Times all classes of (op, dim, dtype) and puts their entries into
    `entries`; the tiny and the huge class get none where the neighbour's shape
    leads."""
    key = f"{op}/{dim}/{dt}"
    named = lambda cls: key if cls == "large" else f"{cls}/{key}"
    for cls in CLASSES:
        other = shape_of(entries[named(BESIDE[cls])]) if cls in BESIDE else None
        in_force = shape_of(entries.pop(named(cls), None)) or other or shape_of(entries.get(key))
        times, sizes = search_range(op, dim, dt, cls, in_force)
        if not times:
            continue
        e = range_entry(times, sizes, cls, in_force)
        if shape_of(e) != other:
            entries[named(cls)] = e
        print(json.dumps({named(cls): entries.get(named(cls))}), flush=True)


SMALL_GRID_CAPS = (0, 2048)
SMALL_MIN_GAIN = 0.02


def search_small(op: str, dim: int, dt: str, n: int, verbose=False, target_bytes: float = 1e9):
    """Tune the small-launch class at n points.  Returns (results sorted as
    [(ms, cfg)], the large configuration's ms at this size, max_n installed
    or 0).  Installs the winner for n <= 2n when it beats the large
    configuration by more than SMALL_MIN_GAIN, else removes the entry."""
    code, dtype = DT[dt]
    es = 8 if dt == "f64" else 4
    sets = max(1, min(64, math.ceil(target_bytes / (bytes_per_point(op, dim, es) * n))))
    fns = [workload(op, dim, dtype, n) for _ in range(sets)]
    one_entry(op, dim, code)
    large = F.fdbb_get_launch_config(op, dim, code)
    F.fdbb_set_small_launch_config(op, dim, code, 0)
    large_ms = time_queued(fns)
    results = []
    for cfg in itertools.product(BLOCKS, PPTS, SMALL_GRID_CAPS, STORE_MODES):
        if F.fdbb_kernel_info(op, dim, code, cfg[1], cfg[3])[1] > 0:
            continue
        try:
            F.fdbb_set_small_launch_config(op, dim, code, n, *cfg)
            ms = time_queued(fns)
        except F.FdbbError:
            continue
        results.append((ms, cfg))
        if verbose:
            print(f"  small {op} {dim}d {dt} n={n} cfg={cfg} {ms * 1e3:.2f} us", file=sys.stderr, flush=True)
    results.sort()
    max_n = 0
    if results and results[0][0] < large_ms * (1 - SMALL_MIN_GAIN) and results[0][1] != large:
        max_n = 2 * n
        F.fdbb_set_small_launch_config(op, dim, code, max_n, *results[0][1])
    else:
        F.fdbb_set_small_launch_config(op, dim, code, 0)
    del fns
    torch.cuda.empty_cache()
    return results, large_ms, max_n


def search(op: str, dim: int, dt: str, n: int, reps: int = 7, space=None, verbose=False):
    """Time every candidate; returns [(ms, (block, ppt, grid_cap, nt))] sorted,
    and leaves the fastest installed."""
    code, dtype = DT[dt]
    fn = workload(op, dim, dtype, n)
    space = space or list(itertools.product(BLOCKS, PPTS, GRID_CAPS, STORE_MODES))
    one_entry(op, dim, code)
    old = F.fdbb_get_launch_config(op, dim, code)
    # a small-launch entry covering n would take over every candidate: lift it
    small = F.fdbb_get_small_launch_config(op, dim, code)
    if small[0] >= n:
        F.fdbb_set_small_launch_config(op, dim, code, 0)
    results = []
    for cfg in space:
        # kernels that spill registers move extra bytes through HBM; skip them
        if F.fdbb_kernel_info(op, dim, code, cfg[1], cfg[3])[1] > 0:
            continue
        try:
            F.fdbb_set_launch_config(op, dim, code, *cfg)
            ms = time_launch(fn, reps)
        except F.FdbbError:
            continue  # a configuration this kernel cannot take (block size, LDS)
        results.append((ms, cfg))
        if verbose:
            print(f"  {op} {dim}d {dt} n={n} cfg={cfg} {ms:.4f} ms", file=sys.stderr, flush=True)
    results.sort()
    F.fdbb_set_launch_config(op, dim, code, *(results[0][1] if results else old))
    if small[0] >= n:
        F.fdbb_set_small_launch_config(op, dim, code, *small)
    return results


def batch_workload(dtype, nblocks: int = 512, seed: int = 2):
    """The batched workload: `nblocks` 3D blocks of sizes log-uniform in
    [10^3, 10^6] points with 5 % near-vacuum points (seeded), each a fused
    pass (flux, Jacobians, invariants) into its own outputs on the device.
    Returns (tasks, points, the tensors the tasks point into)."""
    from . import batch as B
    from . import inputs
    sizes, Vs = inputs.batched(3, nblocks, seed=seed)
    keep, tasks = [], []
    for V in Vs:
        n = V.shape[1]
        Vg = F.to_fields(torch.from_numpy(V).to(dtype).cuda())
        U = F.empty_fields(5, n, dtype)
        F.fdbb_prim2cons(3, GAMMA, Vg, U)
        out = (F.empty_fields(15, n, dtype), F.empty_blocks(3, n, dtype), F.empty_fields(7, n, dtype))
        tasks.append(B.fused_task(U, *out, gamma=GAMMA))
        keep.append((U, out))
        del Vg
    torch.cuda.synchronize()
    return tasks, int(sizes.sum()), keep


BATCH_LISTS = (24, 96, 512)  # blocks of the batched workload


def search_batch(dt: str, reps: int = 5, space=None, verbose=False, lists=BATCH_LISTS):
    """Times every batch configuration on the first blocks of the batched
    workload (graph-captured launches); returns ({(block, ppt, grid_per_cu,
    nt): [ms on each list]}, points of each list) and installs the one that
    `rank` takes."""
    from . import batch as B
    code, dtype = DT[dt]
    es = 8 if dt == "f64" else 4
    tasks, _, keep = batch_workload(dtype, max(lists))
    old = F.fdbb_get_batch_config(code)
    space = space or list(itertools.product(BATCH_BLOCKS, BATCH_PPTS, BATCH_GRID_PER_CU, BATCH_STORE_MODES))
    times = {}
    for cfg in space:
        if cfg[0] * cfg[1] * 25 * es > 160 * 1024:  # 3D Jacobian staging must fit in LDS
            continue
        for k in lists:
            try:
                # through the installed configuration, which chooses kernel and
                # parts by the list; a plan of explicit shape does not
                F.fdbb_set_batch_config(code, *cfg)
                plan = B.Plan(tasks[:k])
            except F.FdbbError:
                times.pop(cfg, None)
                break
            times.setdefault(cfg, []).append(time_launch(lambda: plan.run(graph=True), reps))
            plan.close()
        if verbose:
            print(f"  batch {dt} cfg={cfg} {times.get(cfg)} ms", file=sys.stderr, flush=True)
    F.fdbb_set_batch_config(code, *(rank(times)[0][2] if times else old))
    points = [sum(t.n for t in tasks[:k]) for k in lists]
    del keep, tasks
    torch.cuda.empty_cache()
    return times, points


def serve_workload(batches: int = 24, seed: int = 7, max_batch: int = 64, max_bytes: float = 64e6):
    """Batches as the request server packs them from the serving request mix
    (inputs.request_stream: the server's ops, D in {1, 2, 3}, N log-uniform
    in [10^3, 10^7], FP64 or FP32, inputs viewed from device-resident state
    pools): consecutive requests while a batch holds at most max_batch
    requests and max_bytes moved bytes.  A request larger than that runs
    alone in the server, not in a batch, and is left out.  Returns (task
    lists, moved bytes of one pass, what the tasks point into)."""
    from . import inputs
    from . import serve
    pools = serve.StatePools(pool=10_000_000, seed=4)
    specs = inputs.request_stream(1e6, 40 * batches * max_batch, seed=seed, pool=pools.pool)
    lists, keep, total = [], [pools], 0
    cur, cur_bytes = [], 0
    for spec in specs:
        r = pools.request(spec)
        m = serve.moved_bytes(r.op, r.dim, r.n, r.elem)
        if m > max_bytes:
            continue
        if cur and (len(cur) == max_batch or cur_bytes + m > max_bytes):
            lists.append(cur)
            total += cur_bytes
            cur, cur_bytes = [], 0
            if len(lists) == batches:
                break
        r.out = serve.allocate_output(r, torch.cuda.current_stream())
        keep.append(r)
        cur.append(serve.batch_task(r))
        cur_bytes += m
    torch.cuda.synchronize()
    return lists, total, keep


def search_serve(reps: int = 3, space=None, verbose=False, batches: int = 24):
    """Time every batch configuration on the server's batches (each a direct
    launch of an empty-created plan updated with the batch, as the server
    runs them); returns [(ms per pass over the batches, (block, ppt,
    grid_per_cu, nt))] sorted, the FP64 batch configuration's ms, and the
    moved bytes of one pass, and installs the fastest as the server's."""
    from . import batch as B
    lists, total, keep = serve_workload(batches)
    cus = torch.cuda.get_device_properties(torch.cuda.current_device()).multi_processor_count
    space = space or list(itertools.product(BATCH_BLOCKS, BATCH_PPTS, BATCH_GRID_PER_CU, BATCH_STORE_MODES))
    cap = max(len(t) for t in lists)

    def one(cfg):
        block, ppt, gpc, nt = cfg
        plan = B.Plan([], capacity=cap, block=block, ppt=ppt, grid=cus * (gpc or max(1, 2048 // block)),
                      nontemporal=nt)

        def run():
            for tasks in lists:
                plan.update(tasks)
                plan.run(graph=False)
        try:
            return time_launch(run, reps, 1)
        finally:
            plan.close()

    results = []
    for cfg in space:
        if cfg[0] * cfg[1] * 25 * 8 > 160 * 1024:  # 3D FP64 Jacobian staging must fit in LDS
            continue
        try:
            ms = one(cfg)
        except F.FdbbError:
            continue
        results.append((ms, cfg))
        if verbose:
            print(f"  serve cfg={cfg} {ms:.4f} ms", file=sys.stderr, flush=True)
    results.sort()
    base = F.fdbb_get_batch_config(F.F64)
    base_ms = dict((c, ms) for ms, c in results).get(tuple(base))
    if results:
        F.fdbb_set_server_batch_config(*results[0][1])
    del keep, lists
    torch.cuda.empty_cache()
    return results, base_ms, total


def load_table(path: str = DEFAULT_TABLE):
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return None


def apply_table(path: str = DEFAULT_TABLE, key: str | None = None) -> int:
    """Install the table's configurations for this device; returns how many."""
    table = load_table(path)
    if not table:
        return 0
    if key is None:
        try:
            key = arch_key()
        except Exception:
            return 0
    entries = table.get(key) or {}
    count = 0
    for name, e in entries.items():
        parts = name.split("/")
        try:
            if parts[0] == "serve_batch":
                F.fdbb_set_server_batch_config(e["block"], e["ppt"], e["grid_per_cu"], e["nt"])
                count += 1
                continue
            if parts[0] in ("tiny", "small", "huge") and len(parts) == 4:
                cls, op, dim, dt = parts
                F.fdbb_install_launch_config(op, int(dim), DT[dt][0], CLASSES[cls][0], e["min_n" if cls == "huge" else "max_n"],
                                             e["block"], e["ppt"], e["grid_cap"], e["nt"])
                count += 1
                continue
            op, dim, dt = parts
            code = DT[dt][0]
            if op == "batch":
                F.fdbb_set_batch_config(code, e["block"], e["ppt"], e["grid_per_cu"], e["nt"])
            else:
                F.fdbb_install_launch_config(op, int(dim), code, 2, 0, e["block"], e["ppt"], e["grid_cap"], e["nt"])
        except (F.FdbbError, KeyError, ValueError) as exc:  # an entry this library does not take
            print(f"fdbb: ignoring tuned entry {name}: {exc}", file=sys.stderr)
            continue
        count += 1
    return count


def main(argv=None):
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--ops", default="fused")
    ap.add_argument("--dims", default="3")
    ap.add_argument("--dtypes", default="f64,f32")
    ap.add_argument("--n", default="auto",
                    help="points per launch, or 'auto' for the sizes of both classes")
    ap.add_argument("--reps", type=int, default=7)
    ap.add_argument("--small", type=int, default=0,
                    help="tune the small-launch class at this many points instead of the large one")
    ap.add_argument("--write", default=None, help="merge results into this JSON table")
    ap.add_argument("--verbose", action="store_true")
    args = ap.parse_args(argv)
    torch.cuda.set_device(0)
    key = arch_key()
    table = (load_table(args.write) if args.write else None) or {}
    entries = table.setdefault(key, {})
    for op in args.ops.split(","):
        if op == "serve":
            res, base_ms, total = search_serve(max(3, args.reps - 4), verbose=args.verbose)
            if res:
                best_ms, (block, ppt, gpc, nt) = res[0]
                entries["serve_batch/0/mix"] = {"block": block, "ppt": ppt, "grid_per_cu": gpc, "nt": nt,
                                                "ms": round(best_ms, 5), "bytes": total,
                                                "fp64_batch_config_ms": round(base_ms, 5) if base_ms else None,
                                                "top5": [[round(ms, 5), list(c)] for ms, c in res[:5]]}
                print(json.dumps({"serve_batch/0/mix": entries["serve_batch/0/mix"]}), flush=True)
            continue
        if op == "batch":
            # the batched workload is 3D whatever --dims says
            for dt in args.dtypes.split(","):
                times, points = search_batch(dt, max(3, args.reps - 2), verbose=args.verbose)
                if not times:
                    continue
                rows = rank(times)
                block, ppt, gpc, nt = rows[0][2]
                entries[f"batch/3/{dt}"] = {"block": block, "ppt": ppt, "grid_per_cu": gpc, "nt": nt, "n": points,
                                            "ms": [round(t, 4) for t in times[rows[0][2]]],
                                            "top5": [[round(m, 4), round(w, 4), list(c)] for m, w, c in rows[:5]]}
                print(json.dumps({f"batch/3/{dt}": entries[f"batch/3/{dt}"]}), flush=True)
            continue
        for dim in (int(d) for d in args.dims.split(",")):
            for dt in args.dtypes.split(","):
                if args.small:
                    res, large_ms, max_n = search_small(op, dim, dt, args.small, verbose=args.verbose)
                    name = f"small/{op}/{dim}/{dt}"
                    info = {"n": args.small, "large_us": round(large_ms * 1e3, 3),
                            "top5": [[round(ms * 1e3, 3), list(c)] for ms, c in res[:5]]}
                    if max_n:
                        block, ppt, cap, nt = res[0][1]
                        entries[name] = {"max_n": max_n, "block": block, "ppt": ppt, "grid_cap": cap, "nt": nt,
                                         "us": round(res[0][0] * 1e3, 3), **info}
                    else:
                        entries.pop(name, None)
                    print(json.dumps({name: entries.get(name, {"kept_large": True, **info})}), flush=True)
                    continue
                if args.n == "auto":
                    tune_range(op, dim, dt, entries)
                    continue
                n = int(args.n)
                res = search(op, dim, dt, n, args.reps, verbose=args.verbose)
                if not res:
                    print(f"fdbb: no usable configuration for {op}/{dim}/{dt} (all spill or are refused)",
                          file=sys.stderr, flush=True)
                    continue
                best_ms, (block, ppt, cap, nt) = res[0]
                base = [ms for ms, cfg in res if cfg == (256, 1 if op in ("fused", "flux_jacobian", "viscous_flux") else
                                                         (2 if dt == "f64" else 4), 0, 1)]
                entries[f"{op}/{dim}/{dt}"] = {"block": block, "ppt": ppt, "grid_cap": cap, "nt": nt,
                                               "ms": round(best_ms, 5), "n": n,
                                               "default_ms": round(base[0], 5) if base else None,
                                               "top5": [[round(ms, 5), list(c)] for ms, c in res[:5]]}
                print(json.dumps({f"{op}/{dim}/{dt}": entries[f"{op}/{dim}/{dt}"]}), flush=True)
    if args.write:
        with open(args.write, "w") as f:
            json.dump(table, f, indent=1, sort_keys=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
