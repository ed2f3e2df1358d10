"""The shipped table is what the tuner makes of the times it records, and the
tuner's choice among shapes, on the CPU."""
import json

from paper_1809_09851_amd import fdbb as F
from paper_1809_09851_amd import tune


def test_every_entry_is_its_recorded_winner():
    tables = tune.load_table()
    assert tables
    for table in tables.values():
        for name, e in table.items():
            check(name, e)


def check(key, e):
    if key == "serve_batch/0/mix":
        assert [e["block"], e["ppt"], e["grid_per_cu"], e["nt"]] == e["top5"][0][1]
        assert e["ms"] == e["top5"][0][0] == min(t for t, _ in e["top5"])
        return
    last = "grid_per_cu" if key.startswith("batch/") else "grid_cap"
    lead, *rest = e["top5"]
    assert [e["block"], e["ppt"], e[last], e["nt"]] == lead[2], key
    assert all(lead[0] <= m * (1 + tune.KEEP_MARGIN) + 2e-4 for m, _, _ in rest), key
    if last == "grid_per_cu":
        assert len(e["ms"]) == len(e["n"]) == len(tune.BATCH_LISTS)
        return
    cls = key.split("/")[0] if key.count("/") == 3 else "large"
    level, bound, sizes = tune.CLASSES[cls]
    assert len(e["us"]) == 2 * len(e["sizes"]) and set(e["sizes"]) <= set(sizes)
    assert level == 2 or e["min_n" if level == 3 else "max_n"] == bound


def test_rank_takes_the_steadiest_of_the_near_equal():
    times = {"a": [10.0, 10.0, 14.0], "b": [10.5, 10.5, 12.6], "c": [20.0, 10.0, 10.0], "d": [10.51, 10.49, 12.6]}
    rows = tune.rank(times)
    means = {r[2]: r[0] for r in rows}
    assert min(means, key=means.get) in ("a", "b", "d") and rows[0][2] in ("b", "d")
    assert rows[0][1] <= min(r[1] for r in rows[1:] if r[0] <= min(means.values()) * 1.005)
    assert len(rows) == 4


def test_the_shape_in_force_stays_within_the_margin():
    a, b = (64, 1, 0, 1), (128, 1, 0, 1)
    for slower, kept in ((1.029, b), (1.031, a)):
        times = {a: [1.0, 1.0], b: [slower, slower]}
        assert tune.rank(times, b)[0][2] == kept and tune.rank(times)[0][2] == a


def test_classes_without_a_shape_of_their_own_get_no_entry(monkeypatch):
    a, b = (64, 1, 0, 1), (128, 1, 0, 1)
    seen = {}

    def search(op, dim, dt, cls, in_force=None):
        seen[cls] = in_force
        gain = {"tiny": 1.1, "small": 1.01, "large": 1.0, "huge": 1.02}[cls]  # b's time over a's
        return {a: [1.0, 1.0], b: [gain, gain]}, [10]

    monkeypatch.setattr(tune, "search_range", search)
    entry = {"block": 128, "ppt": 1, "grid_cap": 0, "nt": 1}
    entries = {"flux/2/f64": dict(entry), "huge/flux/2/f64": dict(entry, block=512)}
    tune.tune_range("flux", 2, "f64", entries)
    assert seen == {"large": b, "huge": (512, 1, 0, 1), "small": b, "tiny": b}
    assert {k: tune.shape_of(e) for k, e in entries.items()} == {
        "flux/2/f64": b, "huge/flux/2/f64": a, "small/flux/2/f64": b, "tiny/flux/2/f64": a}


def test_table_round_trip_of_all_classes(tmp_path):
    p, key = tmp_path / "t.json", "gfx950/hiptest"
    op, dim, code = "flux", 2, F.F32
    shapes = {"tiny/": (64, 1), "small/": (128, 1), "": (256, 4), "huge/": (512, 2)}
    bound = {"tiny/": {"max_n": 3 << 17}, "small/": {"max_n": 1 << 21}, "": {}, "huge/": {"min_n": 3 << 23}}
    p.write_text(json.dumps({key: {f"{c}{op}/{dim}/f32": {"block": b, "ppt": q, "grid_cap": 0, "nt": 1, **bound[c]}
                                   for c, (b, q) in shapes.items()}}))
    old = F.fdbb_get_launch_config(op, dim, code)
    small = F.fdbb_get_small_launch_config(op, dim, code)
    try:
        assert tune.apply_table(str(p), key=key) == 4
        at = lambda n: F.fdbb_launch_config_for(op, dim, code, n)[:2]
        for c, n in (("tiny/", 3 << 17), ("small/", (3 << 17) + 1), ("small/", 1 << 21), ("", (1 << 21) + 1),
                     ("", (3 << 23) - 1), ("huge/", 3 << 23)):
            assert at(n) == shapes[c], n
    finally:
        tune.one_entry(op, dim, code)
        F.fdbb_set_launch_config(op, dim, code, *old)
        F.fdbb_set_small_launch_config(op, dim, code, *small)


def test_range_tuning_times_every_size_and_lifts_other_entries(monkeypatch):
    """Shapes far off at the screening sizes are left out; a shape is timed as
    the only entry in force, and the configuration is restored."""
    op, dim, dt, code = "eos", 2, "f64", F.F64
    seen = []

    def workload(o, d, t, n):
        def call():
            return n
        call.n = n
        return call

    def clock(fns, launches, rounds=4):
        n = fns[0].n
        cfg = F.fdbb_launch_config_for(op, dim, code, n)
        seen.append((n, cfg))
        return 10.0 + abs(cfg[0] - 256) / 100 + cfg[1] + (1 if cfg[2] else 0)

    monkeypatch.setattr(tune, "workload", workload)
    monkeypatch.setattr(tune, "time_graph", clock)
    monkeypatch.setattr(F, "fdbb_kernel_info", lambda *a, **k: (64, 0))
    monkeypatch.setattr(tune.torch.cuda, "empty_cache", lambda: None)
    small = F.fdbb_get_small_launch_config(op, dim, code)
    F.fdbb_install_launch_config(op, dim, code, 0, 1 << 30, 64, 1, 0, 1)
    try:
        times, sizes = tune.search_range(op, dim, dt, "small")
        assert sizes == list(tune.CLASSES["small"][2])
        assert tune.rank(times)[0][2] in {(256, 1, 0, 1), (256, 1, 0, 0)}
        assert {n for n, _ in seen} == set(sizes) and all(len(t) == 2 * len(sizes) for t in times.values())
        assert (1024, 4, 0, 1) not in times and (1024, 4, 0, 1) in {c for _, c in seen}
        times, _ = tune.search_range(op, dim, dt, "small", (1024, 4, 2048, 1))
        assert (1024, 4, 2048, 1) in times
        assert F.fdbb_get_small_launch_config(op, dim, code) == small
    finally:
        tune.one_entry(op, dim, code)
