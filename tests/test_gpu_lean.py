"""The fused kernel for scans whose values fit 32 bits (fused_lean.hip): row
counts around a mini block (256), a staged group (1,024) and a header step
(4,096 rows); survivor counts around the dense threshold and the queue's 256;
every width and encoding that takes a path of its own; direct tables in LDS, in
device memory and hash tables; pruned blocks; batches that are split by kernel.
Results against the CPU oracle, exact (every value is an integer)."""
import numpy as np
import pytest

import oracle
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2605_10511_amd import dpf
    assert torch.cuda.is_available()
    return dpf.Context(0)


ENC = {"day": "DELTA", "step": "DELTA", "ramp": "DELTA", "dic": "DICT", "dkey": "DICT"}


def _table(n: int, seed: int) -> dict:
    rng = np.random.default_rng(seed)
    i = np.arange(n, dtype=np.int64)
    return {
        "a": rng.integers(0, 1000, n, dtype=np.int32),           # the filter: a < s keeps s rows in 1000
        "b": rng.integers(-50, 50, n, dtype=np.int32),
        "c": np.where(i // 256 % 3 == 0, 7, rng.integers(0, 1 << 24, n)).astype(np.int32),  # all of some mini blocks
        "w0": np.full(n, -12345, dtype=np.int32),
        "w1": rng.integers(0, 2, n, dtype=np.int32),
        "w25": rng.integers(0, 1 << 25, n, dtype=np.int32),
        "w26": rng.integers(-(1 << 25), 1 << 25, n, dtype=np.int32),
        "w32": rng.integers(-(1 << 31), 1 << 31, n, dtype=np.int64),
        "wide": rng.integers(0, 1 << 40, n, dtype=np.int64),     # not the lean kernel's
        "far": rng.integers((1 << 40), (1 << 40) + 900, n, dtype=np.int64),
        "day": (i // 700).astype(np.int32),                      # DELTA of width 0 and 1
        "step": (i * 3).astype(np.int32),                        # DELTA of width 0
        "ramp": np.cumsum(rng.integers(0, 40, n)).astype(np.int64) % (1 << 31),  # DELTA, wider
        "dic": rng.choice(np.array([-70000, 3, 5, 1 << 20], dtype=np.int32), n),
        "dkey": rng.choice(np.array([11, 12, 400, 90000], dtype=np.int32), n),
        "k6": rng.integers(-3, 3, n, dtype=np.int32),
        "k9k": rng.integers(0, 9000, n, dtype=np.int32),
        "h20": (i * 7919 % (1 << 20)).astype(np.int32),
    }


def _s(col, mul=1, add=0):
    return {"ref": {"col": col}, "mul": mul, "add": add}


def _spec(filters, group_by, aggs):
    return {"fact": "t", "filters": filters, "probes": [], "group_by": [{"col": c} for c in group_by], "aggs": aggs}


def _lt(s):
    return {"col": "a", "op": "LT", "value": s}


SUMS = {
    "plain": [{"op": "COUNT"}] + [{"op": "SUM", "terms": [_s(c)]} for c in ("w0", "w1", "w25", "w26", "far")],
    "wide": [{"op": "SUM", "terms": [_s("w32")]}, {"op": "SUM", "terms": [_s("dic")]}, {"op": "AVG", "terms": [_s("ramp")]},
             {"op": "SUM", "terms": [_s("step", -2, 9)]}],
    "products": [{"op": "SUM", "terms": [_s("a"), _s("b", -1, 60)]},
                 {"op": "SUM", "terms": [_s("a"), _s("b", -1, 60), _s("w1", 1, 3)]},
                 {"op": "SUM", "terms": [_s("b"), _s("b", -3, 2), _s("w26")]},
                 {"op": "SUM", "terms": [_s("a")]}, {"op": "AVG", "terms": [_s("a")]}, {"op": "SUM", "terms": [_s("a")]},
                 {"op": "SUM", "terms": [{"const": 5}]}],
    "general": [{"op": "SUM", "terms": [_s("wide")]}],
}
FILTERS = {
    "none": [], "nothing": [_lt(-1)], "all": [_lt(1000)], "sparse": [_lt(4)], "staged": [_lt(63)],
    "below": [_lt(365)], "dense": [_lt(400)],
    "ne": [_lt(300), {"col": "b", "op": "NE", "value": 7}, {"col": "c", "op": "NE", "value": 7}],
    "in": [{"col": "k6", "op": "IN", "values": [-3, 0, 2]}, {"col": "c", "op": "BETWEEN", "lo": 5, "hi": 1 << 23}],
    "wide": [{"col": "w26", "op": "GT", "value": 0}, {"col": "w32", "op": "LT", "value": 1 << 30}, {"col": "far", "op": "GE", "value": (1 << 40) + 200}],
    "many": [_lt(900), {"col": "b", "op": "GE", "value": -45}, {"col": "w1", "op": "LE", "value": 1},
             {"col": "w25", "op": "GT", "value": 1000}, {"col": "k6", "op": "NE", "value": 1}],
    "delta": [{"col": "ramp", "op": "GE", "value": 300}, {"col": "day", "op": "LE", "value": 11}],
}
GROUPS = {"one": [], "six": ["k6"], "dict": ["dkey", "w1"], "day": ["day"], "hbm": ["k9k"], "hash": ["h20", "k9k"]}
ROWS = [1, 255, 256, 257, 1023, 1025, 4095, 4097, 3 * 4096 + 77]


# every filter with every row count in turn, sums and groups rotating
@pytest.mark.parametrize("filt", sorted(FILTERS))
@pytest.mark.parametrize("group", sorted(GROUPS))
def test_lean_forms(ctx, filt, group):
    k = sorted(FILTERS).index(filt) + 5 * sorted(GROUPS).index(group)
    for r, sums in enumerate(SUMS):
        n = ROWS[(k + 2 * r) % len(ROWS)]
        t = _table(n, 100 * k + r)
        spec = _spec(FILTERS[filt], GROUPS[group], SUMS[sums])
        db = G.make_db(ctx, {"t": t}, {"t": ENC}, chunk_rows=4096)
        want = oracle.run(spec, {"t": t})
        for mode, kw in (("FUSED", {}), ("FUSED", {"waves_per_wg": 16, "max_workgroups": 1}), ("FRAGMENTED", {})):
            G.say(f"lean {filt} {group} {sums} rows={n} {mode} {kw}")
            G.assert_same(G.run_gpu(db, spec, mode=mode, **kw), want, f"{filt} {group} {sums} {mode} {kw}")


def test_lean_pruned_and_large(ctx):
    """Blocks left out by their zone maps, runs of mini blocks that cross block
    edges, and enough rows for several items a workgroup."""
    n = 1_500_007
    t = _table(n, 3)
    db = G.make_db(ctx, {"t": t}, {"t": ENC}, chunk_rows=2048)
    day = [{"col": "day", "op": "BETWEEN", "lo": 300, "hi": 1700}]
    for filters, group in ((day, ["k6"]), (day + [_lt(30)], ["day"]), (day + [{"col": "step", "op": "GE", "value": 2_000_000}], []),
                           ([_lt(125)], ["k6"]), ([], ["day"]), ([{"col": "day", "op": "GT", "value": 1 << 20}], [])):
        spec = _spec(filters, group, SUMS["products"])
        G.say("lean pruned", filters, group)
        G.assert_same(G.run_gpu(db, spec), oracle.run(spec, {"t": t}), f"{filters} {group}")


def test_lean_split_batch_and_replay(ctx):
    """A batch of plans for both kernels, large enough for two launches: once as
    it is, in static scratch, and replayed from a graph with work in between."""
    import torch
    from paper_2605_10511_amd import dpf
    n = 1_100_000
    t = _table(n, 4)
    dim = {"k": np.arange(0, 9000, 2, dtype=np.int32), "p": (np.arange(0, 9000, 2) % 5).astype(np.int32)}
    tables = {"t": t, "d": dim}
    probe = {"fact": "t", "filters": [_lt(500)],
             "probes": [{"fk": "k9k", "dim": "d", "key": "k", "filters": [], "payloads": ["p"]}],
             "group_by": [{"probe": 0, "payload": 0}], "aggs": [{"op": "COUNT"}, {"op": "SUM", "terms": [_s("a")]}]}
    specs = [_spec([_lt(125)], ["k6"], SUMS["plain"]), probe, _spec([], ["dkey"], SUMS["products"]),
             _spec([_lt(999)], [], SUMS["general"]), _spec([_lt(2)], ["day"], SUMS["wide"])]
    db = G.make_db(ctx, tables, {"t": ENC})
    want = [oracle.run(s, tables) for s in specs]
    plans = [db.plan(s) for s in specs]
    for name, run in (("execute", dpf.execute), ("noalloc", dpf.execute_noalloc)):
        G.say("lean split", name)
        res = run(ctx, plans)
        torch.cuda.synchronize()
        for i in range(len(plans)):
            G.assert_same(res.get(i), want[i], f"{name} {i}")
        res.release()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        res = dpf.execute(ctx, plans, stream=s)
    for k in range(3):
        G.say("lean split replay", k)
        g.replay()
        torch.cuda.synchronize()
        for i in range(len(plans)):
            G.assert_same(res.get(i), want[i], f"replay {k} {i}")
        torch.zeros(1 << 20, device="cuda").sum().item()
    res.release()


# grids of one workgroup (it takes every item from all eight ranges), of three,
# and the default; items of the default size and of one mini block a wave
@pytest.mark.parametrize("max_wg, rows_per_item", [(1, 0), (3, 0), (9, 1024), (0, 1024), (0, 0)])
def test_items_taken_once(ctx, max_wg, rows_per_item):
    """Work items of a lone plan: every kernel (32-bit scan, string, semi-join,
    FSST) over a table with pruned blocks and a ragged end."""
    from tests.conftest import to_strings
    n = 40_000 + 77
    t = _table(n, 8)
    rng = np.random.default_rng(8)
    words = [b"alpha", b"beta", b"gamma", b"delta", b"alphabeta"]
    text = to_strings([b" ".join(words[j] for j in rng.integers(0, 5, 4)) for _ in range(n)])
    tables = {"t": {**t, "s": text, "z": text}, "d": {"k": np.arange(0, 9000, 3, dtype=np.int32)}}
    db = G.make_db(ctx, tables, {"t": {**ENC, "z": "FSST"}}, chunk_rows=2048)
    day = [{"col": "day", "op": "BETWEEN", "lo": 9, "hi": 47}]
    like = {"op": "STR_CONTAINS_SEQ", "s1": b"alpha", "s2": b"gamma"}
    semi = {**_spec([], ["k6"], SUMS["plain"]), "probes": [{"fk": "k9k", "dim": "d", "key": "k", "filters": [], "payloads": []}]}
    for name, spec in (("scan", _spec(day, ["k6"], SUMS["plain"])), ("like", _spec(day + [{"col": "s", **like}], ["k6"], SUMS["plain"])),
                       ("like all", _spec([{"col": "s", **like}], [], SUMS["plain"])), ("semi", semi),
                       ("fsst", _spec(day + [{"col": "z", **like}], ["k6"], SUMS["plain"]))):
        G.say(f"items {name} max_wg={max_wg} rows_per_item={rows_per_item}")
        got = G.run_gpu(db, spec, max_workgroups=max_wg, rows_per_item=rows_per_item)
        G.assert_same(got, oracle.run(spec, tables), name)


# the damaged column's part in the query: (filters, group keys, sums), none of
# them an atom on the column
CORRUPT = {
    "delta key": ("day", ["day"], ["a"]),
    "delta value": ("day", ["k6"], ["day"]),
    "wide delta value": ("ramp", ["k6"], ["ramp"]),
    "for value": ("w25", ["k6"], ["w25"]),
    "wide for value": ("w26", ["k6"], ["w26"]),
    "dict value": ("dic", ["k6"], ["dic"]),
    "dict key": ("dkey", ["dkey"], ["b"]),
}


@pytest.mark.parametrize("keep", ["every row", "few rows"])
@pytest.mark.parametrize("what", sorted(CORRUPT))
def test_corrupt_value_header_reported(ctx, what, keep):
    """A damaged header of a column that no atom reads: mini blocks taken in
    place (every row kept) and rows gathered one by one."""
    from paper_2605_10511_amd import dpf
    col, keys, sums = CORRUPT[what]
    t = _table(20_000, 5)
    filters = [] if keep == "every row" else [_lt(40)]
    assert (t["a"][4 * 256:6 * 256] < 40).any()
    spec = _spec(filters, keys, [{"op": "COUNT"}] + [{"op": "SUM", "terms": [_s(c)]} for c in sums])
    want = oracle.run(spec, {"t": t})
    db = G.make_db(ctx, {"t": t}, {"t": ENC}, placement="HOST_MAPPED")
    offs = db.tables["t"][col].debug_offsets()
    saved = int(offs[5])
    G.say(f"corrupt {what}, {keep}")
    offs[5] = saved + 3  # no longer a whole number of 8-word groups
    with pytest.raises(dpf.DpfError) as e:
        G.run_gpu(db, spec)
    assert e.value.code == dpf.DPF_ERR_CORRUPT
    offs[5] = saved
    G.assert_same(G.run_gpu(db, spec), want, "after repair")


def test_refused_split_batch_leaves_no_trace(ctx):
    """A batch for both kernels whose join plan does not fit the workgroup's LDS
    is refused before anything runs: the scan's group table (above 8,192
    entries, written to the host by a launch of its own) stays empty."""
    import torch
    from paper_2605_10511_amd import dpf
    n = 1 << 21
    t = {c: v for c, v in _table(n, 6).items() if c in ("a", "b", "k9k", "h20")}
    big = {"k": np.arange(8192, dtype=np.int32), "p": (np.arange(8192) % 5).astype(np.int32)}     # 128 KB in LDS
    small = {"k": np.arange(1024, dtype=np.int32), "p": (np.arange(1024) % 3).astype(np.int32)}   # 16 KB
    tables = {"t": t, "big": big, "small": small}
    join = {"fact": "t", "filters": [_lt(500)],
            "probes": [{"fk": "k9k", "dim": "big", "key": "k", "filters": [], "payloads": ["p"]},
                       {"fk": "a", "dim": "small", "key": "k", "filters": [], "payloads": ["p"]}],
            "group_by": [{"probe": 0, "payload": 0}, {"probe": 1, "payload": 0}],
            "aggs": [{"op": "COUNT"}, {"op": "SUM", "terms": [_s("b")]}]}
    specs = [_spec([_lt(700)], ["k9k"], [{"op": "COUNT"}, {"op": "SUM", "terms": [_s("b")]}]), join]
    db = G.make_db(ctx, tables)
    want = [oracle.run(s, tables) for s in specs]
    plans = [db.plan(s) for s in specs]
    for run in (dpf.execute, dpf.execute_noalloc):
        G.say("refused split batch", run.__name__)
        before = ctx.info().launches
        with pytest.raises(dpf.DpfError) as e:
            run(ctx, plans, lds_hash_bytes=150 * 1024)
        assert e.value.code == dpf.DPF_ERR_UNSUPPORTED
        assert ctx.info().launches == before
        res = run(ctx, plans)
        torch.cuda.synchronize()
        for i in range(2):
            G.assert_same(res.get(i), want[i], f"{run.__name__} {i}")
        res.release()


# scans beside a join plan: the batch is split once they save enough, 13 of
# them that keep one row in eight, 4 that keep all, one in order of a key whose
# table is in device memory; never for a sum of 64-bit values
@pytest.mark.parametrize("filt, group, col, plans, split", [
    ([_lt(125)], "k6", "b", 13, True), ([_lt(125)], "k6", "b", 12, False), ([], "k6", "b", 4, True),
    ([], "k6", "b", 3, False), ([], "day", "b", 1, True), ([_lt(125)], "k6", "wide", 20, False),
    ([_lt(50)], "k6", "ramp", 20, True), ([_lt(49)], "k6", "ramp", 20, False), ([_lt(49)], "day", "ramp", 20, True),
    ([_lt(125), {"col": "dkey", "op": "IN", "values": [11, 12, 400, 90000]}], "dkey", "dic", 13, True)])
def test_split_launches(ctx, filt, group, col, plans, split):
    import torch
    from paper_2605_10511_amd import dpf
    t = _table(1 << 20, 7)
    dim = {"k": np.arange(0, 9000, 2, dtype=np.int32), "p": (np.arange(0, 9000, 2) % 5).astype(np.int32)}
    tables = {"t": t, "d": dim}
    join = {**_spec([], [], [{"op": "COUNT"}]), "group_by": [{"probe": 0, "payload": 0}, {"probe": 1, "payload": 0}],
            "probes": [{"fk": fk, "dim": "d", "key": "k", "filters": [], "payloads": ["p"]} for fk in ("k9k", "a")]}
    specs = [_spec(filt, [group], [{"op": "COUNT"}, {"op": "SUM", "terms": [_s(col)]}]), join]
    want = [oracle.run(s, tables) for s in specs]
    db = G.make_db(ctx, tables, {"t": ENC})
    batch = [db.plan(specs[0]) for _ in range(plans)] + [db.plan(join)]
    for run in (dpf.execute, dpf.execute_noalloc):
        G.say("split launches", filt, group, col, plans, run.__name__)
        before = ctx.info().launches
        with pytest.raises(dpf.DpfError) as e:  # a table of 128 KB and the waves' own LDS do not fit
            run(ctx, batch, lds_hash_bytes=160 * 1024, waves_per_wg=16)
        assert e.value.code == dpf.DPF_ERR_UNSUPPORTED
        assert ctx.info().launches == before
        res = run(ctx, batch)
        assert ctx.info().launches == before + (2 if split else 1) + (run is dpf.execute_noalloc)
        torch.cuda.synchronize()
        for i in range(len(batch)):
            G.assert_same(res.get(i), want[i == plans], f"{run.__name__} {i}")
        res.release()


# lone string plans whose share of 8 mini blocks and more a workgroup does not
# divide: rounded down, the rest claimed; an XCD's range that ends early or is
# empty; one mini block
@pytest.mark.parametrize("rows, max_wg", [(157 * 256 - 77, 16), (157 * 256, 11), (129 * 256 + 1, 8), (200 * 256, 8), (9 * 256, 0), (1, 0)])
def test_string_items_taken_once(ctx, rows, max_wg):
    from tests.conftest import to_strings
    t = _table(rows, 9)
    rng = np.random.default_rng(9)
    words = [b"alpha", b"beta", b"gamma", b"delta", b"alphabeta"]
    t["s"] = to_strings([b" ".join(words[j] for j in rng.integers(0, 5, 4)) for _ in range(rows)])
    db = G.make_db(ctx, {"t": t}, {"t": ENC}, chunk_rows=2048)
    like = {"col": "s", "op": "STR_CONTAINS_SEQ", "s1": b"alpha", "s2": b"gamma"}
    for filters in ([like], [{"col": "day", "op": "GE", "value": 3}, like], [{"col": "day", "op": "LE", "value": 51}]):
        spec = _spec(filters, ["k6"], SUMS["plain"])
        G.say("string items", rows, max_wg, len(filters))
        got = G.run_gpu(db, spec, max_workgroups=max_wg)
        want = oracle.run(spec, {"t": t})
        if len(want) == 0:
            assert len(got) == 0
        else:
            G.assert_same(got, want, f"{rows} {max_wg} {filters}")


# the widest packed values the 32-bit kernel takes (31 and 32 bits, full-width
# 32-bit columns) and, with 33 bits and full-width 64-bit columns, those it does
# not: atoms at both ends of the range, rows kept densely and sparsely
@pytest.mark.parametrize("col", ["w31", "w32", "s32", "p32", "w33", "p64"])
@pytest.mark.parametrize("rows", [257, 4096 + 1025])
def test_widest_values(ctx, col, rows):
    rng = np.random.default_rng(rows)
    t = _table(rows, 10)
    t["w31"] = rng.integers(-5, (1 << 31) - 5, rows, dtype=np.int64)
    t["w32"] = rng.integers(1 << 40, (1 << 40) + (1 << 32), rows, dtype=np.int64)
    t["s32"] = rng.integers(-(1 << 31), 1 << 31, rows, dtype=np.int64).astype(np.int32)
    t["p32"] = rng.integers(-100, 100, rows, dtype=np.int32)
    t["w33"] = rng.integers(0, 1 << 33, rows, dtype=np.int64)
    t["p64"] = rng.integers(-100, 100, rows, dtype=np.int64)
    lo, hi = {"w31": (-5, (1 << 31) - 6), "w32": (1 << 40, (1 << 40) + (1 << 32) - 1), "s32": (-(1 << 31), (1 << 31) - 1),
              "p32": (-100, 99), "w33": (0, (1 << 33) - 1), "p64": (-100, 99)}[col]
    t[col][:256:2], t[col][1:256:2] = lo, hi
    db = G.make_db(ctx, {"t": t}, {"t": {**ENC, "p32": "PLAIN", "p64": "PLAIN"}}, chunk_rows=4096)
    aggs = [{"op": "COUNT"}, {"op": "SUM", "terms": [_s(col)]}, {"op": "AVG", "terms": [_s("a")]}]
    mid = (lo + hi) // 2
    for f in ([], [_lt(30)], [{"col": col, "op": "GT", "value": lo}], [{"col": col, "op": "LT", "value": hi}],
              [{"col": col, "op": "NE", "value": lo}], [{"col": col, "op": "NE", "value": hi}, _lt(40)],
              [{"col": col, "op": "EQ", "value": hi}], [{"col": col, "op": "GE", "value": mid}, _lt(900)]):
        spec = _spec(f, ["k6"], aggs)
        G.say("widest values", col, rows, f)
        G.assert_same(G.run_gpu(db, spec), oracle.run(spec, {"t": t}), f"{col} {rows} {f}")


# items that the caller wants small: the 32-bit kernel takes them from 2,048
# rows on (two launches), and at any size where every row is kept
@pytest.mark.parametrize("filt, plans, rows_per_item, launches", [
    ([_lt(125)], 20, 1792, 1), ([_lt(125)], 20, 2048, 2), ([], 5, 256, 2)])
def test_small_items(ctx, filt, plans, rows_per_item, launches):
    import torch
    from paper_2605_10511_amd import dpf
    t = _table(1 << 20, 11)
    tables = {"t": t, "d": {"k": np.arange(0, 9000, 2, dtype=np.int32)}}
    semi = {**_spec([_lt(500)], ["k6"], [{"op": "COUNT"}]),
            "probes": [{"fk": "k9k", "dim": "d", "key": "k", "filters": [], "payloads": []}]}
    specs = [_spec(filt, ["k6"], [{"op": "COUNT"}, {"op": "SUM", "terms": [_s("b")]}]), semi]
    want = [oracle.run(s, tables) for s in specs]
    db = G.make_db(ctx, tables, {"t": ENC})
    batch = [db.plan(specs[0]) for _ in range(plans)] + [db.plan(semi)]
    G.say("small items", rows_per_item)
    before = ctx.info().launches
    res = dpf.execute(ctx, batch, rows_per_item=rows_per_item)
    assert ctx.info().launches == before + launches
    torch.cuda.synchronize()
    for i in range(len(batch)):
        G.assert_same(res.get(i), want[i == plans], f"plan {i}")
    res.release()
