"""The two ways a group table goes back to the host: copied whole by the fused
kernel's last workgroup (up to 8,192 entries), or compacted by emit_kernel in
slabs of 8,192 slots.  Sizes at the edges of both, results against the CPU
oracle (exact: every value is an integer), repeated so that a run also sees
what the run before it left in the table."""
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


def _table(card: int, n: int) -> dict:
    """Keys at both ends of the range, around the slab edges, and in between."""
    rng = np.random.default_rng(card)
    k = rng.integers(0, card, n, dtype=np.int32)
    edge = [0, 63, 64, 1023, 1024, 8191, 8192, 8193, 16383, 16384, card - 2, card - 1]
    edge = [e for e in edge if 0 <= e < card]
    k[:len(edge)] = edge
    return {"k": k, "v": rng.integers(-1000, 1000, n, dtype=np.int64), "x": rng.integers(0, 10, n, dtype=np.int32)}


# entries = groups x 2 accumulators: one group; the largest copied table and
# the smallest compacted one; one slab and one slot more; a hash group table
# (a second key of 2^20 values takes the range above 2^22)
@pytest.mark.parametrize("card, rows, hashed", [(1, 700, False), (4096, 5000, False), (4097, 5000, False),
                                                (8192, 20000, False), (8193, 3000, False), (30000, 300, False),
                                                (8192, 20000, True), (5, 40, True)])
def test_emit_sizes(ctx, card, rows, hashed):
    import torch
    from paper_2605_10511_amd import dpf
    t = _table(card, rows)
    keys = [{"col": "k"}]
    if hashed:
        t["h"] = (np.arange(rows, dtype=np.int64) * 7919 % (1 << 20)).astype(np.int32)
        t["h"][:2] = 0, (1 << 20) - 1
        keys = [{"col": "h"}, {"col": "k"}]
    spec = {"fact": "f", "filters": [{"col": "x", "op": "LT", "value": 8}], "probes": [], "group_by": keys,
            "aggs": [{"op": "COUNT"}, {"op": "SUM", "terms": [{"ref": {"col": "v"}}]}]}
    want = oracle.run(spec, {"f": t})
    db = G.make_db(ctx, {"f": t}, chunk_rows=4096)
    for mode in ("FUSED", "FRAGMENTED"):
        G.say(f"emit {card} {rows} hashed={hashed} {mode}")
        G.assert_same(G.run_gpu(db, spec, mode=mode), want, mode)
    plan = db.plan(spec)
    for rep in range(2):
        for run in (dpf.execute, dpf.execute_noalloc):
            if run is dpf.execute_noalloc and hashed and rows > 40:
                continue  # above the 8 MiB scratch or not by the rows alone: test_gpu_hash_agg.py
            res = run(ctx, [plan])
            torch.cuda.synchronize()
            G.assert_same(res.get(0), want, f"{run.__name__} {rep}")
            res.release()
    plan.release()


def test_emit_batch(ctx):
    """Nine plans in one launch (more than a workgroup has waves): copied and
    compacted tables side by side, one of them empty."""
    import torch
    from paper_2605_10511_amd import dpf
    cards = [3, 4097, 1, 64, 9000, 257, 4096, 12, 5000]
    tables = {f"f{i}": _table(c, 2000 + i) for i, c in enumerate(cards)}
    db = G.make_db(ctx, tables, chunk_rows=4096)
    specs = [{"fact": f"f{i}", "filters": [{"col": "x", "op": "LT", "value": 5 if i != 3 else 0}], "probes": [],
              "group_by": [{"col": "k"}], "aggs": [{"op": "COUNT"}, {"op": "SUM", "terms": [{"ref": {"col": "v"}}]}]}
             for i in range(len(cards))]
    plans = [db.plan(s) for s in specs]
    for rep in range(2):
        res = dpf.execute(ctx, plans)
        torch.cuda.synchronize()
        for i, s in enumerate(specs):
            want = oracle.run(s, tables)
            got = res.get(i)
            if len(want) == 0:
                assert len(got) == 0
            else:
                G.assert_same(got, want, f"plan {i} run {rep}")
        res.release()
    for p in plans:
        p.release()
