"""GPU checks of the batched build split around its count (count_batched_async,
then build_batched_counted on the same workspace): the counts equal the
synchronous count, the resumed outputs equal the oracle's grids bit for bit,
and every way the two halves can fail (outputs below NO, pairs beyond the
workspace, a bad vertex index) stops the kernels before they write, with the
status word and the workspace status saying why."""
import numpy as np
import pytest

import oracle
from paper_2403_10647_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_10647_amd import _lib
    _lib.lib()
    return _lib


def _say(*a):
    print(*a, flush=True)


def _batch(seed, sizes):
    out = scenes.make_batch(seed, ngrids=len(sizes), sizes=np.asarray(sizes))
    for s in out:
        if s.ntris == 0:
            s.lo = np.zeros(3, np.float32)
            s.hi = np.ones(3, np.float32)
            s.res = np.asarray([3, 2, 5], np.uint32)
    return out


class _Half:
    """Pinned staging and counts of one split build."""

    def __init__(self, G, n):
        self.stage = torch.empty(2 * int(G.lib().grid_batch_staging_size(n)), dtype=torch.uint8, pin_memory=True)
        self.counts = torch.full((n + 1,), -1, dtype=torch.int64, pin_memory=True)


def _ws_bytes(G, inputs, caps, scale=2):
    arr = G._descs(inputs)
    for d, c in zip(arr, caps):
        d.out.cap_pairs = int(c) * scale
    return int(G.lib().grid_workspace_size_batched(arr, len(inputs)))


def _count(G, inputs, ws, ws_bytes, h, stream=None):
    cap = G.count_batched_async(inputs, ws, ws_bytes, h.stage, h.counts, stream)
    (stream or torch.cuda.current_stream()).synchronize()
    n = len(inputs)
    return cap, [int(x) for x in h.counts[:n].tolist()], int(h.counts[n])


def _filled(G, inputs, caps):
    outs = G.alloc_results(inputs, caps)
    for o in outs:
        o.cells.fill_(-7)
        o.objs.fill_(-7)
        o.ranges.fill_(-7)
    return outs


def _untouched(outs):
    return all(bool((o.cells == -7).all()) and bool((o.objs == -7).all()) and bool((o.ranges == -7).all())
               for o in outs)


def _oracle_equal(outs, batch):
    for o, s in zip(outs, batch):
        oc, oo, orr = oracle.build_scene(s)
        c, ob, r = o.numpy()
        assert np.array_equal(c, oc) and np.array_equal(ob, oo) and np.array_equal(r, orr), s.name


def test_split_build_equals_oracle(G):
    batch = _batch(41, [1, 0, 5000, 17, 90_000, 3, 2049, 777])
    batch[5].res = np.asarray([1, 1, 1], np.uint32)
    _say("split uneven", [s.ntris for s in batch])
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, caps)
    ws.get(wsb)
    h = _Half(G, len(inputs))
    cap, counts, status = _count(G, inputs, ws, wsb, h)
    assert counts == caps and status == 0 and cap >= sum(caps)
    outs = G.alloc_results(inputs, caps)
    G.build_batched_counted(inputs, outs, caps, ws, wsb, h.stage)
    st, total = G.workspace_status(ws)
    assert st == G.GRID_OK and total == sum(caps)
    _oracle_equal(outs, batch)


def test_split_outputs_below_count_are_left_untouched(G):
    batch = _batch(42, [300, 400, 500])
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, caps)
    ws.get(wsb)
    h = _Half(G, 3)
    _, counts, status = _count(G, inputs, ws, wsb, h)
    assert counts == caps and status == 0
    small = list(caps)
    small[1] -= 1
    outs = _filled(G, inputs, small)
    G.build_batched_counted(inputs, outs, small, ws, wsb, h.stage)
    assert G.workspace_status(ws)[0] == G.GRID_E_CAPACITY
    assert _untouched(outs)
    # the same workspace serves the next split build
    _count(G, inputs, ws, wsb, h)
    outs = G.alloc_results(inputs, caps)
    G.build_batched_counted(inputs, outs, caps, ws, wsb, h.stage)
    assert G.workspace_status(ws)[0] == G.GRID_OK
    _oracle_equal(outs, batch)


def test_split_pairs_beyond_the_workspace(G):
    batch = _batch(43, [20_000, 30_000, 25_000])
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, [c // 3 for c in caps], scale=1)   # room for about a third of the pairs
    ws.get(wsb)
    h = _Half(G, 3)
    cap, counts, status = _count(G, inputs, ws, wsb, h)
    _say("split over workspace", cap, sum(caps), status)
    assert cap < sum(caps)
    assert status == G.COUNT_OVER_WORKSPACE
    assert counts == caps                      # the per-grid counts are still exact
    outs = _filled(G, inputs, caps)
    G.build_batched_counted(inputs, outs, caps, ws, wsb, h.stage)
    assert G.workspace_status(ws)[0] == G.GRID_E_CAPACITY
    assert _untouched(outs)


def test_split_bad_index(G):
    batch = _batch(44, [200, 300])
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    bad = batch[1].tris.copy()
    bad[57, 1] = batch[1].verts.shape[1] + 5
    inputs[1] = G.GridInput(inputs[1].verts, torch.from_numpy(bad.view(np.int32)).cuda(), inputs[1].lo,
                            inputs[1].hi, inputs[1].res)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, caps)
    ws.get(wsb)
    h = _Half(G, 2)
    _, _, status = _count(G, inputs, ws, wsb, h)
    assert status & G.COUNT_BAD_INDEX
    outs = _filled(G, inputs, caps)
    G.build_batched_counted(inputs, outs, caps, ws, wsb, h.stage)
    assert G.workspace_status(ws)[0] == G.GRID_E_BADINDEX
    assert _untouched(outs)


def test_split_refuses_other_grids(G):
    batch = _batch(45, [100, 200, 300])
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, caps)
    ws.get(wsb)
    h = _Half(G, 3)
    _count(G, inputs, ws, wsb, h)
    swapped = [inputs[1], inputs[0], inputs[2]]
    outs = G.alloc_results(swapped, [caps[1], caps[0], caps[2]])
    with pytest.raises(G.GridError) as e:
        G.build_batched_counted(swapped, outs, [caps[1], caps[0], caps[2]], ws, wsb, h.stage)
    assert e.value.status == G.GRID_E_INVAL


def test_split_builds_interleaved_on_two_streams(G):
    a = _batch(46, [40_000, 1000, 70_000])
    b = _batch(47, [5, 120_000, 300, 8000])
    ia = [G.GridInput.from_scene(s) for s in a]
    ib = [G.GridInput.from_scene(s) for s in b]
    ca, cb = G.count_batched(ia), G.count_batched(ib)
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    wa, wb = G.Workspace(), G.Workspace()
    ba, bb = _ws_bytes(G, ia, ca), _ws_bytes(G, ib, cb)
    wa.get(ba)
    wb.get(bb)
    ha, hb = _Half(G, 3), _Half(G, 4)
    torch.cuda.synchronize()
    G.count_batched_async(ia, wa, ba, ha.stage, ha.counts, sa)
    G.count_batched_async(ib, wb, bb, hb.stage, hb.counts, sb)
    sb.synchronize()
    assert [int(x) for x in hb.counts[:4].tolist()] == cb
    ob = G.alloc_results(ib, cb)
    G.build_batched_counted(ib, ob, cb, wb, bb, hb.stage, sb)   # b resumes while a may still count
    sa.synchronize()
    assert [int(x) for x in ha.counts[:3].tolist()] == ca
    oa = G.alloc_results(ia, ca)
    G.build_batched_counted(ia, oa, ca, wa, ba, ha.stage, sa)
    assert G.workspace_status(wa, sa)[0] == G.GRID_OK and G.workspace_status(wb, sb)[0] == G.GRID_OK
    _oracle_equal(oa, a)
    _oracle_equal(ob, b)


def test_split_by_records_checks_capacities(G):
    # a batch that is built by records, whose first kernel is where its outputs' capacities are known: every wave
    # checks them by itself, and nothing is written when one is too small
    batch = _batch(48, [60_000, 50_000, 70_000])
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, caps)
    ws.get(wsb)
    h = _Half(G, 3)
    for less in (1, 0):
        _, counts, status = _count(G, inputs, ws, wsb, h)
        assert counts == caps and status == 0
        given = [caps[0], caps[1], caps[2] - less]
        outs = _filled(G, inputs, given)
        _say("split by records", given)
        G.trace_enable(True)
        G.trace_read()
        try:
            G.build_batched_counted(inputs, outs, given, ws, wsb, h.stage)
        finally:
            k = G.trace_read()
            G.trace_enable(False)
        assert "records" in k, sorted(k)
        assert G.workspace_status(ws)[0] == (G.GRID_E_CAPACITY if less else G.GRID_OK)
        if less:
            assert _untouched(outs)
        else:
            _oracle_equal(outs, batch)


def _resumed(G, batch):
    """The kernels of the second half, after the results are checked."""
    inputs = [G.GridInput.from_scene(s) for s in batch]
    caps = G.count_batched(inputs)
    ws = G.Workspace()
    wsb = _ws_bytes(G, inputs, caps)
    ws.get(wsb)
    h = _Half(G, len(batch))
    _, counts, status = _count(G, inputs, ws, wsb, h)
    assert counts == caps and status == 0
    outs = _filled(G, inputs, caps)
    G.trace_enable(True)
    G.trace_read()
    try:
        G.build_batched_counted(inputs, outs, caps, ws, wsb, h.stage)
    finally:
        k = G.trace_read()
        G.trace_enable(False)
    assert G.workspace_status(ws)[0] == G.GRID_OK
    _oracle_equal(outs, batch)
    return k


def test_split_builds_go_by_what_was_counted(G):
    # the second half knows the pairs: few a triangle are sorted as pairs whatever the triangles alone suggest
    rng = np.random.default_rng(49)
    few = []
    for n in (150_000, 90_001):
        c = rng.uniform(0.0, 10.0, (n, 1, 3))
        verts, tris = scenes.soup_from_vertices(c + rng.uniform(-0.01, 0.01, (n, 3, 3)))
        lo, hi = scenes.aabb_bounds(verts)
        few.append(scenes.Scene(f"few{n}", verts, tris, lo, hi, scenes.resolution_rule(lo, hi, n, 4.0, 512)))
    _say("split, few pairs a triangle")
    k = _resumed(G, few)
    assert "finish" not in k and "onesweep_grids" in k, sorted(k)
    _say("split, many pairs a triangle")
    k = _resumed(G, [few[0]] + _batch(50, [120_000, 0, 150_000]))
    assert "finish" in k and "onesweep_grids" not in k, sorted(k)


def test_split_by_records_of_huge_triangles(G):
    # triangles of thousands of records among small ones: the runs of tile owners that the count leaves to the plan
    batch = _batch(51, [40_000, 30_000])
    big = np.asarray([[[0.01, 0.01, 0.01], [9.99, 0.02, 9.98], [5.0, 9.99, 5.0]], [[9.8, 9.7, 2.0], [0.3, 5.0, 9.0], [6.0, 0.2, 4.0]]])
    for s, at in zip(batch, (0, 20_000)):
        for i, b in enumerate(big):
            t = s.tris[at + 9 * i]
            s.verts[:, t] = b.T
        s.res = np.asarray([300, 300, 300], np.uint32)
    _say("split, huge triangles")
    k = _resumed(G, batch)
    assert "finish" in k, sorted(k)
