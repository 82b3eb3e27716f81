"""Builds by records against the CPU oracle, bit for bit, where their pieces change over: segment
widths and row groups, segments at the edges of a wave's, a small and a large workgroup's staging,
short and long stretches of empty segments, outputs aligned to one word, grids of a batch that share
tiles, and the pairs per triangle below which a build keeps sorting pairs.  Tolerance zero."""
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


def _boxes(lo, hi, res, name):
    """Triangles whose cell boxes are [lo, hi] (inclusive cells, [T, 3]) on a grid of unit cells."""
    lo, hi = np.asarray(lo, np.float64), np.asarray(hi, np.float64)
    a, b = lo + 0.25, hi + 0.75
    v = np.stack([a, b, np.stack([a[:, 0], b[:, 1], a[:, 2]], 1)], 1)
    verts, tris = scenes.soup_from_vertices(v)
    res = np.asarray(res, np.uint32)
    return scenes.Scene(name, verts, tris, np.zeros(3, np.float32), res.astype(np.float32), res)


def _random(rng, n, res, most):
    res = np.asarray(res)
    lo = np.stack([rng.integers(0, r, n) for r in res], 1)
    hi = np.minimum(lo + np.stack([rng.integers(0, min(m, r), n) for m, r in zip(most, res)], 1), res - 1)
    return lo, hi


def _same(r, s):
    c, o, rg = r.numpy()
    oc, oo, orr = oracle.build_scene(s)
    assert r.npairs == len(oc)
    assert np.array_equal(c, oc)
    assert np.array_equal(o, oo)
    assert np.array_equal(rg, orr)


def _build(G, s, by_records=True):
    print("build", s.name, s.ntris, list(s.res), flush=True)
    g = G.GridInput.from_scene(s)
    n, _ = G.count(g)
    G.trace_enable(True)
    G.trace_read()
    try:
        r = G.build(g, cap_pairs=n)
    finally:
        k = G.trace_read()
        G.trace_enable(False)
    assert ("finish" in k) == by_records, sorted(k)
    _same(r, s)


@pytest.mark.parametrize("res", [
    (1, 1, 1), (5, 3, 2), (16, 16, 16), (63, 9, 7), (64, 9, 7), (65, 4, 40), (127, 5, 5), (128, 5, 5), (129, 33, 5),
    (256, 7, 9), (257, 2, 30), (1024, 3, 3), (1, 1024, 1), (1, 1, 1024), (3, 1024, 2), (1000, 1, 2)])
def test_segment_shapes(G, res):
    rng = np.random.default_rng(res[0] * 7 + res[1])
    lo, hi = _random(rng, 140_001, res, (40, 40, 40))
    total = np.cumsum(np.prod(hi - lo + 1, 1))
    n = min(int(np.searchsorted(total, 1 << 19)) + 1, len(total))  # as many pairs as a build by records takes
    _build(G, _boxes(lo[:n], hi[:n], res, f"shapes{res}"), by_records=total[n - 1] >= 4 * n)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 999, 1000, 1001, 1999, 2000, 2001, 4095, 4096, 4097, 12289])
def test_pairs_in_one_cell(G, n):
    # n pairs of single cells in one cell, long rows across it, a few elsewhere
    rng = np.random.default_rng(n)
    res = (150, 6, 4)
    hot = np.tile([[70, 2, 1]], (n, 1))
    row_lo, row_hi = np.tile([[0, 2, 1]], (40, 1)), np.tile([[149, 2, 1]], (40, 1))
    lo, hi = _random(rng, 100, res, (3, 2, 2))
    order = rng.permutation(n + 140)
    _build(G, _boxes(np.concatenate([hot, row_lo, lo])[order], np.concatenate([hot, row_hi, hi])[order], res, f"hot{n}"))


def test_many_pairs_with_hot_cells(G):
    # more pairs than one last launch takes, segments of up to 60,000 among them
    rng = np.random.default_rng(5)
    res = (100, 40, 10)
    lo, hi = _random(rng, 60_000, res, (8, 3, 2))
    hot = np.repeat([[10, 5, 5], [11, 5, 5], [99, 39, 9]], [60_000, 3000, 5000], 0)
    order = rng.permutation(len(lo) + len(hot))
    lo, hi = np.concatenate([lo, hot])[order], np.concatenate([hi, hot + [[0, 1, 0]] * np.ones((len(hot), 1), int)])[order]
    _build(G, _boxes(lo, np.minimum(hi, np.asarray(res) - 1), res, "hot cells"))


@pytest.mark.parametrize("at", [0, 1, 2])
def test_empty_stretches(G, at):
    # nothing for thousands, then hundreds of thousands of cells, at the start, inside or at the end
    res = (512, 64, 64)
    z = [(0, 1, 2, 3), (3, 60, 61, 63), (60, 61, 62, 63)][at]
    rng = np.random.default_rng(at)
    lo = np.stack([rng.integers(0, 512, 600), rng.integers(0, 64, 600), rng.choice(z, 600)], 1)
    hi = np.minimum(lo + [[30, 1, 0]], [[511, 63, 63]])
    _build(G, _boxes(lo, hi, res, f"gaps{at}"))


def test_outputs_aligned_to_one_word(G):
    rng = np.random.default_rng(11)
    res = (90, 20, 10)
    s = _boxes(*_random(rng, 60_001, res, (9, 3, 2)), res, "unaligned")
    g = G.GridInput.from_scene(s)
    n, _ = G.count(g)

    def odd(k):
        return torch.zeros(k + 3, dtype=torch.int32, device="cuda")[1:k + 1]
    out = G.GridResult(odd(n), odd(n), odd(2 * g.ncells), 0)
    _same(G.PlainBuild(g, out, G.Workspace())(), s)


def test_batched_grids_share_tiles(G):
    rng = np.random.default_rng(3)
    shapes = [((40, 30, 20), 900), ((1, 1, 1), 3), ((300, 2, 5), 50), ((8, 8, 8), 0), ((16, 16, 16), 20_000), ((200, 100, 9), 20),
              ((64, 64, 4), 36_000), ((2, 2, 2), 2500)]
    ss = [_boxes(*_random(rng, n, res, (12, 4, 3)), res, f"b{i}") if n else
          scenes.Scene("empty", np.zeros((3, 0), np.float32), np.zeros((0, 3), np.uint32), np.zeros(3, np.float32),
                       np.ones(3, np.float32), np.asarray(res, np.uint32)) for i, (res, n) in enumerate(shapes)]
    inputs = [G.GridInput.from_scene(s) for s in ss]
    G.trace_enable(True)
    G.trace_read()
    try:
        results = G.build_batched(inputs)
    finally:
        k = G.trace_read()
        G.trace_enable(False)
    assert "finish" in k, sorted(k)
    for r, s in zip(results, ss):
        torch.cuda.synchronize()
        if s.ntris:
            _same(r, s)
        else:
            assert r.npairs == 0 and not r.ranges.any()


def test_few_pairs_a_triangle_sort_pairs(G):
    # pairs of one cell each: by pairs; more of them in larger boxes: by records; few, unless a pass falls away: by pairs
    rng = np.random.default_rng(8)
    res = (120, 60, 30)
    lo, _ = _random(rng, 300_000, res, (1, 1, 1))
    _build(G, _boxes(lo, lo, res, "points"), by_records=False)
    lo, hi = _random(rng, 160_000, res, (5, 3, 2))
    _build(G, _boxes(lo, hi, res, "boxes"), by_records=True)
    _build(G, _boxes(lo[:40_000], hi[:40_000], res, "fewer boxes"), by_records=False)


@pytest.mark.parametrize("n,over,route", [(200_000, 1, "records"), (200_000, 5, "records"), (150_000, 30, "pairs"), (4000, 100, "compact")])
def test_statistics_choose_among_all_paths(G, n, over, route):
    # build_path 2: by records where the count bears them out, whatever the capacity says
    s = scenes.make_scene("mixed" if route == "records" else "uniform", seed=3, ntris=n)
    g = G.GridInput.from_scene(s)
    no, _ = G.count(g)
    print("statistics", n, no, over, flush=True)
    G.tune_set("build_path", 2)
    G.trace_enable(True)
    G.trace_read()
    try:
        r = G.build(g, cap_pairs=no * over)
        last = G.tune_get("last_path")
    finally:
        k = G.trace_read()
        G.trace_enable(False)
        G.tune_set("build_path", 0)
    assert last == (1 if route == "compact" else 0)
    assert ("finish" in k) == (route == "records") and ("compact_scan" in k) == (route == "compact"), sorted(k)
    _same(r, s)


def _kernels(G, f):
    G.trace_enable(True)
    G.trace_read()
    try:
        r = f()
        torch.cuda.synchronize()
    finally:
        k = G.trace_read()
        G.trace_enable(False)
    return r, k


def test_outputs_with_room_go_by_the_pairs_expected(G):
    # one pair a triangle into outputs of six times as many: by the capacity (records) while nothing better is
    # known, by pairs once the output, or the caller, says how many there are; too many is no answer
    rng = np.random.default_rng(12)
    res = (120, 60, 30)
    lo, _ = _random(rng, 200_000, res, (1, 1, 1))
    s = _boxes(lo, lo, res, "points with room")
    g = G.GridInput.from_scene(s)
    n, _ = G.count(g)
    out = G.alloc_results([g], [6 * n])[0]
    b = G.PlainBuild(g, out, G.Workspace())
    r, k = _kernels(G, b)
    assert "finish" in k
    _same(r, s)
    r, k = _kernels(G, b)
    assert "finish" not in k
    _same(r, s)
    r, k = _kernels(G, lambda: G.build(g, out=out))
    assert "finish" not in k
    _same(r, s)
    out.npairs = 6 * n + 1
    r, k = _kernels(G, lambda: G.build(g, out=out))
    assert "finish" in k
    _same(r, s)
    # batches: the same, and the asynchronous build is told
    outs = G.alloc_results([g, g], [6 * n, 6 * n])
    bb = G.BatchedBuild([g, g], outs, G.Workspace())
    for first in (True, False):
        rs, k = _kernels(G, bb)
        assert ("finish" in k) == first
        for r in rs:
            _same(r, s)
    outs = G.alloc_results([g, g], [6 * n, 6 * n])
    stage = torch.empty(int(G.lib().grid_batch_staging_size(2)), dtype=torch.uint8, pin_memory=True)
    ws = G.Workspace()
    _, k = _kernels(G, lambda: G.build_batched_async([g, g], outs, [n, n], ws, stage))
    assert "finish" not in k and G.workspace_status(ws) == (G.GRID_OK, 2 * n)
    for r in outs:
        _same(r, s)


def test_more_pairs_than_expected(G):
    # an expectation far below the count leaves the result as it is
    s = scenes.make_scene("mixed", seed=8, ntris=150_000)
    g = G.GridInput.from_scene(s)
    n, _ = G.count(g)
    for say in (1, n // 50, n // 2):
        out = G.alloc_results([g], [n + 7])[0]
        out.npairs = say
        _same(G.PlainBuild(g, out, G.Workspace())(), s)
