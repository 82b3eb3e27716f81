"""Builds by records of crowded scenes: a segment's records in chunks (one, several, enough for groups of
chunks, more than the most there can be), chunks whose pairs exceed a workgroup's staging, long stretches of
empty segments in pieces, crowded segments in every grid of a batch and on many task lists.  Against the CPU
oracle bit for bit, tolerance zero; and a scene in a corner of its box takes no multiple of the time that
sorting its pairs does, which is equal work per pair however they lie."""
import numpy as np
import pytest

import oracle
from paper_2403_10647_amd import scenes
from test_gpu_records import _boxes, _build, _random, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_10647_amd import _lib
    _lib.lib()
    return _lib


def _hot(n, cells=4, seed=0):
    # n boxes over the same few cells of one row, and some in other rows
    rng = np.random.default_rng(seed)
    few = n < 4096   # (so that a radix pass falls away by records)
    res = (150, 6, 4) if few else (150, 60, 60)
    lo, hi = _random(rng, 300, (20, 6, 2), (9, 2, 1))
    lo, hi = np.minimum(lo + [0, 0, 2], np.asarray(res) - 1), np.minimum(hi + [0, 0, 2], np.asarray(res) - 1)
    order = rng.permutation(n + 300)
    return _boxes(np.concatenate([np.tile([[70, 2, 1]], (n, 1)), lo])[order],
                  np.concatenate([np.tile([[69 + cells, 2, 1]], (n, 1)), hi])[order], res, f"hot{n}x{cells}")


# pairs of the crowded segment, in chunks of 2048: 1, 2, 63 to 65 (where groups of 32 begin), 95, 96, 128, and beyond the most (2048)
@pytest.mark.parametrize("n", [63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 32_255, 32_256, 32_767, 32_768, 33_280, 49_151, 49_152, 65_537,
                               1_060_003])
def test_chunks_of_a_segment(G, n):
    _build(G, _hot(n))


def test_more_pairs_than_all_chunks_stage(G):
    # 8.6M pairs in one cell's segment: 2048 chunks of more than a workgroup stages, in rounds
    _build(G, _hot(430_001, cells=20, seed=2))


@pytest.mark.parametrize("seed", range(4))
def test_chunks_of_uneven_records(G, seed):
    # bursts of one-cell boxes and of rows across the segment, in object order: chunks of equal records hold
    # between a few and many times the pairs staged
    rng = np.random.default_rng(seed)
    res = (150, 60, 60)
    lo, hi = [], []
    while sum(len(x) for x in lo) < 30_000:
        k = int(rng.integers(1, 600 if seed % 2 else 60))
        long = rng.random() < 0.3
        x0 = rng.integers(0, 20 if long else 150, k)
        x1 = x0 + (rng.integers(60, 130, k) if long else 0)
        yz = np.tile([[2, 1]], (k, 1))
        lo.append(np.column_stack([x0, yz]))
        hi.append(np.column_stack([np.minimum(x1, 149), yz]))
    _build(G, _boxes(np.concatenate(lo), np.concatenate(hi), res, f"uneven{seed}"))


@pytest.mark.parametrize("rows", [(3, 5), (16, 17), (33, 40), (64, 129)])
def test_pieces_of_empty_stretches(G, rows):
    # empty stretches of a few thousand to a few hundred thousand cells before, between and after crowded rows
    rng = np.random.default_rng(rows[0])
    res = (500, 33, 24)
    at = np.concatenate([np.repeat([[r % 33, r // 33]], 3000, 0) for r in (*rows, 33 * 20 + 7)])
    x = rng.integers(0, 490, len(at))
    lo = np.column_stack([x, at])
    hi = np.column_stack([x + rng.integers(3, 10, len(at)), at])
    order = rng.permutation(len(at))
    _build(G, _boxes(lo[order], hi[order], res, f"stretches{rows}"))


def test_crowded_segments_of_a_batch(G):
    # crowded cells in grids of different widths, on either side of shared tiles, with an empty grid between
    rng = np.random.default_rng(3)
    shapes = [((40, 30, 20), 900, 30_000), ((1, 1, 1), 3, 0), ((300, 2, 5), 50, 5000), ((8, 8, 8), 0, 0), ((16, 16, 16), 20_000, 700),
              ((200, 100, 9), 20, 40_000), ((64, 64, 4), 36_000, 2000)]
    ss = []
    for i, (res, n, hot) in enumerate(shapes):
        if n == 0:
            ss.append(scenes.Scene("empty", np.zeros((3, 0), np.float32), np.zeros((0, 3), np.uint32), np.zeros(3, np.float32),
                                   np.ones(3, np.float32), np.asarray(res, np.uint32)))
            continue
        lo, hi = _random(rng, n, res, (12, 4, 3))
        c = np.minimum(np.asarray([res[0] // 2, res[1] - 1, 0]), np.asarray(res) - 1)
        lo = np.concatenate([lo, np.tile(c, (hot, 1))])
        hi = np.concatenate([hi, np.tile(np.minimum(c + [5, 0, 0], np.asarray(res) - 1), (hot, 1))])
        order = rng.permutation(len(lo))
        ss.append(_boxes(lo[order], hi[order], res, f"b{i}"))
    inputs = [G.GridInput.from_scene(s) for s in ss]
    G.trace_enable(True)
    G.trace_read()
    try:
        results = G.build_batched(inputs)
    finally:
        k = G.trace_read()
        G.trace_enable(False)
    assert "finish" in k, sorted(k)
    torch.cuda.synchronize()
    for r, s in zip(results, ss):
        if s.ntris:
            _same(r, s)
        else:
            assert r.npairs == 0 and not r.ranges.any()


def test_many_task_lists(G):
    # a large grid with thousands of crowded segments among sparse ones
    rng = np.random.default_rng(9)
    res = (400, 200, 150)
    lo, hi = _random(rng, 200_000, res, (12, 6, 5))
    at = np.column_stack([rng.integers(0, 390, 300), rng.integers(0, 200, 300), rng.integers(0, 150, 300)])
    hot = np.repeat(at, rng.integers(100, 3000, 300), 0)
    lo, hi = np.concatenate([lo, hot]), np.concatenate([hi, hot + [[3, 0, 0]]])
    order = rng.permutation(len(lo))
    _build(G, _boxes(lo[order], hi[order], res, "many lists"))


def test_a_corner_takes_no_multiple_of_its_pairs_sort(G):
    # half a million boxes of 8 cells over 64 cells of a grid of 2M
    rng = np.random.default_rng(4)
    lo = rng.integers(0, 3, (500_000, 3))
    s = _boxes(lo, lo + 1, (128, 128, 128), "corner")
    g = G.GridInput.from_scene(s)
    n, _ = G.count(g)
    b = G.PlainBuild(g, G.alloc_results([g], [n])[0], G.Workspace())

    def us(fused):
        G.tune_set("fused_expand", fused)
        try:
            t = []
            for _ in range(12):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                b()
                e1.record()
                e1.synchronize()
                t.append(1000 * e0.elapsed_time(e1))
            return sorted(t)[len(t) // 2]
        finally:
            G.tune_set("fused_expand", 0)
    pairs, here = us(1), us(0)
    print("corner", n, "pairs", pairs, here, flush=True)
    _same(b(), s)
    assert here < 3 * pairs   # (one workgroup a segment took 16 times as long)
