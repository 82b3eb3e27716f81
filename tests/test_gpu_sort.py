"""The radix sort of pairs (grid_sort_pairs) where its pieces change over: the tails of the histogram's
tiles, an odd number of passes (whose pairs are copied first) and an even one, and the pair count from
which passes run in 16384-pair tiles.  Against a stable sort on the CPU, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_10647_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("bits", [8, 13, 25, 32])
@pytest.mark.parametrize("n", [1, 1023, 8191, 8192, 8193, "few", "enough"])
def test_sort_pairs_edges(G, n, bits):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if isinstance(n, str):
        n = (cus - 1) * 16384 + (1 if n == "enough" else 0)
    print("sort", n, bits, flush=True)
    rng = np.random.default_rng(n + bits)
    keys = rng.integers(0, 1 << bits, n, dtype=np.uint64).astype(np.uint32)
    vals = np.arange(n, dtype=np.uint32)
    # one word in: arrays aligned to 4 bytes only
    kd = torch.from_numpy(np.concatenate([keys[:1], keys]).view(np.int32)).cuda()[1:]
    vd = torch.from_numpy(np.concatenate([vals[:1], vals]).view(np.int32)).cuda()[1:]
    G.sort_pairs(kd, vd, bits)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(kd.cpu().numpy().view(np.uint32), keys[order])
    assert np.array_equal(vd.cpu().numpy().view(np.uint32), vals[order])


@pytest.mark.parametrize("at", [(9, 16, 0), (9, 16, 1), (1, 1, 0), (1, 1, 1), (3, 2, 0), (3, 2, 1)])
def test_build_at_tile_shape_edges(G, at):
    """Builds that sort pairs, with the last pair count of a tile shape of the passes and the first of the
    next: one cell a triangle, so the pairs are as many as the triangles."""
    import oracle
    from paper_2403_10647_amd import scenes
    num, den, past = at
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = (num * cus - 1) // den if den == 16 else num * cus // den
    n = tiles * 16384 + past
    rng = np.random.default_rng(n)
    res = np.array([64, 50, 40], np.uint32)
    lo = np.stack([rng.integers(0, r, n) for r in res], 1)[:, None, :]
    verts, tris = scenes.soup_from_vertices(lo + rng.uniform(0.2, 0.8, (n, 3, 3)))
    s = scenes.Scene(f"one-cell-{n}", verts, tris, np.zeros(3, np.float32), res.astype(np.float32), res)
    print("build", s.name, flush=True)
    g = G.GridInput.from_scene(s)
    r = G.build(g, cap_pairs=n)
    c, o, rg = r.numpy()
    oc, oo, orr = oracle.build_scene(s)
    assert r.npairs == len(oc) == n
    assert np.array_equal(c, oc) and np.array_equal(o, oo) and np.array_equal(rg, orr)
