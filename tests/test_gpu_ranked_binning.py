"""Ranked binning at the edges of its blocks, tables and range (GPU): tile
lists of given splats without culling equal the oracle's bit for bit, and with
culling the image stays bit-identical.  Cases: one splat, one less, one more
and as many as a block holds; one more than a chunk of blocks; splats with more
rows of super-tiles than the span table's eight and wider than its 255 columns
(whose spans the scatter finds again); the largest grid of super-tiles that the
binning takes and the next one, which is emitted and sorted."""
import numpy as np
import pytest

import oracle
import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h4d():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as m
    oracle.build()
    return m


@pytest.mark.parametrize("tile,W,H,n,max_radius", [
    (16, 60, 50, 1, 20), (8, 203, 131, 255, 40), (16, 203, 131, 256, 40), (32, 700, 500, 257, 300),
    (16, 333, 250, 16385, 8), (8, 600, 520, 300, 250), (8, 4096, 30, 60, 3000),
    (16, 4096, 2048, 257, 300), (16, 4160, 2048, 257, 300)])
def test_lists_at_the_edges(h4d, tile, W, H, n, max_radius):
    print(f"[ranked binning] tile {tile} {W}x{H} n={n} r<={max_radius}", flush=True)
    rec = sg.synthetic_records(n, W, H, seed=31, max_radius=max_radius)
    if n == 1:
        rec["visible"][:] = 1
    full = h4d.Rasterizer(tile=tile, chunk=64, pair_capacity=1 << 22, cull=False)
    img, T, ids, ranges = h4d.rasterize_splats(full, rec, W, H)
    start, ref = oracle.tile_lists(rec, W, H, tile)
    ids, rg = ids.cpu().numpy(), ranges.cpu().numpy()
    assert np.array_equal(rg[:, 1] - rg[:, 0], np.diff(start))
    assert np.array_equal(rg[:, 0], start[:-1]) and np.array_equal(ids[:start[-1]], ref)
    culled = h4d.Rasterizer(tile=tile, chunk=64, pair_capacity=1 << 22, cull=True)
    img1, T1, _, ranges1 = h4d.rasterize_splats(culled, rec, W, H)
    assert torch.equal(img, img1) and torch.equal(T, T1)
    assert int(ranges1[-1, 1]) <= int(ranges[-1, 1])


@pytest.mark.parametrize("n", [63, 64, 65, 2000, 16384, 16385, 24577])
def test_depth_order(h4d, n):
    """Short sorts on both sides of their range (ranks by counting to 16384 keys,
    radix passes that sum their own histograms to 24576): a whole-image tile's
    list is the stable depth order, with many equal depths."""
    print(f"[depth order] n={n}", flush=True)
    rng = np.random.default_rng(n)
    W = H = 16
    rec = sg.synthetic_records(n, W, H, seed=32, max_radius=40)
    rec["u"][:], rec["v"][:], rec["radius"][:] = 8.0, 8.0, 30
    rec["visible"] = (rng.uniform(size=n) > 0.1).astype(np.uint8)
    rec["depth"] = (0.5 + rng.integers(0, max(1, n // 7), size=n) / 64.0).astype(np.float32)
    rast = h4d.Rasterizer(tile=16, chunk=64, pair_capacity=1 << 20, cull=False)
    _, _, ids, ranges = h4d.rasterize_splats(rast, rec, W, H)
    seen = np.nonzero(rec["visible"])[0]
    want = seen[np.argsort(rec["depth"][seen], kind="stable")]
    assert ranges.cpu().numpy().tolist() == [[0, len(want)]]
    assert np.array_equal(ids.cpu().numpy()[:len(want)], want)


@pytest.mark.parametrize("depths", ["spread", "equal", "skewed"])
@pytest.mark.parametrize("n", [13000, 13001, 65537, 262145, 524288, 524289, 1048577])
def test_long_depth_order(h4d, n, depths):
    """Sorts by bins of sampled keys, from the ranks' longest segment to the radix
    sort's shortest (beyond 2^18 keys the workgroups' counts are scanned by a launch
    of their own, beyond 2^19 a workgroup takes 8192 keys, not 4096, and the samples are gathered
    first): a whole-image
    tile's list is the stable depth order, also when most depths are equal or nearly
    so."""
    print(f"[long depth order] n={n} {depths}", flush=True)
    rng = np.random.default_rng(n)
    W = H = 16
    rec = sg.synthetic_records(n, W, H, seed=32, max_radius=40)
    rec["u"][:], rec["v"][:], rec["radius"][:] = 8.0, 8.0, 30
    rec["visible"] = (rng.uniform(size=n) > 0.3).astype(np.uint8)
    if depths == "spread":
        rec["depth"] = (0.5 + rng.integers(0, n // 7, size=n) / 64.0).astype(np.float32)
    elif depths == "equal":
        rec["depth"] = np.full(n, 2.5, np.float32)
    else:
        rec["depth"] = np.exp2(60.0 * rng.uniform(size=n) ** 9).astype(np.float32)
    rast = h4d.Rasterizer(tile=16, chunk=64, pair_capacity=1 << 21, cull=False)
    _, _, ids, ranges = h4d.rasterize_splats(rast, rec, W, H)
    seen = np.nonzero(rec["visible"])[0]
    want = seen[np.argsort(rec["depth"][seen], kind="stable")]
    assert ranges.cpu().numpy().tolist() == [[0, len(want)]]
    assert np.array_equal(ids.cpu().numpy()[:len(want)], want)
