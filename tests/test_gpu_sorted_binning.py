"""Binning by emission and a sort (GPU): views of more super-tiles than the ranked
binning takes, and calls whose capacity leaves its histograms no room.  Images do
not depend on the tile size, and 16-pixel tiles of the same views are binned by
ranks; lists of given splats equal the oracle's."""
import numpy as np
import pytest

import oracle
import scenegen as sg
from sorted_binning import CALLS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h4d():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as m
    oracle.build()
    return m


@pytest.mark.parametrize("name", CALLS)
def test_images_equal_the_ranked_ones(h4d, name):
    sizes, same, n3, n4, tile, batched, cap, _ = CALLS[name]
    print(f"[sorted binning] {name}", flush=True)
    scene = sg.tiny_scene(n3=n3, n4=n4, width=64, height=64, seed=41)
    rng = np.random.default_rng(42)
    for g, n in ((scene.g3, n3), (scene.g4, n4)):
        # small splats, nine in ten too faint for any pixel, as the small capacities need
        g["log_scale"] = (g["log_scale"] - 2.5).astype(np.float32)
        g["opacity"][rng.uniform(size=n) < 0.9] = -9.0
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    views = [sg.look_at((0.0 if same else 0.1 * k, 0.0, -3.0), (0.0, 0.0, 0.0), W, H, t=0.3 + 0.1 * k)
             for k, (W, H) in enumerate(sizes)]
    rast = h4d.Rasterizer(tile=tile, chunk=64, batched=bool(batched), pair_capacity=cap)
    got = rast.forward(g3, g4, views)
    assert rast.capacity == cap  # (the call as it is named)
    want = [h4d.Rasterizer(tile=16, chunk=64).infer(g3, g4, [v]).images[0] for v in views]
    assert all(float((b - b[:, :1, :1]).abs().max()) > 0.1 for b in want)
    for a, b in zip(got.images, want):
        assert torch.equal(a, b)
    # and the views one after another, whose lists the tile lists give
    one = h4d.Rasterizer(tile=tile, chunk=64, pair_capacity=1 << 24)
    h = one.forward(g3, g4, views)
    (ia, ra), (ib, rb) = rast.tile_lists(got), one.tile_lists(h)
    n = int(ra[-1, 1])
    assert n > 1000 and torch.equal(ra, rb) and torch.equal(ia[:n], ib[:n])


def test_lists_of_a_single_pass(h4d):
    sizes, _, n3, n4, tile, _, cap, _ = CALLS["single pass"]
    (W, H), n = sizes[0], n3 + n4
    print("[sorted binning] lists of a single pass", flush=True)
    rec = sg.synthetic_records(n, W, H, seed=43, max_radius=4)
    rec["visible"][np.random.default_rng(44).uniform(size=n) < 0.7] = 0
    rast = h4d.Rasterizer(tile=tile, chunk=64, pair_capacity=cap, cull=False)
    _, _, ids, ranges = h4d.rasterize_splats(rast, rec, W, H)
    assert rast.capacity == cap
    start, ref = oracle.tile_lists(rec, W, H, tile)
    ids, rg = ids.cpu().numpy(), ranges.cpu().numpy()
    assert np.array_equal(rg[:, 0], start[:-1]) and np.array_equal(rg[:, 1], start[1:])
    assert np.array_equal(ids[:start[-1]], ref)
