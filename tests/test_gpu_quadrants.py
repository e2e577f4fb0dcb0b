"""Quadrant blending kernels (GPU): launches of few 16 x 16 tiles blend each tile
as four 8 x 8 quadrants, and their adjoint runs the segments of a tile's list at
the same time from the forward's checkpoints.  Images equal the 8-pixel tiles'
(which never take these kernels) bit for bit; gradients meet the oracle's bars,
also where a list goes past the kept head, without checkpoints (a forward that
counts, a state without room for them) and in the one-wave segments of launches
between the two kernels' ranges."""
import numpy as np
import pytest

import oracle
import scenegen as sg
from parity_util import check_grads, mask_flagged

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h4d():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as m
    oracle.build()
    return m


def _scene(n3, n4, W, H, seed, faint=False):
    scene = sg.tiny_scene(n3=n3, n4=n4, width=W, height=H, seed=seed)
    if faint:  # opacities of about 0.02: lists of hundreds of contributors
        for g in (scene.g3, scene.g4):
            g["opacity"] = (g["opacity"] * 0.2 - 4.0).astype(np.float32)
    return scene


@pytest.mark.parametrize("W,H", [(1, 1), (17, 33), (128, 96), (1024, 512), (1040, 512)])
def test_images_equal_other_tiles(h4d, W, H):
    scene = _scene(900, 600, W, H, 5)
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    v = [scene.views[0].with_time(t) for t in (0.3, 0.7)] if W < 200 else scene.views
    for batched in (False, True):
        a = h4d.Rasterizer(tile=16, batched=batched).infer(g3, g4, v).images
        b = h4d.Rasterizer(tile=8, batched=batched).infer(g3, g4, v).images
        assert all(torch.equal(x, y) for x, y in zip(a, b))


# tiles: 12 (four waves per segment), 1200 (one wave per segment); the faint
# scenes' lists pass the head of 512 entries
@pytest.mark.parametrize("W,H,n3,n4,faint", [(61, 45, 400, 300, False), (640, 480, 1200, 800, False),
                                             (45, 61, 5000, 4000, True), (640, 480, 30000, 20000, True)])
def test_gradients_match_oracle(h4d, W, H, n3, n4, faint):
    print(f"[quadrants] {W}x{H} n={n3}+{n4} faint={faint}", flush=True)
    scene = _scene(n3, n4, W, H, 6, faint)
    v = scene.views[0]
    ref = oracle.render(scene, v)
    dl = mask_flagged(sg.upstream_grads([v], seed=7)[0], ref["amb"])
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    rast = h4d.Rasterizer()
    h = rast.forward(g3, g4, [v])
    if faint and W < 200:
        # every pixel of the middle blends far past the head
        _, rg = rast.tile_lists(h)
        assert int((rg[:, 1] - rg[:, 0]).max()) > 1000
    gr3, gr4 = rast.backward(h, g3, g4, [torch.as_tensor(dl, device="cuda")])
    r3, r4 = oracle.render_bwd(scene, [v], [dl])
    check_grads(scene, gr3, gr4, r3, r4, np.zeros(n3 + n4, bool))


@pytest.mark.parametrize("how", ["counting", "small state"])
def test_gradients_without_checkpoints(h4d, how):
    """The same gradients up to the order of the sums and the rounding of the
    colour behind a segment (normwise 1e-5: a few hundred float32 roundings)."""
    W, H = 61, 45
    scene = _scene(5000, 4000, W, H, 8, True)
    v = scene.views[0]
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    dl = [torch.as_tensor(sg.upstream_grads([v], seed=9)[0], device="cuda")]
    rast = h4d.Rasterizer()
    h = rast.forward(g3, g4, [v])
    want = [x.clone() for d in rast.backward(h, g3, g4, dl) for x in d.values()]
    img = h.images[0].clone()
    if how == "counting":
        rast.stats(True)
        h = rast.forward(g3, g4, [v])
        rast.stats(False)
    else:
        tiles = ((W + 15) // 16) * ((H + 15) // 16)
        st, _ = rast.sizes(scene.n3, scene.n4, h.views, 1)
        rast._state = rast._state[:st - 16 * 7 * 256 * tiles - 4 * 256 * tiles].clone()
        rast._ensure = lambda *a: None
        h = rast.forward(g3, g4, [v])
    assert torch.equal(img, h.images[0])
    got = [x for d in rast.backward(h, g3, g4, dl) for x in d.values()]
    for a, b in zip(want, got):
        assert float((a - b).norm()) <= 1e-5 * float(a.norm())
