"""A backward given another sufficient state size than its forward (GPU): the list
heads and checkpoints lie where the forward's size puts them, so that the backward
walks the lists again.  The same gradients up to the order of the sums and the
rounding of the colour behind a segment (normwise 1e-5: a few hundred float32
roundings), in one pass of each kernel's range (12 and 1200 tiles) and with lists
past the heads."""
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n3,n4,faint", [(61, 45, 5000, 4000, True), (61, 45, 400, 300, False),
                                             (640, 480, 1200, 800, False)])
@pytest.mark.parametrize("forward,backward", [("full", "least"), ("least", "full")])
def test_backward_with_another_state_size(forward, backward, W, H, n3, n4, faint):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as h4d
    print(f"[state sizes] {W}x{H} n={n3}+{n4} forward {forward}, backward {backward}", flush=True)
    scene = sg.tiny_scene(n3=n3, n4=n4, width=W, height=H, seed=12)
    if faint:  # opacities of about 0.02: lists of hundreds of contributors
        for g in (scene.g3, scene.g4):
            g["opacity"] = (g["opacity"] * 0.2 - 4.0).astype("float32")
    v = scene.views[0]
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    dl = [torch.as_tensor(sg.upstream_grads([v], seed=13)[0], device="cuda")]
    rast = h4d.Rasterizer()
    h = rast.forward(g3, g4, [v])
    want = [x.clone() for d in rast.backward(h, g3, g4, dl) for x in d.values()]
    img = h.images[0].clone()
    st, _ = rast.sizes(n3, n4, h.views, 1)
    tiles = ((W + 15) // 16) * ((H + 15) // 16)
    # 256 entries of a head more and 7 x 256 checkpoints of 16 bytes per tile
    state = {"full": torch.zeros(st, dtype=torch.uint8, device="cuda")}
    state["least"] = state["full"][:st - 16 * 7 * 256 * tiles - 4 * 256 * tiles]
    rast._ensure = lambda *a: None
    rast._state = state[forward]
    h = rast.forward(g3, g4, [v])
    assert torch.equal(img, h.images[0])
    h.state = state[backward]
    got = [x for d in rast.backward(h, g3, g4, dl) for x in d.values()]
    for a, b in zip(want, got):
        assert float((a - b).norm()) <= 1e-5 * float(a.norm())
