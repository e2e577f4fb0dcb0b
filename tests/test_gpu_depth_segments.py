"""Depth sorts of several segments (GPU): a batched call's lists equal its views'
one after another, whose orders the tests of single segments pin.  Short segments
of 4D Gaussians beside long ones of a camera's 3D ones; several segments whose
samples are gathered first (8192 and more in all) and whose workgroups' counts are
scanned by a launch of their own (beyond 2^18 keys)."""
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _views(n, W, H, same):
    return [sg.look_at((0.0 if same else 0.05 * k - 0.1, 0.0, -3.0), (0.0, 0.0, 0.0), W, H, t=0.1 + 0.8 * k / n)
            for k in range(n)]


@pytest.mark.parametrize("n3,n4,V,same", [(14000, 100, 16, True), (13001, 1, 32, True), (60, 13001, 2, True),
                                          (60000, 40000, 5, False), (20000, 7000, 3, False), (262200, 300, 2, False),
                                          (300000, 262200, 2, True)])
def test_batched_lists_equal_one_view_at_a_time(n3, n4, V, same):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as h4d
    print(f"[depth segments] n={n3}+{n4} views {V} same camera {same}", flush=True)
    scene = sg.tiny_scene(n3=n3, n4=n4, width=64, height=64, seed=21)
    for g in (scene.g3, scene.g4):  # many equal depths
        g["mean"][2] = (g["mean"][2] * 64).round() / 64
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    views = _views(V, 64, 64, same)
    one = h4d.Rasterizer(batched=False, pair_capacity=1 << 20)
    all_ = h4d.Rasterizer(batched=True, pair_capacity=1 << 20)
    ha, hb = one.forward(g3, g4, views), all_.forward(g3, g4, views)
    assert all(torch.equal(a, b) for a, b in zip(ha.images, hb.images))
    (ia, ra), (ib, rb) = one.tile_lists(ha), all_.tile_lists(hb)
    n = int(ra[-1, 1])
    assert n > 1000 and torch.equal(ra, rb) and torch.equal(ia[:n], ib[:n])
