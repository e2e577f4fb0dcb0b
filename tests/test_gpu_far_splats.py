"""Vast splats whose centre lies far off the image, and splats without a centre (GPU):
images do not depend on culling or the tile size, and hold what the splats blend."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("distance", [1e4, 3e6, 1e8])
def test_images_do_not_depend_on_culling(distance):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as h4d
    print(f"[far splats] distance {distance:g}", flush=True)
    n, W, H = 24, 203, 131
    rng = np.random.default_rng(3)
    th = rng.uniform(0, 2 * np.pi, n)
    s = distance * rng.uniform(0.4, 1.5, n)  # round splats
    f = lambda x: np.asarray(x, np.float32)
    sp = dict(u=f(distance * np.cos(th)), v=f(distance * np.sin(th)), conic=f(np.stack([s ** -2.0, 0 * s, s ** -2.0])),
              opacity=f(np.full(n, 0.3)), rgb=f(rng.uniform(0, 1, (3, n))), radius=np.ceil(3 * s).astype(np.int32),
              depth=f(rng.uniform(1, 5, n)), visible=np.ones(n, np.uint8))
    want = h4d.rasterize_splats(h4d.Rasterizer(tile=8, cull=False), sp, W, H)[:2]
    # (0.3 exp(-0.5 / 0.4^2) = 0.013 at the least, where 1/255 suffices)
    assert float(want[1].max()) < 0.9
    for tile in (8, 16, 32):
        for cull in (False, True):
            got = h4d.rasterize_splats(h4d.Rasterizer(tile=tile, cull=cull), sp, W, H)[:2]
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (tile, cull)


def test_splats_without_a_centre():
    """A centre that is not a number: the pixels of the splat's square pass the power
    test (no comparison fails), and the quadrants keep all of them as the other
    kernels do."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as h4d
    print("[far splats] no centre", flush=True)
    n, W, H = 3, 40, 150
    f = lambda x: np.asarray(x, np.float32)
    sp = dict(u=f([np.nan, 20.0, 12.0]), v=f([70.0, np.nan, 40.0]), conic=f([[0.01] * n, [0.0] * n, [0.01] * n]),
              opacity=f([0.5, 0.6, 0.7]), rgb=f(np.arange(9).reshape(3, 3) / 9.0), radius=np.full(n, 60, np.int32),
              depth=f([1.0, 2.0, 3.0]), visible=np.ones(n, np.uint8))
    def render(tile, cull, some=slice(None)):
        return torch.cat([x.reshape(-1, H, W) for x in h4d.rasterize_splats(
            h4d.Rasterizer(tile=tile, cull=cull), {k: v[..., some] for k, v in sp.items()}, W, H)[:2]]).nan_to_num(7.0)

    assert torch.equal(render(16, False), render(8, False))
    # culling leaves a splat without a column out of every tile
    for tile in (8, 16, 32):
        assert torch.equal(render(tile, True), render(tile, True, slice(1, None)))
        assert not torch.equal(render(tile, True), render(tile, True, slice(2, None)))
