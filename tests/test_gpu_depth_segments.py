"""Depth sorts of several segments (GPU): a batched call's lists equal its views'
one after another, whose orders the tests of single segments pin.  Short segments
of 4D Gaussians beside long ones of a camera's 3D ones; several segments whose
samples are gathered first (8192 and more in all) and whose workgroups' counts are
scanned by a launch of their own (beyond 2^18 keys)."""
import numpy as np
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


def _sample_places(n, lg):
    """Where the bins' samples lie: a hashed place of each of 2^lg equal stretches."""
    out = []
    for j in range(1 << lg):
        lo, hi = (j * n) >> lg, ((j + 1) * n) >> lg
        h = (j * 0x9E3779B1) & 0xFFFFFFFF
        h ^= h >> 15
        h = (h * 0x85EBCA77) & 0xFFFFFFFF
        h ^= h >> 13
        out.append(min(lo + ((h * max(1, hi - lo)) >> 32), n - 1))
    return np.array(out)


@pytest.mark.parametrize("n,lg_bins", [(13001, 6), (65537, 9)])
@pytest.mark.parametrize("depths", ["spread", "equal"])
def test_a_bin_of_most_keys(n, lg_bins, depths):
    """The samples at the extreme depths and every other key between them: one bin
    takes all of those (12,745 and 63,489 keys, where a workgroup holds 4096), and is
    ordered block against block."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as h4d
    print(f"[depth bin] n={n} {depths}", flush=True)
    rng = np.random.default_rng(n)
    rec = sg.synthetic_records(n, 16, 16, seed=32, max_radius=40)
    rec["u"][:], rec["v"][:], rec["radius"][:], rec["visible"][:] = 8.0, 8.0, 30, 1
    at = _sample_places(n, lg_bins + 2)
    assert len(set(at)) == len(at)
    key = 2.0 + rng.integers(0, n // 7, n) / 65536.0 if depths == "spread" else np.full(n, 2.0)
    key[at] = np.where(np.arange(len(at)) % 2 == 0, 1.0, 9.0) + np.arange(len(at)) / 65536.0
    rec["depth"] = key.astype(np.float32)
    rast = h4d.Rasterizer(tile=16, chunk=64, pair_capacity=1 << 21, cull=False)
    _, _, ids, ranges = h4d.rasterize_splats(rast, rec, 16, 16)
    want = np.argsort(rec["depth"], kind="stable")
    assert ranges.cpu().numpy().tolist() == [[0, n]]
    assert np.array_equal(ids.cpu().numpy()[:n], want)
