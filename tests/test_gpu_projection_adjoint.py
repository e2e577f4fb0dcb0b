"""The projection adjoint's workgroups (64 Gaussians, one wave for their colour and one
for the rest) at the edges: sets that do not fill a workgroup, an empty set, one
view and several, cameras repeated at several times; every gradient against the
oracle within the tolerance of the parity tests."""
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
    m._lib.load()
    return m


@pytest.mark.parametrize("n3,n4", [(0, 65), (64, 0), (1, 63), (65, 129), (300, 64)])
@pytest.mark.parametrize("times,batched", [((0.5,), False), ((0.2, 0.6, 0.9), False), ((0.2, 0.6, 0.9), True)])
def test_set_sizes(h4d, n3, n4, times, batched):
    print(f"[projection adjoint] n3 {n3}, n4 {n4}, times {times}, batched {batched}", flush=True)
    scene = sg.tiny_scene(n3=n3, n4=n4, seed=101 + n3, box=1.5)
    views = [scene.views[0].with_time(t) for t in times]
    views.append(sg.look_at((1.5, 0.0, -2.0), (0.0, 0.0, 0.0), 80, 61, t=0.4))
    rast = h4d.Rasterizer(batched=batched)
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    refs = [oracle.render(scene, v) for v in views]
    dls = [mask_flagged(d, r["amb"]) for d, r in zip(sg.upstream_grads(views, seed=102), refs)]
    h = rast.forward(g3, g4, views)
    gr3, gr4 = rast.backward(h, g3, g4, [torch.as_tensor(d, device="cuda") for d in dls])
    torch.cuda.synchronize()
    r3, r4 = oracle.render_bwd(scene, views, dls)
    check_grads(scene, gr3, gr4, r3, r4, np.zeros(n3 + n4, bool))


def test_unseen_rows_of_infinite_extent(h4d):
    """A 4D Gaussian that no view sees takes no gradient of its times, however its
    covariance came to be infinite."""
    print("[projection adjoint] unseen, infinite extent", flush=True)
    scene = sg.tiny_scene(n3=10, n4=70, seed=103)
    scene.g4["opacity"][5:60:7] = -30.0  # below 1/255 in every view
    scene.g4["log_scale"][3, 5:60:7] = np.inf
    rast = h4d.Rasterizer()
    g3, g4 = h4d.to_device(scene.g3), h4d.to_device(scene.g4)
    h = rast.forward(g3, g4, scene.views)
    _, gr4 = rast.backward(h, g3, g4, [torch.ones_like(im) for im in h.images])
    for k in ("mean", "mean_t", "opacity", "sh"):
        assert float(gr4[k][..., 5:60:7].abs().max()) == 0.0, k
