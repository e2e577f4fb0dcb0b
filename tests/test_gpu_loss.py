"""The L1 loss and its gradient over views of different sizes in one launch, and with
one output buffer for all of them (which then holds the last view's)."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[(5, 7)], [(333, 250), (64, 64), (5, 7)], [(16, 16)] * 32])
@pytest.mark.parametrize("shared", [False, True])
def test_l1_loss_over_views(sizes, shared):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_13215_amd as h4d
    print(f"[l1 loss] {len(sizes)} views, shared output {shared}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    views = [sg.look_at((0.0, 0.0, -3.0), (0.0, 0.0, 0.0), w, h, t=0.5) for w, h in sizes]
    img = [torch.randn((3, h, w), generator=g, device="cuda") for w, h in sizes]
    tgt = [torch.randn((3, h, w), generator=g, device="cuda") for w, h in sizes]
    for a, b in zip(img, tgt):
        a.view(-1)[::5] = b.view(-1)[::5]
    room = torch.full((max(3 * w * h for w, h in sizes),), float("nan"), device="cuda")
    dl = [room[:3 * w * h].view(3, h, w) if shared else torch.full((3, h, w), float("nan"), device="cuda")
          for w, h in sizes]
    loss = torch.full((1,), float("nan"), device="cuda")
    h4d.l1_loss_grad(h4d.Rasterizer(), img, tgt, views, dl, loss)
    n = len(sizes)
    want = np.mean([(a.double() - b.double()).abs().mean().item() for a, b in zip(img, tgt)])
    assert abs(loss.item() - want) <= 1e-5 * want
    for k in ([n - 1] if shared else range(n)):
        scale = np.float32(1.0 / (float(img[k].numel()) * n))
        assert torch.equal(dl[k], torch.sign(img[k] - tgt[k]) * float(scale))
