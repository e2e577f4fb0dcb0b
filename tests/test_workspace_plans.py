"""Every call that the workspace was sized for is enqueued (host code over a
recording HIP runtime, no GPU): the depth sorts' scratch holds the plan of every
job, also of short segments beside long ones."""
import pytest

import hip_record
from test_read_back import stub  # noqa: F401 (a fixture)


def test_short_segments_beside_long_ones(stub):  # noqa: F811
    """Shared static binning: the views' few 4D Gaussians are segments of their own
    beside the group's many 3D ones."""
    hip_record.run(stub, """
for n3, n4, V, W, H, cap in [(14000, 1000, 32, 64, 64, 1 << 22), (20000, 500, 32, 128, 96, 1 << 20),
                             (20000, 500, 32, 333, 250, 1 << 18), (14000, 100, 16, 64, 64, 1 << 22),
                             (20000, 100, 32, 500, 500, 1 << 22), (13001, 1, 32, 16, 16, 1 << 10),
                             (1, 13001, 32, 16, 16, 1 << 10)]:
    rc = render(n3, n4, cameras(V, W, H, same=True), V, L.Config(16, 64, 1, 1, cap))
    assert rc == L.H4D_OK, (n3, n4, V, W, H, cap, error())
""")


def test_no_call_is_refused_for_its_workspace(stub):  # noqa: F811
    hip_record.run(stub, """
rng = random.Random(5)
def log(a, b):
    return int(a * (b / a) ** rng.random())
for _ in range(4000):
    V = rng.randint(1, 32)
    n3, n4 = (0 if rng.random() < 0.1 else log(1, 2000000) for _ in range(2))
    W, H = log(1, 3000), log(1, 2200)
    a = cameras(V, W, H, same=rng.random() < 0.5)
    if rng.random() < 0.5:  # some of the cameras repeated
        for k in range(V):
            a[k] = a[rng.randrange(k + 1)]
    cfg = L.Config(rng.choice([8, 16, 32]), 64, rng.randint(0, 1), rng.randint(0, 1),
                   rng.choice([0, log(1, 1 << 24), 1 << 22]))
    rc = render(n3, n4, a, V, cfg, rng.choice(["h4dgs_render_fwd", "h4dgs_render_infer"]))
    assert rc == L.H4D_OK, (n3, n4, V, W, H, cfg.tile, cfg.batched, cfg.cull, cfg.pair_capacity, error())
    R.record_clear()
""")


def test_grids_stay_within_the_launch_limits(stub):  # noqa: F811
    """A batched call of more than 2^30 (view, Gaussian) pairs: no grid of more than
    65535 in y or z, nor of 2^32 threads in x."""
    hip_record.run(stub, """
for n3, n4, same, cull in [(33600000, 0, False, 0), (1000, 33600000, True, 0), (33600000, 0, False, 1)]:
    rc = render(n3, n4, cameras(32, 64, 64, same), 32, L.Config(16, 64, 1, cull, 1 << 22))
    assert rc == L.H4D_OK, error()
    got = calls()
    assert any("k_bin_scatter" in k for k in kernels(got))
    for c in got:
        gx, gy, gz, bx = map(int, c[2:])
        assert 0 < gx and gx * bx < 1 << 32 and 0 < gy <= 65535 and 0 < gz <= 65535, c
""")
