"""The kernels that calls launch (host code over a recording HIP runtime, no GPU):
the paths that the GPU tests name are the ones they take."""
import pytest

import hip_record
from sorted_binning import CALLS
from test_read_back import stub  # noqa: F401 (a fixture)


@pytest.mark.parametrize("name", CALLS)
def test_emitted_and_sorted(stub, name):  # noqa: F811
    sizes, same, n3, n4, tile, batched, cap, want = CALLS[name]
    out = hip_record.run(stub, f"""
import re
views = L.view_array([sg.look_at((0.0 if {same} else 0.1 * k, 0.0, -3.0), (0.0, 0.0, 0.0), W, H, t=0.3 + 0.1 * k)
                      for k, (W, H) in enumerate({sizes})])
assert render({n3}, {n4}, views, len(views), L.Config({tile}, 64, {batched}, 1, {cap})) == L.H4D_OK, error()
for k in kernels(calls()):
    print(re.search("\\\\d+(k_[a-z0-9_]*?[a-z0-9])(?=[EI])", k).group(1))
""").split()
    assert set(want) <= set(out) and not any(k.startswith("k_bin_") for k in out), out
    assert ("k_ranges" in out) == ("k_ranges" in want), out
    assert ("k_coarse_top" in out) == ("k_coarse_top" in want), out
