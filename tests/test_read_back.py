"""Reading a call's status and row counts back (host code over a recording HIP
runtime, no GPU)."""
import pytest

import hip_record


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    from paper_2505_13215_amd import _lib, build
    import os
    if not os.path.exists(_lib.LIB_PATH):
        build.build()
    return hip_record.build(str(tmp_path_factory.mktemp("hip_record")))


STATE = """
state = (C.c_uint64 * 64)()
need = C.c_int64(-1)
def check():
    return ctx.L.h4dgs_check(ctx.h, C.cast(state, C.c_void_p), C.sizeof(state), C.byref(need), None)
state[1] = 7
assert check() == L.H4D_OK and need.value == 7
state[0], state[1] = 1, 9
assert check() == L.H4D_ERR_CAPACITY and need.value == 9
"""


def test_a_copy_that_does_not_launch_is_an_error(stub):
    """A refused launch leaves the words of an earlier read-back where this one's
    belong: they are not this call's status."""
    hip_record.run(stub, STATE + """
state[0], state[1] = 0, 5
need.value = -1
R.record_set(719, 0, 0, 0)
assert check() == L.H4D_ERR_HIP and need.value == -1
R.record_set(0, 0, 0, 0)
assert check() == L.H4D_OK and need.value == 5
ctx.close()
got = [c[0] for c in calls()]
assert got.count("malloc") == 1 == got.count("free"), got
""")
