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


def test_a_state_of_another_device_is_copied(stub):
    """A kernel on the stream's device may have no access to another device's
    memory: such a state is read by a copy."""
    hip_record.run(stub, STATE + """
calls()
R.record_set(0, 0, 1, 0)  # the state on device 1, the stream on device 0
state[0], state[1] = 0, 11
assert check() == L.H4D_OK and need.value == 11
assert calls() == [["sync"], ["memcpy"]]
R.record_set(0, 0, 1, 1)
state[1] = 12
assert check() == L.H4D_OK and need.value == 12
assert [c[0] for c in calls()] == ["launch", "sync"]
""")


def test_without_pinned_memory(stub):
    hip_record.run(stub, """
R.record_set(0, 2, 0, 0)  # (out of memory)
""" + STATE + """
assert not kernels(calls())
""")


def test_nothing_is_thrown(stub):
    """A context keeps its pinned blocks without host allocations that could throw
    across the C entry."""
    hip_record.run(stub, """
R.record_new_fails(1)
""" + STATE.replace("state[0], state[1] = 1, 9", "state[1] = 9").replace("H4D_ERR_CAPACITY", "H4D_OK") + """
R.record_new_fails(0)
""")


def test_under_capture(stub):
    """Refused before anything is recorded into the graph or kept for it."""
    hip_record.run(stub, STATE + """
calls()
R.record_capturing(1)
for _ in range(3):
    assert check() == L.H4D_ERR_HIP
assert calls() == [["sync"]] * 3
R.record_capturing(0)
assert check() == L.H4D_ERR_CAPACITY
assert [c[0] for c in calls()] == ["launch", "sync"]
""")
