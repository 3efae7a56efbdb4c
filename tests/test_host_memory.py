"""What making a context does on the host, on a stand-in for the HIP runtime: running out of memory is
a status, not a C++ exception through the C interface (which ends the process), and the device gets no
more than the populations to clear and the initial state (and the lists of the two-step passes)."""
import pytest

from hip_calls import run

SCRIPT = r"""
p = lbm.make_params(W.random_case(3, {nx}, {ny}))
n = lib.lbm_workspace_bytes(C.byref(p))
keep, ws = memory(n)
h = C.c_void_p()
for left in range(6):
    print(left, flush=True)
    log()
    calls.calls_fail_new(left)
    st = lib.lbm_init(C.byref(p), ws, n, None, C.byref(h))
    calls.calls_fail_new(-1)
    assert (st == 2 and not h) or (st == 0 and h), st
    lib.lbm_destroy(h)
assert st == 0
"""


@pytest.mark.parametrize("nx,ny", [(20, 6), (4, 7), (400, 7), (150, 6)])
def test_init_without_host_memory(tmp_path, nx, ny):
    run(SCRIPT.format(nx=nx, ny=ny), tmp_path)


CALLS = r"""
Sim(W.cavity(12))
for n, lists in (((20, 6), []), ((40, 40), ["copy"])):
    log()
    s = Sim(W.random_case(3, *n))
    got = log()
    assert got == lists + ["set", "launch k_init"], got
"""


def test_device_calls_of_init(tmp_path):
    run(CALLS, tmp_path)
