"""Failed device allocations are reported once, by the call that made them: the
launches that follow succeed, and a transfer doesn't report one made elsewhere."""

import ctypes as C

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import say
from paper_2205_11052_amd import DGWError, Solver, _lib

pytestmark = pytest.mark.gpu

TOO_MUCH = 1 << 60                      # bytes; no device has them


def fail_malloc():
    """A failed hipMalloc through the runtime that the library is linked to."""
    p = C.c_void_p()
    fn = _lib.load().hipMalloc
    fn.restype = C.c_int
    assert fn(C.byref(p), C.c_size_t(TOO_MUCH)) != 0


def test_refused_scratch_is_not_the_next_launch_s_error():
    refuse = [False]

    def alloc(nbytes, user):
        if refuse[0]:
            fail_malloc()
            return None
        return torch.cuda.caching_allocator_alloc(int(nbytes))

    mesh = W.kuhn_cube(2)
    K = mesh["etov"].shape[0]
    s = Solver(3, 64, 1, torch_allocator=False)
    s._callbacks = (_lib.ALLOC_FN(alloc), _lib.FREE_FN(
        lambda p, user: torch.cuda.caching_allocator_delete(p)))
    s._check(s.lib.dgw_set_allocator(s._ctx, s._callbacks[0], s._callbacks[1], None),
             "dgw_set_allocator")
    s.set_mesh_dict(mesh)
    s.set_material(np.ones(K), np.ones(K), np.ones(K))
    s.set_dt(1e-3)
    s.set_fields(0, np.random.default_rng(1).standard_normal((K, 9, s.Np)))
    refuse[0] = True
    say("case autotune without memory for its scratch")
    with pytest.raises(DGWError) as e:
        s.autotune()
    assert e.value.status == "DGW_ENOMEM"
    refuse[0] = False
    say("case step after it")
    s.step(1)
    s.check_finite()
    s.close()


def test_transfer_does_not_report_another_call_s_failure():
    mesh = W.kuhn_cube(13)              # 10 M values: converted on the device both ways
    K = mesh["etov"].shape[0]
    s = Solver(6, 32, 1)
    s.set_mesh_dict(mesh)
    q = np.random.default_rng(2).standard_normal((K, 9, s.Np))
    fail_malloc()
    try:
        s.set_fields(0, q)
        got = s.get_fields(0)
    finally:
        last = _lib.load().hipGetLastError
        last.restype = C.c_int
        left = last()                   # still the caller's to see
    assert left != 0
    np.testing.assert_array_equal(got, q.astype(np.float32))
    s.close()
