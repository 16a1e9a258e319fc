"""Large FP32 transfers (converted on the device) take no device memory of their
own and disturb nothing: a run with fields read and written between its steps,
and a gradient with fields read between forward and reverse, give the same
bits as without."""

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import say
from paper_2205_11052_amd import Solver, _lib

pytestmark = pytest.mark.gpu

N, CELLS = 6, 13                        # 13182 elements, 10 M values a shot


def _solver(nshots, hook=None, layer=False):
    mesh = W.kuhn_cube(CELLS)
    K = mesh["etov"].shape[0]
    s = Solver(N, 32, nshots, torch_allocator=hook is None)
    if hook is not None:
        s._callbacks = (_lib.ALLOC_FN(hook), _lib.FREE_FN(
            lambda p, user: torch.cuda.caching_allocator_delete(p)))
        s._check(s.lib.dgw_set_allocator(s._ctx, s._callbacks[0], s._callbacks[1], None),
                 "dgw_set_allocator")
    s.set_mesh_dict(mesh)
    s.set_material(np.ones(K), np.ones(K), np.ones(K))
    s.set_dt(1e-4)
    if layer:
        el = np.arange(1500, dtype=np.int32)      # 2.3 M memory variables
        s.set_pml(el, np.random.default_rng(3).uniform(0, 5, (el.size, 6, s.Np)))
    return s, K


def _fields(K, n, seed):
    return np.random.default_rng(seed).standard_normal((n, K, 9, (N + 1) * (N + 2) * (N + 3) // 6))


def test_no_memory_is_taken():
    asked = []

    def alloc(nbytes, user):
        asked.append(nbytes)
        return torch.cuda.caching_allocator_alloc(int(nbytes))

    s, K = _solver(1, alloc, layer=True)
    q = _fields(K, 1, 1)[0]
    s.step(1)
    before = len(asked)
    s.set_fields(0, q)
    s.get_fields(0)
    s.set_pml_memory(0, s.pml_memory(0) + 0.5)
    assert asked[before:] == []
    s.close()


@pytest.mark.parametrize("kernel,layer", [(0, False), (1, False), (2, False), (1, True)])
def test_transfers_between_steps(kernel, layer):
    say("case kernel %d layer %s" % (kernel, layer))
    out = []
    for between in (False, True):
        s, K = _solver(2, layer=layer)
        s.set_launch(kernel)
        q = _fields(K, 3, 2)
        s.set_fields(0, q[0])
        s.set_fields(1, q[1] if not between else q[2])
        if between:
            s.set_fields(1, q[1])
        s.step(1)
        mid = s.get_fields(0) if between else None
        s.step(1)
        r = [s.get_fields(0), s.get_fields(1)]
        if layer:
            r.append(s.pml_memory(1))
        out.append(r)
        assert mid is None or not np.array_equal(mid, r[0])
        s.close()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def test_fields_read_before_the_reverse_sweep():
    grads = []
    for between in (False, True):
        s, K = _solver(1)
        x = W.element_centroids(W.kuhn_cube(CELLS))
        s.set_source(0, x[K // 2], 3.0, 0.0)
        s.set_receivers(0, x[[K // 2, K // 2 + 1]], 4)
        s.zero_fields()
        s.forward_checkpointed(4, 2, np.zeros((1, 2, 3, 4)))
        if between:
            s.get_fields(0)
        grads.append(s.adjoint())
        s.close()
    assert any(np.abs(g).max() > 0 for g in grads[0])
    for a, b in zip(*grads):
        np.testing.assert_array_equal(a, b)
