"""Setting a mesh takes no more allocations than the mesh, the operators (one)
and the shots need, and per-face-node tables only where they are read: the
node table in the order of face-0 preimages belongs to FP64 from order 3."""

import pytest
import torch

import workloads as W
from paper_2205_11052_amd import Solver, _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6])
def test_set_mesh_allocations(N, prec):
    sizes = []

    def alloc(nbytes, user):
        sizes.append(nbytes)
        return torch.cuda.caching_allocator_alloc(int(nbytes))

    mesh = W.kuhn_cube(3)
    K = mesh["etov"].shape[0]
    s = Solver(N, prec, 1, torch_allocator=False)
    s._callbacks = (_lib.ALLOC_FN(alloc), _lib.FREE_FN(
        lambda p, user: torch.cuda.caching_allocator_delete(p)))
    s._check(s.lib.dgw_set_allocator(s._ctx, s._callbacks[0], s._callbacks[1], None),
             "dgw_set_allocator")
    s.set_mesh_dict(mesh)
    s.close()
    sym = prec == 64 and N >= 3
    # five mesh tables, the operators, the reordered node table, nine of the shots
    assert len(sizes) == (16 if sym else 15)
    # bytes K x 4 Nfp: neighbour volume nodes, neighbour face nodes, the former reordered
    assert sizes.count(K * 4 * s.Nfp) == (3 if sym else 2)
