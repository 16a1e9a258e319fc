"""Orders 5 and 6 on the full 82944-element mesh, where the oracle is too slow
for a whole run: the oracle steps the elements within six faces of a few
elements, and one step (five stages, one ring of faces each) gives those and
their neighbours exactly.  Every block choice, plain and persistent, FP64
<= 1e-12 and FP32 <= 1e-5 against it.  The elements are at corners, edges, the
free surface, the source, and the first and last blocks."""

import numpy as np
import pytest

import workloads as W
from gpu_helpers import oracle_problem, oracle_run, random_fields, rel_l2, say
from paper_2205_11052_amd import Solver

pytestmark = pytest.mark.gpu

RINGS = 6
SHAPES = {(5, 64): [(1, 6, 0), (1, 3, 0), (1, 6, 2)],
          (6, 64): [(1, 4, 0), (1, 2, 0), (1, 4, 2)],
          (5, 32): [(0, 0, 0), (1, 7, 0), (1, 3, 2)],
          (6, 32): [(0, 0, 0), (1, 7, 0), (1, 3, 2)]}


def neighbours(etov):
    """[K, 4] element across each face, -1 at the boundary."""
    K = etov.shape[0]
    tri = np.sort(np.stack([np.delete(etov, f, 1) for f in range(4)], 1), 2).reshape(-1, 3)
    order = np.lexsort(tri.T)
    same = (tri[order[1:]] == tri[order[:-1]]).all(1)
    out = np.full(4 * K, -1)
    a, b = order[:-1][same], order[1:][same]
    out[a], out[b] = b // 4, a // 4
    return out.reshape(K, 4)


def ball(nb, k, rings):
    """Elements within `rings` faces of element k, and their distances."""
    dist = {k: 0}
    front = [k]
    for r in range(1, rings + 1):
        front = sorted({int(j) for i in front for j in nb[i] if j >= 0 and int(j) not in dist})
        dist.update((j, r) for j in front)
    el = np.array(sorted(dist))
    return el, np.array([dist[i] for i in el])


@pytest.mark.parametrize("N", [5, 6])
def test_full_size_against_the_oracle_around_sampled_elements(N):
    w = W.build_workload("c1_layered_n24", N=N)
    mesh, K = w["mesh"], w["K"]
    Np = (N + 1) * (N + 2) * (N + 3) // 6
    nb = neighbours(mesh["etov"])
    cen = W.element_centroids(mesh)
    src = K // 2 + 1234
    q0 = random_fields(K, Np, 17)
    near = lambda *x: int(np.argmin(((cen - np.array(x)) ** 2).sum(1)))
    picks = [0, K - 1, K - 7, src, near(10, 10, 10), near(5, 5, 10), near(0, 5, 5), near(3, 7, 4)]
    dt = None
    want = []
    for (n, prec), shapes in sorted(SHAPES.items(), reverse=True):
        if n != N:
            continue
        s = Solver(N, prec, 1)
        s.set_mesh_dict(mesh)
        s.set_material(w["rho"], w["lam"], w["mu"])
        if dt is None:
            dt = s.suggest_dt(w["cfl"])
            for k in picks:
                el, dist = ball(nb, k, RINGS)
                sub = dict(vxyz=mesh["vxyz"], etov=mesh["etov"][el], vertex_periodic_id=None,
                           face_bc=np.where(nb[el] < 0, mesh["face_bc"][el], 2).astype(np.int8))
                P = oracle_problem(sub, N)
                if src in el:
                    P.set_source(cen[src], w["f0"], 0.05, w["amp"])
                q, _ = oracle_run(P, q0[el], w["rho"][el], w["lam"][el], w["mu"][el], dt, 1)
                say("case order %d element %d, %d around it" % (N, k, len(el)))
                keep = dist <= 1
                want.append((el[keep], q[keep]))
        s.set_dt(dt)
        s.set_source(0, cen[src], w["f0"], 0.05, w["amp"])
        for shape in shapes:
            s.set_launch(*shape)
            s.set_fields(0, q0)
            s.step(1)
            got = s.get_fields(0)
            err = max(rel_l2(got[el], q) for el, q in want)
            say("order %d fp%d shape %s, %d elements: %.3e" %
                (N, prec, shape, sum(len(el) for el, _ in want), err))
            assert err <= (1e-12 if prec == 64 else 1e-5)
        s.close()
