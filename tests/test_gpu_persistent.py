"""Persistent grids that really loop: shots enough for more blocks than
work-groups, of uneven length (the later step runs over the shot map), each
order, precision, block choice and isotropic and anisotropic elements, against
the oracle: FP64 relative L2 <= 1e-12, FP32 <= 1e-5.  And kernel 0 in FP64
from order 2 on, which runs kernel 1's code."""

import functools

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import oracle_problem, oracle_run, random_fields, rel_l2, say
from paper_2205_11052_amd import DGWError, Solver

pytestmark = pytest.mark.gpu

# elements per block of kernel 1; kernel 0 has at most 64 (one thread per
# element and node, 256 threads, at least 4 nodes)
BLOCKS = {(1, 64): (7, 3), (2, 64): (7, 3), (3, 64): (7, 3), (4, 64): (7, 3),
          (5, 64): (6, 3), (6, 64): (4, 2),
          (1, 32): (14, 7), (2, 32): (14, 7), (3, 32): (14, 7), (4, 32): (14, 7),
          (5, 32): (7, 3), (6, 32): (7, 3)}


def _medium(K, N, aniso):
    if aniso:
        rho, C = W.random_stiffness(K, 50 + N)
        return rho, np.ones(K), np.ones(K), C
    rng = np.random.default_rng(60 + N)
    cp = rng.uniform(1.5, 3.0, K)
    return W.lame_from_velocities(cp, cp / rng.uniform(1.5, 2.2, K),
                                  rng.uniform(1.0, 3.0, K)) + (None,)


@functools.lru_cache(maxsize=2)
def _reference(N, aniso):
    """mesh, medium, dt, source, two initial states and what 1 and 2 steps make of them."""
    mesh = W.general_mesh(3, L=1.0, seed=40 + N)
    K = mesh["etov"].shape[0]
    rho, lam, mu, C = _medium(K, N, aniso)
    P = oracle_problem(mesh, N)
    bound = 2.0 * np.linalg.eigvalsh(C).max(axis=1) if aniso else lam
    dt = P.suggest_dt(rho, bound, 0 * mu if aniso else mu, 0.5)
    if aniso:
        P.stiffness = torch.as_tensor(C)
    src = W.element_centroids(mesh)[K // 2]
    P.set_source(src, 3.0, 0.0, 2.0)
    q0 = [random_fields(K, P.Np, 70 + i) for i in range(2)]
    want = {(i, n): oracle_run(P, q0[i], rho, lam, mu, dt, n)[0]
            for i in range(2) for n in (1, 2)}
    return mesh, (rho, lam, mu, C), dt, src, q0, want


def _check(N, prec, aniso, kernel, be, wpc, shots):
    mesh, (rho, lam, mu, C), dt, src, q0, want = _reference(N, aniso)
    s = Solver(N, prec, shots)
    s.set_mesh_dict(mesh)
    s.set_material(rho, lam, mu)
    if aniso:
        s.set_stiffness(C)
    s.set_dt(dt)
    steps = [1 if i % 3 == 2 else 2 for i in range(shots)]
    for i in range(shots):
        s.set_source(i, src, 3.0, 0.0, 2.0, nsteps=steps[i])
        s.set_fields(i, q0[i % 2])
    s.set_launch(kernel, be, wpc)
    s.step(2)
    err = max(rel_l2(s.get_fields(i), want[i % 2, steps[i]]) for i in range(shots))
    s.close()
    say("N=%d fp%d aniso=%s shape (%d, %d, %d) %d shots %.3e" %
        (N, prec, aniso, kernel, be, wpc, shots, err))
    assert err <= (1e-12 if prec == 64 else 1e-5)


def _shots(be, wpc):
    """Shots for which two thirds of them have more blocks than the grid has
    work-groups."""
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    grid = (ncu * wpc + 7) // 8 * 8
    blocks = -(-162 // be)
    shots = 3 * (grid // blocks // 2 + 2)
    assert blocks * (shots - shots // 3) > grid
    return shots


@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("prec", [64, 32])
def test_kernel_1(N, prec, aniso):
    for be in BLOCKS[N, prec]:
        _check(N, prec, aniso, 1, be, 1, _shots(be, 1))


@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("N,prec", [(1, 64)] + [(N, 32) for N in range(1, 7)])
def test_kernel_0(N, prec, aniso):
    _check(N, prec, aniso, 0, 0, 1, _shots(64, 1))


@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 6])
def test_kernel_0_runs_kernel_1_in_fp64(N, aniso):
    """The same bits whatever the block, and blocks that kernel 0 doesn't have
    refused; both against the oracle."""
    mesh, (rho, lam, mu, C), dt, src, q0, want = _reference(N, aniso)
    s = Solver(N, 64, 1)
    s.set_mesh_dict(mesh)
    s.set_material(rho, lam, mu)
    if aniso:
        s.set_stiffness(C)
    s.set_dt(dt)
    s.set_source(0, src, 3.0, 0.0, 2.0)
    with pytest.raises(DGWError):
        s.set_launch(0, 99, 0)
    out = []
    for shape in [(0, 0, 0), (0, 0, 1)] + [(1, be, 0) for be in BLOCKS[N, 64]]:
        s.set_launch(*shape)
        s.set_fields(0, q0[0])
        s.step(2)
        out.append(s.get_fields(0))
    s.close()
    assert rel_l2(out[0], want[0, 2]) <= 1e-12
    for o in out[1:]:
        np.testing.assert_array_equal(out[0], o)
