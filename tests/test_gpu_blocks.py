"""The matrix-core stage kernel on meshes smaller than a block, of one block
and a remainder, and of many blocks, at every block choice of orders 3 to 6,
against the oracle: FP64 relative L2 <= 1e-12, FP32 <= 1e-5 (the bounds of
the other parity tests)."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import pml as OP
from gpu_helpers import oracle_problem, oracle_run, random_fields, rel_l2, say
from paper_2205_11052_amd import Solver

pytestmark = pytest.mark.gpu

BLOCKS = {(3, 64): (7, 3), (4, 64): (7, 3), (5, 64): (6, 3), (6, 64): (4, 2),
          (3, 32): (14, 7), (4, 32): (14, 7), (5, 32): (7, 3), (6, 32): (7, 3)}


@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("N,prec", sorted(BLOCKS))
def test_blocks(N, prec, n, aniso):
    mesh = W.general_mesh(n, L=1.0, seed=40 + N)
    K = mesh["etov"].shape[0]
    P = oracle_problem(mesh, N)
    if aniso:
        rho, C = W.random_stiffness(K, 50 + N)
        P.stiffness = torch.as_tensor(C)
        lam = 2.0 * np.linalg.eigvalsh(C).max(axis=1)   # bounds the speeds
        mu = np.zeros(K)
    else:
        rng = np.random.default_rng(60 + N)
        cp = rng.uniform(1.5, 3.0, K)
        rho, lam, mu = W.lame_from_velocities(cp, cp / rng.uniform(1.5, 2.2, K),
                                              rng.uniform(1.0, 3.0, K))
    dt = P.suggest_dt(rho, lam, mu, 0.5)
    if aniso:
        lam, mu = np.ones(K), np.ones(K)
    q0 = random_fields(K, P.Np, 70 + n)
    src = W.element_centroids(mesh)[K // 2]
    P.set_source(src, 3.0, 0.0, 2.0)
    q_ora, _ = oracle_run(P, q0, rho, lam, mu, dt, 3)
    s = Solver(N, prec, 1)
    s.set_mesh_dict(mesh)
    s.set_material(rho, lam, mu)
    if aniso:
        s.set_stiffness(C)
    s.set_dt(dt)
    s.set_source(0, src, 3.0, 0.0, 2.0)
    for be in BLOCKS[N, prec]:
        for wpc in (0, 1):
            s.set_launch(1, be, wpc)
            s.set_fields(0, q0)
            s.step(3)
            err = rel_l2(s.get_fields(0), q_ora)
            say("N=%d fp%d K=%d be=%d wpc=%d aniso=%s %.3e" % (N, prec, K, be, wpc, aniso, err))
            assert err <= (1e-12 if prec == 64 else 1e-5)


@pytest.mark.parametrize("m", [1, 3, 7, 8, 23])
@pytest.mark.parametrize("N", [3, 4, 5, 6])
def test_layer_blocks(N, m):
    """The layer kernel in FP64 on one element, less than a block, a block, a
    block and a remainder, and several: fields and memory variables against
    the oracle (<= 1e-12)."""
    mesh = W.general_mesh(2, L=1.0, seed=80 + N)
    K = mesh["etov"].shape[0]
    P = oracle_problem(mesh, N)
    rng = np.random.default_rng(90 + m)
    cp = rng.uniform(1.5, 3.0, K)
    rho, lam, mu = W.lame_from_velocities(cp, cp / rng.uniform(1.5, 2.2, K),
                                          rng.uniform(1.0, 3.0, K))
    dt = P.suggest_dt(rho, lam, mu, 0.5)
    el = np.sort(rng.choice(K, m, replace=False)).astype(np.int32)
    prof = rng.uniform(0.0, 5.0, (m, 6, P.Np))
    d, a = np.zeros((K, 3, P.Np)), np.zeros((K, 3, P.Np))
    d[el], a[el] = prof[:, :3], prof[:, 3:]
    q0 = random_fields(K, P.Np, 95 + N)
    t = torch.as_tensor
    q_ora, m_ora, _ = OP.run(P, t(q0).clone(), t(rho), t(lam), t(mu), t(d), t(a), dt, 3)
    s = Solver(N, 64, 1)
    s.set_mesh_dict(mesh)
    s.set_material(rho, lam, mu)
    s.set_dt(dt)
    s.set_pml(el, prof)
    s.set_fields(0, q0)
    s.step(3)
    err = rel_l2(s.get_fields(0), q_ora.numpy())
    merr = rel_l2(s.pml_memory(0), m_ora.numpy()[el])
    say("N=%d layer elements %d fields %.3e memory %.3e" % (N, m, err, merr))
    assert err <= 1e-12 and merr <= 1e-12


@pytest.mark.parametrize("N,n,kernel", [(1, 9, 1), (1, 10, 0), (2, 10, 1), (3, 8, 1), (3, 9, 0),
                                        (4, 5, 0), (4, 6, 1), (4, 7, 0), (4, 9, 1), (5, 9, 1),
                                        (5, 10, 0), (6, 4, 0), (6, 17, 1)])
def test_fp32_kernel_is_not_timed(N, n, kernel):
    """The FP32 kernel follows from order and size: both sides of each line."""
    mesh = W.kuhn_cube(n)
    K = mesh["etov"].shape[0]
    s = Solver(N, 32, 1)
    s.set_mesh_dict(mesh)
    s.set_material(np.ones(K), np.ones(K), np.ones(K))
    s.set_dt(1e-3)
    assert s.autotune()[0] == kernel
    s.close()
