"""set_fields and get_fields of an FP32 context at sizes converted by the host,
by the device on the way in, and by the device both ways in pieces: FP64
fields come back as rounded to FP32 (IEEE, to nearest), bit for bit, each shot
its own."""

import numpy as np
import pytest

import workloads as W
from paper_2205_11052_amd import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 8, 13])      # 36288, 2.3 M and 10 M values
def test_fp32_fields_round_once(n):
    mesh = W.kuhn_cube(n)
    K = mesh["etov"].shape[0]
    s = Solver(6, 32, 2)
    s.set_mesh_dict(mesh)
    s.set_material(np.ones(K), np.ones(K), np.ones(K))
    s.set_dt(1e-3)
    rng = np.random.default_rng(n)
    q = rng.standard_normal((2, K, 9, 84)) * 10.0 ** rng.integers(-44, 38, (2, K, 9, 84))
    q.reshape(2, -1)[:, :4] = [np.inf, -np.inf, np.nan, 1e300]
    with np.errstate(over="ignore"):
        want = q.astype(np.float32).astype(np.float64)
    q = q.reshape((2,) + s.get_fields(0).shape)
    for shot in (0, 1):
        s.set_fields(shot, q[shot])
    for shot in (0, 1):
        np.testing.assert_array_equal(s.get_fields(shot).ravel(), want[shot].ravel())
    s.close()
