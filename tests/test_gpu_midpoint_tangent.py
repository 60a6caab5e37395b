"""The midpoint solves' polynomial for tan(theta) / theta: step angles on both sides of every
change of its number of terms, against the oracle.

Tolerances are those of the other parity tests: 1e-12 per point in FP64, 1e-5 in FP32.
"""
import numpy as np
import pytest

import oracle
from paper_1607_03062_amd import workloads as wl

from .test_gpu_parity import FP32_N_ABS, FP64_N_ABS, run

pytestmark = pytest.mark.gpu


# largest step angle dt E of the grid; second order changes its terms near .015, .072 and .18
# (FP32) and near .015, .03 and .092 (FP64); past .20 the cosine form takes over
@pytest.mark.parametrize("theta", [1e-5, 0.0150, 0.0178, 0.0185, 0.030, 0.036, 0.095, 0.108, 0.19, 0.26])
@pytest.mark.parametrize("scheme", ["midpoint", "midpoint4"])
@pytest.mark.parametrize("ellipticity", [0.0, 0.5])
def test_step_angles(gpu, theta, scheme, ellipticity):
    g = {"nx": 17, "ny": 40, "px": (-1.3, 2.1), "py": (-0.9, 1.7)}
    f, N = wl.constant(0.05, 40.0, ellipticity), 600
    s = gpu.Solver.for_grid(g, "fp64", scheme)
    e_max = s.check_field(f, N)["E_max"]
    s.close()
    f = wl.constant(0.05, theta * N / e_max, ellipticity)
    n_o = oracle.solve_grid(f, g, N, scheme)[0]
    for precision, tol in (("fp64", FP64_N_ABS), ("fp32", FP32_N_ABS)):
        n, _, info = run(gpu, g, f, N, precision, scheme)
        assert np.max(np.abs(n - n_o)) <= tol, (precision, info["taylor_order"])
