"""The Strang solves by rows: grids of fewer than 32 rows and step angles past the column
kernel's, in every way their kernel reads the field's rows, and as members of a batch beside
solves by columns.

Tolerances are those of the other parity tests: 1e-12 per point in FP64, 1e-5 in the FP32
forms, against the oracle; ways to run the same solve agree bit for bit.
"""
import numpy as np
import pytest

import oracle
from paper_1607_03062_amd import workloads as wl

from .test_gpu_parity import FP32_N_ABS, FP64_N_ABS, run

pytestmark = pytest.mark.gpu

THIN = {"nx": 37, "ny": 29, "px": (-1.3, 2.1), "py": (-0.9, 1.7)}
TALL = {"nx": 37, "ny": 53, "px": (-1.3, 2.1), "py": (-0.9, 1.7)}
PULSE = wl.sin2(0.3, 0.6, 3)
PRECISIONS = ["fp64", "fp32", "fp32fast"]


def _tol(precision):
    return FP64_N_ABS if precision == "fp64" else FP32_N_ABS


def _large(pd, grid, scheme, versine, ellipticity=0.0):
    """(field, N) whose largest half angle is 0.95, past pi/4, in shear form, or 1.95, past it."""
    f = wl.constant(0.05, 40.0, ellipticity)
    s = pd.Solver.for_grid(grid, "fp64", scheme)
    e_max = s.check_field(f, 1000)["E_max"]
    s.close()
    N = int(40.0 * e_max * (1.0 if scheme == "strang" else 4 / (4 - 4 ** (1 / 3)) - 1) / (1.95 if versine else 0.95))
    return f, N


# thin grids; and many rows with steps too large for one rotation about x, in both forms
@pytest.mark.parametrize("case", ["thin", "large", "versine"])
@pytest.mark.parametrize("scheme,ellipticity", [("strang", 0.0), ("strang4", 0.0), ("strang", 0.5), ("strang4", 0.5)])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_every_launch_shape(gpu, case, scheme, ellipticity, precision):
    grid = THIN if case == "thin" else TALL
    if case == "thin":
        field, N = wl.sin2(0.3, 0.6, 3, ellipticity), 1111
    else:
        field, N = _large(gpu, grid, scheme, case == "versine", ellipticity)
    n_o = oracle.solve_grid(field, grid, N, scheme)[0]
    ref = None
    for ppl, block, stage, chunk in [(1, 64, 2, 0), (2, 256, 2, 0), (4, 128, 2, 0), (2, 128, 1, 64), (4, 256, 1, 1024),
                                     (1, 64, 1, 256)]:
        n, rho, info = run(gpu, grid, field, N, precision, scheme, ppl, block, stage=stage, chunk_steps=chunk)
        if ref is None:
            ref = n, rho
            assert np.max(np.abs(n - n_o)) <= _tol(precision)
            assert info["rotation_form"] == (1 if case == "versine" else 0)
        assert np.array_equal(n, ref[0]) and rho == ref[1], (ppl, block, stage, chunk)


# ranges of steps with no whole group, one, an odd and an even number of them, from every phase,
# by the scalar unit and from the LDS
@pytest.mark.parametrize("scheme,ellipticity", [("strang", 0.0), ("strang4", 0.0), ("strang", 0.5), ("strang4", 0.5)])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_short_chunks(gpu, scheme, ellipticity, precision):
    chunks = [5, 8, 16, 24, 17, 15, 9, 33, 64, 7, 40, 3, 32, 1, 31, 48, 4, 12, 20, 2]
    field = wl.sin2(0.3, 0.6, 3, ellipticity)
    single = run(gpu, THIN, field, sum(chunks), precision, scheme)
    assert np.max(np.abs(single[0] - oracle.solve_grid(field, THIN, sum(chunks), scheme)[0])) <= _tol(precision)
    for stage in (1, 2):
        n, rho, _ = run(gpu, THIN, field, sum(chunks), precision, scheme, chunks=chunks, stage=stage, chunk_steps=64)
        assert np.array_equal(n, single[0]) and rho == single[1], stage


def test_batch_of_rows_and_columns(gpu):
    """Members by rows (thin, in each precision; versine in each precision) and by columns in one
    captured graph, replayed, and in epochs with uneven limits: the solves alone, bit for bit."""
    specs = [({"nx": 41, "ny": 20, "px": (-2.0, 2.0), "py": (-1.0, 1.0)}, wl.sin2(0.2, 0.5, 3), 1300 + 170 * q, p)
             for q, p in enumerate(PRECISIONS)]
    specs += [(TALL, *_large(gpu, TALL, "strang", True), p) for p in PRECISIONS]
    specs += [(wl.grid(64, 2.0), wl.sin2(0.1, 0.5, 4), 900 + 400 * q, p) for q, p in enumerate(PRECISIONS)]
    ms, refs = [], []
    for g, f, N, p in specs:
        s = gpu.Solver.for_grid(g, p).set_field(f, N)
        n = np.empty(s.nx * s.ny)
        rho = s.solve(n_out=n)
        n_o = oracle.solve_grid(f, g, N)[0]
        assert np.max(np.abs(n - n_o)) <= _tol(p)
        refs.append((n, rho))
        ms.append(s.rewind())
    assert [s.info()["rotation_form"] for s in ms] == [0, 0, 0, 1, 1, 1, 0, 0, 0]

    def check(rho):
        for s, r, (n_ref, rho_ref), spec in zip(ms, rho, refs, specs):
            n = np.empty(s.nx * s.ny)
            s.density(n_out=n, want_rho=False)
            assert r == rho_ref and np.array_equal(n, n_ref), spec

    b = gpu.Batch(ms)
    for _ in range(3):
        check(b.run())
        gpu.Solver.for_grid(wl.grid(40, 1.5), "fp64").set_field(PULSE, 200).solve()  # eager work between replays
    for s in ms:
        s.rewind()
    done, rho = np.zeros(len(ms), dtype=bool), np.full(len(ms), np.nan)
    for e in range(40):
        r, done = b.step_each([(137 + 91 * ((i + e) % 4)) if (i + e) % 5 else 0 for i in range(len(ms))])
        rho = np.where(np.isnan(r), rho, r)
        if done.all():
            break
    assert done.all()
    check(rho)
    b.close()
    for s in ms:
        s.close()
