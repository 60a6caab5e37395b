"""The Strang solves by columns (grids of at least 32 rows, half angles up to pi/4) at the
sizes where their tiling and their step loop can go wrong, against the oracle, and against
the row kernel that grids of fewer rows take.

Tolerances are those of the other parity tests: 1e-12 per point in FP64, 1e-5 in the FP32
forms; two FP64 paths may each be 1e-12 off, so they agree to 2e-12.
"""
import math

import numpy as np
import pytest

import oracle
from paper_1607_03062_amd import workloads as wl

from .test_gpu_parity import FP32_N_ABS, FP64_N_ABS, run

pytestmark = pytest.mark.gpu


def _grid(nx, ny):
    return {"nx": nx, "ny": ny, "px": (-1.3, 2.1), "py": (-0.9, 1.7)}


# one column; columns that do not fill a group of 16; rows that leave part of a band, of a
# wave and of the last wave empty, for every number of rows a lane takes
@pytest.mark.parametrize("nx,ny", [(1, 32), (2, 33), (15, 63), (16, 64), (17, 65), (5, 127), (33, 100), (3, 513)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32fast"])
def test_edges_of_the_tiling(gpu, nx, ny, precision):
    g, f, N = _grid(nx, ny), wl.sin2(0.3, 0.6, 3), 700  # a chunk of 512 steps, then a part of one
    n_o = oracle.solve_grid(f, g, N)[0]
    ref = run(gpu, g, f, N, precision)
    assert np.max(np.abs(ref[0] - n_o)) <= (FP64_N_ABS if precision == "fp64" else FP32_N_ABS)
    for ppl, block in ((1, 64), (2, 128), (4, 256)):
        n, rho, _ = run(gpu, g, f, N, precision, "strang", ppl, block)
        assert np.array_equal(n, ref[0]) and rho == ref[1], (ppl, block)


# eight points per lane, which large grids take where they fill the device evenly
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32fast"])
def test_eight_points_per_lane(gpu, precision):
    nx, ny = 1019, 1021
    g, f, N = _grid(nx, ny), wl.sin2(0.3, 0.6, 3), 700
    ref = run(gpu, g, f, N, precision)
    assert ref[2]["points_per_lane"] == 8
    n, rho, _ = run(gpu, g, f, N, precision, "strang", 1, 256)
    assert np.array_equal(n, ref[0]) and rho == ref[1]
    idx = np.unique(np.concatenate([np.arange(40), np.arange(nx * ny - 40, nx * ny),
                                    np.random.default_rng(3).integers(0, nx * ny, 200)]))
    n_o = oracle.solve_grid(f, g, N, idx=idx)[0]
    assert np.max(np.abs(n[idx] - n_o)) <= (FP64_N_ABS if precision == "fp64" else FP32_N_ABS)


# runs of steps with nothing but single steps, one group, a group and single steps, a
# chunk's end, the renormalisation at 1024 steps; cut anywhere
@pytest.mark.parametrize("N", [1, 2, 3, 5, 9, 17, 24, 513, 1026])
@pytest.mark.parametrize("scheme,ellipticity", [("strang", 0.0), ("strang4", 0.0), ("strang", 0.5), ("strang4", 0.5)])
def test_step_counts(gpu, N, scheme, ellipticity):
    g = _grid(18, 70)
    f = wl.sin2(0.2, 0.9, 2, ellipticity) if N > 20 else wl.constant(0.2, 0.05 * N, ellipticity)
    n_o = oracle.solve_grid(f, g, N, scheme)[0]
    for precision in ("fp64", "fp32", "fp32fast"):
        n, rho, _ = run(gpu, g, f, N, precision, scheme)
        assert np.max(np.abs(n - n_o)) <= (FP64_N_ABS if precision == "fp64" else FP32_N_ABS), precision
        if N > 2:
            c = run(gpu, g, f, N, precision, scheme, chunks=[N // 3, N // 2, N - N // 3 - N // 2])
            assert np.array_equal(c[0], n) and c[1] == rho, precision


# step angles dt |p + A| up to: series of 3, 5, 8 terms, the loop, and past pi/4, where the
# rows kernel takes over
@pytest.mark.parametrize("phase", [0.01, 0.04, 0.12, 0.3, 0.7, 0.78, 0.8, 1.2])
@pytest.mark.parametrize("scheme", ["strang", "strang4"])
@pytest.mark.parametrize("ellipticity", [0.0, 0.5])
def test_step_angles(gpu, phase, scheme, ellipticity):
    g = _grid(17, 40)
    f = wl.constant(0.05, 40.0, ellipticity)
    s = gpu.Solver.for_grid(g, "fp64", scheme)
    e_max = s.check_field(f, 400)["E_max"]
    s.close()
    cmax = 1.0 if scheme == "strang" else abs(1 - 4 / (4 - 4 ** (1 / 3)))
    N = math.ceil(40.0 * e_max * cmax / phase)
    for precision in ("fp64", "fp32", "fp32fast"):
        n, _, info = run(gpu, g, f, N, precision, scheme)
        n_o = oracle.solve_grid(f, g, N, scheme)[0]
        assert np.max(np.abs(n - n_o)) <= (FP64_N_ABS if precision == "fp64" else FP32_N_ABS), (N, precision)


@pytest.mark.parametrize("scheme,ellipticity,valley", [("strang", 0.0, "both"), ("strang", 0.4, "K-"),
                                                       ("strang4", 0.0, "K-"), ("strang4", 0.4, "both")])
def test_columns_agree_with_rows(gpu, scheme, ellipticity, valley):
    """48 rows at once (by columns) and the same rows as three grids of 16 (the row kernel),
    with snapshots on the way."""
    ny, part, nx, N, k = 48, 16, 21, 900, 411
    dy = 2.4 / ny
    f = wl.sin2(0.25, 0.7, 3, ellipticity)

    def solve(py0, rows):
        g = {"nx": nx, "ny": rows, "px": (-1.5, 1.25), "py": (py0, py0 + rows * dy)}
        s = gpu.Solver.for_grid(g, "fp64", scheme, valley).set_field(f, N)
        mid, end = np.empty(nx * rows), np.empty(nx * rows)
        s.propagate(k)
        s.snapshot(n_out=mid)
        s.propagate(-1)
        s.density(n_out=end)
        s.close()
        return mid, end

    whole = solve(-1.1, ny)
    parts = [solve(-1.1 + i * part * dy, part) for i in range(ny // part)]
    for a, b in zip(whole, (np.concatenate(x) for x in zip(*parts))):
        assert np.max(np.abs(a - b)) <= 2 * FP64_N_ABS


def test_valleys_are_mirrored(gpu):
    """K- is K+ with every angle negated: the same bits, dithered coefficients included."""
    g, f, N = {"nx": 24, "ny": 36, "px": (-1.2, 1.2), "py": (-1.0, 1.0)}, wl.sin2(0.2, 0.6, 4), 1500
    for precision in ("fp64", "fp32", "fp32fast"):
        got = []
        for valley in ("K+", "K-"):
            s = gpu.Solver.for_grid(g, precision, "strang", valley).set_field(f, N)
            n = np.empty(24 * 36)
            s.propagate(-1)
            s.density(n_out=n)
            s.close()
            got.append(n)
        assert np.array_equal(*got), precision


@pytest.mark.parametrize("precision,arrangement", [("fp32", "once"), ("fp32fast", "fast")])
@pytest.mark.parametrize("ny", [24, 48])
def test_fp32_roundings_are_the_models(gpu, precision, arrangement, ny):
    """The FP32 forms' roundings one by one, by rows (24) and by columns (48): PD_FP32 rounds each
    component once in every rotation.  The CPU model of that arithmetic gives the same n(p),
    projected in FP64, except where a double rounding of its emulated multiply-adds (about
    1 in 2^28) or a coefficient at a tie falls differently: at most 1 point in 100 over the
    600 steps' 8 roundings of 3 components.  Another arrangement of them leaves no point in ten."""
    from tests import fp32_model

    g, f, N = {"nx": 40, "ny": ny, "px": (-1.7, 2.0), "py": (-1.9, 1.6)}, wl.sin2(0.2, 0.6, 2), 600
    n = run(gpu, g, f, N, precision)[0]
    model = fp32_model.solve_grid(f, g, N, arrangement=arrangement)
    ok = np.isfinite(model)
    assert np.mean(np.abs(n - model)[ok] > 1e-12) <= 0.01


def test_eight_points_per_lane_as_reported(gpu):
    """The points per lane that a handle reports can be set on it; eight stay with the solves by
    columns: not for a smaller grid, nor for a field that takes the handle to the other kernel."""
    g, f, N = _grid(1019, 1021), wl.sin2(0.3, 0.6, 3), 700
    big, wide = gpu.Solver.for_grid(g, "fp64").set_field(f, N), wl.constant(0.05, 40.0)
    shape = big.info()["points_per_lane"]
    assert shape == 8
    rho = big.solve()
    assert big.set_launch(shape).rewind().solve() == rho and big.info()["points_per_lane"] == 8

    small = gpu.Solver.for_grid(_grid(20, 40), "fp64").set_field(f, N)
    with pytest.raises(gpu.PDError):
        small.set_launch(8)
    small.close()

    steps = math.ceil(40.0 * big.check_field(wide, 400)["E_max"])  # dt |p + A| up to 1
    big.set_field(wide, steps)
    assert big.info()["points_per_lane"] == 4
    other = gpu.Solver.for_grid(g, "fp64").set_field(wide, steps)
    assert big.solve() == other.solve()
    with pytest.raises(gpu.PDError):
        big.set_launch(8)
    big.close()
    other.close()
