"""The library's side-by-side sampling of the analytic fields at the sizes and pulse shapes
where its blocks of 256 samples and its pieces (rise, flat, fall) change over, against the
oracle.  4e-15 of the field's scale, as for the other sampling tests; past a phase of 2^20,
where single samples are evaluated instead, the rounding of the phase itself."""
import numpy as np
import pytest

import oracle
from paper_1607_03062_amd import _lib

PULSE = {"kind": "pulse", "E0": 0.8, "omega": 0.5, "phi": 0.4, "omega_rise": 0.07, "omega_fall": 0.11,
         "duration": 60.0, "ellipticity": 0.6}
FIELDS = {
    "sin2": {"kind": "sin2", "E0": 0.3, "omega": 0.4, "cycles": 3, "ellipticity": 0.5},
    "sin2_two_cycles": {"kind": "sin2", "E0": 0.3, "omega": 0.4, "cycles": 2, "ellipticity": -0.5},
    "constant": {"kind": "constant", "E0": 0.2, "t_end": 31.0, "ellipticity": 0.3},
    "pulse": PULSE,
    "pulse_no_flat_part": dict(PULSE, duration=np.pi / 0.14 + np.pi / 0.22),
    "pulse_resonant_rise": dict(PULSE, omega=0.14),  # the lower side band of the rise at zero frequency
    "pulse_resonant_fall": dict(PULSE, omega=0.22),
}


@pytest.mark.parametrize("N", [1, 2, 7, 255, 256, 257, 1000, 40000])
@pytest.mark.parametrize("kind", sorted(FIELDS))
@pytest.mark.parametrize("scheme", ["strang", "strang4"])
def test_samples_match_the_oracle(kind, N, scheme):
    f = FIELDS[kind]
    Ax, Ay, _ = _lib.sample_field_xy(f, N, scheme)
    ox, oy = oracle.field_table(f, N, scheme)[0], oracle.field_table_y(f, N, scheme)[0]
    scale = max(1.0, np.abs(ox).max(), np.abs(oy).max())
    assert np.max(np.abs(Ax - ox)) <= 4e-15 * scale and np.max(np.abs(Ay - oy)) <= 4e-15 * scale


def test_large_phases():
    f = dict(PULSE, phi=3e6, ellipticity=0.0)
    Ax = _lib.sample_field_xy(f, 500, "strang")[0]
    assert np.max(np.abs(Ax - oracle.field_table(f, 500, "strang")[0])) <= 8 * 3e6 * 2.0 ** -52


@pytest.mark.parametrize("omega_rise", [np.inf, 1e308])
@pytest.mark.parametrize("omega_fall", [0.11, np.inf])
@pytest.mark.parametrize("N", [1, 7, 300])
def test_a_pulse_without_a_finite_rise_is_refused(omega_rise, omega_fall, N):
    """Also where no sample lies in a part whose integral is not finite."""
    for ellipticity in (0.0, 0.6):
        with pytest.raises(_lib.PDError) as e:
            _lib.sample_field_xy(dict(PULSE, omega_rise=omega_rise, omega_fall=omega_fall, ellipticity=ellipticity), N)
        assert e.value.status == _lib.PD_ERR_INVALID


def _integral(f, phase, t):
    """-E0 int_0^t env(s) cos(omega s + phase) ds at the increasing times t: Gauss-Legendre
    rules of 16 nodes between the times, the corners of the envelope and 400 even steps, summed
    in extended precision."""
    L = np.longdouble
    pi = L("3.14159265358979323846264338")
    W = [L(f["omega_rise"]), L(f["omega_fall"])]
    corners = [pi / (2 * W[0]), L(f["duration"]) - pi / (2 * W[1])]
    x, w = np.polynomial.legendre.leggauss(16)
    edges = np.sort(np.concatenate([corners, t.astype(L), np.linspace(0, f["duration"], 401).astype(L)]))
    a, h = edges[:-1, None], np.diff(edges)[:, None] / 2
    s = a + h * (1 + x.astype(L))
    env = np.where(s < corners[0], np.sin(W[0] * s) ** 2, np.where(s > corners[1], np.cos(W[1] * (s - corners[1])) ** 2, 1))
    parts = (h * w.astype(L) * env * np.cos(L(f["omega"]) * s + L(phase))).sum(axis=1)
    total = np.concatenate([[L(0)], np.cumsum(parts)])
    return -L(f["E0"]) * total[np.searchsorted(edges, t.astype(L), side="right") - 1]


# a side band at a frequency near zero, in the rise and in the fall, and a carrier of far less
# than a period: what divides by the small frequency has to lose nothing to it
@pytest.mark.parametrize("detuning", [5e-17, 1e-12, 1e-9, 1e-6, 1e-4, 1e-2, 0.2])
@pytest.mark.parametrize("part", ["omega_rise", "omega_fall", "omega"])
@pytest.mark.parametrize("N", [3, 300])
def test_slow_parts_of_a_pulse(detuning, part, N):
    f = {"kind": "pulse", "E0": 0.8, "omega": 0.6, "phi": 0.4, "omega_rise": 0.07, "omega_fall": 0.11,
         "duration": 60.0, "ellipticity": 1.0}
    if part == "omega":
        f["omega"] = 0.6 * detuning
    else:
        f[part] = 0.1 * 3 * (1 + detuning)  # 0.1 * 3 is not 0.3: off the resonance by a rounding
    got, of_oracle = _lib.sample_field_xy(f, N), (oracle.field_table(f, N)[0], oracle.field_table_y(f, N)[0])
    t = (np.arange(N) + 0.5) * (f["duration"] / N)
    # a rounding of each term's phase (up to 80 here), once per end of each of three parts
    w, span = f["omega"], np.pi / 2 / 0.07
    size = min(1 / w, 60.0) + 0.25 / (w + 0.14) + span / 4
    tol = 3 * 2.0 ** -52 * (1 + 60 * (w + 0.62)) * f["E0"] * size
    ends = np.array([f["duration"]])
    for samples, other, end, phase in zip(got, of_oracle, (got[2][3], got[2][5]), (0.4, 0.4 - 0.5 * np.pi)):
        want = _integral(f, phase, t)
        assert np.max(np.abs(samples - want)) <= tol and np.max(np.abs(other - want)) <= tol
        assert abs(end - _integral(f, phase, ends)[0]) <= tol
