// Host side of the field: the vector potential A(t) of each supported field
// kind (both components), sampled at the times the scheme uses, and the per-step
// rows and per-point rotation coefficients the kernels read.
//
// Gauge A_0 = 0, E = -dA/dt, A(t) = -int_{t_i}^{t} E (Sec. II, after Eq. (2));
// A is sampled at the step midpoints t_i + (k + 1/2) dt (Sec. III, Eqs. (11)-(12)),
// or for the fourth-order composition at the stage midpoints t_i + (k + sigma_j) dt.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "pd_internal.h"

namespace pdx {
namespace {

constexpr double kPi = 3.14159265358979323846;

// Phase below which the sines at the ends of an interval are not subtracted: their
// difference, divided by the frequency, has lost some 1 / phase of its digits.
constexpr double kShortPhase = 0.5;

// 2 sin^2(x/2) = 1 - cos x without cancellation at small x.
double versine(double x) {
  double s = std::sin(0.5 * x);
  return 2.0 * s * s;
}

// sin^2-envelope pulse E0 sin^2(pi t / T) sin(w t) on [0, T]: with W = 2 pi / T,
// E = (E0/2) sin(w t) - (E0/4) sin((w + W) t) - (E0/4) sin((w - W) t), whose
// integral from 0 is a sum of versines.  Elliptic: E_y = e E0 sin^2(pi t/T) cos(w t)
// = (e E0/2) cos(w t) - (e E0/4)[cos((w + W) t) + cos((w - W) t)], integral a sum of sines.
struct Sin2Pulse {
  double E0, w, W, T, e;
  double A(double t) const {
    if (t <= 0.0) return 0.0;
    if (t > T) t = T;
    double I = versine(w * t) / (2.0 * w) - versine((w + W) * t) / (4.0 * (w + W)) -
               versine((w - W) * t) / (4.0 * (w - W));
    return -E0 * I;
  }
  double Ay(double t) const {
    if (t <= 0.0) return 0.0;
    if (t > T) t = T;
    double I = std::sin(w * t) / (2.0 * w) - std::sin((w + W) * t) / (4.0 * (w + W)) -
               std::sin((w - W) * t) / (4.0 * (w - W));
    return -e * E0 * I;
  }
};

// The laser pulse of Sec. IV, Eq. (14): carrier cos(w t + phi) under an envelope
// that rises as sin^2(Wr t) over [0, tr], tr = pi/(2 Wr), is flat, and falls as
// cos^2(Wf (t - ta)) over [ta, D], ta = D - pi/(2 Wf).  Its y component (elliptic)
// has the carrier sin(w t + phi) = cos(w t + phi - pi/2).
struct LaserPulse {
  double E0, w, phi, Wr, Wf, D;
  double tr() const { return kPi / (2.0 * Wr); }
  double ta() const { return D - kPi / (2.0 * Wf); }
  // int_a^b cos(w t + q) dt: the difference of the sines, or over less than kShortPhase the
  // interval times the cosine at its middle times sin(h) / h, h half the phase it covers,
  // which loses nothing to a small w.
  static double carrier(double w, double q, double a, double b) {
    const double h = 0.5 * (w * (b - a));
    if (std::fabs(2.0 * h) < kShortPhase)
      return (b - a) * (h != 0.0 ? std::sin(h) / h : 1.0) * std::cos(w * (0.5 * (a + b)) + q);
    return (std::sin(w * b + q) - std::sin(w * a + q)) / w;
  }
  double carrier(double q, double a, double b) const { return carrier(w, q, a, b); }
  // int_a^b cos(2 W (t - c)) cos(w t + q) dt, the side bands w + 2 W and w - 2 W
  double beat(double q, double W, double c, double a, double b) const {
    return 0.5 * (carrier(w + 2.0 * W, q - 2.0 * W * c, a, b) + carrier(w - 2.0 * W, q + 2.0 * W * c, a, b));
  }
  // -E0 int_0^t env(s) cos(w s + q) ds
  double A_phase(double q, double t) const {
    if (t <= 0.0) return 0.0;
    if (t > D) t = D;
    double r = tr(), a = ta(), I = 0.0;
    double e1 = std::fmin(t, r);  // rise: sin^2 = (1 - cos 2 Wr t) / 2
    I += 0.5 * carrier(q, 0.0, e1) - 0.5 * beat(q, Wr, 0.0, 0.0, e1);
    if (t > r) {
      double e2 = std::fmin(t, a);
      if (e2 > r) I += carrier(q, r, e2);
      if (t > a) I += 0.5 * carrier(q, a, t) + 0.5 * beat(q, Wf, a, a, t);  // fall: cos^2 = (1 + cos 2 Wf (t - a)) / 2
    }
    return -E0 * I;
  }
};

bool finite(double x) { return std::isfinite(x); }

// (A_x, A_y) of an analytic field kind at time t (the kind is validated).
void eval_A(const pd_field& f, double t, double* ax, double* ay) {
  switch (f.kind) {
    case PD_FIELD_SIN2: {
      double T = f.cycles * 2.0 * kPi / f.omega;
      Sin2Pulse s{f.E0, f.omega, 2.0 * kPi / T, T, f.ellipticity};
      *ax = s.A(t);
      *ay = f.ellipticity != 0.0 ? s.Ay(t) : 0.0;
      return;
    }
    case PD_FIELD_CONSTANT: {
      double u = t <= 0.0 ? 0.0 : (t < f.t_end ? t : f.t_end);
      *ax = -f.E0 * u;
      *ay = f.ellipticity != 0.0 ? -f.ellipticity * f.E0 * u : 0.0;
      return;
    }
    case PD_FIELD_PULSE: {
      LaserPulse p{f.E0, f.omega, f.phi, f.omega_rise, f.omega_fall, f.duration};
      *ax = p.A_phase(f.phi, t);
      *ay = f.ellipticity != 0.0 ? f.ellipticity * p.A_phase(f.phi - 0.5 * kPi, t) : 0.0;
      return;
    }
    default:
      *ax = 0.0;
      *ay = 0.0;
  }
}

// A component of A over [begin, end] as c0 + lin t + sum_i amp_i f(freq_i t + phase_i), f the
// sine or its square: what an analytic field is between the corners of its envelope.  Many
// samples of it are evaluated side by side (sample_span).
struct SineSum {
  double end = 0, c0 = 0, lin = 0;
  bool squared = false;
  bool slow = false;  // a sine covers less than kShortPhase: c0 cancels it
  int n = 0;
  double amp[3] = {}, freq[3] = {}, phase[3] = {};
  void add(double a, double w, double q) {
    amp[n] = a;
    freq[n] = w;
    phase[n++] = q;
  }
  // c0 such that the value at t is `value`
  void pass_through(double t, double value) {
    double v = lin * t;
    for (int i = 0; i < n; ++i) v += amp[i] * std::sin(freq[i] * t + phase[i]);
    c0 = value - v;
  }
};

// pi in three parts of 33, 33 and 53 bits: a multiple below 2^20 of the first two is exact.
constexpr double kPiA = 0x1.921fb54400000p+1, kPiB = 0x1.0b4611a600000p-33, kPiC = 0x1.3198a2e037073p-68;

// sin x to 4e-16 for |x| < 2^20 (the samples' arguments are rounded by far more): x less the nearest multiple k pi,
// the Taylor series to x^23 (its next term is 5e-21 at pi/2), the sign of an odd k.  Without
// branches or library calls, so that a loop over it runs in vector registers.
inline __attribute__((always_inline)) double sin_lane(double x) {
  constexpr double kMagic = 0x1.8p52;  // adding it rounds to a whole number, in its low bits
  const double m = x * (1.0 / kPi) + kMagic, k = m - kMagic;
  const double r = ((x - k * kPiA) - k * kPiB) - k * kPiC, z = r * r;
  // in pairs, pairs of pairs and so on: short chains, which loops over it overlap
  const double z2 = z * z, z4 = z2 * z2, z8 = z4 * z4;
  const double p0 = -1.0 / 6.0 + z * (1.0 / 120.0), p1 = -1.0 / 5040.0 + z * (1.0 / 362880.0);
  const double p2 = -1.0 / 39916800.0 + z * (1.0 / 6227020800.0);
  const double p3 = -1.0 / 1307674368000.0 + z * (1.0 / 355687428096000.0);
  const double p4 = -1.0 / 121645100408832000.0 + z * (1.0 / 51090942171709440000.0);
  const double p = ((p0 + z2 * p1) + z4 * (p2 + z2 * p3)) + z8 * (p4 - z2 * (1.0 / 25852016738884976640000.0));
  const double v = r + r * (z * p);
  uint64_t odd, bits;
  std::memcpy(&odd, &m, sizeof odd);
  std::memcpy(&bits, &v, sizeof bits);
  bits ^= odd << 63;
  double out;
  std::memcpy(&out, &bits, sizeof out);
  return out;
}
constexpr double kSinLaneMax = 0x1p20;

// out[i * stride] = the component at t0 + (first + i + sigma) dt, i < n <= kSpan.
constexpr int kSpan = 256;
inline __attribute__((always_inline)) void span_body(const SineSum& f, double t0, double first, double sigma,
                                                     double dt, int n, double* out, int stride) {
  double t[kSpan], v[kSpan];
  for (int i = 0; i < n; ++i) {
    t[i] = t0 + ((first + (double)i) + sigma) * dt;
    v[i] = f.c0 + f.lin * t[i];
  }
  for (int q = 0; q < f.n; ++q) {
    const double a = f.amp[q], w = f.freq[q], p = f.phase[q];
    if (f.squared)
      for (int i = 0; i < n; ++i) {
        const double y = sin_lane(w * t[i] + p);
        v[i] += a * (y * y);
      }
    else
      for (int i = 0; i < n; ++i) v[i] += a * sin_lane(w * t[i] + p);
  }
  for (int i = 0; i < n; ++i) out[(size_t)i * stride] = v[i];
}
// Twice, for four and for two doubles to a register.  Neither contracts a multiply and an
// add (no FMA in the target, -ffp-contract=off), so both give the same values.
__attribute__((target("avx2"))) void span_avx2(const SineSum& f, double t0, double first, double sigma, double dt,
                                               int n, double* out, int stride) {
  span_body(f, t0, first, sigma, dt, n, out, stride);
}
void span_base(const SineSum& f, double t0, double first, double sigma, double dt, int n, double* out, int stride) {
  span_body(f, t0, first, sigma, dt, n, out, stride);
}
void span(const SineSum& f, double t0, double first, double sigma, double dt, int n, double* out, int stride) {
  static const bool avx2 = __builtin_cpu_supports("avx2");
  (avx2 ? span_avx2 : span_base)(f, t0, first, sigma, dt, n, out, stride);
}

// The pieces of a component of an analytic field (validated), in time order.
int pieces_of(const pd_field& f, bool y, SineSum out[3]) {
  switch (f.kind) {
    case PD_FIELD_SIN2: {
      // see Sin2Pulse
      const double T = f.cycles * 2.0 * kPi / f.omega, W = 2.0 * kPi / T, w = f.omega;
      SineSum& p = out[0];
      p.end = T;
      if (y) {
        const double a = -f.ellipticity * f.E0;
        p.add(a / (2.0 * w), w, 0.0);
        p.add(-a / (4.0 * (w + W)), w + W, 0.0);
        p.add(-a / (4.0 * (w - W)), w - W, 0.0);
      } else {
        p.squared = true;
        p.add(-f.E0 / w, 0.5 * w, 0.0);
        p.add(f.E0 / (2.0 * (w + W)), 0.5 * (w + W), 0.0);
        p.add(f.E0 / (2.0 * (w - W)), 0.5 * (w - W), 0.0);
      }
      return 1;
    }
    case PD_FIELD_CONSTANT:
      out[0].end = f.t_end;
      out[0].lin = y ? -f.ellipticity * f.E0 : -f.E0;
      return 1;
    default: {
      // see LaserPulse: rise, flat, fall, each a carrier with or without its two side bands
      const double a = y ? f.ellipticity * f.E0 : f.E0, q = y ? f.phi - 0.5 * kPi : f.phi, w = f.omega;
      const LaserPulse lp{f.E0, w, f.phi, f.omega_rise, f.omega_fall, f.duration};
      const double ends[3] = {lp.tr(), lp.ta(), lp.D};
      double t = 0.0, value = 0.0;
      int m = 0;
      for (int part = 0; part < 3; ++part) {
        if (!(ends[part] > t)) continue;  // no flat part
        SineSum& p = out[m++];
        p.end = ends[part];
        if (part == 1) {
          p.add(-a / w, w, q);
        } else {
          // the side bands of cos(2 W (t - c)) cos(w t + q), subtracted in the rise and added in the fall
          const double W = part == 0 ? lp.Wr : lp.Wf, c = part == 0 ? 0.0 : lp.ta(), sign = part == 0 ? 0.25 : -0.25;
          const double w1 = w + 2.0 * W, w2 = w - 2.0 * W;
          p.add(-0.5 * a / w, w, q);
          p.add(sign * a / w1, w1, q - 2.0 * W * c);
          if (w2 != 0.0)
            p.add(sign * a / w2, w2, q + 2.0 * W * c);
          else
            p.lin = sign * a * std::cos(q + 2.0 * W * c);
        }
        for (int i = 0; i < p.n; ++i) p.slow = p.slow || std::fabs(p.freq[i] * (p.end - t)) < kShortPhase;
        p.pass_through(t, value);
        t = p.end;
        value = (y ? f.ellipticity * lp.A_phase(q, t) : lp.A_phase(q, t));
      }
      return m;
    }
  }
}

// Samples [k0, k1) of every stage of one component into `out` (stage stride S).  One by one
// where a sine of a piece is slow (its amplitude over a small frequency and c0 cancel) or a
// phase is past sin_lane's range.
void sample_component(const pd_field& f, bool y, double t_i, double dt, const Composition& comp, long long k0,
                      long long k1, double* out) {
  SineSum p[3];
  const int m = pieces_of(f, y, p);
  const int S = comp.stages;
  bool in_range = true;
  for (int i = 0; i < m; ++i)
    for (int q = 0; q < p[i].n; ++q)
      in_range = in_range && std::fabs(p[i].freq[q]) * p[i].end + std::fabs(p[i].phase[q]) < kSinLaneMax;
  const auto side_by_side = [&](const SineSum& f) { return in_range && !f.slow; };
  for (int j = 0; j < S; ++j) {
    const auto time = [&](long long k) { return t_i + ((double)k + comp.sigma[j]) * dt; };
    long long k = k0;
    for (int i = 0; i < m && k < k1; ++i) {
      // the samples up to the piece's end (the last piece takes the rest)
      long long e = k1;
      if (i + 1 < m) {
        e = std::min(k1, std::max(k, (long long)((p[i].end - t_i) / dt - comp.sigma[j])));
        while (e < k1 && time(e) <= p[i].end) ++e;
        while (e > k && time(e - 1) > p[i].end) --e;
      }
      for (; k < e; k += kSpan) {
        const int n = (int)std::min<long long>(kSpan, e - k);
        if (side_by_side(p[i])) {
          span(p[i], t_i, (double)k, comp.sigma[j], dt, n, out + (size_t)k * S + j, S);
        } else {
          double ax, ay;
          for (int v = 0; v < n; ++v) {
            eval_A(f, time(k + v), &ax, &ay);
            out[(size_t)(k + v) * S + j] = y ? ay : ax;
          }
        }
      }
      k = e;
    }
  }
}

// Whether every value is finite, and the range of the values with what *lo, *hi hold.
bool value_range(const std::vector<double>& v, double* lo, double* hi) {
  constexpr int kLanes = 8;
  double a[kLanes], b[kLanes], bad = 0.0;
  for (int i = 0; i < kLanes; ++i) {
    a[i] = *lo;
    b[i] = *hi;
  }
  const size_t n = v.size(), whole = n / kLanes * kLanes;
  double nan[kLanes] = {};
  for (size_t i = 0; i < whole; i += kLanes)
    for (int q = 0; q < kLanes; ++q) {
      const double x = v[i + q];
      a[q] = x < a[q] ? x : a[q];
      b[q] = x > b[q] ? x : b[q];
      nan[q] += x - x;  // 0 for a finite value, else NaN from here on
    }
  for (size_t i = whole; i < n; ++i) {
    a[0] = v[i] < a[0] ? v[i] : a[0];
    b[0] = v[i] > b[0] ? v[i] : b[0];
    bad += v[i] - v[i];
  }
  for (int q = 0; q < kLanes; ++q) {
    bad += nan[q];
    *lo = a[q] < *lo ? a[q] : *lo;
    *hi = b[q] > *hi ? b[q] : *hi;
  }
  return bad == 0.0;
}

}  // namespace

Composition composition_of(int scheme) {
  Composition c;
  if (scheme == PD_SCHEME_STRANG4 || scheme == PD_SCHEME_MIDPOINT4) {
    const double p = 1.0 / (4.0 - std::cbrt(4.0));
    c.stages = 5;
    const double v[5] = {p, p, 1.0 - 4.0 * p, p, p};
    double start = 0.0;
    c.cmax = 0.0;
    for (int j = 0; j < 5; ++j) {
      c.c[j] = v[j];
      c.sigma[j] = start + 0.5 * v[j];
      start += v[j];
      c.cmax = std::fmax(c.cmax, std::fabs(v[j]));
    }
  }
  return c;
}

bool sample_field(const pd_field& f, long long n_steps, const Composition& comp, FieldTables* out,
                  std::string* err) {
  if (n_steps < 1) {
    *err = "n_steps must be >= 1";
    return false;
  }
  if (n_steps > (1LL << 31)) {
    *err = "n_steps must be <= 2^31";
    return false;
  }
  const int S = comp.stages;
  const size_t n_samples = (size_t)n_steps * (size_t)S;
  FieldTables t;
  t.A_mid = std::move(out->A_mid);  // the buffers of what *out holds, used again
  t.Ay_mid = std::move(out->Ay_mid);
  t.n_steps = n_steps;
  t.comp = comp;
  t.spec = f;
  t.spec.A_mid = nullptr;
  t.spec.Ay_mid = nullptr;
  if (f.kind != PD_FIELD_TABLE && !finite(f.ellipticity)) {
    *err = "ellipticity must be finite";
    return false;
  }
  switch (f.kind) {
    case PD_FIELD_SIN2:
      if (!finite(f.E0) || !finite(f.omega) || f.omega <= 0.0) {
        *err = "sin2 field needs finite E0 and omega > 0";
        return false;
      }
      if (f.cycles < 2) {
        *err = "sin2 field needs cycles >= 2";
        return false;
      }
      t.t_i = 0.0;
      t.t_f = f.cycles * 2.0 * kPi / f.omega;
      break;
    case PD_FIELD_CONSTANT:
      if (!finite(f.E0) || !finite(f.t_end) || f.t_end <= 0.0) {
        *err = "constant field needs finite E0 and t_end > 0";
        return false;
      }
      t.t_i = 0.0;
      t.t_f = f.t_end;
      break;
    case PD_FIELD_PULSE: {
      LaserPulse p{f.E0, f.omega, f.phi, f.omega_rise, f.omega_fall, f.duration};
      if (!finite(f.E0) || !finite(f.omega) || !finite(f.phi) || f.omega <= 0.0 || !(f.omega_rise > 0.0) ||
          !(f.omega_fall > 0.0) || !finite(f.duration)) {
        *err = "pulse field needs finite E0, phi, duration and omega, omega_rise, omega_fall > 0";
        return false;
      }
      // a pulse with no flat part (duration = rise + fall window) is valid: allow rounding
      if (p.ta() < p.tr() - 1e-12 * std::fabs(f.duration)) {
        *err = "pulse duration shorter than its rise plus fall windows";
        return false;
      }
      t.t_i = 0.0;
      t.t_f = f.duration;
      break;
    }
    case PD_FIELD_TABLE:
      if (!f.A_mid || f.n_table != (long long)n_samples) {
        *err = S == 1 ? "table field needs A_mid with n_table == n_steps values"
                      : "table field needs A_mid with n_table == 5 * n_steps values (one per stage)";
        return false;
      }
      if (!finite(f.t_i) || !finite(f.t_f) || !(f.t_f > f.t_i) || !finite(f.A_in) || !finite(f.A_out)) {
        *err = "table field needs finite t_i < t_f, A_in, A_out";
        return false;
      }
      if (f.Ay_mid && (!finite(f.Ay_in) || !finite(f.Ay_out))) {
        *err = "table field with Ay_mid needs finite Ay_in, Ay_out";
        return false;
      }
      t.t_i = f.t_i;
      t.t_f = f.t_f;
      break;
    default:
      *err = "unknown field kind";
      return false;
  }
  t.dt = (t.t_f - t.t_i) / (double)n_steps;
  t.elliptic = f.kind == PD_FIELD_TABLE ? f.Ay_mid != nullptr : f.ellipticity != 0.0;
  t.A_mid.resize(n_samples);
  t.Ay_mid.resize(t.elliptic ? n_samples : 0);
  if (f.kind == PD_FIELD_TABLE) {
    std::memcpy(t.A_mid.data(), f.A_mid, n_samples * sizeof(double));
    if (t.elliptic) std::memcpy(t.Ay_mid.data(), f.Ay_mid, n_samples * sizeof(double));
    t.A_in = f.A_in;
    t.A_out = f.A_out;
    t.Ay_in = t.elliptic ? f.Ay_in : 0.0;
    t.Ay_out = t.elliptic ? f.Ay_out : 0.0;
  } else {
    // a thread is worth its start for some 30000 samples (3 ns each)
    parallel_ranges(n_steps, 32768 / S, [&](long long k0, long long k1) {
      sample_component(f, false, t.t_i, t.dt, comp, k0, k1, t.A_mid.data());
      if (t.elliptic) sample_component(f, true, t.t_i, t.dt, comp, k0, k1, t.Ay_mid.data());
    });
    eval_A(f, t.t_i, &t.A_in, &t.Ay_in);
    eval_A(f, t.t_f, &t.A_out, &t.Ay_out);
  }
  t.A_min = std::fmin(t.A_in, t.A_out);
  t.A_max = std::fmax(t.A_in, t.A_out);
  t.Ay_min = std::fmin(t.Ay_in, t.Ay_out);
  t.Ay_max = std::fmax(t.Ay_in, t.Ay_out);
  const bool x_ok = value_range(t.A_mid, &t.A_min, &t.A_max), y_ok = value_range(t.Ay_mid, &t.Ay_min, &t.Ay_max);
  // The end values by themselves: fmin and fmax pass over a NaN, and a pulse whose rise has
  // no finite integral need not have a sample there.
  if (!x_ok || !y_ok || !finite(t.A_in) || !finite(t.A_out) || !finite(t.Ay_in) || !finite(t.Ay_out)) {
    *err = "field has a non-finite value";
    return false;
  }
  if (!finite(t.A_min) || !finite(t.A_max) || !finite(t.Ay_min) || !finite(t.Ay_max) || !(t.dt > 0.0)) {
    *err = "field sampling produced non-finite values";
    return false;
  }
  *out = std::move(t);
  return true;
}

void boundary_A(const FieldTables& t, long long k, double* ax, double* ay) {
  const long long S = t.comp.stages;
  if (k <= 0) {
    *ax = t.A_in;
    *ay = t.Ay_in;
  } else if (k >= t.n_steps) {
    *ax = t.A_out;
    *ay = t.Ay_out;
  } else if (t.spec.kind == PD_FIELD_TABLE) {
    *ax = 0.5 * (t.A_mid[(size_t)(k * S - 1)] + t.A_mid[(size_t)(k * S)]);
    *ay = t.elliptic ? 0.5 * (t.Ay_mid[(size_t)(k * S - 1)] + t.Ay_mid[(size_t)(k * S)]) : 0.0;
  } else {
    eval_A(t.spec, t.t_i + (double)k * t.dt, ax, ay);
    if (!t.elliptic) *ay = 0.0;
  }
}

void field_extent(const Grid& g, FieldTables* t) {
  // |p + A| is largest at a corner of the box [grid range] x [A range], per component.
  double x0 = g.px(0), x1 = g.px(g.nx - 1);
  double y0 = g.py(0), y1 = g.py(g.ny - 1);
  double X = std::fmax(std::fmax(std::fabs(x0 + t->A_min), std::fabs(x0 + t->A_max)),
                       std::fmax(std::fabs(x1 + t->A_min), std::fabs(x1 + t->A_max)));
  double Y = std::fmax(std::fmax(std::fabs(y0 + t->Ay_min), std::fabs(y0 + t->Ay_max)),
                       std::fmax(std::fabs(y1 + t->Ay_min), std::fabs(y1 + t->Ay_max)));
  t->E_max = std::sqrt(X * X + Y * Y);
}

long long count_masked(const Grid& g, const FieldTables& t) {
  // |P| = sqrt(Px^2 + Py^2) is 0 only where Py^2 == 0; scan those rows.
  long long m = 0;
  for (int j = 0; j < g.ny; ++j) {
    double py = g.py(j);
    double Pyi = py + t.Ay_in, Pyo = py + t.Ay_out;
    if (Pyi * Pyi != 0.0 && Pyo * Pyo != 0.0) continue;
    for (int i = 0; i < g.nx; ++i) {
      double px = g.px(i);
      double Pi = px + t.A_in, Po = px + t.A_out;
      double Ei = std::sqrt(Pi * Pi + Pyi * Pyi), Eo = std::sqrt(Po * Po + Pyo * Pyo);
      if (Ei == 0.0 || Eo == 0.0) ++m;
    }
  }
  return m;
}

size_t table_row_values(int scheme, int elliptic) {
  const size_t S = (size_t)composition_of(scheme).stages;
  const size_t per = base_scheme(scheme) == PD_SCHEME_MIDPOINT ? 1 : 2;
  return per * S * (elliptic ? 2 : 1);
}

size_t table_row_bytes(int scheme, int precision, int elliptic) {
  size_t v = (base_scheme(scheme) == PD_SCHEME_STRANG && is_fp32(precision)) ? sizeof(float) : sizeof(double);
  return table_row_values(scheme, elliptic) * v;
}

long long table_rows(int scheme, int elliptic, long long n_steps) {
  return (base_scheme(scheme) == PD_SCHEME_STRANG && elliptic) ? n_steps + 1 : n_steps;
}

void rotation_coefficients(double half, int form, double* a, double* s) {
  double sh = std::sin(half), ch = std::cos(half);
  *s = 2.0 * sh * ch;
  *a = form == kFormShear ? sh / ch : -2.0 * sh * sh;
}

namespace {

template <typename R>
void put(std::vector<unsigned char>* bytes, size_t offset, size_t index, double v) {
  reinterpret_cast<R*>(bytes->data() + offset)[index] = (R)v;
}

}  // namespace

void build_step_table(const FieldTables& t, int scheme, int precision, int form, bool columns, double vsign,
                      std::vector<unsigned char>* rows) {
  const long long N = t.n_steps;
  const int S = t.comp.stages;
  const int ell = t.elliptic ? 1 : 0;
  const size_t W = table_row_values(scheme, ell);
  const long long R = table_rows(scheme, ell, N);
  const double* c = t.comp.c;
  // The y half steps of neighbouring stages (and of the last stage of a step and
  // the first of the next) are merged; the field part of the merged rotation
  // after stage j has half angle dt (c_j A_y,j + c_j+1 A_y,j+1) / 2.
  auto y_half = [&](long long k, int j) {
    auto ay = [&](long long kk, int jj) { return t.Ay_mid[(size_t)kk * S + jj]; };
    double sum;
    if (j + 1 < S)
      sum = c[j] * ay(k, j) + c[j + 1] * ay(k, j + 1);
    else if (k + 1 < N)
      sum = c[j] * ay(k, j) + c[0] * ay(k + 1, 0);
    else
      sum = c[j] * ay(k, j);  // closing half step
    return vsign * 0.5 * t.dt * sum;
  };
  const double open = ell ? vsign * 0.5 * t.dt * (c[0] * t.Ay_mid[0]) : 0.0;  // opening half step
  if (columns) {
    // half angles in FP64: per stage c_j dt A_x, then those of the y rotations' field parts
    const size_t V = (size_t)S * (ell ? 2 : 1);
    rows->resize((size_t)R * V * sizeof(double));
    double* d = reinterpret_cast<double*>(rows->data());
    for (int j = 0; j < S; ++j) {
      const double scale = vsign * (c[j] * t.dt);
      for (long long k = 0; k < N; ++k) d[(size_t)k * V + j] = scale * t.A_mid[(size_t)k * S + j];
    }
    if (ell) {
      for (long long k = 0; k < N; ++k)
        for (int j = 0; j < S; ++j) d[(size_t)k * V + S + j] = y_half(k, j);
      std::fill_n(d + (size_t)N * V, V, 0.0);
      d[(size_t)N * V + S] = open;
    }
    return;
  }
  rows->resize((size_t)R * table_row_bytes(scheme, precision, ell));
  std::fill(rows->end() - (std::ptrdiff_t)table_row_bytes(scheme, precision, ell), rows->end(), 0);
  if (base_scheme(scheme) == PD_SCHEME_MIDPOINT) {
    // per stage the phase increment c_j dt A at the stage midpoint (then c_j dt A_y)
    double* d = reinterpret_cast<double*>(rows->data());
    for (long long k = 0; k < N; ++k)
      for (int j = 0; j < S; ++j) {
        d[(size_t)k * W + j] = vsign * (c[j] * t.dt) * t.A_mid[(size_t)k * S + j];
        if (ell) d[(size_t)k * W + S + j] = vsign * (c[j] * t.dt) * t.Ay_mid[(size_t)k * S + j];
      }
    return;
  }
  // Strang.  exp(-i h A sigma_x) rotates the Bloch vector by 2h A about x: store the
  // coefficients of the rotation by 2 * half, half = c_j dt A (valley sign included).
  auto store = [&](long long row, size_t slot, double half) {
    double a, s;
    rotation_coefficients(half, form, &a, &s);
    if (is_fp32(precision)) {
      put<float>(rows, 0, (size_t)row * W + 2 * slot, a);
      put<float>(rows, 0, (size_t)row * W + 2 * slot + 1, s);
    } else {
      put<double>(rows, 0, (size_t)row * W + 2 * slot, a);
      put<double>(rows, 0, (size_t)row * W + 2 * slot + 1, s);
    }
  };
  for (long long k = 0; k < N; ++k)
    for (int j = 0; j < S; ++j) store(k, (size_t)j, vsign * (c[j] * t.dt) * t.A_mid[(size_t)k * S + j]);
  if (!ell) return;
  for (long long k = 0; k < N; ++k)
    for (int j = 0; j < S; ++j) store(k, (size_t)(S + j), y_half(k, j));
  store(N, (size_t)S, open);
}

size_t point_coefficient_pairs_x(int scheme, int precision) {
  return (composition_of(scheme).stages == 5 ? 2 : 1) * (size_t)coefficient_phases(precision);
}
size_t point_coefficient_pairs_y(int scheme, int precision) {
  return (composition_of(scheme).stages == 5 ? 2 : 1) * (size_t)coefficient_phases(precision) + 1;
}

namespace {

// The `phases` FP32 values of a coefficient x: the FP32 neighbours of |x| below
// and above it, the upper one in round(phases * f) of the phases, f being where |x|
// lies between them, with the sign of x (so that -x gives the negated values: the
// rotations of the K- valley are those of K+ with every angle negated); the phases
// that take the upper value are spread over the cycle (order 0, 2, 1, 3 for four
// phases), so that partial sums over the cycle stay close to x too.
void dither(double x, int phases, float* out) {
  if (x < 0.0) {
    dither(-x, phases, out);
    for (int h = 0; h < phases; ++h) out[h] = -out[h];
    return;
  }
  // neighbours of a float >= 0 differ by one in their bits
  float lo = (float)x, hi;
  uint32_t bits;
  std::memcpy(&bits, &lo, sizeof bits);
  if ((double)lo > x) --bits;
  std::memcpy(&lo, &bits, sizeof bits);
  ++bits;
  std::memcpy(&hi, &bits, sizeof bits);
  const double f = (x - (double)lo) / ((double)hi - (double)lo);
  const int up = (int)(f * phases + 0.5);
  for (int h = 0; h < phases; ++h) {
    // rank of phase h in the bit-reversed order of the cycle
    int r = 0;
    for (int b = 1, v = h; b < phases; b <<= 1, v >>= 1) r = (r << 1) | (v & 1);
    out[h] = r < up ? hi : lo;
  }
}

}  // namespace

void build_point_coefficients(const Grid& g, const FieldTables& t, int scheme, int precision, int form, bool columns,
                              double vsign, std::vector<unsigned char>* bytes, size_t* col_offset,
                              size_t* row_offset) {
  const bool f32 = is_fp32(precision);
  const size_t v = f32 ? sizeof(float) : sizeof(double);
  const int H = coefficient_phases(precision);
  const size_t nxp = point_coefficient_pairs_x(scheme, precision), nyp = point_coefficient_pairs_y(scheme, precision);
  auto align = [](size_t n) { return (n + 255) / 256 * 256; };
  *col_offset = align(bytes->size());
  *row_offset = align(*col_offset + (columns ? 0 : 2 * nxp * v * (size_t)g.nx));
  bytes->resize(align(*row_offset + 2 * nyp * v * (size_t)g.ny));
  // pair `pair` of `entry` (column or row) from the exact coefficients (a, s): one
  // value per phase in FP32 (dithered), the value itself in FP64
  auto store_pair = [&](size_t off, size_t entry, size_t per_entry, size_t pair, int phases, double a, double s) {
    float da[kDitherFP32], ds[kDitherFP32];
    if (f32 && phases > 1) {
      dither(a, phases, da);
      dither(s, phases, ds);
    }
    for (int h = 0; h < phases; ++h) {
      const size_t idx = 2 * (per_entry * entry + pair + (size_t)h);
      if (!f32) {
        put<double>(bytes, off, idx, a);
        put<double>(bytes, off, idx + 1, s);
      } else if (phases > 1) {
        put<float>(bytes, off, idx, da[h]);
        put<float>(bytes, off, idx + 1, ds[h]);
      } else {
        put<float>(bytes, off, idx, a);
        put<float>(bytes, off, idx + 1, s);
      }
    }
  };
  // Half-angle multipliers of dt px and dt py: x rotation of stage j: c_j; y
  // rotation after stage j: (c_j + c_j+1) / 2 (cyclic); opening / closing half: c_1 / 2.
  const double* c = t.comp.c;
  double mx[2], my[3];
  int nmx, nmy;  // distinct multipliers (the half step excluded)
  if (t.comp.stages == 5) {
    mx[0] = c[0];
    mx[1] = c[2];
    my[0] = 0.5 * (c[0] + c[1]);
    my[1] = 0.5 * (c[1] + c[2]);
    my[2] = 0.5 * c[0];
    nmx = nmy = 2;
  } else {
    mx[0] = 1.0;
    my[0] = 1.0;
    my[1] = 0.5;
    nmx = nmy = 1;
  }
  double a, s;
  for (int i = 0; i < (columns ? 0 : g.nx); ++i)
    for (int q = 0; q < nmx; ++q) {
      rotation_coefficients(vsign * (mx[q] * t.dt) * g.px(i), form, &a, &s);
      store_pair(*col_offset, (size_t)i, nxp, (size_t)q * H, H, a, s);
    }
  for (int j = 0; j < g.ny; ++j) {
    for (int q = 0; q < nmy; ++q) {
      rotation_coefficients(vsign * (my[q] * t.dt) * g.py(j), form, &a, &s);
      store_pair(*row_offset, (size_t)j, nyp, (size_t)q * H, H, a, s);
    }
    // the opening / closing half step: applied twice per solve, one value
    rotation_coefficients(vsign * (my[nmy] * t.dt) * g.py(j), form, &a, &s);
    store_pair(*row_offset, (size_t)j, nyp, (size_t)nmy * H, 1, a, s);
  }
}

int strang_form(const Grid& g, const FieldTables& t) {
  // Bloch rotation angles of a stage: 2 c dt A_x, 2 c dt px, at most 2 c dt py and
  // 2 c dt A_y (merged halves), c <= cmax.
  double amax = std::fmax(std::fabs(t.A_min), std::fabs(t.A_max));
  double aymax = std::fmax(std::fabs(t.Ay_min), std::fabs(t.Ay_max));
  double pxmax = std::fmax(std::fabs(g.px(0)), std::fabs(g.px(g.nx - 1)));
  double pymax = std::fmax(std::fabs(g.py(0)), std::fabs(g.py(g.ny - 1)));
  double phi = 2.0 * t.comp.cmax * t.dt * std::fmax(std::fmax(amax, aymax), std::fmax(pxmax, pymax));
  return phi <= kShearMaxAngle ? kFormShear : kFormVersine;
}

namespace {

// Times of a stage of a Strang solve for one wave, ns: alone on its SIMD (`single` + `single_point`
// per point of a lane; by rows `rows_single`), and its share of a SIMD's time among many
// (`wave` + `point` per point of a lane; by rows `rows_wave`), the kernel by rows with the points
// per lane it has by default, four in FP64 and one in FP32.  Measured over 860 drawn solves of
// 1000 to 3 million points, 16 to 40000 columns and 32 to 8000 rows, each by both kernels and with
// 1, 2, 4 and (some) 8 points per lane, in repeated passes of the step loop.  The faster of the two
// kernels by them was within 5% of the faster one on all but 9 of 1100 further solves.
struct StageTimes {
  double single, single_point, wave, point, rows_single, rows_wave;
};
constexpr StageTimes kStageTimes[3][2][2] = {
    // second order, fourth order; the second line with a y component
    {{{9.6, 10.6, 2.9, 11.8, 64.0, 66.5}, {10.0, 10.4, 3.6, 11.5, 84.0, 73.0}},  // PD_FP64
     {{12.0, 16.4, 6.5, 16.9, 86.5, 87.0}, {13.5, 15.6, 6.8, 16.8, 107.6, 95.0}}},
    {{{7.0, 13.9, 1.7, 8.55, 22.7, 12.4}, {11.0, 13.5, 2.6, 9.0, 40.0, 13.3}},  // PD_FP32
     {{8.3, 21.4, 3.6, 12.8, 32.9, 16.8}, {12.5, 20.5, 4.5, 13.7, 50.0, 17.8}}},
    {{{6.8, 10.7, 3.0, 6.55, 19.6, 9.4}, {10.5, 10.4, 2.9, 6.6, 34.7, 10.2}},  // PD_FP32_FAST
     {{8.2, 16.2, 5.6, 9.35, 25.8, 13.3}, {13.0, 15.4, 6.0, 9.4, 43.6, 14.0}}}};

// Waves that the fullest SIMD works through, of `units` dealt in blocks of four to 256 compute
// units (past eight, where blocks follow one another, their mean), and what the last of them
// take more than their share: FP32 instructions of two waves issue together, so that one without
// a partner takes its turn alone.
double simd_load(long long units, bool fp32) {
  const long long blocks = (units + 3) / 4;
  const double n = blocks <= 8 * 256 ? (double)((blocks + 255) / 256) : (double)units / 1024.0;
  return n + (fp32 ? std::min(0.2 * n, 0.8) : std::min(0.08 * n, 0.6));
}

// Units of a launch by columns with 2^cshift columns to a wave.
ColumnGeometry columns_at(const Grid& g, int precision, int stages, int elliptic, int ppl, int cshift) {
  const int pair = is_fp32(precision) ? 8 : 16, lanes = 64 >> cshift;
  const long long bands = (g.ny + ppl - 1) / ppl;
  const long long supers = (g.nx + (1 << kColumnSuperShift) - 1) >> kColumnSuperShift;
  const int spaces = (1 << cshift) + (elliptic ? 1 : 0);  // columns of coefficients in the LDS
  ColumnGeometry c{};
  c.cshift = cshift;
  c.segs = (int)((bands + lanes - 1) / lanes);
  c.units = (int)((supers * c.segs) << (kColumnSuperShift - cshift));
  c.chunk = std::min(kColumnEntries, kColumnPairBytes / pair / spaces) / stages / 4 * 4;
  return c;
}
constexpr int most_columns(int stages) { return stages == 5 ? 3 : 4; }  // largest cshift

// Time of a stage of a solve by columns alone on the device, ns.  A further column of a wave
// costs it the evaluation and the reads of another column's coefficients, evaluated 64 at a time
// (short chunks leave lanes without one: 2874 x 40 in FP64 with a y component took 137 ns a stage
// with 16 columns to a wave, 28 steps to a chunk, and 89 by rows).
double column_time(const Grid& g, int precision, int stages, int elliptic, int ppl, int cshift) {
  const StageTimes& t = kStageTimes[precision][elliptic ? 1 : 0][stages == 5 ? 1 : 0];
  const bool f32 = is_fp32(precision);
  const ColumnGeometry c = columns_at(g, precision, stages, elliptic, ppl, cshift);
  const int entries = c.chunk * stages;
  const double more = ((1 << cshift) - 1) * (double)((entries + 63) / 64 * 64) / entries;
  const double one = t.single + t.single_point * ppl + 1.8 * more;
  const double many = t.wave + t.point * ppl + (f32 ? 1.0 : 1.5) * more;
  return std::max(one, simd_load(c.units, f32) * many);
}

// The same by rows, with the default points per lane and blocks of 256.
double row_time(const Grid& g, int precision, int stages, int elliptic) {
  const StageTimes& t = kStageTimes[precision][elliptic ? 1 : 0][stages == 5 ? 1 : 0];
  const bool f32 = is_fp32(precision);
  const long long tile = f32 ? 256 : 1024;
  return std::max(t.rows_single, simd_load((g.points() + tile - 1) / tile * 4, f32) * t.rows_wave);
}

// Most points per lane by columns: in FP32, eight with a y component or in the fourth order take
// so many registers that one wave is left to a SIMD (3110 x 298 in the fourth order: 292 ns a
// stage, 190 with four).
int most_points(int precision, int stages, int elliptic) {
  return is_fp32(precision) && (elliptic || stages == 5) ? 4 : 8;
}

// The points per lane of the fastest launch by columns, and its time.  Within 2%, less than the
// times are good for, the most: the fewest waves that evaluate coefficients.
int column_points(const Grid& g, int precision, int stages, int elliptic, double* time) {
  double of[4], least = 0.0;
  int count = 0;
  for (int ppl = 1; ppl <= most_points(precision, stages, elliptic); ppl *= 2, ++count) {
    of[count] = column_time(g, precision, stages, elliptic, ppl, 0);
    for (int s = 1; s <= most_columns(stages); ++s)
      of[count] = std::min(of[count], column_time(g, precision, stages, elliptic, ppl, s));
    least = count ? std::min(least, of[count]) : of[count];
  }
  *time = least;
  while (of[--count] > 1.02 * least) {
  }
  return 1 << count;
}

}  // namespace

int column_series(const Grid& g, const FieldTables& t, int precision) {
  if (g.ny < kColumnMinRows || strang_form(g, t) != kFormShear) return 0;
  // half angles of a stage: c dt (px + A_x), and at most c dt |A_y| for the field part of a
  // y rotation
  const double aymax = std::fmax(std::fabs(t.Ay_min), std::fabs(t.Ay_max));
  const double h = t.comp.cmax * t.dt * std::fmax(t.E_max, aymax);
  if (!(h <= 0.25 * kPi)) return 0;
  // By columns a step has fewer instructions, but lanes stay idle where the rows do not fill a
  // wave's bands, and each wave evaluates its columns' coefficients: the step loop of some grids
  // is faster by rows (fast FP32 1184 x 108 x 8000 steps: 0.20 ms by rows, 0.30 by columns).  A
  // new field costs the row kernel more, though: a sine and a cosine a step and a column on the
  // host (15 ns a step, 27 with a y component, 40 and 14 a column), and its scalar unit waits
  // for rows that no pass has brought near yet (18 and 35 ns a step).  What counts is the call
  // with a new field (1403 x 38 x 14714 in FP32 with a y component: 2.47 ms by rows, 0.72 by
  // columns, of which 0.50 and 0.63 the step loop).
  double by_columns = 0.0;
  const int S = t.comp.stages, ell = t.elliptic ? 1 : 0;
  const double n = (double)t.n_steps * S;
  const double set_up = n * (ell ? 62.0 : 33.0) + (double)g.nx * (S == 5 ? 2 : 1) * (is_fp32(precision) ? 40.0 : 14.0);
  column_points(g, precision, S, ell, &by_columns);
  if (n * by_columns > 0.95 * n * row_time(g, precision, S, ell) + set_up) return 0;
  // the omitted terms, relative to the leading one: tan as in taylor_order; sin(2h)
  // alternates, so at most its first.  FP32: small against the dithering's 1/8 of a spacing.
  const double x = h * h, r = 4.0 * x / (kPi * kPi);
  const double tol = is_fp32(precision) ? 0x1p-30 : 0x1p-56;
  for (int J : {3, 5, 8, 12, 16, 20, 24}) {
    const double e = tan_series_coef(J + 1) * std::pow(x, J) / (1.0 - r);
    if (e <= tol && std::fabs(sin2_series_coef(J + 1)) * std::pow(x, J) <= tol) return J;
  }
  return kSeriesMax;
}

ColumnGeometry column_geometry(const Grid& g, int precision, int stages, int elliptic, int points_per_lane,
                               bool alone) {
  // Fewer columns to a wave: fewer coefficients to evaluate; more: fewer lanes without a
  // row where the bands do not fill 64 lanes.  A solve alone on the device: what is fastest;
  // one of a batch: least issue time, a column's coefficients and reads taking a wave about 1/4
  // (FP32) or 1/8 of a point's step.
  int best = 0;
  double best_cost = 0.0;
  for (int s = 0; s <= most_columns(stages); ++s) {
    double cost;
    if (alone) {
      cost = column_time(g, precision, stages, elliptic, points_per_lane, s);
    } else {
      const int segs = columns_at(g, precision, stages, elliptic, points_per_lane, s).segs;
      const double waves = (double)segs * (double)((g.nx + (1 << s) - 1) >> s);
      cost = waves * (points_per_lane + ((1 << s) + (elliptic ? 1 : 0)) * (is_fp32(precision) ? 1.0 / 4 : 1.0 / 8));
    }
    if (s == 0 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return columns_at(g, precision, stages, elliptic, points_per_lane, best);
}

int auto_points_per_lane(const Grid& g, int scheme, int precision, int stages, int elliptic) {
  double time = 0.0;
  if (base_scheme(scheme) != PD_SCHEME_MIDPOINT) return column_points(g, precision, stages, elliptic, &time);
  // Midpoint.  Time of a launch in issue slots of a point's step: the waves of the fullest of the
  // device's 1024 SIMDs, one after another, a wave without a partner (FP32 instructions of two
  // issue together) more than its turn, and what a lane's points have in common, the column's
  // phase (with its conversion, unpaired, 4 of 36 FP32 slots; FP64 as measured on large grids).
  // Measured, 1 / 2 / 4 points: FP64 64^2 x 4000 0.15 / 0.27 / 0.51 ms, 700 x 511 x 8000 1.71 /
  // 1.65 / 2.05, 22403 x 249 x 5377 - / 17.8 / 17.1; FP32 256^2 x 4000 0.21 / 0.31 / 0.55,
  // 1024^2 x 10000 3.24 / 3.08 / 3.00.
  const bool f32 = is_fp32(precision);
  int best = 1;
  for (int ppl = 1; ppl <= 4; ppl *= 2) {
    const long long waves = ((g.ny + ppl - 1) / ppl * (long long)g.nx + 63) / 64, n = (waves + 1023) / 1024;
    const double turns = n == 1 ? (f32 ? 1.8 : 1.12) : n + (f32 && n % 2 ? 0.4 : 0.0);
    const double cost = turns * (ppl + (f32 ? 0.11 : 0.14));
    if (ppl == 1 || cost < time) {
      best = ppl;
      time = cost;
    }
  }
  return best;
}

int taylor_order(double x_max, int precision, int form) {
  // Orders compiled into the midpoint kernels.
  static const int kCos64[] = {5, 8, 14};
  static const int kCos32[] = {3, 5, 9};
  static const int kTan64[] = {5, 7, 10};
  static const int kTan32[] = {2, 3, 5};
  const bool f32 = is_fp32(precision);
  const int* orders = form == kMidTangent ? (f32 ? kTan32 : kTan64) : (f32 ? kCos32 : kCos64);
  double tol = f32 ? 0x1p-27 : 0x1p-56;
  for (int q = 0; q < 3; ++q) {
    int J = orders[q];
    if (form == kMidTangent) {
      // a_n > 0 and a_{n+1} / a_n < 4 / pi^2, so the omitted terms sum to at most
      // a_{J+1} x^J / (1 - 4 x / pi^2), relative to tan(x)/x >= 1
      double r = 4.0 * x_max / (kPi * kPi);
      if (r < 1.0 && tan_series_coef(J + 1) * std::pow(x_max, J) / (1.0 - r) <= tol) return J;
      continue;
    }
    // relative size of the first omitted terms: 2 x^J / (2J+2)! for cos - 1 and
    // x^(J+1) / (2J+3)! for sin(x)/x
    double f = 1.0;
    for (int m = 2; m <= 2 * J + 2; ++m) f *= m;
    double e1 = 2.0 * std::pow(x_max, J) / f;
    double e2 = std::pow(x_max, J + 1) / (f * (2 * J + 3));
    if (e1 <= tol && e2 <= tol) return J;
  }
  return -1;
}

// The series' coefficients, to the terms that double precision holds for the angles of the
// tangent form.  A table: evaluated on each call they took 10 us of a field's set-up.
constexpr int kTanTerms = 28;
struct TanCoefficients {
  double a[kTanTerms];
  constexpr TanCoefficients() : a() {
    for (int n = 1; n < kTanTerms; ++n) a[n] = tan_series_coef(n);
  }
};
constexpr TanCoefficients kTan;

TanPolynomial tan_polynomial(double x_max, int precision) {
  static const int k64[] = {4, 5, 6, 8}, k32[] = {2, 3, 4, 5};
  const bool f32 = is_fp32(precision);
  const double tol = f32 ? 0x1p-30 : 0x1p-58;
  const int* orders = f32 ? k32 : k64;
  const int count = 4;
  // q(x) = sum_{k >= 0} b_k x^k
  constexpr int kTerms = kTanTerms - 2;
  const double* b = kTan.a + 2;
  TanPolynomial p{};
  const int taylor = taylor_order(x_max, precision, kMidTangent);
  for (int o = 0; o < count; ++o) {
    const int J = orders[o], m = J - 2;  // q by a polynomial of degree m
    p.terms = J;
    double r = 4.0 * x_max / (kPi * kPi);
    for (int n = 2; n <= J; ++n) p.c[n] = kTan.a[n];
    if (kTan.a[J + 1] * std::pow(x_max, J) / (1.0 - r) <= tol) return p;
    // Chebyshev nodes: |q - polynomial| <= max |q^(m+1)| / (m+1)! (x_max / 4)^(m+1) 2, and all
    // derivatives of q grow with x
    long double deriv = 0, binom = 1, power = 1;  // C(k, m+1) x_max^(k-m-1)
    for (int k = m + 1; k < kTerms; ++k) {
      deriv += binom * b[k] * power;
      binom = binom * (k + 1) / (k - m);
      power *= x_max;
    }
    const double bound = (double)(deriv * std::pow(0.25L * x_max, m + 1) * 2.0L * x_max);
    // of two FP32 terms always the series' own, which the kernel has as a literal: 2^-27 holds there
    if (J == taylor && (bound > tol || (f32 && J == 2))) return p;
    if (bound > tol && o + 1 < count) continue;
    // Newton's divided differences at the nodes, expanded
    long double node[kTanTermsMax], diff[kTanTermsMax], c[kTanTermsMax] = {};
    for (int i = 0; i <= m; ++i) {
      node[i] = 0.5L * x_max * (1.0L + std::cos((2 * i + 1) * 3.14159265358979323846L / (2 * m + 2)));
      diff[i] = 0;
      for (int k = kTerms - 1; k >= 0; --k) diff[i] = diff[i] * node[i] + b[k];
    }
    for (int w = 1; w <= m; ++w)
      for (int i = m; i >= w; --i) diff[i] = (diff[i] - diff[i - 1]) / (node[i] - node[i - w]);
    for (int i = m; i >= 0; --i) {
      for (int k = m; k >= 1; --k) c[k] = c[k - 1] - node[i] * c[k];
      c[0] = diff[i] - node[i] * c[0];
    }
    for (int k = 0; k <= m; ++k) p.c[k + 2] = (double)c[k];
    return p;
  }
  return p;
}

int midpoint_form(const FieldTables& t, int precision) {
  // every stage angle is at most theta = cmax dt E_max; a step of S stages grows
  // the state by at most (1 / cos theta)^S
  const double theta = t.comp.cmax * t.dt * t.E_max;
  if (!(theta < 0.5 * kPi)) return kMidCosine;
  const double growth_log2 = (double)kRenormEvery * t.comp.stages * -std::log2(std::cos(theta));
  if (growth_log2 > 32.0) return kMidCosine;
  return taylor_order(theta * theta, precision, kMidTangent) > 0 ? kMidTangent : kMidCosine;
}

}  // namespace pdx
