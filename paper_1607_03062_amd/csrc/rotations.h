// Plane rotations, point coordinates and the stage layout of the Strang kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "pd_internal.h"

namespace pdx {
namespace {

// Rotation of (u, v) by phi: u' = u cos - v sin, v' = u sin + v cos.
// Shear form, t = tan(phi/2), s = sin(phi): u -= t v; v += s u; u -= t v.
template <typename R>
__device__ __forceinline__ void rotate_shear(R& u, R& v, R t, R s) {
  u = fma(-t, v, u);
  v = fma(s, u, v);
  u = fma(-t, v, u);
}

// Versine form, h = cos - 1: u' = u + h u - s v,  v' = v + h v + s u.
__device__ __forceinline__ void rotate_versine(double& u, double& v, double h, double s) {
  double nu = fma(h, u, fma(-s, v, u));
  double nv = fma(h, v, fma(s, u, v));
  u = nu;
  v = nv;
}

// FP32 versine form: the small increment is formed first and added once, so the
// state sees a single rounding per component per rotation.
__device__ __forceinline__ void rotate_versine(float& u, float& v, float h, float s) {
  float du = fmaf(h, u, -(s * v));
  float dv = fmaf(h, v, s * u);
  u = u + du;
  v = v + dv;
}

template <int FORM, typename R>
__device__ __forceinline__ void rotate(R& u, R& v, R a, R s) {
  if (FORM == kFormShear)
    rotate_shear(u, v, a, s);
  else
    rotate_versine(u, v, a, s);
}


// Shear form with every component rounded once per rotation: the two u shears
// add up to u - t (v + v'), so u is updated from its value before the rotation
// (3 FMA + 1 add).  In FP32 the state's rounding errors are the whole error of a
// solve, and the second rounding of u per rotation dominates them (its increments
// are small, and the roundings of a slowly varying state accumulate); rounding each
// component once halves the worst-point error of the FP32 form on the benchmark
// workloads, for a quarter more instructions.
__device__ __forceinline__ void rotate_shear_once(float& u, float& v, float t, float s) {
  float u1 = fmaf(-t, v, u);
  float v1 = fmaf(s, u1, v);
  float w = v + v1;
  u = fmaf(-t, w, u);
  v = v1;
}

// The same shear rotation with the roles of u and v exchanged: v += t u; u -= s v;
// v += t u.  Now v is the component rounded twice.
template <typename R>
__device__ __forceinline__ void rotate_shear_vu(R& u, R& v, R t, R s) {
  v = fma(t, u, v);
  u = fma(-s, v, u);
  v = fma(t, u, v);
}

// Two rotations in one plane, by a and then by b, as five shears: the last shear of
// the first triple and the first of the second act on the same component, so they
// merge into one with the summed coefficient (one add).  Both orientations.
template <typename R>
__device__ __forceinline__ void rotate_two_shear(R& u, R& v, R ta, R sa, R tb, R sb) {
  u = fma(-ta, v, u);
  v = fma(sa, u, v);
  u = fma(-(ta + tb), v, u);
  v = fma(sb, u, v);
  u = fma(-tb, v, u);
}

template <typename R>
__device__ __forceinline__ void rotate_two_shear_vu(R& u, R& v, R ta, R sa, R tb, R sb) {
  v = fma(ta, u, v);
  u = fma(-sa, v, u);
  v = fma(ta + tb, u, v);
  u = fma(-sb, v, u);
  v = fma(tb, u, v);
}

// Shear variants (FP32 forms):
//   kShearPlain  u -= t v; v += s u; u -= t v (u rounded twice per rotation);
//   kShearOnce   each component rounded once (rotate_shear_once, 4 instructions);
//   kShearAlt    plain shears with the orientation alternating from one stage to the
//                next (u-v-u, then v-u-v; the parity of the absolute stage index), so
//                that the doubly rounded component alternates and the systematic part
//                of the roundings largely cancels between neighbouring stages; the
//                stage's two rotations in one plane (field and per-point parts) run as
//                five shears (rotate_two_shear), which rounds less for the same count:
//                3 instructions per rotation.
constexpr int kShearPlain = 0;
constexpr int kShearOnce = 1;
constexpr int kShearAlt = 2;

// A rotation in the solve's form and shear variant SH; odd: the stage's parity
// (kShearAlt only; a compile-time constant wherever the steps are unrolled).
template <int FORM, int SH, typename R>
__device__ __forceinline__ void rot(R& u, R& v, R a, R s, bool odd = false) {
  if constexpr (FORM == kFormShear && SH == kShearOnce && sizeof(R) == 4) {
    rotate_shear_once(u, v, a, s);
  } else if constexpr (FORM == kFormShear && SH == kShearAlt) {
    if (odd)
      rotate_shear_vu(u, v, a, s);
    else
      rotate_shear(u, v, a, s);
  } else {
    rotate<FORM>(u, v, a, s);
  }
}

struct PointCoords {
  int i, j;
  double px, py;
};

__device__ __forceinline__ PointCoords coords(const SolveParams& p, long long idx) {
  long long j = idx / p.nx;
  long long i = idx - j * p.nx;
  PointCoords c;
  c.i = (int)i;
  c.j = (int)j;
  c.px = p.px_min + (double)i * p.dx;
  c.py = p.py_min + (double)j * p.dy;
  return c;
}

// Rotation layout of one step of a composition with NS stages.  Stage j applies
// the x rotation by its field part (table) and by its per-point part (class
// xcls(j) of the column coefficients), then the y rotation that follows it: its
// per-point part (class ycls(j) of the row coefficients) and, with a y component
// of the field (POL), its field part (table).  The y rotations of neighbouring
// stages, and of the last stage of a step and the first of the next, are merged;
// the solve opens and closes with a half step (the last row class).
template <int NS>
struct Layout;
template <>
struct Layout<1> {
  static constexpr int NX = 1, NY = 2;  // y classes: full, half
  __device__ static constexpr int xcls(int) { return 0; }
  __device__ static constexpr int ycls(int) { return 0; }
};
template <>
struct Layout<5> {
  // c = (p, p, q, p, p): x classes {p, q}; y classes {(p + p)/2, (p + q)/2, half}
  static constexpr int NX = 2, NY = 3;
  __device__ static constexpr int xcls(int j) { return j == 2 ? 1 : 0; }
  __device__ static constexpr int ycls(int j) { return (j == 1 || j == 2) ? 1 : 0; }
};

// Coefficient phases of the per-point rotations (host: coefficient_phases): the
// FP32 forms cycle through kDitherFP32 values of each coefficient, step k using
// value k mod kDitherFP32.
template <typename R>
constexpr int phases_of() {
  return sizeof(R) == 4 ? kDitherFP32 : 1;
}

// Period of a solve's step pattern: the coefficient phases and, for alternating
// shears, the orientation parity.  Steps run in groups that start at multiples of
// it, so inside a group every step's pattern is a compile-time constant.
template <typename R, int SH>
constexpr int step_period() {
  return (SH == kShearAlt && phases_of<R>() % 2 != 0) ? 2 * phases_of<R>() : phases_of<R>();
}

}  // namespace
}  // namespace pdx
