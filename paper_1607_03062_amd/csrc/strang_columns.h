// Strang solves by columns.
//
// The two rotations about x of a step, by 2 dt A_k (field) and by 2 dt px (point), add up
// to one by 2 dt (px + A_k), whose coefficients (tan, sin) depend on the column and the
// step only.  A wave therefore owns points of few columns (one, for grids of some size):
// it evaluates the coefficients of its columns for a chunk of steps into its own part of
// the LDS, one (step, column) per lane, and then runs the chunk, every lane reading its
// column's entry (a broadcast).  A step is then two rotations of three shears, 6 FMAs a
// point, where the field and point parts apart take 9.  The table the kernel reads is the
// half angle vsign c_j dt A of each step and stage in FP64.
//
// What bounds it: the vector ALU, at the clock the power limit leaves (FP64: 0.96 of the
// issue slots are taken).  Evaluating an entry takes about 30 FP64 instructions for the 64
// lanes' PPL points (3-4% of an FP32 solve's time, 1-2% of an FP64 one's), reading it back a
// 16-byte LDS read per FP64 step, or per two FP32 steps, for 6 PPL FMAs (3-4%); hence up to 8
// points per lane.  The waves of a block do not wait for each other: an entry is written and
// read by the same wave.  Lanes take consecutive rows, so n(p) and a chunk's state are read
// and written with the grid's width between lanes; neighbouring columns are in flight
// together on one XCD, whose L2 joins their lines.
//
// Measured against the row kernel on one machine, whole calls with the steps around it:
// 2048^2 x 80000 steps fast FP32 51.6 -> 38.6 ms (this kernel alone 54.9 -> 41.9, before the
// points per lane followed the launch), 1500 x 2047 x 12000 FP32 8.34 -> 5.90 ms, 1024^2 x 40000
// FP64 13.4 -> 8.7 ms, fourth order 512^2 x 4000 FP64 4.40 -> 1.31 ms, with a y component 1024^2 x
// 4000 FP32 8.3 -> 5.6 ms.  Fast FP32 issues 1.56-1.63 VALU instructions of 2 per SIMD
// quad-cycle, PD_FP32 1.68-1.70.
//
// The FP32 forms' roundings.  PD_FP32 rounds each component once in every rotation (8
// instructions for a point's step; the row kernel's three rotations 12).  PD_FP32_FAST: plain
// shears, both rotations turned over together from stage to stage (6; 9).  Two rotations a
// step round less than three: over 225 solves (64 full grids of 256^2 to 2048^2 points and 5000
// to 80000 steps, the 2048^2 x 80000 solve, 160 drawn ones with fourth order and a y component
// among them) the rms error against FP64 is 0.80 of the row kernel's in PD_FP32 (worst solve
// 0.96) and 0.86 in PD_FP32_FAST (1.05), the worst point's 0.79 (1.28) and 0.84 (1.57), the
// worst of all points 1.45e-5 after 1.80e-5 and 3.14e-5 after 3.15e-5.  Plain shears about y
// alone in PD_FP32 (7 instructions) had a worst point of 2.75e-5, and 2.0 times the row
// kernel's in one solve.
#pragma once

#include <hip/hip_runtime.h>

#include "pd_internal.h"
#include "rotations.h"

namespace pdx {
namespace {

// Rotation coefficients tan(h) and sin(2 h), h the half angle.
template <typename R>
struct alignas(2 * sizeof(R)) Pair {
  R t, s;
};

// tan(h) and sin(2h) by their Taylor series in x = h^2, the leading term added last so
// that the rounding of the series is relative to its own size.  J terms of
// tan(h) / h = sum a_n x^(n-1); sin(2h) / (2h) needs no more.  J = 0: `series` terms, 8 and
// a multiple of 4; those past the eighth come from a table, four to a trip (the larger step
// angles; unrolled for every length they cost the step loop its registers).
struct SeriesTable {
  double c[kSeriesMax + 1][2];
  constexpr SeriesTable() : c() {
    for (int n = 1; n <= kSeriesMax; ++n) {
      c[n][0] = tan_series_coef(n);
      c[n][1] = sin2_series_coef(n);
    }
  }
};
__constant__ const SeriesTable kSeries = SeriesTable();

template <int J>
__device__ __forceinline__ void half_angle_coefficients(int series, double h, double& t, double& s) {
  constexpr int kLast = J ? J : 8;  // terms from here on are unrolled
  const double x = h * h;
  double a, b;
  if constexpr (J == 0) {
    a = kSeries.c[series][0];
    b = kSeries.c[series][1];
#pragma unroll 1
    for (int n = series - 4; n >= kLast; n -= 4) {
#pragma unroll
      for (int m = 3; m >= 0; --m) {
        a = fma(a, x, kSeries.c[n + m][0]);
        b = fma(b, x, kSeries.c[n + m][1]);
      }
    }
  } else {
    a = tan_series_coef(J);
    b = sin2_series_coef(J);
  }
#pragma unroll
  for (int n = kLast - 1; n >= 2; --n) {
    a = fma(a, x, tan_series_coef(n));
    b = fma(b, x, sin2_series_coef(n));
  }
  const double h2 = h + h;
  t = fma(h, x * a, h);
  s = fma(h2, x * b, h2);
}

// f(constant J) for the solve's number of terms.
template <int N>
struct Constant {
  static constexpr int value = N;
};
template <typename F>
__device__ __forceinline__ void with_series(int series, F f) {
  switch (series) {
    case 3: f(Constant<3>()); return;
    case 5: f(Constant<5>()); return;
    case 8: f(Constant<8>()); return;
    default: f(Constant<0>()); return;
  }
}

// A coefficient in the solve's precision.  FP32: ordered dithering over four steps, the
// value rounded after a shift of `shift` * 2^-23 of its own power of two (3/8, -1/8, 1/8,
// -3/8 of a spacing for steps 0 .. 3 modulo 4), so that the mean over four steps of a
// slowly varying coefficient is within 1/8 of a spacing of it, as with the per-point
// coefficients' phases (kDitherFP32).  Odd in the value: the K- valley's coefficients are
// the K+ ones negated.
__device__ __forceinline__ void round_coefficient(double v, double, double* out) { *out = v; }
__device__ __forceinline__ void round_coefficient(double v, double shift, float* out) {
  const double scale = __hiloint2double(__double2hiint(v) & (int)0xfff00000, 0);  // +-2^e
  *out = (float)fma(scale, shift, v);
}
__device__ __forceinline__ double dither_shift(int phase) {
  const double d = (phase & 1) ? ((phase & 2) ? -0.375 : -0.125) : ((phase & 2) ? 0.125 : 0.375);
  return d * 0x1p-23;
}

template <typename R, int J>
__device__ __forceinline__ Pair<R> column_entry(int series, double h, double shift) {
  double t, s;
  half_angle_coefficients<J>(series, h, t, s);
  Pair<R> e;
  round_coefficient(t, shift, &e.t);
  round_coefficient(s, shift, &e.s);
  return e;
}

// The signs a pair takes in the two orientations, (-t, s) or (t, -s), so that each shear
// is a multiply-add without a negation.
template <typename R>
__device__ __forceinline__ Pair<R> oriented(Pair<R> e, bool vu) {
  return vu ? Pair<R>{e.t, -e.s} : Pair<R>{-e.t, e.s};
}

// The rotation of an oriented pair (a, b): plain shears, or (ONCE, orientation u-v-u) each
// component rounded once as in rotate_shear_once.
template <bool ONCE, typename R>
__device__ __forceinline__ void rotate_oriented(R& u, R& v, R a, R b, bool vu) {
  if constexpr (ONCE) {
    const R u1 = fma(a, v, u);
    const R v1 = fma(b, u1, v);
    const R w = v + v1;
    u = fma(a, w, u);
    v = v1;
  } else if (vu) {
    v = fma(a, u, v);
    u = fma(b, v, u);
    v = fma(a, u, v);
  } else {
    u = fma(a, v, u);
    v = fma(b, u, v);
    u = fma(a, v, u);
  }
}

// Orientation (false: u-v-u, true: v-u-v) of the rotations about x and y at a stage of
// parity `odd`.
template <int SH>
__device__ __forceinline__ constexpr bool orientation_x(int odd) {
  return SH == kShearAlt && odd != 0;
}
template <int SH>
__device__ __forceinline__ constexpr bool orientation_y(int odd) {
  return SH == kShearAlt && odd != 0;
}

// The Bloch vectors of a lane's points, PPL consecutive rows of one column, and the
// per-row coefficients of their rotations about y.
template <typename R, int PPL, int NS, int POL, int SH>
struct ColumnLanes {
  using L = Layout<NS>;
  static constexpr int D = phases_of<R>();
  // the row coefficients are held oriented where a coefficient phase meets one orientation only
  static constexpr bool kOrientedY = NS == 1 && !POL;
  static constexpr int kPol = POL;
  R x[PPL], y[PPL], z[PPL];
  R aY[L::NY - 1][D][PPL], sY[L::NY - 1][D][PPL];

  // Stage J of a step; ex: its entry, ef (POL): the field part of the rotation about y;
  // PH = the step's absolute index modulo 4.  LAST: the rotation after the last stage is
  // the closing half step (ha, hs per point).
  template <bool LAST, int PH, int J>
  __device__ __forceinline__ void stage(const Pair<R>& ex, const Pair<R>& ef, const R* ha, const R* hs) {
    constexpr int h = PH % D, o = (PH + J) & 1, c = L::ycls(J);
    constexpr bool closing = LAST && J == NS - 1;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      rotate_oriented<SH == kShearOnce>(y[q], z[q], ex.t, ex.s, orientation_x<SH>(o));
      if constexpr (kOrientedY && !closing) {
        rotate_oriented<SH == kShearOnce>(z[q], x[q], aY[c][h][q], sY[c][h][q], orientation_y<SH>(o));
      } else {
        const R ya = closing ? ha[q] : aY[c][h][q], ys = closing ? hs[q] : sY[c][h][q];
        if constexpr (POL && SH == kShearAlt) {
          if (orientation_y<SH>(o))
            rotate_two_shear_vu(z[q], x[q], ya, ys, ef.t, ef.s);
          else
            rotate_two_shear(z[q], x[q], ya, ys, ef.t, ef.s);
        } else {
          rot<kFormShear, SH>(z[q], x[q], ya, ys, orientation_y<SH>(o));
          if constexpr (POL) rot<kFormShear, SH>(z[q], x[q], ef.t, ef.s);
        }
      }
    }
  }

  template <bool LAST, int PH, int J = 0>
  __device__ __forceinline__ void step(const Pair<R>* ex, const Pair<R>* ef, const R* ha, const R* hs) {
    if constexpr (J < NS) {
      stage<LAST, PH, J>(ex[J], ef[POL ? J : 0], ha, hs);
      step<LAST, PH, J + 1>(ex, ef, ha, hs);
    }
  }

  // A step whose index modulo 4 is known only at run time (uniform over the wave).
  template <bool LAST>
  __device__ __forceinline__ void step_at(const Pair<R>* ex, const Pair<R>* ef, int phase, const R* ha = nullptr,
                                          const R* hs = nullptr) {
    if constexpr (D == 1) {
      step<LAST, 0>(ex, ef, ha, hs);
    } else {
      switch (phase & 3) {
        case 0: step<LAST, 0>(ex, ef, ha, hs); break;
        case 1: step<LAST, 1>(ex, ef, ha, hs); break;
        case 2: step<LAST, 2>(ex, ef, ha, hs); break;
        default: step<LAST, 3>(ex, ef, ha, hs); break;
      }
    }
  }

  __device__ __forceinline__ void renormalise() {
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      double X = x[q], Y = y[q], Z = z[q];
      double nr = sqrt(X * X + Y * Y + Z * Z);
      if (nr > 0.0) {
        x[q] = (R)(X / nr);
        y[q] = (R)(Y / nr);
        z[q] = (R)(Z / nr);
      }
    }
  }
};

// How the entries of a run of steps come into registers: SUB stages at a time (16 bytes, or
// one entry), DEPTH such pieces ahead of their use in a ring.  A wave alone on its SIMD
// waits out the latency of the LDS unless it reads about 16 steps ahead; with several
// points per lane 8 steps are enough, and the reads, one piece between two steps' FMAs,
// cost the vector ALU least that way.  A group is a whole number of ring turns and of four
// steps.
template <typename R, int PPL, int NS>
struct Pieces {
  static constexpr int SUB = (sizeof(R) == 4 && NS == 1) ? 2 : 1;
  static constexpr int STEPS = NS == 1 ? (PPL == 1 ? 16 : 8) : 4;
  static constexpr int COUNT = STEPS * NS / SUB;  // pieces of a group
  static constexpr int DEPTH = NS == 1 ? (sizeof(R) == 8 && PPL == 8 ? 4 : COUNT) : 10;
};
template <typename R, int POL, int SUB>
struct Piece {
  Pair<R> x[SUB], f[POL ? SUB : 1];
  __device__ __forceinline__ void load(const Pair<R>* ex, const Pair<R>* ef) {
#pragma unroll
    for (int m = 0; m < SUB; ++m) x[m] = ex[m];
    if constexpr (POL) {
#pragma unroll
      for (int m = 0; m < SUB; ++m) f[m] = ef[m];
    }
  }
};

// Pieces V .. of a group that starts at a multiple of 4 steps; each piece's registers take
// the piece DEPTH further on (at the end of a chunk, what lies behind it, which is not used).
template <typename PP, typename Lanes, typename Ring, int NS, int V, typename R>
__device__ __forceinline__ void column_group(Lanes& L, const Pair<R>* ex, const Pair<R>* ef, Ring& ring) {
  if constexpr (V < PP::COUNT) {
    constexpr int m = V * PP::SUB, slot = V % PP::DEPTH;
    L.template stage<false, m / NS % 4, m % NS>(ring[slot].x[0], ring[slot].f[0], nullptr, nullptr);
    if constexpr (PP::SUB == 2)
      L.template stage<false, (m + 1) / NS % 4, (m + 1) % NS>(ring[slot].x[1], ring[slot].f[Lanes::kPol], nullptr,
                                                              nullptr);
    __builtin_amdgcn_sched_barrier(0);
    ring[slot].load(ex + (V + PP::DEPTH) * PP::SUB, ef + (V + PP::DEPTH) * PP::SUB);
    __builtin_amdgcn_sched_barrier(0);
    column_group<PP, Lanes, Ring, NS, V + 1>(L, ex, ef, ring);
  }
}

// The value, of which the compiler knows nothing: what is computed from it is computed there.
__device__ __forceinline__ int untraced(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// One wave's share of a Strang solve by columns: unit `unit` of the grid's column
// geometry, steps [p.k_begin, p.k_end).  lds: the wave's kColumnLdsWave bytes.
template <typename R, int PPL, int NS, int POL, int SH>
__device__ __forceinline__ void column_tile(const SolveParams& p, const int unit, unsigned char* lds) {
  using Lanes = ColumnLanes<R, PPL, NS, POL, SH>;
  using LY = Layout<NS>;
  constexpr int D = Lanes::D;
  constexpr int CY = 2 * ((LY::NY - 1) * D + 1);  // per row: the phased pairs, then the half step
  constexpr int HALF = 2 * (LY::NY - 1) * D;      // offset of the half-step pair in a row
  constexpr int W = NS * (1 + POL);               // table values per step
  const R* __restrict__ rowc = static_cast<const R*>(p.row_coef);
  const double* __restrict__ tab = static_cast<const double*>(p.table);

  // unit -> (16 columns, rows of a wave, columns of a wave): neighbouring units lie beside
  // each other, so that the 16 columns of a 128-byte line are in flight together
  const ColumnGeometry& g = p.columns;
  const int lane = threadIdx.x & 63;
  const int group_shift = kColumnSuperShift - g.cshift;
  const int super_units = g.segs << group_shift;
  const int super = unit / super_units, rest = unit - super * super_units;
  const int ncols = 1 << g.cshift;
  const int col0 = (super << kColumnSuperShift) + ((rest & ((1 << group_shift) - 1)) << g.cshift);
  if (unit >= g.units || col0 >= p.nx) return;  // uniform over the wave
  const int seg = rest >> group_shift;
  // Where a lane's points lie.  `at` is evaluated anew after the step loop from a lane index
  // the compiler cannot trace, here and for the entries: it would else keep addresses,
  // momenta and more of them in some 60 registers through the loop.
  struct Place {
    int ccol, col, band;
    bool col_valid;
    double px;
  };
  const auto at = [&](int ln) {
    Place w;
    w.ccol = ln & (ncols - 1);
    w.band = seg * (64 >> g.cshift) + (ln >> g.cshift);
    w.col_valid = col0 + w.ccol < p.nx;
    w.col = w.col_valid ? col0 + w.ccol : p.nx - 1;
    w.px = p.px_min + (double)w.col * p.dx;
    return w;
  };
  // row of point q; rows past the last one recompute it and store nothing
  const auto row_of = [&](const Place& w, int q) {
    const long long j = (long long)w.band * PPL + q;
    return j < p.ny ? (int)j : p.ny - 1;
  };
  const auto stored = [&](const Place& w, int q) { return w.col_valid && (long long)w.band * PPL + q < p.ny; };
  Lanes L;

  const Place w0 = at(lane);
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    const int j = row_of(w0, q);
    const long long idx = (long long)j * p.nx + w0.col;
#pragma unroll
    for (int m = 0; m < LY::NY - 1; ++m)
#pragma unroll
      for (int h = 0; h < D; ++h) {
        L.aY[m][h][q] = rowc[(size_t)CY * j + 2 * (m * D + h)];
        L.sY[m][h][q] = rowc[(size_t)CY * j + 2 * (m * D + h) + 1];
        if constexpr (Lanes::kOrientedY) {
          const Pair<R> e = oriented(Pair<R>{L.aY[m][h][q], L.sY[m][h][q]}, orientation_y<SH>(h & 1));
          L.aY[m][h][q] = e.t;
          L.sY[m][h][q] = e.s;
        }
      }
    if (p.load_state) {
      const R* st = static_cast<const R*>(p.state);
      L.x[q] = st[idx];
      L.y[q] = st[p.npts + idx];
      L.z[q] = st[2 * p.npts + idx];
    } else {
      // v_in: negative-energy eigenvector of the valley Hamiltonian vsign sigma.P_in,
      // Bloch vector -vsign P_in/|P_in|
      const double py = p.py_min + (double)j * p.dy;
      double Px = w0.px + p.A_in, Py = py + p.Ay_in;
      double E = sqrt(Px * Px + Py * Py);
      double rx = 0.0, ry = 0.0;
      if (E > 0.0) {
        rx = -p.vsign * Px / E;
        ry = -p.vsign * Py / E;
      }
      L.x[q] = (R)rx;
      L.y[q] = (R)ry;
      L.z[q] = (R)0;
      // opening half step about y: per-point part, then (POL) the field part
      rot<kFormShear, SH>(L.z[q], L.x[q], rowc[(size_t)CY * j + HALF], rowc[(size_t)CY * j + HALF + 1]);
      if (POL) {
        with_series(p.series, [&](auto terms) {
          double t, s;
          half_angle_coefficients<decltype(terms)::value>(p.series, tab[(size_t)p.n_steps * W + NS], t, s);
          rot<kFormShear, SH>(L.z[q], L.x[q], (R)t, (R)s);
        });
      }
    }
  }

  constexpr int kPad = 16 / (int)sizeof(Pair<R>);  // columns 16 bytes apart in the banks
  Pair<R>* ent = reinterpret_cast<Pair<R>*>(lds);
  const int stride = g.chunk * NS + kPad;
  const Pair<R>* ex = ent + w0.ccol * stride;
  const Pair<R>* ef = ent + (POL ? ncols * stride : 0);
  const long long k_full = p.k_end < p.n_steps ? p.k_end : p.n_steps - 1;
  long long k = p.k_begin;
  // The loads so far are waited for here, once, so that the step loop's wait counts are not
  // made to cover them.
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  while (k < k_full) {
    // steps [k, kend) of the chunk that starts at k0, a multiple of 4
    const long long k0 = k & ~3LL;
    long long kend = k0 + g.chunk;
    if (sizeof(R) == 4) {
      const long long next = (k / kRenormEvery + 1) * kRenormEvery;
      if (next < kend) kend = next;
    }
    if (kend > k_full) kend = k_full;
    const int cnt = (int)(kend - k0);
    // The chunk's entries, up to kSide to a lane side by side.  Lanes without one write to the
    // last slot of the wave's LDS (no branch).  The angles are loaded here and not before the
    // previous chunk's steps: their latency, once in some hundred steps, is less than the
    // registers they would hold through the loop.
    constexpr int kSide = PPL <= 2 ? 4 : 2;  // more points per lane: fewer registers to spare
    const int total = cnt * NS;
    const auto evaluate = [&](auto terms, auto entries, int e0) {
      constexpr int J = decltype(terms)::value, N = decltype(entries)::value;
      constexpr int kDump = kColumnLdsWave / (int)sizeof(Pair<R>) - 1;
      const int ln = untraced(lane);
      double dx[N], dy[N], shift[N], hx[N];
      bool vu[N];
#pragma unroll
      for (int r = 0; r < N; ++r) {
        int e = e0 + ln + 64 * r;
        if (e >= total) e = total - 1;
        const int ke = e / NS, j = e - ke * NS;
        const double* row = tab + (k0 + ke) * W + j;
        dx[r] = row[0];
        if constexpr (POL) dy[r] = row[NS];
        shift[r] = dither_shift(ke + j);
        hx[r] = NS == 5 && j == 2 ? p.hx[1] : p.hx[0];
        vu[r] = orientation_x<SH>((ke + j) & 1);
      }
#pragma unroll 1
      for (int c = 0; c < ncols + POL; ++c) {
        const bool field_y = POL && c == ncols;
        const double pc = p.px_min + (double)(col0 + c < p.nx ? col0 + c : p.nx - 1) * p.dx;
        Pair<R> v[N];
#pragma unroll
        for (int r = 0; r < N; ++r) v[r] = column_entry<R, J>(p.series, field_y ? dy[r] : hx[r] * pc + dx[r], shift[r]);
#pragma unroll
        for (int r = 0; r < N; ++r) {
          const int e = e0 + ln + 64 * r;
          ent[e < total ? c * stride + e : kDump] = field_y ? v[r] : oriented(v[r], vu[r]);
        }
      }
    };
    with_series(p.series, [&](auto terms) {
      int e0 = 0;
#pragma unroll 1
      for (; total - e0 > 64 * (kSide - 1); e0 += 64 * kSide) evaluate(terms, Constant<kSide>(), e0);
#pragma unroll 1
      for (; total - e0 > 0; e0 += 64) evaluate(terms, Constant<1>(), e0);
    });
    // the wave's own writes, read by its other lanes: the LDS serves a wave in order, the
    // compiler has to keep that order too
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // nothing but the prefetched entries is in flight below, so that the compiler counts
    // them instead of waiting for all
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    int i = (int)(k - k0);
    for (; (i & 3) != 0 && i < cnt; ++i) L.template step_at<false>(ex + i * NS, ef + i * NS, i);
    using PP = Pieces<R, PPL, NS>;
    if (i + PP::STEPS <= cnt) {
      Piece<R, POL, PP::SUB> ring[PP::DEPTH];
#pragma unroll
      for (int v = 0; v < PP::DEPTH; ++v) {
        ring[v].load(ex + i * NS + v * PP::SUB, ef + i * NS + v * PP::SUB);
        __builtin_amdgcn_sched_barrier(0);  // in the loop's order, so that its wait counts hold here too
      }
      for (; i + PP::STEPS <= cnt; i += PP::STEPS)
        column_group<PP, Lanes, decltype(ring), NS, 0>(L, ex + i * NS, ef + i * NS, ring);
    }
    for (; i < cnt; ++i) L.template step_at<false>(ex + i * NS, ef + i * NS, i);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    k = kend;
    if (sizeof(R) == 4 && (k % kRenormEvery) == 0) L.renormalise();
  }

  const Place w = at(untraced(lane));
  if (p.k_end == p.n_steps) {
    // last step: its y rotation after the last stage is the closing half step
    const long long kl = p.n_steps - 1;
    R ha[PPL], hs[PPL];
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      const int j = row_of(w, q);
      ha[q] = rowc[(size_t)CY * j + HALF];
      hs[q] = rowc[(size_t)CY * j + HALF + 1];
    }
    Pair<R> lx[NS], lf[NS];
    with_series(p.series, [&](auto terms) {
      constexpr int J = decltype(terms)::value;
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        const double shift = dither_shift((int)(kl & 3) + j);
        const double hx = NS == 5 && j == 2 ? p.hx[1] : p.hx[0];
        lx[j] = oriented(column_entry<R, J>(p.series, hx * w.px + tab[kl * W + j], shift), orientation_x<SH>((int)(kl + j) & 1));
        if (POL) lf[j] = column_entry<R, J>(p.series, tab[kl * W + NS + j], shift);
      }
    });
    L.template step_at<true>(lx, lf, (int)(kl & 3), ha, hs);
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      const int j = row_of(w, q);
      const double py = p.py_min + (double)j * p.dy;
      // projection on u_out: n = (1 + vsign r.P_out / |P_out|) / 2 with r normalised
      double Pxi = w.px + p.A_in, Pyi = py + p.Ay_in;
      double Pxo = w.px + p.A_out, Pyo = py + p.Ay_out;
      double Ei = sqrt(Pxi * Pxi + Pyi * Pyi), Eo = sqrt(Pxo * Pxo + Pyo * Pyo);
      double X = L.x[q], Y = L.y[q], Z = L.z[q];
      double nr = sqrt(X * X + Y * Y + Z * Z);
      double n = 0.0;
      if (Ei > 0.0 && Eo > 0.0 && nr > 0.0) {
        double dot = (Pxo * X + Pyo * Y) / nr;
        n = (Eo + p.vsign * dot) / (2.0 * Eo);
      }
      if (stored(w, q)) p.n_out[(long long)j * p.nx + w.col] = n;
    }
  } else if (p.store_state) {
    R* st = static_cast<R*>(p.state);
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      if (stored(w, q)) {
        const long long idx = (long long)row_of(w, q) * p.nx + w.col;
        st[idx] = L.x[q];
        st[p.npts + idx] = L.y[q];
        st[2 * p.npts + idx] = L.z[q];
      }
    }
  }
}

// The wave's unit of a launch of whole blocks: blocks go round the XCDs in turn, so block
// b takes tile (b mod 8) * (blocks / 8) + b / 8 and each XCD's L2 sees neighbouring tiles.
template <typename R, int PPL, int NS, int POL, int SH>
__global__ void __launch_bounds__(256) column_kernel(const SolveParams p) {
  extern __shared__ __align__(16) unsigned char pd_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned tile = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int unit = (int)p.first + (int)(tile * (blockDim.x >> 6)) + wave;
  column_tile<R, PPL, NS, POL, SH>(p, unit, pd_lds + wave * kColumnLdsWave);
}

// Launch over all units in slices of at most kMaxLanes lanes (p.first: the slice's first
// unit), each a multiple of 8 blocks.
template <typename R, int PPL, int NS, int POL, int SH>
hipError_t launch_columns(int block, const SolveParams& p, hipStream_t stream) {
  const long long waves = block / 64;
  const long long blocks = (p.columns.units + waves - 1) / waves;
  const long long max_blocks = kMaxLanes / block;
  SolveParams q = p;
  for (long long b0 = 0; b0 < blocks; b0 += max_blocks) {
    q.first = b0 * waves;
    const long long nb = blocks - b0 < max_blocks ? blocks - b0 : max_blocks;
    hipLaunchKernelGGL((column_kernel<R, PPL, NS, POL, SH>), dim3((unsigned)((nb + 7) / 8 * 8)), dim3(block),
                       (size_t)(waves * kColumnLdsWave), stream, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename R, int NS, int POL, int SH>
hipError_t columns_ppl(int ppl, int block, const SolveParams& p, hipStream_t stream) {
  switch (ppl) {
    case 1: return launch_columns<R, 1, NS, POL, SH>(block, p, stream);
    case 2: return launch_columns<R, 2, NS, POL, SH>(block, p, stream);
    case 4: return launch_columns<R, 4, NS, POL, SH>(block, p, stream);
    default: return launch_columns<R, 8, NS, POL, SH>(block, p, stream);
  }
}

template <typename R, int SH>
hipError_t columns_variant(int stages, int elliptic, int ppl, int block, const SolveParams& p, hipStream_t stream) {
  if (stages == 5)
    return elliptic ? columns_ppl<R, 5, 1, SH>(ppl, block, p, stream) : columns_ppl<R, 5, 0, SH>(ppl, block, p, stream);
  return elliptic ? columns_ppl<R, 1, 1, SH>(ppl, block, p, stream) : columns_ppl<R, 1, 0, SH>(ppl, block, p, stream);
}

}  // namespace
}  // namespace pdx
