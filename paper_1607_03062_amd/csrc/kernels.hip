// gfx950 kernels of libpd: split-operator propagation of one state per momentum
// point, projection on the final positive-energy state, and the density sum.
//
// One lane per momentum point (points_per_lane of them, strided by the block
// size so loads and stores stay coalesced).  The per-step field row is the same
// for every lane: it is either staged through LDS in time chunks (every lane then
// reads it into VGPRs) or read by the scalar unit into SGPRs.
//
// Most Strang solves run by columns (strang_columns.h); the Strang kernel of this file takes
// grids of fewer than 32 rows and the steps too large for that.
//
// Strang scheme (Sec. III, Eqs. (11)-(12), with the midpoint Hamiltonian
// sigma_x P_x + sigma_y p_y split into its two parts):
//   U_k = exp(-i dt py sy / 2) exp(-i dt (px + A_k) sx) exp(-i dt py sy / 2).
// The kernel propagates the Bloch vector r of the pure state, psi psi^dagger =
// (1 + r.sigma) / 2, which carries everything n(p) depends on (the global
// phase of psi is unobservable): exp(-i a sx) rotates r by 2a about x and
// exp(-i b sy) by 2b about y.  Since exp(-i dt (px + A_k) sx) =
// exp(-i dt px sx) exp(-i dt A_k sx), every step is three plane rotations:
// by 2 dt A_k about x (table row, the same for all lanes), by 2 dt px about x
// and by 2 dt py about y (per-point constants computed once); the half steps of
// neighbouring steps are merged.
//
// A plane rotation by phi is applied either as three shears (Paeth's
// decomposition; one FMA each, coefficients tan(phi/2) and sin(phi)), or, when
// some angle of the solve is too large for the shears to stay well conditioned,
// in versine form with h = cos(phi) - 1 and s = sin(phi).  The fast FP32 form runs
// two successive rotations in one plane (a stage's field and per-point parts) as
// five shears, the two adjacent shears of the same component merged.
// The projection on u_out is n = |u_out^dagger psi|^2 = (1 + r.r_u) / 2 with
// r_u = P_out / |P_out| the Bloch vector of u_out (Sec. II, Eqs. (1), (3)); r
// is normalised first (the exact steps are unitary, Sec. III).
//
// Midpoint scheme (Sec. III, Eq. (13)): per step the closed 2x2 form
//   U = cos(dt E) I - i sigma.P sin(dt E) / E,  P = p + A_k,
// acting on the spinor (a1 + i b1, a2 + i b2).  For the small step angles of
// most solves the kernel applies U / cos(dt E) = I - i tan(dt E) sigma.P / E, one
// even series (tan(x)/x) instead of two and one rounding per component; the
// state's norm then grows by 1 / cos(dt E) per step and is renormalised every
// kRenormEvery steps (n divides it out).  Otherwise cos - 1 and sin(x)/x are
// evaluated.  The series are Taylor series in x = (dt E)^2 of an order chosen
// by the host.
//
// Both kernels are templated on the composition (NS = 1 second-order step, or
// NS = 5 stages of Suzuki's fourth-order composition, each a second-order step
// over c_j dt with the field at its own sub-interval midpoint) and on a y
// component of the field (POL: sigma_y (p_y + A_y) in place of sigma_y p_y; the
// Strang kernel then adds the field part of each y rotation from the table).
// The K- valley (H = -sigma.P) arrives as negated table and coefficient angles
// plus the sign vsign of the initial state and of the projection.
#include <hip/hip_runtime.h>

#include <mutex>

#include "pd_internal.h"
#include "rotations.h"
#include "strang_columns.h"

namespace pdx {
namespace {

// The Bloch vectors of a lane's points and their per-point rotations.
template <typename R, int PPL, int FORM, int NS, int POL, int SH>
struct BlochLanes {
  using L = Layout<NS>;
  static constexpr int kRow = 2 * NS * (1 + POL);  // table values per step
  static constexpr int D = phases_of<R>();
  static constexpr int P = step_period<R, SH>();
  R x[PPL], y[PPL], z[PPL];
  R aX[L::NX][D][PPL], sX[L::NX][D][PPL];          // x rotations by 2 c dt px, per phase
  R aY[L::NY - 1][D][PPL], sY[L::NY - 1][D][PPL];  // y rotations after the stages, by (c_j + c_j+1) dt py

  // One step; row = the step's table values; PH = the step's absolute index modulo
  // P (phase PH % D of the coefficients; with alternating shears stage j of step k
  // has parity k + j, NS odd).  LAST: the y rotation after the last stage is the
  // closing half step (ha, hs per point).
  template <bool LAST, int PH>
  __device__ __forceinline__ void step(const R* row, const R* ha, const R* hs) {
    constexpr int h = PH % D;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const bool o = ((PH & 1) != 0) != ((j & 1) != 0);
#pragma unroll
      for (int q = 0; q < PPL; ++q) {
        const R ya = (LAST && j == NS - 1) ? ha[q] : aY[L::ycls(j)][h][q];
        const R ys = (LAST && j == NS - 1) ? hs[q] : sY[L::ycls(j)][h][q];
        if constexpr (FORM == kFormShear && SH == kShearAlt) {
          // the x rotations by the field part and the point's part, then the y rotation
          // by the point's part and (POL) the field part, each pair as five shears
          if (o)
            rotate_two_shear_vu(y[q], z[q], row[2 * j], row[2 * j + 1], aX[L::xcls(j)][h][q], sX[L::xcls(j)][h][q]);
          else
            rotate_two_shear(y[q], z[q], row[2 * j], row[2 * j + 1], aX[L::xcls(j)][h][q], sX[L::xcls(j)][h][q]);
          if constexpr (POL) {
            if (o)
              rotate_two_shear_vu(z[q], x[q], ya, ys, row[2 * NS + 2 * j], row[2 * NS + 2 * j + 1]);
            else
              rotate_two_shear(z[q], x[q], ya, ys, row[2 * NS + 2 * j], row[2 * NS + 2 * j + 1]);
          } else {
            rot<FORM, SH>(z[q], x[q], ya, ys, o);
          }
        } else {
          rot<FORM, SH>(y[q], z[q], row[2 * j], row[2 * j + 1], o);
          rot<FORM, SH>(y[q], z[q], aX[L::xcls(j)][h][q], sX[L::xcls(j)][h][q], o);
          rot<FORM, SH>(z[q], x[q], ya, ys, o);
          if (POL) rot<FORM, SH>(z[q], x[q], row[2 * NS + 2 * j], row[2 * NS + 2 * j + 1], o);
        }
      }
    }
  }

  // A step whose pattern index k mod P is known only at run time (uniform over the wave).
  template <bool LAST>
  __device__ __forceinline__ void step_at(const R* row, long long k, const R* ha = nullptr, const R* hs = nullptr) {
    switch ((int)(k % P)) {
      case 0: step<LAST, 0>(row, ha, hs); break;
      case 1: if constexpr (P > 1) step<LAST, 1 % P>(row, ha, hs); break;
      case 2: if constexpr (P > 2) step<LAST, 2 % P>(row, ha, hs); break;
      case 3: if constexpr (P > 3) step<LAST, 3 % P>(row, ha, hs); break;
      case 4: if constexpr (P > 4) step<LAST, 4 % P>(row, ha, hs); break;
      case 5: if constexpr (P > 5) step<LAST, 5 % P>(row, ha, hs); break;
      case 6: if constexpr (P > 6) step<LAST, 6 % P>(row, ha, hs); break;
      default: if constexpr (P > 7) step<LAST, 7 % P>(row, ha, hs); break;
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

template <typename R, int W>
struct RowN {
  R v[W];
};

// Steps U of a group that starts at a multiple of the step period, with the
// pattern index of each known at compile time.
template <typename Lanes, typename Row, int U, int G>
__device__ __forceinline__ void group_steps(Lanes& L, const Row* r) {
  if constexpr (U < G) {
    L.template step<false, U % Lanes::P>(r[U].v, nullptr, nullptr);
    group_steps<Lanes, Row, U + 1, G>(L, r);
  }
}

// Steps U of a group whose rows are long (fourth order, y component), each row loaded
// one step ahead: row U + 1 (or the next group's first, `after`) is requested before step
// U's arithmetic, so two rows are live instead of two groups of them.
template <typename Lanes, typename Row, int U, int G>
__device__ __forceinline__ void group_steps_ahead(Lanes& L, const Row* __restrict__ g, const Row* __restrict__ after,
                                                  Row& cur) {
  if constexpr (U < G) {
    const Row nxt = (U + 1 < G) ? g[U + 1] : after[0];
    __builtin_amdgcn_sched_barrier(0);
    L.template step<false, U % Lanes::P>(cur.v, nullptr, nullptr);
    __builtin_amdgcn_sched_barrier(0);
    cur = nxt;
    group_steps_ahead<Lanes, Row, U + 1, G>(L, g, after, cur);
  }
}

// Steps [k, k_full) with the table rows read by the scalar unit (SGPR operands).
template <typename R, int PPL, int FORM, int NS, int POL, int SH>
__device__ __forceinline__ void steps_scalar(BlochLanes<R, PPL, FORM, NS, POL, SH>& L, const R* __restrict__ table,
                                             long long k, long long k_full) {
  using Lanes = BlochLanes<R, PPL, FORM, NS, POL, SH>;
  using Row = RowN<R, Lanes::kRow>;
  constexpr int P = Lanes::P;
  const Row* __restrict__ tab = reinterpret_cast<const Row*>(table);
  constexpr int kRows = Lanes::kRow >= 8 ? 1 : 8 / (Lanes::kRow / 2);  // rows fetched together
  constexpr int kGroup = (kRows + P - 1) / P * P;                     // whole periods
  // two sets of a group's rows fit the scalar registers for short rows, or groups of one
  // row; the long rows of the FP32 forms (groups of a whole coefficient period) go one
  // row ahead instead
  constexpr bool kTwoSets = kGroup == 1 || kGroup * Lanes::kRow * (int)sizeof(R) <= 32 * 4;
  while (k < k_full) {
    long long seg = k_full;
    if (sizeof(R) == 4) {
      long long next = (k / kRenormEvery + 1) * kRenormEvery;
      seg = next < k_full ? next : k_full;
    }
    // up to the first multiple of the period (renormalisation steps are multiples of it)
    for (; (k % P) != 0 && k < seg; ++k) {
      const Row r = tab[k];
      L.template step_at<false>(r.v, k);
    }
    // whole groups: a 32-bit trip count, so the loop test stays on the scalar unit, and
    // two row sets in turn.  Each set is loaded right after the other set's first step
    // (scalar loads complete out of order, so the wait before a set's first use covers
    // every load in flight) and its latency is hidden behind that set's other steps; the
    // scheduling barriers keep the loads there.  The clamped index re-reads the last
    // group instead of branching.
    if constexpr (!kTwoSets) {
      // long rows: one row ahead.  Rows k .. k + n kGroup are read; the last of them is
      // at most seg <= the last step's row, so every read is inside the table.
      while (k + kGroup <= seg) {
        const long long left = (seg - k) / kGroup;
        const int n = left < (1 << 30) ? (int)left : (1 << 30);
        const Row* __restrict__ g = tab + k;
        Row cur = g[0];
        for (int i = 0; i < n; ++i) {
          const Row* __restrict__ gi = g + (long long)i * kGroup;
          group_steps_ahead<Lanes, Row, 0, kGroup>(L, gi, gi + kGroup, cur);
        }
        k += (long long)n * kGroup;
      }
    }
    while (kTwoSets && k + kGroup <= seg) {
      const long long left = (seg - k) / kGroup;
      const int n = left < (1 << 30) ? (int)left : (1 << 30);
      const Row* __restrict__ g = tab + k;
      Row a[kGroup], b[kGroup];
#pragma unroll
      for (int u = 0; u < kGroup; ++u) a[u] = g[u];
      int i = 0;
      for (; i + 1 < n; i += 2) {
        group_steps<Lanes, Row, 0, 1>(L, a);
        __builtin_amdgcn_sched_barrier(0);
        const Row* __restrict__ gb = g + (long long)(i + 1) * kGroup;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) b[u] = gb[u];
        __builtin_amdgcn_sched_barrier(0);
        group_steps<Lanes, Row, 1, kGroup>(L, a);
        group_steps<Lanes, Row, 0, 1>(L, b);
        __builtin_amdgcn_sched_barrier(0);
        const Row* __restrict__ ga = g + (long long)(i + 2 < n ? i + 2 : n - 1) * kGroup;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) a[u] = ga[u];
        __builtin_amdgcn_sched_barrier(0);
        group_steps<Lanes, Row, 1, kGroup>(L, b);
      }
      if (i < n) group_steps<Lanes, Row, 0, kGroup>(L, a);
      k += (long long)n * kGroup;
    }
    for (; k < seg; ++k) {
      const Row r = tab[k];
      L.template step_at<false>(r.v, k);
    }
    if (sizeof(R) == 4 && (k % kRenormEvery) == 0) L.renormalise();
  }
}

// Steps [k, k_full) with the table staged through LDS in chunks of `chunk` rows
// (absolute chunk boundaries; a power of two dividing the renormalisation period
// in the FP32 form, and a multiple of the step period), so every lane reads its
// rotation from VGPRs.
template <typename R, int PPL, int FORM, int NS, int POL, int SH>
__device__ __forceinline__ void steps_lds(BlochLanes<R, PPL, FORM, NS, POL, SH>& L, const R* __restrict__ table,
                                          long long k, long long k_full, long long chunk) {
  using Lanes = BlochLanes<R, PPL, FORM, NS, POL, SH>;
  using Row = RowN<R, Lanes::kRow>;
  constexpr int P = Lanes::P;
  const Row* __restrict__ tab = reinterpret_cast<const Row*>(table);
  extern __shared__ __align__(16) unsigned char pd_lds[];
  Row* rows = reinterpret_cast<Row*>(pd_lds);
  while (k < k_full) {
    long long cend = (k / chunk + 1) * chunk;
    if (cend > k_full) cend = k_full;
    const int cnt = (int)(cend - k);
    __syncthreads();  // every wave has finished with the previous chunk
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) rows[t] = tab[k + t];
    __syncthreads();
    int t = 0;
    for (; ((k + t) % P) != 0 && t < cnt; ++t) {
      const Row r = rows[t];
      L.template step_at<false>(r.v, k + t);
    }
    if constexpr (P == 1) {
#pragma unroll 8
      for (; t < cnt; ++t) {
        const Row r = rows[t];
        L.template step<false, 0>(r.v, nullptr, nullptr);
      }
    } else {
#pragma unroll 2
      for (; t + P <= cnt; t += P) {
        Row r[P];
#pragma unroll
        for (int u = 0; u < P; ++u) r[u] = rows[t + u];
        group_steps<Lanes, Row, 0, P>(L, r);
      }
      for (; t < cnt; ++t) {
        const Row r = rows[t];
        L.template step_at<false>(r.v, k + t);
      }
    }
    k = cend;
    if (sizeof(R) == 4 && (k % kRenormEvery) == 0) L.renormalise();
  }
}

// One tile of a Strang solve: the block's lanes own points base + q * blockDim.x,
// q < PPL; steps [p.k_begin, p.k_end).
template <typename R, int PPL, int STAGE, int FORM, int NS, int POL, int SH>
__device__ __forceinline__ void strang_tile(const SolveParams& p, const long long base) {
  using Lanes = BlochLanes<R, PPL, FORM, NS, POL, SH>;
  using LY = Layout<NS>;
  constexpr int D = Lanes::D;
  constexpr int CX = 2 * LY::NX * D;                // coefficient values per column
  constexpr int CY = 2 * ((LY::NY - 1) * D + 1);    // per row: the phased pairs, then the half step
  constexpr int HALF = 2 * (LY::NY - 1) * D;        // offset of the half-step pair in a row
  const R* __restrict__ colc = static_cast<const R*>(p.col_coef);
  const R* __restrict__ rowc = static_cast<const R*>(p.row_coef);
  const R* __restrict__ table = static_cast<const R*>(p.table);
  Lanes L;

#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    long long idx = base + (long long)q * blockDim.x;
    if (idx >= p.npts) idx = p.npts - 1;  // tail lanes recompute a valid point and store nothing
    PointCoords c = coords(p, idx);
#pragma unroll
    for (int m = 0; m < LY::NX; ++m)
#pragma unroll
      for (int h = 0; h < D; ++h) {
        L.aX[m][h][q] = colc[CX * c.i + 2 * (m * D + h)];
        L.sX[m][h][q] = colc[CX * c.i + 2 * (m * D + h) + 1];
      }
#pragma unroll
    for (int m = 0; m < LY::NY - 1; ++m)
#pragma unroll
      for (int h = 0; h < D; ++h) {
        L.aY[m][h][q] = rowc[CY * c.j + 2 * (m * D + h)];
        L.sY[m][h][q] = rowc[CY * c.j + 2 * (m * D + h) + 1];
      }
    if (p.load_state) {
      const R* st = static_cast<const R*>(p.state);
      L.x[q] = st[idx];
      L.y[q] = st[p.npts + idx];
      L.z[q] = st[2 * p.npts + idx];
    } else {
      // v_in: negative-energy eigenvector of the valley Hamiltonian vsign sigma.P_in,
      // Bloch vector -vsign P_in/|P_in|
      double Px = c.px + p.A_in, Py = c.py + p.Ay_in;
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
      rot<FORM, SH>(L.z[q], L.x[q], rowc[CY * c.j + HALF], rowc[CY * c.j + HALF + 1]);
      if (POL) {
        const R* open = table + (size_t)p.n_steps * Lanes::kRow + 2 * NS;
        rot<FORM, SH>(L.z[q], L.x[q], open[0], open[1]);
      }
    }
  }

  const long long k_full = p.k_end < p.n_steps ? p.k_end : p.n_steps - 1;
  if (STAGE == 1)
    steps_lds(L, table, p.k_begin, k_full, p.chunk_steps);
  else
    steps_scalar(L, table, p.k_begin, k_full);

  if (p.k_end == p.n_steps) {
    // last step: its y rotation after the last stage is the closing half step
    R ha[PPL], hs[PPL];
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      long long idx = base + (long long)q * blockDim.x;
      if (idx >= p.npts) idx = p.npts - 1;
      PointCoords c = coords(p, idx);
      ha[q] = rowc[CY * c.j + HALF];
      hs[q] = rowc[CY * c.j + HALF + 1];
    }
    const R* last = table + (size_t)(p.n_steps - 1) * Lanes::kRow;
    L.template step_at<true>(last, p.n_steps - 1, ha, hs);
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      long long idx = base + (long long)q * blockDim.x;
      bool valid = idx < p.npts;
      if (!valid) idx = p.npts - 1;
      PointCoords c = coords(p, idx);
      // projection on u_out: n = (1 + vsign r.P_out / |P_out|) / 2 with r normalised
      double Pxi = c.px + p.A_in, Pyi = c.py + p.Ay_in;
      double Pxo = c.px + p.A_out, Pyo = c.py + p.Ay_out;
      double Ei = sqrt(Pxi * Pxi + Pyi * Pyi), Eo = sqrt(Pxo * Pxo + Pyo * Pyo);
      double X = L.x[q], Y = L.y[q], Z = L.z[q];
      double nr = sqrt(X * X + Y * Y + Z * Z);
      double n = 0.0;
      if (Ei > 0.0 && Eo > 0.0 && nr > 0.0) {
        double dot = (Pxo * X + Pyo * Y) / nr;
        n = (Eo + p.vsign * dot) / (2.0 * Eo);
      }
      if (valid) p.n_out[idx] = n;
    }
  } else if (p.store_state) {
    R* st = static_cast<R*>(p.state);
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      long long idx = base + (long long)q * blockDim.x;
      if (idx < p.npts) {
        st[idx] = L.x[q];
        st[p.npts + idx] = L.y[q];
        st[2 * p.npts + idx] = L.z[q];
      }
    }
  }
}

template <typename R, int PPL, int STAGE, int FORM, int NS, int POL, int SH>
__global__ void __launch_bounds__(256) strang_kernel(const SolveParams p) {
  strang_tile<R, PPL, STAGE, FORM, NS, POL, SH>(p, p.first + (long long)blockIdx.x * blockDim.x * PPL + threadIdx.x);
}

// ---------------------------------------------------------------------------
// Batched Strang solves in one persistent launch.  Every block takes the next
// work item (one tile of one solve) from a global counter until none is left;
// the host orders the items longest first.  An item's arithmetic is the same as
// in the single-solve kernel, so each solve's result does not depend on the
// batch it runs in.

__global__ void batch_reset(unsigned int* counter) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *counter = 0u;
}

// A tile of a solve by rows: the block's points from `base`.
template <int PPL>
__device__ __forceinline__ void batch_rows(const BatchSolve& s, long long base) {
  if (s.precision == PD_FP32) {
    if (s.form == kFormShear)
      strang_tile<float, PPL, 0, kFormShear, 1, 0, kShearOnce>(s.p, base);
    else
      strang_tile<float, PPL, 0, kFormVersine, 1, 0, kShearPlain>(s.p, base);
  } else if (s.precision == PD_FP32_FAST) {
    if (s.form == kFormShear)
      strang_tile<float, PPL, 0, kFormShear, 1, 0, kShearAlt>(s.p, base);
    else
      strang_tile<float, PPL, 0, kFormVersine, 1, 0, kShearPlain>(s.p, base);
  } else {
    if (s.form == kFormShear)
      strang_tile<double, PPL, 0, kFormShear, 1, 0, kShearPlain>(s.p, base);
    else
      strang_tile<double, PPL, 0, kFormVersine, 1, 0, kShearPlain>(s.p, base);
  }
}

// A wave's unit of a solve by columns.
template <int PPL>
__device__ __forceinline__ void batch_columns(const BatchSolve& s, int unit, unsigned char* lds) {
  if (s.precision == PD_FP32)
    column_tile<float, PPL, 1, 0, kShearOnce>(s.p, unit, lds);
  else if (s.precision == PD_FP32_FAST)
    column_tile<float, PPL, 1, 0, kShearAlt>(s.p, unit, lds);
  else
    column_tile<double, PPL, 1, 0, kShearPlain>(s.p, unit, lds);
}

template <int PPL>
__global__ void __launch_bounds__(256) batch_kernel(const BatchSolve* __restrict__ solves,
                                                    const BatchItem* __restrict__ items, int n_items,
                                                    unsigned int* counter) {
  __shared__ int next;
  for (;;) {
    __syncthreads();  // every lane has read the previous item index
    if (threadIdx.x == 0) next = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int it = next;
    if (it >= n_items) return;  // uniform over the block
    const BatchItem w = items[it];
    batch_rows<PPL>(solves[w.solve], w.base + threadIdx.x);
  }
}

// The same for solves by columns, in a kernel of its own: its 128 registers let four blocks
// of 256 threads stay on a compute unit, where both kinds of tile in one kernel take 168 and
// let three.  Sixteen FP32 solves of 128^2 to 1024^2 points, whole passes: 5.55 ms by rows, 4.07
// by columns.
template <int PPL>
__global__ void __launch_bounds__(256, 4) batch_columns_kernel(const BatchSolve* __restrict__ solves,
                                                               const BatchItem* __restrict__ items, int n_items,
                                                               unsigned int* counter) {
  __shared__ int next;
  extern __shared__ __align__(16) unsigned char pd_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (;;) {
    __syncthreads();  // every lane has read the previous item index
    if (threadIdx.x == 0) next = (int)atomicAdd(counter, 1u);
    __syncthreads();
    // told uniform, so that the item, the solve's parameters and with them the loops'
    // bounds stay in scalar registers
    const int it = __builtin_amdgcn_readfirstlane(next);
    if (it >= n_items) return;
    const BatchItem w = items[it];
    const BatchSolve s = solves[w.solve];
    batch_columns<PPL>(s, (int)w.base + wave, pd_lds + wave * kColumnLdsWave);
  }
}

// Items of both kinds from one queue.  Two kernels side by side, one of each kind, had their
// blocks dealt to the same compute units while others stood idle: six solves of 138 x 207 to
// 208 x 460 points in three precisions, two of them by rows, 0.66 ms, all by rows 0.47, from one
// queue 0.44.
template <int PPL>
__global__ void __launch_bounds__(256, 3) batch_mixed_kernel(const BatchSolve* __restrict__ solves,
                                                             const BatchItem* __restrict__ items, int n_items,
                                                             unsigned int* counter) {
  __shared__ int next;
  extern __shared__ __align__(16) unsigned char pd_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (;;) {
    __syncthreads();  // every lane has read the previous item index
    if (threadIdx.x == 0) next = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(next);
    if (it >= n_items) return;
    const BatchItem w = items[it];
    if (solves[w.solve].p.series) {
      const BatchSolve s = solves[w.solve];
      batch_columns<PPL>(s, (int)w.base + wave, pd_lds + wave * kColumnLdsWave);
    } else {
      batch_rows<PPL>(solves[w.solve], w.base + threadIdx.x);
    }
  }
}

// ---------------------------------------------------------------------------
// Midpoint scheme: spinor state, series coefficients per point and step.

template <int J>
struct Taylor {
  // cos(sqrt x) - 1 = sum_{j>=1} (-x)^j / (2j)!;  sin(sqrt x)/sqrt x = sum_{j>=0} (-x)^j / (2j+1)!
  __device__ __forceinline__ static double h(double x) {
    double acc = coef_h(J);
#pragma unroll
    for (int j = J - 1; j >= 1; --j) acc = fma(acc, x, coef_h(j));
    return acc * x;
  }
  __device__ __forceinline__ static double s(double x) {
    double acc = coef_s(J);
#pragma unroll
    for (int j = J - 1; j >= 0; --j) acc = fma(acc, x, coef_s(j));
    return acc;
  }
  __device__ __forceinline__ static float h(float x) {
    float acc = (float)coef_h(J);
#pragma unroll
    for (int j = J - 1; j >= 1; --j) acc = fmaf(acc, x, (float)coef_h(j));
    return acc * x;
  }
  __device__ __forceinline__ static float s(float x) {
    float acc = (float)coef_s(J);
#pragma unroll
    for (int j = J - 1; j >= 0; --j) acc = fmaf(acc, x, (float)coef_s(j));
    return acc;
  }
  // (-1)^j / (2j)!  and  (-1)^j / (2j+1)!, folded by the compiler
  __device__ __forceinline__ static constexpr double coef_h(int j) {
    double f = 1.0;
    for (int m = 2; m <= 2 * j; ++m) f *= m;
    return (j % 2 ? -1.0 : 1.0) / f;
  }
  __device__ __forceinline__ static constexpr double coef_s(int j) {
    double f = 1.0;
    for (int m = 2; m <= 2 * j + 1; ++m) f *= m;
    return (j % 2 ? -1.0 : 1.0) / f;
  }
};

// psi1' = c psi1 + (-i al - be) psi2 ;  psi2' = c psi2 + (be - i al) psi1, with c = 1 + h.
__device__ __forceinline__ void midpoint_update(double& a1, double& b1, double& a2, double& b2, double h, double al,
                                                double be) {
  double na1 = fma(h, a1, fma(-be, a2, fma(al, b2, a1)));
  double nb1 = fma(h, b1, fma(-be, b2, fma(-al, a2, b1)));
  double na2 = fma(h, a2, fma(be, a1, fma(al, b1, a2)));
  double nb2 = fma(h, b2, fma(be, b1, fma(-al, a1, b2)));
  a1 = na1;
  b1 = nb1;
  a2 = na2;
  b2 = nb2;
}

__device__ __forceinline__ void midpoint_update(float& a1, float& b1, float& a2, float& b2, float h, float al,
                                                float be) {
  float da1 = fmaf(h, a1, fmaf(-be, a2, al * b2));
  float db1 = fmaf(h, b1, fmaf(-be, b2, -(al * a2)));
  float da2 = fmaf(h, a2, fmaf(be, a1, al * b1));
  float db2 = fmaf(h, b2, fmaf(be, b1, -(al * a1)));
  a1 += da1;
  b1 += db1;
  a2 += da2;
  b2 += db2;
}

// tan(sqrt x) / sqrt x - 1 = sum_{n=2}^{J} c_n x^(n-1), the solve's coefficients c
// (tan_polynomial).  The kernel is bound by VALU issue, so each term saved is one instruction
// of about 17 a point's step: 700 x 511 points, 8000 FP64 steps, angles up to .055 take 6 terms
// where the Taylor polynomial took 7 and 1.59 instead of 1.72 ms.  The 1 is left out so that
// the rounding of the sum is relative to its own small size; the caller adds it exactly, as
// (al, be) = fma(tau - 1, (X, Y), (X, Y)).
template <int J, typename R>
struct TanSeries {
  R c[J + 1];
  __device__ __forceinline__ explicit TanSeries(const TanPolynomial& p) {
#pragma unroll
    for (int n = 2; n <= J; ++n) {
      c[n] = (R)p.c[n];
      // FP32 pairs only with its operands in vector registers
      if constexpr (sizeof(R) == 4) asm("" : "+v"(c[n]));
    }
  }
  __device__ __forceinline__ R minus1(R x) const {
    // two FP32 terms are always the series' own (tan_polynomial): 1/3 as a literal takes no
    // register port and pairs more often, 2048 x 2048 points, 80000 steps 91.2 ms, from a
    // register 94.1
    if constexpr (sizeof(R) == 4 && J == 2) return (R)tan_series_coef(2) * x;
    R acc = c[J];
#pragma unroll
    for (int n = J - 1; n >= 2; --n) acc = fma(acc, x, c[n]);
    return acc * x;
  }
};

// Tangent form: psi += (-i al sigma_x - i be sigma_y) psi with (al, be) = tan(theta) (X, Y) / theta,
// i.e. U / cos(theta).  FP32: each component rounded once (the increment is formed
// first).  FP64: two chained FMAs per component (two roundings at 2^-53 stay far below
// the 1e-12 target and save a third of the update's instructions).
__device__ __forceinline__ void midpoint_update_tan(float& a1, float& b1, float& a2, float& b2, float al, float be) {
  float da1 = fmaf(-be, a2, al * b2);
  float db1 = fmaf(-be, b2, -(al * a2));
  float da2 = fmaf(be, a1, al * b1);
  float db2 = fmaf(be, b1, -(al * a1));
  a1 += da1;
  b1 += db1;
  a2 += da2;
  b2 += db2;
}

__device__ __forceinline__ void midpoint_update_tan(double& a1, double& b1, double& a2, double& b2, double al,
                                                    double be) {
  double na1 = fma(-be, a2, fma(al, b2, a1));
  double nb1 = fma(-be, b2, fma(-al, a2, b1));
  double na2 = fma(be, a1, fma(al, b1, a2));
  double nb2 = fma(be, b1, fma(-al, a1, b2));
  a1 = na1;
  b1 = nb1;
  a2 = na2;
  b2 = nb2;
}

// Stage layout of the midpoint kernel: stage j of a step of the NS-stage
// composition uses the per-point phase of class mcls(j) (c = p or q).
template <int NS>
__device__ __forceinline__ constexpr int mcls(int j) {
  return NS == 5 && j == 2 ? 1 : 0;
}

// Point q of a lane of the midpoint kernel: the lane owns column i of the band of
// PPL consecutive rows band * PPL .. band * PPL + PPL - 1, so all its points share
// p_x and with it the FP64 phase c dt (p_x + A_k) of every step (and its FP32
// rounding), computed once per lane.  Consecutive lanes take consecutive columns,
// so loads and stores stay coalesced.  Rows past the last one recompute a valid
// point (the last row) and store nothing.
struct BandPoint {
  long long idx;
  bool valid;
};

__device__ __forceinline__ BandPoint band_point(const SolveParams& p, long long band, int i, int ppl, int q) {
  const long long ny = p.npts / p.nx;
  long long j = band * ppl + q;
  BandPoint b;
  b.valid = j < ny;
  if (!b.valid) j = ny - 1;
  b.idx = j * p.nx + i;
  return b;
}

// TAN: the tangent form (U / cos(theta), one series); otherwise the cosine form.
template <typename R, int J, int PPL, int NS, int POL, int TAN>
__global__ void __launch_bounds__(256) midpoint_kernel(const SolveParams p) {
  constexpr int NC = NS == 5 ? 2 : 1;  // distinct stage coefficients
  constexpr int W = NS * (1 + POL);    // table values per step
  constexpr bool kRenorm = sizeof(R) == 4 || TAN;  // renormalise every kRenormEvery steps
  constexpr int kUnroll = NS == 1 ? 4 : 1;
  // p.first counts lanes here: lane -> (band of rows, column)
  long long lane = p.first + (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long bands = (p.npts / p.nx + PPL - 1) / PPL;
  if (lane >= bands * p.nx) lane = bands * p.nx - 1;  // tail lanes recompute a valid lane's points
  const long long band = lane / p.nx;
  const int col = (int)(lane - band * p.nx);
  const bool lane_valid = p.first + (long long)blockIdx.x * blockDim.x + threadIdx.x < bands * p.nx;
  const double px = p.px_min + (double)col * p.dx;
  R a1[PPL], b1[PPL], a2[PPL], b2[PPL];
  double X0[NC], Y0[NC][PPL], Y2[NC][PPL];
#pragma unroll
  for (int m = 0; m < NC; ++m) X0[m] = p.hx[m] * px;  // vsign c dt px, shared by the lane's points
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    const long long idx = band_point(p, band, col, PPL, q).idx;
    const double py = p.py_min + (double)(idx / p.nx) * p.dy;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      Y0[m][q] = p.hx[m] * py;
      Y2[m][q] = Y0[m][q] * Y0[m][q];
    }
    if (p.load_state) {
      const R* st = static_cast<const R*>(p.state);
      a1[q] = st[idx];
      b1[q] = st[p.npts + idx];
      a2[q] = st[2 * p.npts + idx];
      b2[q] = st[3 * p.npts + idx];
    } else {
      // v_in = (-Px + i Py, E) / (sqrt(2) E) (Sec. II, Eq. (3), unit norm); the K-
      // spinor of Eq. (4) is the same with P -> -P
      double Px = p.vsign * (px + p.A_in), Py = p.vsign * (py + p.Ay_in);
      double E = sqrt(Px * Px + Py * Py);
      double d = 1.4142135623730951 * E;
      bool ok = E > 0.0;
      a1[q] = ok ? (R)(-Px / d) : (R)0;
      b1[q] = ok ? (R)(Py / d) : (R)0;
      a2[q] = ok ? (R)(E / d) : (R)0;
      b2[q] = (R)0;
    }
  }
  const double* __restrict__ tab = static_cast<const double*>(p.table);
  const TanSeries<TAN ? J : 2, R> series(p.tan);
  long long k = p.k_begin;
  while (k < p.k_end) {
    long long seg = p.k_end;
    if (kRenorm) {
      long long next = (k / kRenormEvery + 1) * kRenormEvery;
      seg = next < p.k_end ? next : p.k_end;
    }
    // one step: the stages of table row `row` (W values)
    auto one_step = [&](const double* row) {
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        const double d = row[j];
        const double dy = POL ? row[NS + j] : 0.0;
        const double X = X0[mcls<NS>(j)] + d;  // vsign c dt (px + A_x), FP64 in both forms, once per lane
        const float Xs = (float)X;              // its FP32 rounding (FP32 tangent form)
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
          double Y = POL ? Y0[mcls<NS>(j)][q] + dy : Y0[mcls<NS>(j)][q];
          if constexpr (TAN && sizeof(R) == 4) {
            // the series is evaluated in FP32, so (c dt E)^2 is formed from the rounded
            // phases (a relative error of the size of the coefficient's own rounding)
            float Xr = Xs, Yr = (float)Y;
            float x = POL ? fmaf(Xr, Xr, Yr * Yr) : fmaf(Xr, Xr, (float)Y2[mcls<NS>(j)][q]);
            float t1 = series.minus1(x);  // tan(c dt E) / (c dt E) - 1
            midpoint_update_tan(a1[q], b1[q], a2[q], b2[q], fmaf(t1, Xr, Xr), fmaf(t1, Yr, Yr));
          } else if constexpr (TAN) {
            double x = POL ? fma(X, X, Y * Y) : fma(X, X, Y2[mcls<NS>(j)][q]);
            double t1 = series.minus1(x);
            midpoint_update_tan(a1[q], b1[q], a2[q], b2[q], fma(t1, X, X), fma(t1, Y, Y));
          } else {
            double x = POL ? fma(X, X, Y * Y) : fma(X, X, Y2[mcls<NS>(j)][q]);  // (c dt E)^2
            R xr = (R)x;
            R h = Taylor<J>::h(xr);
            R sp = Taylor<J>::s(xr);  // sin(c dt E) / (c dt E)
            R al = sp * (R)X, be = sp * (R)Y;
            midpoint_update(a1[q], b1[q], a2[q], b2[q], h, al, be);
          }
        }
      }
    };
    if constexpr (NS == 1) {
      // groups of kUnroll steps as in the Strang kernel: a 32-bit trip count (a scalar
      // loop test) and two row sets in turn, each loaded right after the other set's
      // first step and pinned there, so its latency is hidden behind that set's other
      // steps; the clamped index re-reads the last group instead of branching
      constexpr int kG = kUnroll, kV = kUnroll * W;
      while (k + kG <= seg) {
        const long long left = (seg - k) / kG;
        const int n = left < (1 << 30) ? (int)left : (1 << 30);
        const double* __restrict__ g = tab + k * W;
        double ra[kV], rb[kV];
#pragma unroll
        for (int u = 0; u < kV; ++u) ra[u] = g[u];
        int i = 0;
        for (; i + 1 < n; i += 2) {
          one_step(ra);
          __builtin_amdgcn_sched_barrier(0);
          const double* __restrict__ gb = g + (long long)(i + 1) * kV;
#pragma unroll
          for (int u = 0; u < kV; ++u) rb[u] = gb[u];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 1; u < kG; ++u) one_step(ra + u * W);
          one_step(rb);
          __builtin_amdgcn_sched_barrier(0);
          const double* __restrict__ ga = g + (long long)(i + 2 < n ? i + 2 : n - 1) * kV;
#pragma unroll
          for (int u = 0; u < kV; ++u) ra[u] = ga[u];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 1; u < kG; ++u) one_step(rb + u * W);
        }
        if (i < n) {
#pragma unroll
          for (int u = 0; u < kG; ++u) one_step(ra + u * W);
        }
        k += (long long)n * kG;
      }
    }
#pragma unroll kUnroll
    for (; k < seg; ++k) one_step(tab + k * W);
    if (kRenorm && (k % kRenormEvery) == 0 && k < p.n_steps) {
#pragma unroll
      for (int q = 0; q < PPL; ++q) {
        double A1 = a1[q], B1 = b1[q], A2 = a2[q], B2 = b2[q];
        double nr = sqrt(A1 * A1 + B1 * B1 + A2 * A2 + B2 * B2);
        if (nr > 0.0) {
          a1[q] = (R)(A1 / nr);
          b1[q] = (R)(B1 / nr);
          a2[q] = (R)(A2 / nr);
          b2[q] = (R)(B2 / nr);
        }
      }
    }
  }
  if (p.k_end == p.n_steps) {
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      const BandPoint b = band_point(p, band, col, PPL, q);
      PointCoords c = coords(p, b.idx);
      double Pxi = c.px + p.A_in, Pyi = c.py + p.Ay_in;
      double Pxo = p.vsign * (c.px + p.A_out), Pyo = p.vsign * (c.py + p.Ay_out);
      double Ei = sqrt(Pxi * Pxi + Pyi * Pyi), Eo = sqrt(Pxo * Pxo + Pyo * Pyo);
      double A1 = a1[q], B1 = b1[q], A2 = a2[q], B2 = b2[q];
      double n = 0.0;
      if (Ei > 0.0 && Eo > 0.0) {
        // u_out = (E, Px + i Py) / (sqrt(2) E):  sqrt(2) E amp = (E a1 + Px a2 + Py b2) + i (E b1 + Px b2 - Py a2)
        double re = (Eo * A1 + Pxo * A2) + Pyo * B2;
        double im = (Eo * B1 + Pxo * B2) - Pyo * A2;
        n = (re * re + im * im) / (2.0 * Eo * Eo);
        if (kRenorm) n = n / (A1 * A1 + B1 * B1 + A2 * A2 + B2 * B2);
      }
      if (lane_valid && b.valid) p.n_out[b.idx] = n;
    }
  } else if (p.store_state) {
    R* st = static_cast<R*>(p.state);
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      const BandPoint b = band_point(p, band, col, PPL, q);
      if (lane_valid && b.valid) {
        st[b.idx] = a1[q];
        st[p.npts + b.idx] = b1[q];
        st[2 * p.npts + b.idx] = a2[q];
        st[3 * p.npts + b.idx] = b2[q];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Snapshots: the state after k steps (in the state buffer, or v_in at k = 0)
// projected on the positive-energy state of sigma.(p + A(t_k)); a point's value as a
// source of the density pass below.

template <typename R, int POL>
struct StrangSnapshot {
  SolveParams p;
  SnapshotParams s;
  int half_offset, row_stride;
  __device__ __forceinline__ double operator()(long long idx) const {
    PointCoords c = coords(p, idx);
    double Pxi = c.px + p.A_in, Pyi = c.py + p.Ay_in;
    double Px = c.px + s.Ax, Py = c.py + s.Ay;
    double Ei = sqrt(Pxi * Pxi + Pyi * Pyi), E = sqrt(Px * Px + Py * Py);
    double n = 0.0;
    if (Ei > 0.0 && E > 0.0) {
      double X, Y, Z;
      if (p.load_state) {
        const R* st = static_cast<const R*>(p.state);
        R x = st[idx], y = st[p.npts + idx], z = st[2 * p.npts + idx];
        // the stored state is ahead by the opening half step of step k: undo it
        // (field part first, then the per-point part, each by its inverse rotation)
        const R* rowc = static_cast<const R*>(p.row_coef);
        R ha = rowc[(size_t)row_stride * c.j + half_offset], hs = rowc[(size_t)row_stride * c.j + half_offset + 1];
        if (POL) {
          if (p.form == kFormShear)
            rotate_shear(z, x, (R)s.undo_a, (R)s.undo_s);
          else
            rotate_versine(z, x, (R)s.undo_a, (R)s.undo_s);
        }
        if (p.form == kFormShear)
          rotate_shear(z, x, -ha, -hs);
        else
          rotate_versine(z, x, ha, -hs);
        X = x;
        Y = y;
        Z = z;
      } else {
        X = -p.vsign * Pxi / Ei;
        Y = -p.vsign * Pyi / Ei;
        Z = 0.0;
      }
      double nr = sqrt(X * X + Y * Y + Z * Z);
      if (nr > 0.0) n = (E + p.vsign * (Px * X + Py * Y) / nr) / (2.0 * E);
  }
  return n;
  }
};

template <typename R>
struct MidpointSnapshot {
  SolveParams p;
  SnapshotParams s;
  __device__ __forceinline__ double operator()(long long idx) const {
    PointCoords c = coords(p, idx);
    double Pxi = p.vsign * (c.px + p.A_in), Pyi = p.vsign * (c.py + p.Ay_in);
    double Px = p.vsign * (c.px + s.Ax), Py = p.vsign * (c.py + s.Ay);
    double Ei = sqrt(Pxi * Pxi + Pyi * Pyi), E = sqrt(Px * Px + Py * Py);
    double n = 0.0;
    if (Ei > 0.0 && E > 0.0) {
      double A1, B1, A2, B2;
      if (p.load_state) {
        const R* st = static_cast<const R*>(p.state);
        A1 = st[idx];
        B1 = st[p.npts + idx];
        A2 = st[2 * p.npts + idx];
        B2 = st[3 * p.npts + idx];
      } else {
        double d = 1.4142135623730951 * Ei;
        A1 = -Pxi / d;
        B1 = Pyi / d;
        A2 = Ei / d;
        B2 = 0.0;
      }
      double re = (E * A1 + Px * A2) + Py * B2;
      double im = (E * B1 + Px * B2) - Py * A2;
      n = (re * re + im * im) / (2.0 * E * E) / (A1 * A1 + B1 * B1 + A2 * A2 + B2 * B2);
  }
  return n;
  }
};

// ---------------------------------------------------------------------------
// Density: rho = scale * sum n, in a fixed order that depends only on npts.

constexpr int kRedThreads = 256;
constexpr int kRedPerThread = 8;
constexpr long long kRedTile = (long long)kRedThreads * kRedPerThread;

__device__ __forceinline__ double block_sum(double v) {
  __shared__ double wave_part[kRedThreads / 64];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) wave_part[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < kRedThreads / 64; ++w) s += wave_part[w];
  }
  return s;
}

// Sum of tile `tile` of n (2048 points), valid in thread 0.
__device__ __forceinline__ double tile_sum(const double* __restrict__ n, long long npts, long long tile) {
  const long long base = tile * kRedTile + threadIdx.x;
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kRedPerThread; ++q) {
    long long i = base + (long long)q * kRedThreads;
    if (i < npts) s += n[i];
  }
  return block_sum(s);
}

// Sum of the tile partials, valid in thread 0.
__device__ __forceinline__ double partials_sum(const double* __restrict__ partial, long long count) {
  double s = 0.0;
  for (long long i = threadIdx.x; i < count; i += kRedThreads) s += partial[i];
  return block_sum(s);
}

// A stored n(p).
struct StoredDensity {
  const double* __restrict__ n;
  __device__ __forceinline__ double operator()(long long i) const { return n[i]; }
};

// One pass over the points: a point's value from `value`, kept in n_store and copied to
// n_copy (each may be null), its tile's sum into partial[tile].  `done` (null: a second
// launch sums the partials): the blocks count themselves there, and the last one sums the
// partials and writes rho.  The count goes round modulo the number of blocks: every pass
// that counts there has as many (one handle's grid), so it is 0 again after any number of
// them, also where two overlapped and mixed their counts.
//
// What bounds it: for small grids its own launch and the wait for it, so one launch does
// what took four (values, tile sums, their sum, the copy of n) and the copy of rho to the
// host; for large ones the memory, each value read and copied once.
template <typename Value>
__global__ void __launch_bounds__(kRedThreads) density_pass(const Value value, long long npts, double* n_store,
                                                            double* n_copy, double* partial, unsigned* done,
                                                            double scale, double* rho, double* rho_host) {
  const long long tile = blockIdx.x, base = tile * kRedTile + threadIdx.x;
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kRedPerThread; ++q) {
    const long long i = base + (long long)q * kRedThreads;
    if (i < npts) {
      const double v = value(i);
      s += v;
      if (n_store) n_store[i] = v;
      if (n_copy) n_copy[i] = v;
    }
  }
  s = block_sum(s);
  if (!done) {
    if (threadIdx.x == 0) partial[tile] = s;
    return;
  }
  __shared__ bool last;
  if (threadIdx.x == 0) {
    __hip_atomic_store(partial + tile, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();  // the sum before the count, and the count before the others' sums
    last = atomicInc(done, gridDim.x - 1u) == gridDim.x - 1u;
    __threadfence();
  }
  __syncthreads();
  if (!last) return;
  double r = 0.0;
  for (unsigned i = threadIdx.x; i < gridDim.x; i += kRedThreads)
    r += __hip_atomic_load(partial + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();  // the first sum's shared values have been read
  r = block_sum(r);
  if (threadIdx.x == 0) {
    *rho = scale * r;
    if (rho_host) *rho_host = scale * r;
  }
}

__global__ void __launch_bounds__(kRedThreads) density_finish(const double* __restrict__ partial, long long count,
                                                              double scale, double* __restrict__ rho,
                                                              double* __restrict__ rho_host) {
  double s = partials_sum(partial, count);
  if (threadIdx.x == 0) {
    *rho = scale * s;
    if (rho_host) *rho_host = scale * s;
  }
}

// Batched densities: the tiles of every job in one launch (block -> job by
// binary search over the jobs' first tiles), then one block per job.
__global__ void __launch_bounds__(kRedThreads) batch_density_tiles(const DensityJob* __restrict__ jobs, int n_jobs) {
  const long long b = blockIdx.x;
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) / 2;
    if (jobs[mid].tile_begin <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  const DensityJob& j = jobs[lo];
  const long long tile = b - j.tile_begin;
  double s = tile_sum(j.n, j.npts, tile);
  if (threadIdx.x == 0) j.partial[tile] = s;
}

__global__ void __launch_bounds__(kRedThreads) batch_density_finish(const DensityJob* __restrict__ jobs) {
  const DensityJob& j = jobs[blockIdx.x];
  double s = partials_sum(j.partial, (j.npts + kRedTile - 1) / kRedTile);
  if (threadIdx.x == 0) {
    *j.rho = j.scale * s;
    if (j.rho_copy) *j.rho_copy = j.scale * s;
  }
}

// A larger grid than kMaxLanes points (up to 65536 x 65536 at one point per lane) runs as
// consecutive launches over point ranges, each starting at a multiple of the block's span,
// so every point sees the same tile as in one launch.
// Launch `launch(q, blocks)` over the grid in slices of at most kMaxLanes lanes,
// q.first being the slice's first point.
template <typename F>
hipError_t sliced_launch(const SolveParams& p, int block, int ppl, F launch) {
  const long long span = (long long)block * ppl;
  const long long blocks = (p.npts + span - 1) / span;
  const long long max_blocks = kMaxLanes / block;
  SolveParams q = p;
  for (long long b0 = 0; b0 < blocks; b0 += max_blocks) {
    q.first = b0 * span;
    launch(q, (unsigned)(blocks - b0 < max_blocks ? blocks - b0 : max_blocks));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename R, int PPL, int FORM, int NS, int POL, int SH>
hipError_t launch_strang(int block, const SolveParams& p, hipStream_t stream) {
  if (p.stage == 1) {
    const size_t lds = (size_t)p.chunk_steps * BlochLanes<R, PPL, FORM, NS, POL, SH>::kRow * sizeof(R);
    return sliced_launch(p, block, PPL, [&](const SolveParams& q, unsigned nb) {
      hipLaunchKernelGGL((strang_kernel<R, PPL, 1, FORM, NS, POL, SH>), dim3(nb), dim3(block), lds, stream, q);
    });
  }
  return sliced_launch(p, block, PPL, [&](const SolveParams& q, unsigned nb) {
    hipLaunchKernelGGL((strang_kernel<R, PPL, 0, FORM, NS, POL, SH>), dim3(nb), dim3(block), 0, stream, q);
  });
}

template <typename R, int FORM, int NS, int POL, int SH>
hipError_t strang_ppl(int ppl, int block, const SolveParams& p, hipStream_t stream) {
  switch (ppl) {
    case 1: return launch_strang<R, 1, FORM, NS, POL, SH>(block, p, stream);
    case 2: return launch_strang<R, 2, FORM, NS, POL, SH>(block, p, stream);
    default: return launch_strang<R, 4, FORM, NS, POL, SH>(block, p, stream);
  }
}

template <typename R, int FORM, int SH>
hipError_t strang_variant(int stages, int elliptic, int ppl, int block, const SolveParams& p, hipStream_t stream) {
  if (stages == 5)
    return elliptic ? strang_ppl<R, FORM, 5, 1, SH>(ppl, block, p, stream)
                    : strang_ppl<R, FORM, 5, 0, SH>(ppl, block, p, stream);
  return elliptic ? strang_ppl<R, FORM, 1, 1, SH>(ppl, block, p, stream)
                  : strang_ppl<R, FORM, 1, 0, SH>(ppl, block, p, stream);
}

// The midpoint kernel's lanes cover bands of PPL rows column by column (band_point):
// ceil(ny / PPL) * nx lanes, launched in slices of at most kMaxLanes, q.first being
// the slice's first lane.
template <typename R, int J, int PPL, int NS, int POL, int TAN>
hipError_t launch_midpoint(int block, const SolveParams& p, hipStream_t stream) {
  const long long lanes = (p.npts / p.nx + PPL - 1) / PPL * p.nx;
  const long long blocks = (lanes + block - 1) / block;
  const long long max_blocks = kMaxLanes / block;
  SolveParams q = p;
  for (long long b0 = 0; b0 < blocks; b0 += max_blocks) {
    q.first = b0 * block;
    const unsigned nb = (unsigned)(blocks - b0 < max_blocks ? blocks - b0 : max_blocks);
    hipLaunchKernelGGL((midpoint_kernel<R, J, PPL, NS, POL, TAN>), dim3(nb), dim3(block), 0, stream, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename R, int J, int NS, int POL, int TAN>
hipError_t midpoint_ppl(int ppl, int block, const SolveParams& p, hipStream_t stream) {
  switch (ppl) {
    case 1: return launch_midpoint<R, J, 1, NS, POL, TAN>(block, p, stream);
    case 2: return launch_midpoint<R, J, 2, NS, POL, TAN>(block, p, stream);
    default: return launch_midpoint<R, J, 4, NS, POL, TAN>(block, p, stream);
  }
}

template <typename R, int J, int TAN>
hipError_t midpoint_variant(int stages, int elliptic, int ppl, int block, const SolveParams& p, hipStream_t stream) {
  if (stages == 5)
    return elliptic ? midpoint_ppl<R, J, 5, 1, TAN>(ppl, block, p, stream)
                    : midpoint_ppl<R, J, 5, 0, TAN>(ppl, block, p, stream);
  return elliptic ? midpoint_ppl<R, J, 1, 1, TAN>(ppl, block, p, stream)
                  : midpoint_ppl<R, J, 1, 0, TAN>(ppl, block, p, stream);
}

}  // namespace

size_t state_values_per_point(int scheme) { return base_scheme(scheme) == PD_SCHEME_MIDPOINT ? 4 : 3; }

long long density_partials(long long npts) { return (npts + kRedTile - 1) / kRedTile; }

hipError_t launch_propagate(int scheme, int precision, int ppl, int block, int taylor, int elliptic,
                            const SolveParams& p, hipStream_t stream) {
  const int S = (scheme == PD_SCHEME_STRANG4 || scheme == PD_SCHEME_MIDPOINT4) ? 5 : 1;
  if (base_scheme(scheme) == PD_SCHEME_STRANG && p.series) {
    if (precision == PD_FP32) return columns_variant<float, kShearOnce>(S, elliptic, ppl, block, p, stream);
    if (precision == PD_FP32_FAST) return columns_variant<float, kShearAlt>(S, elliptic, ppl, block, p, stream);
    return columns_variant<double, kShearPlain>(S, elliptic, ppl, block, p, stream);
  }
  if (base_scheme(scheme) == PD_SCHEME_STRANG) {
    if (precision == PD_FP32)
      return p.form == kFormShear ? strang_variant<float, kFormShear, kShearOnce>(S, elliptic, ppl, block, p, stream)
                                  : strang_variant<float, kFormVersine, kShearPlain>(S, elliptic, ppl, block, p, stream);
    if (precision == PD_FP32_FAST)
      return p.form == kFormShear ? strang_variant<float, kFormShear, kShearAlt>(S, elliptic, ppl, block, p, stream)
                                  : strang_variant<float, kFormVersine, kShearPlain>(S, elliptic, ppl, block, p, stream);
    return p.form == kFormShear ? strang_variant<double, kFormShear, kShearPlain>(S, elliptic, ppl, block, p, stream)
                                : strang_variant<double, kFormVersine, kShearPlain>(S, elliptic, ppl, block, p, stream);
  }
  // series orders: those tan_polynomial() and taylor_order() choose from
  if (p.form == kMidTangent) {
    if (is_fp32(precision)) {
      switch (p.tan.terms) {
        case 2: return midpoint_variant<float, 2, 1>(S, elliptic, ppl, block, p, stream);
        case 3: return midpoint_variant<float, 3, 1>(S, elliptic, ppl, block, p, stream);
        case 4: return midpoint_variant<float, 4, 1>(S, elliptic, ppl, block, p, stream);
        default: return midpoint_variant<float, 5, 1>(S, elliptic, ppl, block, p, stream);
      }
    }
    switch (p.tan.terms) {
      case 4: return midpoint_variant<double, 4, 1>(S, elliptic, ppl, block, p, stream);
      case 5: return midpoint_variant<double, 5, 1>(S, elliptic, ppl, block, p, stream);
      case 6: return midpoint_variant<double, 6, 1>(S, elliptic, ppl, block, p, stream);
      default: return midpoint_variant<double, 8, 1>(S, elliptic, ppl, block, p, stream);
    }
  }
  if (is_fp32(precision)) {
    switch (taylor) {
      case 3: return midpoint_variant<float, 3, 0>(S, elliptic, ppl, block, p, stream);
      case 5: return midpoint_variant<float, 5, 0>(S, elliptic, ppl, block, p, stream);
      default: return midpoint_variant<float, 9, 0>(S, elliptic, ppl, block, p, stream);
    }
  }
  switch (taylor) {
    case 5: return midpoint_variant<double, 5, 0>(S, elliptic, ppl, block, p, stream);
    case 8: return midpoint_variant<double, 8, 0>(S, elliptic, ppl, block, p, stream);
    default: return midpoint_variant<double, 14, 0>(S, elliptic, ppl, block, p, stream);
  }
}

namespace {

// Tiles up to which the pass's last block sums the partials: beyond, the blocks' counting
// costs more than the launch it saves.
constexpr long long kOnePassTiles = 256;

template <typename Value>
hipError_t launch_pass(const Value& value, long long npts, double* n_store, const DensityOut& o, hipStream_t stream) {
  const long long tiles = density_partials(npts);
  unsigned* done = tiles <= kOnePassTiles ? o.done : nullptr;
  hipLaunchKernelGGL((density_pass<Value>), dim3((unsigned)tiles), dim3(kRedThreads), 0, stream, value, npts, n_store,
                     o.n_copy, o.partial, done, o.scale, o.rho, o.rho_host);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || done) return e;
  hipLaunchKernelGGL(density_finish, dim3(1), dim3(kRedThreads), 0, stream, o.partial, tiles, o.scale, o.rho,
                     o.rho_host);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_snapshot(int scheme, int precision, int elliptic, const SolveParams& p, const SnapshotParams& q,
                           const DensityOut& o, hipStream_t stream) {
  if (base_scheme(scheme) == PD_SCHEME_STRANG) {
    // per row: (stage classes) x (coefficient phases) pairs, then the half-step pair
    const int classes = scheme == PD_SCHEME_STRANG4 ? 2 : 1;
    const int half = 2 * classes * coefficient_phases(precision), stride = half + 2;
    if (is_fp32(precision))
      return elliptic ? launch_pass(StrangSnapshot<float, 1>{p, q, half, stride}, p.npts, p.n_out, o, stream)
                      : launch_pass(StrangSnapshot<float, 0>{p, q, half, stride}, p.npts, p.n_out, o, stream);
    return elliptic ? launch_pass(StrangSnapshot<double, 1>{p, q, half, stride}, p.npts, p.n_out, o, stream)
                    : launch_pass(StrangSnapshot<double, 0>{p, q, half, stride}, p.npts, p.n_out, o, stream);
  }
  return is_fp32(precision) ? launch_pass(MidpointSnapshot<float>{p, q}, p.npts, p.n_out, o, stream)
                            : launch_pass(MidpointSnapshot<double>{p, q}, p.npts, p.n_out, o, stream);
}

// ---------------------------------------------------------------------------
// Static scratch of the no-allocation density (pd_density_static): the tile partials
// of one reduction, then its sum.  Each device holds its own copy until the process
// ends; every call on a device shares it, so nothing in it outlasts a call: every partial is
// written before it is read, and the blocks are counted in the handle's own memory.

static_assert(kRedTile * kStaticPartials == kStaticMaxPoints, "static scratch sized for the reduction's tiles");
static __device__ __align__(256) double scratch[kStaticPartials + 1];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(int device, double** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    // the array's device address, looked up once per device with that device current
    int prev = -1;
    hipError_t e = hipGetDevice(&prev);
    if (e != hipSuccess) return e;
    if (prev != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (prev != device) (void)hipSetDevice(prev);
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

hipError_t launch_density(const double* n, long long npts, const DensityOut& o, hipStream_t stream) {
  return launch_pass(StoredDensity{n}, npts, nullptr, o, stream);
}

hipError_t launch_batch_density(const DensityJob* jobs, int n_jobs, long long total_tiles, hipStream_t stream) {
  if (n_jobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(batch_density_tiles, dim3((unsigned)total_tiles), dim3(kRedThreads), 0, stream, jobs, n_jobs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(batch_density_finish, dim3((unsigned)n_jobs), dim3(kRedThreads), 0, stream, jobs);
  return hipGetLastError();
}

namespace {
size_t batch_lds(int kind, int block) { return kind == kBatchRows ? 0 : (size_t)(block / 64) * kColumnLdsWave; }

using BatchKernel = void (*)(const BatchSolve*, const BatchItem*, int, unsigned int*);
BatchKernel batch_kernel_of(int kind, int ppl) {
  if (kind == kBatchColumns)
    return ppl == 1 ? batch_columns_kernel<1> : ppl == 2 ? batch_columns_kernel<2> : batch_columns_kernel<4>;
  if (kind == kBatchMixed)
    return ppl == 1 ? batch_mixed_kernel<1> : ppl == 2 ? batch_mixed_kernel<2> : batch_mixed_kernel<4>;
  return ppl == 1 ? batch_kernel<1> : ppl == 2 ? batch_kernel<2> : batch_kernel<4>;
}
}  // namespace

hipError_t launch_batch(int kind, int ppl, int block, int grid_blocks, const BatchSolve* solves,
                        const BatchItem* items, int n_items, unsigned int* counter, hipStream_t stream) {
  hipLaunchKernelGGL(batch_reset, dim3(1), dim3(64), 0, stream, counter);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(batch_kernel_of(kind, ppl), dim3(grid_blocks), dim3(block), batch_lds(kind, block), stream, solves,
                     items, n_items, counter);
  return hipGetLastError();
}

int batch_blocks_per_cu(int kind, int ppl, int block) {
  int n = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &n, reinterpret_cast<const void*>(batch_kernel_of(kind, ppl)), block, batch_lds(kind, block));
  return (e == hipSuccess && n > 0) ? n : 1;
}

}  // namespace pdx
