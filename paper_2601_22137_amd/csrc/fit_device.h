// Device code of the fit (see fit.hip): coefficients of the objective, their minimiser with the stop rule, and the chain of a
// matrix by a cluster of workgroups.  Shared by fit.hip (a launch per iteration) and flow.hip (all iterations in one
// launch).
#pragma once
#include "common.h"

namespace prism {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;

constexpr int NT = 256;
constexpr int MAXC = 2 * PRISM_MAX_ROOT + 1;  // coefficients of m

// x plus what the lanes that CTRL selects hold (lanes it does not reach: 0)
template <int CTRL, int ROWS> __device__ inline double add_dpp(double x) {
  const u32x2 w = __builtin_bit_cast(u32x2, x);
  u32x2 v;
  v[0] = __builtin_amdgcn_update_dpp(0, (int)w[0], CTRL, ROWS, 0xF, true);
  v[1] = __builtin_amdgcn_update_dpp(0, (int)w[1], CTRL, ROWS, 0xF, true);
  return x + __builtin_bit_cast(double, v);
}
// Sum over the wave, in lane 63: rows of 16 lanes by shifts, then row by row.  Without a trip to the LDS crossbar per step.
__device__ inline double wave_sum(double x) {
  x = add_dpp<0x111, 0xF>(x);   // row_shr 1, 2, 4, 8
  x = add_dpp<0x112, 0xF>(x);
  x = add_dpp<0x114, 0xF>(x);
  x = add_dpp<0x118, 0xF>(x);
  x = add_dpp<0x142, 0xA>(x);   // row_bcast 15 into rows 1 and 3
  return add_dpp<0x143, 0xC>(x);   // row_bcast 31 into rows 2 and 3
}
__device__ inline double read_lane(double x, int lane) {
  const u32x2 w = __builtin_bit_cast(u32x2, x);
  u32x2 v;
  v[0] = (unsigned)__builtin_amdgcn_readlane((int)w[0], lane);
  v[1] = (unsigned)__builtin_amdgcn_readlane((int)w[1], lane);
  return __builtin_bit_cast(double, v);
}

__device__ inline double horner(const double* c, int deg, double x) {
  double v = c[deg];
  for (int i = deg - 1; i >= 0; --i) v = v * x + c[i];
  return v;
}

// Blocks<d>: Newton-Schulz family (polar, square root, sign).  BlocksInv<p>: coupled inverse
// Newton.  BlocksCheb: Chebyshev inverse.
template <int KIND> struct Blocks;
template <> struct Blocks<1> {
  static constexpr int NV = 3, NW = 3;
  __device__ static void make(const double* v, double* w) {  // v[j-1] = V_j
    w[0] = v[0];
    w[1] = -2.0 * (v[0] - v[1]);
    w[2] = -(v[1] - v[2]);
  }
};
template <> struct Blocks<2> {
  static constexpr int NV = 5, NW = 3;
  __device__ static void make(const double* v, double* w) {
    w[0] = (3.0 * v[1] + v[2]) * 0.25;
    w[1] = -((2.0 * v[1] + v[2]) - (2.0 * v[2] + v[3]));
    w[2] = -(v[3] - v[4]);
  }
};
struct BlocksCheb {   // App. A.4: W_0 = R^2 S^T, W_1 = -(R^2 - R^3) S^T
  static constexpr int NV = 3, NW = 2;
  __device__ static void make(const double* v, double* w) {
    w[0] = v[1];
    w[1] = -(v[1] - v[2]);
  }
};
template <int P> struct BlocksInv {
  static constexpr int NV = P + 1, NW = P + 1;
  __device__ static void make(const double* v, double* w) {
    w[0] = v[0];
    double binom = 1.0;
#pragma unroll
    for (int i = 1; i <= P; ++i) {
      binom = binom * (double)(P - i + 1) / (double)i;  // C(P, i), exact for P <= 8
      w[i] = -binom * (v[i - 1] - v[i]);
    }
  }
};

template <class BL>
__device__ void accumulate_coefficients(const SolveArgs& a, int b, int grp, int ngrp, double* c_out /* global, MAXC */) {
  constexpr int NV = BL::NV, NW = BL::NW, NC = 2 * NW - 1;
  double c[NC];
#pragma unroll
  for (int s = 0; s < NC; ++s) c[s] = 0.0;
  const long long total = (long long)a.rows * a.ld;
  const float* base = a.V + (long long)b * a.bstride;
  for (long long idx = (long long)grp * NT + threadIdx.x; idx < total; idx += (long long)ngrp * NT) {
    double v[NV], w[NW];
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = (double)base[(long long)j * a.vstride + idx];
    BL::make(v, w);
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
      for (int l = 0; l < NW; ++l) c[i + l] += w[i] * w[l];
  }
  __shared__ double red[4][MAXC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int s = 0; s < NC; ++s) {
    const double x = wave_sum(c[s]);
    if (lane == 63) red[wave][s] = x;
  }
  __syncthreads();
  if (threadIdx.x < MAXC) {
    const int s = threadIdx.x;
    c_out[s] = (s < NC) ? (red[0][s] + red[1][s] + red[2][s] + red[3][s]) : 0.0;
  }
}

__device__ void accumulate_for(const SolveArgs& a, int b, int grp, int ngrp, double* out) {
  if (a.fn == PRISM_FN_INV_ROOT) {
    switch (a.p) {
      case 1: accumulate_coefficients<BlocksInv<1>>(a, b, grp, ngrp, out); break;
      case 2: accumulate_coefficients<BlocksInv<2>>(a, b, grp, ngrp, out); break;
      case 3: accumulate_coefficients<BlocksInv<3>>(a, b, grp, ngrp, out); break;
      case 4: accumulate_coefficients<BlocksInv<4>>(a, b, grp, ngrp, out); break;
      case 5: accumulate_coefficients<BlocksInv<5>>(a, b, grp, ngrp, out); break;
      case 6: accumulate_coefficients<BlocksInv<6>>(a, b, grp, ngrp, out); break;
      case 7: accumulate_coefficients<BlocksInv<7>>(a, b, grp, ngrp, out); break;
      default: accumulate_coefficients<BlocksInv<8>>(a, b, grp, ngrp, out); break;
    }
  } else if (a.fn == PRISM_FN_INVERSE) {
    accumulate_coefficients<BlocksCheb>(a, b, grp, ngrp, out);
  } else if (a.d == 1) {
    accumulate_coefficients<Blocks<1>>(a, b, grp, ngrp, out);
  } else {
    accumulate_coefficients<Blocks<2>>(a, b, grp, ngrp, out);
  }
}

// Values that other workgroups of the launch write or go on with: past the caches that are not coherent between XCDs
template <bool COH, typename T> __device__ inline T coh_load(const T* p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}
template <bool COH, typename T, typename V> __device__ inline void coh_store(T* p, V v) {
  if constexpr (COH) __hip_atomic_store(p, (T)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

// The root of f in [xa, xb], f(xa) = fa and f(xb) of opposite signs; eval(x, f, df) gives f and its derivative.  Newton's steps, each
// from a point that has at most half the |f| of the one before it and to a point inside what the signs have left of the interval;
// anywhere else the middle of that.  So every other evaluation at least halves |f| or the interval.  A step of 1e-9 is the last one:
// it leaves an error of its square (over the distance to the next root).  The quotient f / f' is taken with the
// hardware's reciprocal (relative error 2^-24, which scales that last step only; an exact division was half the time of
// an evaluation).
template <typename E> __device__ inline double bracketed_root(double xa, double xb, double fa, E eval) {
  double at = 0.5 * (xa + xb), before = __builtin_inf();
  for (int evals = 0; evals < 200; ++evals) {
    double f, slope;
    eval(at, f, slope);
    if (f == 0.0) break;
    if ((f < 0.0) == (fa < 0.0)) xa = at;
    else xb = at;
    double next = at - f * __builtin_amdgcn_rcp(slope);
    const bool inside = next > xa && next < xb;
    if (fabs(next - at) <= 1.0e-9 * fabs(at)) return inside ? next : at;
    if (!inside || !(2.0 * fabs(f) <= before)) next = 0.5 * (xa + xb);
    if (!(next > xa && next < xb)) break;          // neighbouring numbers
    before = fabs(f);
    at = next;
  }
  return at;
}

// Narrows the bracket [xa, xb] of a root of f (the sign changes once in it; neg: f(xa) < 0) by a whole wave: 64 points at a
// time, twice, so that Newton's method starts within 1/4000 of the bracket's width and needs two or three steps instead of
// seven to ten.
template <typename F> __device__ inline void narrow_bracket(double& xa, double& xb, bool neg, F f) {
  const double at = (double)((threadIdx.x & 63) + 1) * (1.0 / 65.0);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double w = xb - xa;
    const u64 same = __ballot((f(xa + w * at) < 0.0) == neg);
    const int cnt = ~same ? __builtin_ctzll(~same) : 64;     // points on xa's side of the root
    const double l = xa + w * ((double)cnt * (1.0 / 65.0)), h = xa + w * ((double)(cnt + 1) * (1.0 / 65.0));
    if (cnt > 0) xa = l;
    if (cnt < 64) xb = h;
  }
}

// Minimiser of a quartic on [lo, hi], ties to the smallest: one wave, everything in registers (through LDS, level by
// level of the derivative chain, the same took 2 us more per iteration in barriers and LDS round trips).  The roots of
// m' lie between lo, the roots of m'' (closed form, the larger in magnitude first and the other from their product)
// and hi.
__device__ inline double minimise_quartic(double c0, double c1, double c2, double c3, double c4, double lo, double hi) {
  const double q0 = c1, q1 = 2.0 * c2, q2 = 3.0 * c3, q3 = 4.0 * c4;
  const double b0 = q1, b1 = 2.0 * q2, b2 = 3.0 * q3;
  auto value = [&](double x) { return (((c4 * x + c3) * x + c2) * x + c1) * x + c0; };
  auto slope1 = [&](double x) { return ((q3 * x + q2) * x + q1) * x + q0; };
  auto slope = [&](double x, double& f, double& df) {
    f = slope1(x);
    df = (b2 * x + b1) * x + b0;
  };
  double e0 = hi, e1 = hi;                     // roots of m'' inside (lo, hi), in order; hi: none
  if (b2 == 0.0) {
    if (b1 != 0.0) e0 = -b0 / b1;
  } else {
    const double disc = b1 * b1 - 4.0 * b2 * b0;
    if (disc >= 0.0) {
      const double q = -0.5 * (b1 + (b1 < 0.0 ? -sqrt(disc) : sqrt(disc)));
      const double r0 = q / b2, r1 = q != 0.0 ? b0 / q : r0;
      e0 = r0 < r1 ? r0 : r1;
      e1 = r0 < r1 ? r1 : r0;
    }
  }
  e0 = e0 < lo ? lo : (e0 > hi ? hi : e0);
  e1 = e1 < lo ? lo : (e1 > hi ? hi : e1);
  double best = lo, bestv = value(lo);
  double xa = lo, fa = slope1(lo);
  for (int i = 0; i < 3; ++i) {
    const double xb = i == 0 ? e0 : (i == 1 ? e1 : hi);
    const double fb = slope1(xb);
    if ((fa < 0.0) != (fb < 0.0)) {
      double x;
      if (fa == 0.0) x = xa;
      else if (fb == 0.0) x = xb;
      else {
        double l = xa, h = xb;
        narrow_bracket(l, h, fa < 0.0, slope1);
        x = bracketed_root(l, h, fa, slope);
      }
      const double v = value(x);
      if (v < bestv) { bestv = v; best = x; }
    }
    xa = xb;
    fa = fb;
  }
  const double vh = value(hi);
  if (vh < bestv) best = hi;
  return best;
}

// Minimiser of m(alpha) = sum_s c[s] alpha^s, s < nc, on [lo, hi], ties to the smallest, by one wave (all lanes get it); false: c is
// not usable (not finite, or nothing but zeros).  c: LDS.
__device__ inline bool minimise(const double* c, int nc, double lo, double hi, double& best) {
  const int t = threadIdx.x & 63;
  const int deg = nc - 1;   // degree of m
  const int dq = deg - 1;   // degree of m'
  bool bad = false, some = false;
  if (t < nc) {
    const double v = c[t];
    bad = !(v == v) || fabs(v) > 1.0e300;
    some = fabs(v) >= 1.0e-300;
  }
  if (__any(bad) || !__any(some)) return false;
  if (deg == 2) {   // Chebyshev inverse
    best = lo;
    double bestv = horner(c, 2, lo);
    const double x = -0.5 * c[1] / c[2];
    if (c[2] != 0.0 && x >= lo && x <= hi && horner(c, 2, x) < bestv) { bestv = horner(c, 2, x); best = x; }
    if (horner(c, 2, hi) < bestv) best = hi;
    return true;
  }
  if (deg == 4) {   // Newton-Schulz family, DB Newton
    best = minimise_quartic(c[0], c[1], c[2], c[3], c[4], lo, hi);
    return true;
  }
  auto slope1 = [&](double x) {
    double f = 0.0;
    for (int i = deg; i >= 1; --i) f = f * x + (double)i * c[i];
    return f;
  };
  // Without or with one root of m' inside, by the theorem of Budan and Fourier: the roots in (lo, hi] are as many as the sign
  // changes of the derivatives of m' at lo less those at hi, or fewer by an even number.  Then nothing or one bracket is left
  // to search; level by level, below, that took 8 us more per iteration at p = 4.
  {
    const int j = t;                            // derivative j of m' over (j + 1)!
    double at[2] = {0.0, 0.0}, power[2] = {1.0, 1.0}, binom = 1.0;
#pragma unroll
    for (int i = 0; i < 2 * PRISM_MAX_ROOT; ++i) {
      if (i > dq) break;                        // uniform
      const double v = i + j <= dq ? c[i + j + 1] * binom : 0.0;
      at[0] += v * power[0]; at[1] += v * power[1];
      power[0] *= lo; power[1] *= hi;
      binom *= (double)(i + j + 2) * (1.0 / (double)(i + 1));
    }
    int changes[2];
    bool exact = true;
    for (int e = 0; e < 2; ++e) {
      const u64 neg = __ballot(j <= dq && at[e] < 0.0);
      exact = exact && !__any(j <= dq && !(at[e] < 0.0 || at[e] > 0.0));   // a zero: left to the search below
      changes[e] = __popcll((neg ^ (neg >> 1)) & ((1ull << dq) - 1));
    }
    const int roots = changes[0] - changes[1];
    if (exact && (roots == 0 || roots == 1)) {
      best = lo;
      double bestv = horner(c, deg, lo);
      if (roots == 1) {
        const double fa = read_lane(at[0], 0);
        double l = lo, h = hi;
        narrow_bracket(l, h, fa < 0.0, slope1);
        const double x = bracketed_root(l, h, fa, [&](double y, double& f, double& df) {
          f = 0.0; df = 0.0;
          for (int i = deg; i >= 1; --i) { df = df * y + f; f = f * y + (double)i * c[i]; }
        });
        const double v = horner(c, deg, x);
        if (v < bestv) { bestv = v; best = x; }
      }
      if (horner(c, deg, hi) < bestv) best = hi;
      return true;
    }
  }
  // derivative chain: s_q[j] = (j+1)-th derivative of m, degree deg-1-j; a lane per interval, all in one wave
  __shared__ double s_q[2 * PRISM_MAX_ROOT][MAXC];
  __shared__ double s_roots[2][MAXC + 2];
  __shared__ int s_nroots[2];
  auto sync = []() {           // LDS written by other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (t == 0) {
    for (int i = 0; i <= dq; ++i) s_q[0][i] = (double)(i + 1) * c[i + 1];
    for (int j = 1; j < dq; ++j)
      for (int i = 0; i <= dq - j; ++i) s_q[j][i] = (double)(i + 1) * s_q[j - 1][i + 1];
    // linear level j = dq-1: a0 + a1 x
    const double a0 = s_q[dq - 1][0], a1 = s_q[dq - 1][1];
    int n0 = 0;
    if (a1 != 0.0) {
      const double r = -a0 / a1;
      if (r >= lo && r <= hi) s_roots[(dq - 1) & 1][n0++] = r;
    }
    s_nroots[(dq - 1) & 1] = n0;
  }
  sync();
  for (int j = dq - 2; j >= 0; --j) {
    const int src = (j + 1) & 1, dst = j & 1;
    const int nr = s_nroots[src];
    const int pdeg = dq - j;
    double found = 0.0;
    bool has = false;
    if (t <= nr) {  // interval t between consecutive roots of the next derivative
      const double xa = (t == 0) ? lo : s_roots[src][t - 1];
      const double xb = (t == nr) ? hi : s_roots[src][t];
      double fa = horner(s_q[j], pdeg, xa);
      const double fb = horner(s_q[j], pdeg, xb);
      if (fa == 0.0) { found = xa; has = true; }
      else if (t == nr && fb == 0.0) { found = xb; has = true; }
      else if ((fa < 0.0) != (fb < 0.0) && fb != 0.0) {
        const double x = bracketed_root(xa, xb, fa, [&](double y, double& f, double& df) {
          f = horner(s_q[j], pdeg, y);
          df = horner(s_q[j + 1], pdeg - 1, y);   // the derivative of level j is level j + 1 of the chain
        });
        found = x;
        has = true;
      }
    }
    const u64 all = __ballot(has);
    if (has) s_roots[dst][__popcll(all & ((1ull << t) - 1))] = found;
    if (t == 0) s_nroots[dst] = __popcll(all);
    sync();
  }
  const int lvl = (dq >= 2) ? 0 : ((dq - 1) & 1);
  const int nr = s_nroots[lvl & 1];
  best = lo;
  double bestv = horner(c, deg, lo);
  for (int i = 0; i < nr; ++i) {
    const double x = s_roots[lvl & 1][i];
    const double v = horner(c, deg, x);
    if (v < bestv) { bestv = v; best = x; }
  }
  const double vh = horner(c, deg, hi);
  if (vh < bestv) best = hi;
  return true;
}

// The interval of the fit
__device__ inline void fit_interval(int fn, int p, int d, double& lo, double& hi) {
  if (fn == PRISM_FN_INV_ROOT) { lo = 1.0 / p; hi = 2.0 / p; }
  else if (fn == PRISM_FN_INVERSE) { lo = 0.5; hi = 2.0; }
  else if (fn == PRISM_FN_SQRT_NEWTON) { lo = 0.0; hi = 1.0; }
  else if (d == 1) { lo = 0.5; hi = 1.0; }
  else { lo = 0.375; hi = 1.45; }
}

// One workgroup (NT threads or more), matrix b: stop rule and coefficient of iteration a.k.  Every return but the last is taken
// by all threads of the workgroup together.
// c_local (LDS, MAXC doubles): the moments are accumulated right here.
// ctl_local (LDS): the matrix's control block, when the caller keeps it on chip; it is not done then.  (Nobody may look: thread 0
// can have set `done` before a late wave gets to the test, and that wave would leave alone.)
// COH: the partials come from workgroups of the same launch, the report is continued by others of it.
template <bool COH = false>
__device__ void solve_body(const SolveArgs& a, int b, double* c_local = nullptr, Ctrl* ctl_local = nullptr) {
  const int t = threadIdx.x;
  Ctrl* ctl = ctl_local ? ctl_local : &a.ctrl[b];
  const int done = ctl_local ? 0 : ctl->done;
  const float res0 = ctl->res0, res1 = ctl->res1, res2 = ctl->res2;   // in the shadow of the first load
  if (done) return;
  prism_info* info = a.info + b;
  __shared__ int s_stop;
  __shared__ double s_c[MAXC];

  // residual: sum of the per-tile partials, every thread a strided share, then a fixed tree
  __shared__ double s_rho[4];
  double part = 0.0;
  for (int i = t; t < NT && i < a.nparts; i += NT) part += (double)coh_load<COH>(a.rho_part + (long long)b * a.nparts + i);
  part = wave_sum(part);
  if (t < NT && (t & 63) == 63) s_rho[t >> 6] = part;
  __syncthreads();
  if (a.phase == 2) {
    if (t == 0) s_stop = 0;          // coefficient only: the stop test of this k has been taken
  } else if (t == 0) {
    const double rho = (s_rho[0] + s_rho[1]) + (s_rho[2] + s_rho[3]);
    const double res = sqrt(rho / (double)a.n);
    coh_store<COH>(&info->residual[a.k], (float)res);
    int status = -1;
    if (!(res == res) || res > 1.0e300) status = PRISM_INFO_DIVERGED;
    else if (a.tol > 0.0 && res <= a.tol) status = PRISM_INFO_CONVERGED;
    else if (a.k == a.max_iters) status = PRISM_INFO_BUDGET;
    else if (a.tol > 0.0 && a.k >= 2 && res > (double)res1 && res1 > res2 && res > (double)res0)
      status = PRISM_INFO_DIVERGED;
    // one lane is active, so the status is uniform; told so, the compiler keeps the two sets of stores below apart
    // (with a branch on the lane's own value it merged their addresses and the report went to the wrong block)
    status = __builtin_amdgcn_readfirstlane(status);
    if (status >= 0) {
      ctl->status = status;
      ctl->iters = a.k;
      ctl->done = 1;
      coh_store<COH>(&info->status, status);
      coh_store<COH>(&info->iters, a.k);
      s_stop = 1;
    } else {
      if (a.k == 0) ctl->res0 = (float)res;
      ctl->res2 = res1;
      ctl->res1 = (float)res;
      ctl->iters = a.k + 1;     // the update of this iteration is already enqueued behind us
      coh_store<COH>(&info->iters, a.k + 1);
      s_stop = 0;
    }
  }
  __syncthreads();
  if (s_stop || a.phase == 1) return;

  if (a.fn == PRISM_FN_SQRT_NEWTON) {
    // The fp32 inverse N_k loses about cond(M_k) * eps * sqrt(n) of its accuracy and X, Y inherit
    // that; once it is worthless the iteration would still drive M_k to I and report convergence.
    // Slot 16 of the partials holds ||M_k N_k v - v||^2 for a probe vector v of +-1 entries, an
    // estimate of ||M_k N_k - I||_F^2: above 10 % relative the matrix stops as diverged, before the
    // update that would use N_k.
    if (t < 64) {
      double e2 = 0.0;
      for (int gidx = t; gidx < a.ngroups; gidx += 64) e2 += a.cpart[((long long)b * a.ngroups + gidx) * MAXC + 16];
      e2 = wave_sum(e2);
      if (t == 63 && !(e2 <= 0.01 * (double)a.n)) {
        ctl->status = PRISM_INFO_DIVERGED; ctl->iters = a.k; ctl->done = 1;
        coh_store<COH>(&info->status, PRISM_INFO_DIVERGED); coh_store<COH>(&info->iters, a.k);
        s_stop = 1;
      }
    }
    __syncthreads();
    if (s_stop) return;
  }

  double lo, hi;
  fit_interval(a.fn, a.p, a.d, lo, hi);

  if (a.mode != 0) {
    if (t == 0) {
      // without a fit: the Taylor coefficient, which is l except for the Chebyshev inverse (1)
      // (and the DB Newton iteration, whose classical coefficient is 1/2)
      const double taylor = (a.fn == PRISM_FN_INVERSE) ? 1.0 : (a.fn == PRISM_FN_SQRT_NEWTON ? 0.5 : lo);
      const float al = (a.mode == 3) ? a.sched_alpha : (float)((a.mode == 1) ? taylor : hi);
      ctl->alpha = al;
      coh_store<COH>(&info->alpha[a.k], al);
    }
    return;
  }

  const int nc = (a.fn == PRISM_FN_INV_ROOT) ? 2 * a.p + 1 : (a.fn == PRISM_FN_INVERSE ? 3 : 5);
  if (c_local) {   // moments straight into LDS
    accumulate_for(a, b, 0, 1, c_local);
    __syncthreads();
    if (t < MAXC) s_c[t] = c_local[t];
  } else {
    // coefficient s = sum of the group partials: thread (share, s) adds up every SHARES-th group, then the shares
    // in order
    constexpr int SHARES = NT / MAXC;
    __shared__ double s_share[SHARES][MAXC];
    if (t < SHARES * MAXC) {
      double v = 0.0;
      for (int gidx = t / MAXC; gidx < a.ngroups; gidx += SHARES) v += coh_load<COH>(a.cpart + ((long long)b * a.ngroups + gidx) * MAXC + t % MAXC);
      s_share[t / MAXC][t % MAXC] = v;
    }
    __syncthreads();
    if (t < MAXC) {
      double v = 0.0;
      for (int q = 0; q < SHARES && q < a.ngroups; ++q) v += s_share[q][t];
      s_c[t] = v;
    }
  }
  __syncthreads();

  // ---- minimise m(alpha) = sum_s c_s alpha^s on [lo, hi] ----
  if (t >= 64) return;
  double best = lo;
  const bool usable = minimise(s_c, nc, lo, hi, best);
  if (t == 0) {
    ctl->alpha = (float)best;
    coh_store<COH>(&info->alpha[a.k], (float)best);
    // The fit has left the upper end of its interval: no eigenvalue of R is close to 1 any more,
    // i.e. no singular value of the iterate is small.  The bf16 polar path stops carrying the low
    // half of the iterate from here on (it exists for the small singular values only).
    if (usable && best < hi - 1e-6) ctl->plain = 1;
  }
}

// ---- chain, moments and solve of one iteration in one launch ----
// The chain V_j = R V_{j-1} of a matrix, up to order 2048, by a cluster of G = n / (16 RB) workgroups: each owns 16 RB
// rows of R, fetches them once, keeps them in registers for all products (its waves take the chunks of 64 k by
// turns) and hands its rows of V_j to the others through memory; then every workgroup forms the moments of its rows
// and the one that arrives last solves for alpha.
// What bounds it: latency, 4 to 5 us per product (hand-over 2.6 us, products, partial sums).  Order 320: 26 us, 768: 31 us,
// 16 matrices of order 1024 (fp32): 76 us in one launch, where the chain products, the moments and the solve took seven
// of 6 to 25 us each, and 2.6 us instead of 18 us for every iteration enqueued past convergence.
// Calls: fp32 polar 6 x 500 x 299 1.29 -> 0.77 ms, mixed small inverse roots 9.3 -> 5.4, sign 4 x 1000^2 3.02 -> 2.57, one
// 768 x 3072 bf16 gradient 0.56 -> 0.50.
// Hand-over: V and the coefficient partials are written and read past the caches that are not coherent between XCDs
// (agent scope), and a wave has seen its stores complete (vmcnt) before its workgroup
// counts itself in.  Agent-scope fences instead write back and invalidate whole L2s: 8 to 25 us per hand-over
// with 256 workgroups.
// Nobody depends on a workgroup that is not running: a wait is bounded (a.polls), and a workgroup whose partners' rows
// are still missing then (they may have no place on the chip: other launches, fewer CUs) computes those rows itself,
// block by block, with the same sums in the same order.  The partner writes the same bits again when it gets to run:
// every V_j has memory of its own, and what it reads has not changed.  Behind the chain nobody waits.
// sync: per matrix and block of rows the last product done, counted through all launches of a call (epoch + j; zeroed by
// the prepare step); and a counter of the products that workgroups have done for their own rows.  G j of them: all rows of
// V_j are there, because a workgroup goes on to product j + 1 only when they are.  The counter is what is polled (all
// flags of a matrix at every poll: 1 us more per product).
//   V_0 .. V_{nv-1} in memory: [n / 16][LD / 16][lane][4], lane (lr, lq) with rows 4 lq + r,
//   r = 0..3, of column lr of the 16 x 16 block: what a lane holds of a product's result is its operand of the next, and a
//   wave moves 1 KiB without gaps.
// The order of all sums is a function of n and the sketch width alone (the moments are kept per 16 rows), so the bits
// do not depend on RB.
template <bool B16> struct RRow;   // four consecutive k of one row of R
template <> struct RRow<false> {
  typedef float elem;
  f32x4 v;
  __device__ void load(const float* p) { v = *(const f32x4*)p; }
  __device__ float get(int e) const { return v[e]; }
};
template <> struct RRow<true> {
  typedef unsigned short elem;
  u32x2 v;
  __device__ void load(const unsigned short* p) { v = *(const u32x2*)p; }
  __device__ float get(int e) const { return __uint_as_float((e & 1) ? (v[e >> 1] & 0xFFFF0000u) : (v[e >> 1] << 16)); }
};
// 16 bytes past the caches that are not coherent between XCDs (sc1, as agent-scope atomics have it; those exist up
// to 8 bytes only); `bytes` bounds the array
__device__ inline f32x4 load_shared16(const float* base, int bytes, int offset) {
  const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00027000);
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, offset, 0, 16));
}
__device__ inline void store_shared16(float* base, int bytes, int offset, f32x4 v) {
  const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00027000);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, offset, 0, 16);
}

// coefficient partials of 16 rows (own[j * stride + element]), by one wave
template <class BL>
__device__ void block_moments(const float* own, int stride, int count, double* out) {
  constexpr int NV = BL::NV, NW = BL::NW, NC = 2 * NW - 1;
  const int lane = threadIdx.x & 63;
  double c[NC];
#pragma unroll
  for (int s = 0; s < NC; ++s) c[s] = 0.0;
  for (int idx = lane; idx < count; idx += 64) {
    double v[NV], w[NW];
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = (double)own[j * stride + idx];
    BL::make(v, w);
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
      for (int l = 0; l < NW; ++l) c[i + l] += w[i] * w[l];
  }
#pragma unroll
  for (int s = 0; s < NC; ++s) c[s] = wave_sum(c[s]);
  if (lane == 63) {
#pragma unroll
    for (int s = 0; s < MAXC; ++s) {
      const double v = s < NC ? c[s < NC ? s : 0] : 0.0;
      __hip_atomic_store((u64*)out + s, __builtin_bit_cast(u64, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}
__device__ __noinline__ void block_moments_for(int fn, int p, int d, const float* own, int stride, int count, double* out) {
  if (fn == PRISM_FN_INV_ROOT) {
    switch (p) {
      case 1: block_moments<BlocksInv<1>>(own, stride, count, out); break;
      case 2: block_moments<BlocksInv<2>>(own, stride, count, out); break;
      case 3: block_moments<BlocksInv<3>>(own, stride, count, out); break;
      case 4: block_moments<BlocksInv<4>>(own, stride, count, out); break;
      case 5: block_moments<BlocksInv<5>>(own, stride, count, out); break;
      case 6: block_moments<BlocksInv<6>>(own, stride, count, out); break;
      case 7: block_moments<BlocksInv<7>>(own, stride, count, out); break;
      default: block_moments<BlocksInv<8>>(own, stride, count, out); break;
    }
  } else if (fn == PRISM_FN_INVERSE) {
    block_moments<BlocksCheb>(own, stride, count, out);
  } else if (d == 1) {
    block_moments<Blocks<1>>(own, stride, count, out);
  } else {
    block_moments<Blocks<2>>(own, stride, count, out);
  }
}

// Workgroup `mine` of the G of matrix b.  KW waves, each with every KW-th chunk of 64 k, NCH chunks at most (n <= 64 KW NCH).
// True, for all threads, in the workgroup that arrives last: it goes on to the solve.
template <bool B16, int LD, int RB, int NCH, int KW>
__device__ __forceinline__ bool fit_rows(const FitArgs& a, int b, int batch, int mine, int G, float* fit_lds) {
  constexpr int NBLK = LD / 16, NQ = RB * NBLK, ROWS = 16 * RB;
  constexpr int NACC = NBLK == 1 ? 4 : (NBLK == 2 && KW == 4 ? 2 : 1);   // independent accumulators (the same for every RB)
  constexpr int CG = NBLK == 1 && RB == 1 ? 2 : 1;            // chunks whose operands are requested together
  f32x4 (*red)[NQ][64] = (f32x4 (*)[NQ][64])fit_lds;          // [KW] partial sums
  float* own = fit_lds + KW * NQ * 256;                       // [nv][ROWS][LD]: this workgroup's rows of V_1 .. V_nv
  __shared__ float dfix[ROWS];
  __shared__ int s_next;
  const SolveArgs& sv = a.sv;
  const int n = sv.rows;
  const int t = threadIdx.x, lane = t & 63, lr = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nchunks = n / 64;
  typedef typename RRow<B16>::elem elem;
  RRow<B16> ra[RB][NCH][4];
  auto load_rows = [&](int row0) {
    const elem* R = (const elem*)a.R + (long long)b * a.strideR + (long long)row0 * a.ldr;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
      if (w + KW * i < nchunks) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int s = 0; s < 4; ++s) ra[rb][i][s].load(R + (16 * rb + lr) * a.ldr + (w + KW * i) * 64 + 16 * s + 4 * lq);
      }
    if (B16 && t < ROWS) {   // exact diagonal minus the rounded one
      const unsigned short h = ((const unsigned short*)R)[t * a.ldr + row0 + t];
      dfix[t] = a.D[(long long)b * a.strideD + (long long)(row0 + t) * a.ldd] - __uint_as_float((unsigned)h << 16);
    }
    if (B16) __syncthreads();
  };
  int held = mine;              // whose rows of R the registers hold
  load_rows(mine * ROWS);
  unsigned* done = a.sync + (long long)b * FIT_SYNC_WORDS;   // products done, by block of rows
  unsigned* count = done + FIT_MAX_CLUSTER;                   // ... and counted over the workgroups, each for its own rows
  const int vbytes = n * LD * 4;
#pragma unroll 1
  for (int j = 1; j <= a.nv; ++j) {
    const float* Vin = j == 1 ? a.V0 : a.V + ((long long)(j - 2) * batch + b) * n * LD;        // V_{j-1}
    float* Vout = a.V + ((long long)(j - 1) * batch + b) * n * LD;
#pragma unroll 1
    for (int blk = mine; blk >= 0;) {   // this workgroup's rows, then others that are missing
      const int row0 = blk * ROWS;
      if (blk != held) { held = blk; load_rows(row0); }
      if constexpr (B16) {   // widened at each use: the compiler would keep the fp32 values of all products instead
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int i = 0; i < NCH; ++i)
#pragma unroll
            for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(ra[rb][i][s].v));
      }
      f32x4 acc[RB][NBLK][NACC];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int q = 0; q < NBLK; ++q)
#pragma unroll
          for (int u = 0; u < NACC; ++u) acc[rb][q][u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      f32x4 vf[2][CG][NBLK][4];
      auto request = [&](int i0) {
#pragma unroll
        for (int i = 0; i < CG; ++i)
          if (i0 + i < NCH && w + KW * (i0 + i) < nchunks) {
#pragma unroll
            for (int q = 0; q < NBLK; ++q)
#pragma unroll
              for (int s = 0; s < 4; ++s) vf[(i0 / CG) & 1][i][q][s] = load_shared16(Vin, vbytes, (((w + KW * (i0 + i)) * 4 + s) * NBLK + q) * 1024 + lane * 16);
          }
      };
      request(0);
#pragma unroll
      for (int i0 = 0; i0 < NCH; i0 += CG) {
        if (i0 + CG < NCH) request(i0 + CG);
#pragma unroll
        for (int i = 0; i < CG; ++i)
          if (i0 + i < NCH && w + KW * (i0 + i) < nchunks) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int q = 0; q < NBLK; ++q)
#pragma unroll
                  for (int rb = 0; rb < RB; ++rb)
                    acc[rb][q][(4 * s + e) % NACC] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        ra[rb][i0 + i < NCH ? i0 + i : 0][s].get(e), vf[(i0 / CG) & 1][i][q][s][e], acc[rb][q][(4 * s + e) % NACC], 0, 0, 0);
          }
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int q = 0; q < NBLK; ++q) {
#pragma unroll
          for (int h = NACC / 2; h > 0; h >>= 1)
#pragma unroll
            for (int u = 0; u < h; ++u) acc[rb][q][u] += acc[rb][q][u + h];
          red[w][rb * NBLK + q][lane] = acc[rb][q][0];
        }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < (NQ + KW - 1) / KW; ++i) {
        const int x = w + KW * i;
        if (x < NQ) {
          const int row = 16 * (x / NBLK) + 4 * lq, col = 16 * (x % NBLK) + lr;
          f32x4 v = (red[0][x][lane] + red[1][x][lane]) + (red[2][x][lane] + red[3][x][lane]);
          if constexpr (KW == 8) v += (red[4][x][lane] + red[5][x][lane]) + (red[6][x][lane] + red[7][x][lane]);
          const int vo = (row0 / 16 * NBLK + x) * 1024 + lane * 16;   // these entries in V
          if (B16) {
            f32x4 prev;
            if (j == 1 || blk != mine) prev = load_shared16(Vin, vbytes, vo);
            else {
#pragma unroll
              for (int r = 0; r < 4; ++r) prev[r] = own[((j - 2) * ROWS + row + r) * LD + col];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] += dfix[row + r] * prev[r];
          }
          if (j < a.nv) store_shared16(Vout, vbytes, vo, v);
          if (blk == mine) {
#pragma unroll
            for (int r = 0; r < 4; ++r) own[((j - 1) * ROWS + row + r) * LD + col] = v[r];
          }
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores have reached memory
      __syncthreads();
      if (j == a.nv || G == 1) break;
      if (w == 0) {
        const unsigned want = a.epoch + j;
        int next = -1;
        if (lane == 0) {
          __hip_atomic_fetch_max(done + blk, want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (blk == mine) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          bool all = false;
          for (int i = blk == mine ? a.polls : 0; i > 0 && !all; --i) {
            all = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= (unsigned)(G * j);
            if (!all) __builtin_amdgcn_s_sleep(1);
          }
          next = all ? -1 : 0;
        }
        if (__builtin_amdgcn_readfirstlane(next) == 0) {   // whose rows are missing?  The next behind this workgroup's own, round about
          const unsigned have = lane < G ? __hip_atomic_load(done + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : want;
          u64 missing = __ballot(have < want && lane != mine && lane != blk);
          missing = missing >> mine | missing << ((64 - mine) & 63);
          next = missing ? (mine + __builtin_ctzll(missing)) & 63 : -1;
        }
        if (lane == 0) s_next = next;
      }
      __syncthreads();
      blk = __builtin_amdgcn_readfirstlane(s_next);
    }
  }
  for (int rb = w; rb < RB; rb += KW)
    block_moments_for(sv.fn, sv.p, sv.d, own + rb * 16 * LD, ROWS * LD, 16 * LD,
                      sv.cpart + ((long long)b * sv.ngroups + mine * RB + rb) * MAXC);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (t == 0) {
    const int last = G == 1 || __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(G * a.nv - 1);
    if (last && G > 1) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    s_next = last;
  }
  __syncthreads();
  return s_next != 0;
}

// ---- a fit and, beside it, the tiles of the product that needs its coefficient at the end only (Q = R / 2 + alpha R^2) ----
// The fit is latency (hand-overs, a serial solve) on a few workgroups; the product runs on the rest of the chip meanwhile, its
// tiles keep their sums in registers and wait for the coefficient.  Per matrix `tiles` workgroups more than the fit has; which of the steps
// one takes is decided by a counter, rows of the fit first: a tile waits for steps that were taken before it, by workgroups that
// run, so nothing depends on workgroups being resident together.  (Rows wait for each other bounded, see fit_rows.)
// Words of FitArgs::sync: counter (every launch that leaves the matrix live takes as many numbers as it has steps), then iteration + 1 and
// beside it the bits of alpha or SQUARE_STOPPED.
constexpr int SQUARE_TICKET = FIT_MAX_CLUSTER + 32, SQUARE_STATE = FIT_MAX_CLUSTER + 64;
constexpr unsigned SQUARE_STOPPED = 0xFFFFFFFFu;
template <bool B16, int LD, int RB, int NCH, class TILE>
__device__ __forceinline__ void fit_and_tiles(const FitArgs& f, int batch, int tiles, unsigned char* smem, TILE tile) {
  __shared__ int s_step;
  __shared__ u64 s_state;
  const int t = threadIdx.x, G = f.sv.rows / (16 * RB);
  // the rows of all matrices are dispatched before the tiles
  const int b = (int)blockIdx.x < G * batch ? blockIdx.x / G : (blockIdx.x - G * batch) / tiles;
  unsigned* sync = f.sync + (long long)b * FIT_SYNC_WORDS;
  // Whether the matrix is done is one thread's to see, for the whole workgroup: whoever solves sets it while others of this launch
  // may only be starting, and waves that look for themselves could part ways (those that stay would find no step in LDS).
  // The step is taken in the same breath, wanted or not: nobody counts on the numbers of a matrix that is done.
  if (t == 0) {
    const unsigned ticket = __hip_atomic_fetch_add(sync + SQUARE_TICKET, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int done = coh_load<true>(&f.sv.ctrl[b].done);
    s_step = done ? -1 : (int)(ticket % (unsigned)(G + tiles));
  }
  __syncthreads();
  const int step = __builtin_amdgcn_readfirstlane(s_step);
  if (step < 0) return;
  u64* state = (u64*)(sync + SQUARE_STATE);
  if (step < G) {
    if (!fit_rows<B16, LD, RB, NCH, 4>(f, b, batch, step, G, (float*)smem)) return;
    solve_body<true>(f.sv, b);
    __syncthreads();
    if (t == 0) {
      const Ctrl& c = f.sv.ctrl[b];
      unsigned bits = __float_as_uint(c.alpha);
      if (bits == SQUARE_STOPPED) bits ^= 1u;            // a NaN like another
      coh_store<true>(state, (u64)(c.done ? SQUARE_STOPPED : bits) << 32 | (unsigned)(f.sv.k + 1));
    }
    return;
  }
  tile(b, step - G, [&](float& alpha) {
    if (t == 0) {
      u64 v;
      while ((unsigned)(v = coh_load<true>(state)) != (unsigned)(f.sv.k + 1)) __builtin_amdgcn_s_sleep(1);
      s_state = v;
    }
    __syncthreads();
    const unsigned bits = __builtin_amdgcn_readfirstlane((unsigned)(s_state >> 32));
    alpha = __uint_as_float(bits);
    return bits != SQUARE_STOPPED;
  });
}

}  // namespace
}  // namespace prism
