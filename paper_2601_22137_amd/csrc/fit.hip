// The per-iteration coefficient fit of PRISM (paper Section 4.2, eq. (4); App. A.1, A.3 and A.4)
// after the sketch chain V_j = R V_{j-1} has been formed:
//   moments_kernel (a few workgroups per matrix) forms the blocks W_i = u_i(R) S^T from the chain
//      (the factor (1 - xi) = G = I - R is applied as V_j - V_{j+1}) and accumulates
//         c_s = sum_{i+l=s} <W_i, W_l>,  m(alpha) = || sum_i alpha^i W_i ||_F^2,
//      in fp64 with a fixed reduction order (results are run-to-run identical);
//   solve_kernel (one workgroup per matrix)
//   1. sums the residual partials, applies the stop rule and records the residual;
//   2. adds up the coefficient partials;
//   3. minimises m over [l, u]: all real roots of m' in the interval are bracketed between the
//      roots of m'' (recursively down to the linear derivative) and found by Newton's method
//      safeguarded by bisection, then m
//      is compared at the end points and those roots; the smallest alpha wins ties.
// Nothing returns to the host: alpha_k, the done flag and the report stay on the device.
//   fit_kernel: chain, moments and solve in one launch, where launches do not fill the chip.
//   small_root_kernel: the whole coupled inverse Newton iteration of a matrix of padded order 64.
//   small_polar_kernel: for fp32 polar factors whose padded iterate is 64 x 64, the whole method
//   (residual, chain, fit, update, for all iterations) in one workgroup per matrix.
#include "common.h"

namespace prism {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;
constexpr int MAXC = 2 * PRISM_MAX_ROOT + 1;  // coefficients of m

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
    double x = c[s];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    if (lane == 0) red[wave][s] = x;
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

// grid (groups, batch): partial coefficient sums of one matrix, groups interleaved over the elements
__global__ __launch_bounds__(NT) void moments_kernel(SolveArgs a) {
  const int b = blockIdx.y, grp = blockIdx.x, ngrp = gridDim.x;
  if (a.ctrl[b].done) return;
  accumulate_for(a, b, grp, ngrp, a.cpart + ((long long)b * ngrp + grp) * MAXC);
}

// The root of f in [xa, xb], f(xa) = fa and f(xb) of opposite signs: Newton's method kept inside the bracket [l, h] (f(l) has
// the sign of fa); a step that would leave the bracket, or that shrinks too slowly, is replaced by a bisection step.
// eval(x, f, df) gives f and its derivative.
template <typename E> __device__ inline double bracketed_root(double xa, double xb, double fa, E eval) {
  double l = xa, h = xb;
  double x = 0.5 * (l + h), dx = h - l, dxold = dx, fx, dfx;
  eval(x, fx, dfx);
  for (int it = 0; it < 200; ++it) {
    if (fx == 0.0) break;
    if ((fx < 0.0) == (fa < 0.0)) l = x; else h = x;
    const bool leaves = !((((x - h) * dfx - fx) * ((x - l) * dfx - fx)) < 0.0);
    const bool slow = fabs(2.0 * fx) > fabs(dxold * dfx);
    dxold = dx;
    double xn;
    if (leaves || slow) { dx = 0.5 * (h - l); xn = l + dx; }
    else { dx = fx / dfx; xn = x - dx; }
    if (xn == x || !(xn > l && xn < h)) break;   // the bracket is down to neighbouring numbers
    x = xn;
    if (fabs(dx) <= 2.0e-16 * fabs(x)) break;
    eval(x, fx, dfx);
  }
  return x;
}

// Minimiser of a quartic on [lo, hi], ties to the smallest: one thread, everything in registers (through LDS, level by
// level of the derivative chain, the same took 2 us more per iteration in barriers and LDS round trips: one 64 x 32 polar
// factor 158 -> 139 us, fp32 polar 6 x 500 x 299 760 -> 735).  The roots of
// m' lie between lo, the roots of m'' (closed form, the larger in magnitude first and the other from their product)
// and hi.
__device__ inline double minimise_quartic(double c0, double c1, double c2, double c3, double c4, double lo, double hi) {
  const double q0 = c1, q1 = 2.0 * c2, q2 = 3.0 * c3, q3 = 4.0 * c4;
  const double b0 = q1, b1 = 2.0 * q2, b2 = 3.0 * q3;
  auto value = [&](double x) { return (((c4 * x + c3) * x + c2) * x + c1) * x + c0; };
  auto slope = [&](double x, double& f, double& df) {
    f = ((q3 * x + q2) * x + q1) * x + q0;
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
  double xa = lo, fa, df;
  slope(lo, fa, df);
  for (int i = 0; i < 3; ++i) {
    const double xb = i == 0 ? e0 : (i == 1 ? e1 : hi);
    double fb;
    slope(xb, fb, df);
    if ((fa < 0.0) != (fb < 0.0)) {
      const double x = fa == 0.0 ? xa : (fb == 0.0 ? xb : bracketed_root(xa, xb, fa, slope));
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

// One workgroup (NT threads or more), matrix b: stop rule and coefficient of iteration a.k.  Every return is taken by all
// threads of the workgroup together.
// rho_local (LDS, one double) stands in for the residual partials in global memory and c_local
// (LDS, MAXC doubles) for the coefficient partials when the caller has them on chip.
// ctl_local (LDS): the matrix's control block, when the caller keeps it on chip; it is not done then.  (Nobody may look: thread 0
// can have set `done` before a late wave gets to the test, and that wave would leave alone.)
__device__ void solve_body(const SolveArgs& a, int b, const double* rho_local = nullptr, double* c_local = nullptr,
                           Ctrl* ctl_local = nullptr) {
  const int t = threadIdx.x;
  Ctrl* ctl = ctl_local ? ctl_local : &a.ctrl[b];
  const int done = ctl_local ? 0 : ctl->done;
  const float res0 = ctl->res0, res1 = ctl->res1, res2 = ctl->res2;   // in the shadow of the first load
  if (done) return;
  prism_info* info = a.info + b;
  __shared__ int s_stop;
  __shared__ double s_c[MAXC];
  __shared__ double s_q[2 * PRISM_MAX_ROOT][MAXC];   // derivative chain of m'
  __shared__ double s_roots[2][MAXC + 2];
  __shared__ int s_nroots[2];

  // residual: sum of the per-tile partials, every thread a strided share, then a fixed tree
  __shared__ double s_rho[4];
  if (!rho_local) {
    double part = 0.0;
    for (int i = t; t < NT && i < a.nparts; i += NT) part += (double)a.rho_part[(long long)b * a.nparts + i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
    if (t < NT && (t & 63) == 0) s_rho[t >> 6] = part;
    __syncthreads();
  }
  if (a.phase == 2) {
    if (t == 0) s_stop = 0;          // coefficient only: the stop test of this k has been taken
  } else if (t == 0) {
    const double rho = rho_local ? *rho_local : (s_rho[0] + s_rho[1]) + (s_rho[2] + s_rho[3]);
    const double res = sqrt(rho / (double)a.n);
    info->residual[a.k] = (float)res;
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
      info->status = status;
      info->iters = a.k;
      s_stop = 1;
    } else {
      if (a.k == 0) ctl->res0 = (float)res;
      ctl->res2 = res1;
      ctl->res1 = (float)res;
      ctl->iters = a.k + 1;     // the update of this iteration is already enqueued behind us
      info->iters = a.k + 1;
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
    if (t == 0) {
      double e2 = 0.0;
      for (int gidx = 0; gidx < a.ngroups; ++gidx) e2 += a.cpart[((long long)b * a.ngroups + gidx) * MAXC + 16];
      if (!(e2 <= 0.01 * (double)a.n)) {
        ctl->status = PRISM_INFO_DIVERGED; ctl->iters = a.k; ctl->done = 1;
        info->status = PRISM_INFO_DIVERGED; info->iters = a.k;
        s_stop = 1;
      }
    }
    __syncthreads();
    if (s_stop) return;
  }

  double lo, hi;
  if (a.fn == PRISM_FN_INV_ROOT) { lo = 1.0 / a.p; hi = 2.0 / a.p; }
  else if (a.fn == PRISM_FN_INVERSE) { lo = 0.5; hi = 2.0; }
  else if (a.fn == PRISM_FN_SQRT_NEWTON) { lo = 0.0; hi = 1.0; }
  else if (a.d == 1) { lo = 0.5; hi = 1.0; }
  else { lo = 0.375; hi = 1.45; }

  if (a.mode != 0) {
    if (t == 0) {
      // without a fit: the Taylor coefficient, which is l except for the Chebyshev inverse (1)
      // (and the DB Newton iteration, whose classical coefficient is 1/2)
      const double taylor = (a.fn == PRISM_FN_INVERSE) ? 1.0 : (a.fn == PRISM_FN_SQRT_NEWTON ? 0.5 : lo);
      const float al = (a.mode == 3) ? a.sched_alpha : (float)((a.mode == 1) ? taylor : hi);
      ctl->alpha = al;
      info->alpha[a.k] = al;
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
      for (int gidx = t / MAXC; gidx < a.ngroups; gidx += SHARES) v += a.cpart[((long long)b * a.ngroups + gidx) * MAXC + t % MAXC];
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
  const int deg = nc - 1;   // degree of m
  const int dq = deg - 1;   // degree of m'
  bool usable = true;
  {
    bool all_tiny = true;
    for (int s = 0; s < nc; ++s) {
      const double v = s_c[s];
      if (!(v == v) || fabs(v) > 1.0e300) usable = false;
      if (fabs(v) >= 1.0e-300) all_tiny = false;
    }
    if (all_tiny) usable = false;
  }
  if (!usable) {
    if (t == 0) { ctl->alpha = (float)lo; info->alpha[a.k] = (float)lo; }
    return;
  }
  if (deg == 4) {   // Newton-Schulz family, DB Newton
    if (t == 0) {
      const double best = minimise_quartic(s_c[0], s_c[1], s_c[2], s_c[3], s_c[4], lo, hi);
      ctl->alpha = (float)best;
      info->alpha[a.k] = (float)best;
      if (best < hi - 1e-6) ctl->plain = 1;   // as below
    }
    return;
  }
  // derivative chain: s_q[j] = (j+1)-th derivative of m, degree deg-1-j
  if (t == 0) {
    for (int i = 0; i <= dq; ++i) s_q[0][i] = (double)(i + 1) * s_c[i + 1];
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
  __syncthreads();
  for (int j = dq - 2; j >= 0; --j) {
    const int src = (j + 1) & 1, dst = j & 1;
    const int nr = s_nroots[src];
    const int pdeg = dq - j;
    double found = 0.0;
    int has = 0;
    if (t <= nr) {  // interval t between consecutive roots of the next derivative
      const double xa = (t == 0) ? lo : s_roots[src][t - 1];
      const double xb = (t == nr) ? hi : s_roots[src][t];
      double fa = horner(s_q[j], pdeg, xa);
      const double fb = horner(s_q[j], pdeg, xb);
      if (fa == 0.0) { found = xa; has = 1; }
      else if (t == nr && fb == 0.0) { found = xb; has = 1; }
      else if ((fa < 0.0) != (fb < 0.0) && fb != 0.0) {
        const double x = bracketed_root(xa, xb, fa, [&](double y, double& f, double& df) {
          f = horner(s_q[j], pdeg, y);
          df = horner(s_q[j + 1], pdeg - 1, y);   // the derivative of level j is level j + 1 of the chain
        });
        found = x;
        has = 1;
      }
    }
    __syncthreads();
    __shared__ double s_tmp[MAXC + 2];
    __shared__ int s_has[MAXC + 2];
    if (t <= nr) { s_tmp[t] = found; s_has[t] = has; }
    __syncthreads();
    if (t == 0) {
      int cnt = 0;
      for (int i = 0; i <= nr; ++i)
        if (s_has[i]) s_roots[dst][cnt++] = s_tmp[i];
      s_nroots[dst] = cnt;
    }
    __syncthreads();
  }
  if (t == 0) {
    const int lvl = (dq >= 2) ? 0 : ((dq - 1) & 1);
    const int nr = s_nroots[lvl & 1];
    double best = lo, bestv = horner(s_c, deg, lo);
    for (int i = 0; i < nr; ++i) {
      const double x = s_roots[lvl & 1][i];
      const double v = horner(s_c, deg, x);
      if (v < bestv) { bestv = v; best = x; }
    }
    const double vh = horner(s_c, deg, hi);
    if (vh < bestv) { bestv = vh; best = hi; }
    ctl->alpha = (float)best;
    info->alpha[a.k] = (float)best;
    // The fit has left the upper end of its interval: no eigenvalue of R is close to 1 any more,
    // i.e. no singular value of the iterate is small.  The bf16 polar path stops carrying the low
    // half of the iterate from here on (it exists for the small singular values only).
    if (best < hi - 1e-6) ctl->plain = 1;
  }
}

__global__ __launch_bounds__(NT) void solve_kernel(SolveArgs a) {
  __shared__ double coef[MAXC];   // small matrices: the moments are accumulated right here
  solve_body(a, blockIdx.x, nullptr, a.ngroups == 1 && a.fn != PRISM_FN_SQRT_NEWTON ? coef : nullptr);
}

// ---- fp32 polar factor, padded iterate 64 x 64: all iterations in one workgroup ----
// The products run on v_mfma_f32_16x16x4_f32 (A operand: lane l holds A[m = l % 16][k = l / 16], B
// operand B[k = l / 16][n = l % 16], result register r of lane l is D[4 (l / 16) + r][l % 16]); each
// of the four waves owns a 32 x 32 quadrant of a 64 x 64 result (2 x 2 blocks), or 16 rows of a chain
// product.  LDS: X [64][SX], R [64][SR], and a third area for the two chain buffers [64][ldv] and
// later Q [64][SR].  R and Q are symmetric, so they are always read with k as the row index; SR = 80 and
// the chain stride ld + 16 put the four k rows of a fragment read into different banks, SX = 68
// does the same for the reads of X along its rows in X Q.
constexpr int SN = 64, SX = 68, SR = 80;
__host__ __device__ inline int small_ldv(int ld) { return ld == 16 ? 16 : ld + 16; }
// the third area holds Q [64][SR] or the two chain buffers [64][ldv], whichever is larger (58 KiB in
// all for 16 sketch columns, so that two workgroups share a CU; 77 KiB for 64 columns)
// (16 sketch columns: V_0 .. V_5 all stay in LDS, 6 x [64][16], and the moments are taken from there)
inline int small_lds_floats(int ld) {
  const int chain = ld == 16 ? 6 * SN * 16 : 2 * SN * small_ldv(ld);
  return SN * SX + SN * SR + (chain > SN * SR ? chain : SN * SR);
}

// acc[i][j] += sum_k A(k, m) B(k, n) over k = 0 .. 63 for the wave's quadrant; A(k, m) sits at
// As[k * sak + m * sam], B(k, n) at Bs[k * ldb + n]
__device__ inline void small_mma(const float* As, int sak, int sam, const float* Bs, int ldb, int wm0, int wn0,
                                 f32x4 (&acc)[2][2]) {
  const int lr = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int k0 = 0; k0 < SN; k0 += 4) {
    float av[2], bv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) av[i] = As[(k0 + lk) * sak + (wm0 + i * 16 + lr) * sam];
#pragma unroll
    for (int j = 0; j < 2; ++j) bv[j] = Bs[(k0 + lk) * ldb + wn0 + j * 16 + lr];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
  }
}

// Vout = R Vin (R symmetric): wave w forms rows 16 w .. 16 w + 15, all LD columns; the result goes to
// the other LDS buffer and, densely ([64][LD]), to global memory for the moments
template <int LD>
__device__ inline void small_chain_step(const float* Rs, const float* Vin, float* Vout, float* Vglobal) {
  constexpr int NB = LD / 16;
  const int ldv = LD == 16 ? 16 : LD + 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
  f32x4 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k0 = 0; k0 < SN; k0 += 4) {
    const float av = Rs[(k0 + lk) * SR + 16 * wave + lr];
#pragma unroll
    for (int j = 0; j < NB; ++j)
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, Vin[(k0 + lk) * ldv + 16 * j + lr], acc[j], 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * wave + 4 * lk + r, col = 16 * j + lr;
      Vout[row * ldv + col] = acc[j][r];
      if (Vglobal) Vglobal[row * LD + col] = acc[j][r];
    }
}

__global__ __launch_bounds__(NT) void small_polar_kernel(SmallPolarArgs a) {
  extern __shared__ float small_lds[];
  float* Xs = small_lds;
  float* Rs = Xs + SN * SX;
  float* Ts = Rs + SN * SR;
  __shared__ double s_part[4];
  __shared__ double s_rho;
  __shared__ double s_coef[MAXC];
  __shared__ Ctrl s_ctl;             // the control block: in memory, every iteration would wait for it several times
  const int b = blockIdx.x, t = threadIdx.x;
  SolveArgs sv = a.sv;
  if (sv.ctrl[b].done) return;   // zero or non-finite input: reported by the prepare step
  if (t == 0) s_ctl = sv.ctrl[b];
  Ctrl* ctl = &s_ctl;
  if (sv.ld == 16) { sv.V = Ts + SN * 16; sv.vstride = SN * 16; sv.bstride = 0; }
  const int lane = t & 63, wave = t >> 6, lr = lane & 15, lk = lane >> 4;
  const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;   // this wave's quadrant of a 64 x 64 result
  {
    const float* Xg = a.X[0] + (long long)b * SN * SN;
    for (int idx = t; idx < SN * SN / 4; idx += NT) {
      const int r = idx >> 4, c = (idx & 15) * 4;
      *(f32x4*)&Xs[r * SX + c] = *(const f32x4*)&Xg[r * SN + c];
    }
  }
  __syncthreads();
  f32x4 acc[2][2];
  for (int k = 0; k <= sv.max_iters; ++k) {
    if (k == sv.max_iters && sv.tol <= 0.0) break;
    // R = I - X^T X, zero outside the leading n x n block; rho = ||R||_F^2
    small_mma(Xs, SX, 1, Xs, SX, wm0, wn0, acc);
    double part = 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wm0 + i * 16 + 4 * lk + r, col = wn0 + j * 16 + lr;
          const float rv = (row < sv.n && col < sv.n) ? ((row == col ? 1.0f : 0.0f) - acc[i][j][r]) : 0.0f;
          Rs[row * SR + col] = rv;
          part += (double)rv * (double)rv;
        }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
    if (lane == 0) s_part[wave] = part;
    __syncthreads();
    if (t == 0) s_rho = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);

    // sketch chain V_j = R V_{j-1}, V_0 = S_k^T; the V_j also go to global memory for the moments
    if (a.p_s > 0 && k >= a.first_fit && k < sv.max_iters) {
      const int ld = sv.ld, ldv = small_ldv(ld);
      const float* v0 = a.V0 + (long long)(k - a.first_fit) * SN * ld;
      for (int idx = t; idx < SN * ld / 4; idx += NT) {
        const int r = (idx * 4) / ld, c = (idx * 4) % ld;
        *(f32x4*)&Ts[r * ldv + c] = *(const f32x4*)&v0[idx * 4];
      }
      __syncthreads();
      // between the products only the LDS copies must be in place; the stores to global memory stay
      // in flight until the full barrier below
      auto lds_barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      };
      if (ld == 16) {   // V_j at Ts + j * 1024: the moments read them from LDS
        for (int j = 1; j <= a.nv; ++j) {
          small_chain_step<16>(Rs, Ts + (j - 1) * SN * 16, Ts + j * SN * 16, nullptr);
          lds_barrier();
        }
      } else {
        float* vin = Ts;
        float* vout = Ts + SN * ldv;
        for (int j = 1; j <= a.nv; ++j) {
          float* vg = const_cast<float*>(a.sv.V) + (long long)(j - 1) * a.sv.vstride + (long long)b * a.sv.bstride;
          if (ld == 32) small_chain_step<32>(Rs, vin, vout, vg);
          else small_chain_step<64>(Rs, vin, vout, vg);
          lds_barrier();
          float* tmp = vin; vin = vout; vout = tmp;
        }
      }
    }
    __threadfence_block();
    __syncthreads();

    sv.k = k;
    sv.mode = k < a.sched_len ? 3 : (a.p_s == 0 ? 1 : (k < a.warm ? 2 : 0));
    sv.sched_alpha = k < a.sched_len ? a.sched[k] : 0.0f;
    solve_body(sv, b, &s_rho, s_coef, ctl);
    __syncthreads();
    if (ctl->done) break;
    const float alpha = ctl->alpha;

    const float* Bm = Rs;
    float wa = alpha;
    if (sv.d == 2) {   // Q = R / 2 + alpha R^2
      small_mma(Rs, SR, 1, Rs, SR, wm0, wn0, acc);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = wm0 + i * 16 + 4 * lk + r, col = wn0 + j * 16 + lr;
            Ts[row * SR + col] = 0.5f * Rs[row * SR + col] + alpha * acc[i][j][r];
          }
      __syncthreads();
      Bm = Ts;
      wa = 1.0f;
    }
    // X <- X + wa X B: every wave reads whole rows of X, so all reads end before the first store
    small_mma(Xs, 1, SX, Bm, SR, wm0, wn0, acc);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wm0 + i * 16 + 4 * lk + r, col = wn0 + j * 16 + lr;
          Xs[row * SX + col] += wa * acc[i][j][r];
        }
    __syncthreads();
  }
  {
    if (t == 0) sv.ctrl[b] = s_ctl;
    float* Xg = a.X[ctl->iters & 1] + (long long)b * SN * SN;
    for (int idx = t; idx < SN * SN / 4; idx += NT) {
      const int r = idx >> 4, c = (idx & 15) * 4;
      *(f32x4*)&Xg[r * SN + c] = *(const f32x4*)&Xs[r * SX + c];
    }
  }
}

// ---- coupled inverse Newton iteration (p <= 4), padded order 64: all iterations in one workgroup ----
// The launches of the general path (fit, update of X, one or two factor products, M) by one workgroup per matrix that
// keeps X, R, the factors E (fp32) and M (fp64) in LDS, all operands and roundings as there.  Products on
// v_mfma_f32_16x16x4_f32 / v_mfma_f64_16x16x4_f64, one 32 x 32 quadrant per wave.
// What bounds it: latency of one workgroup (22 us per iteration at p = 4: chain, serial solve, four products of 64^3).  The general path took five launches for each of the budgeted iterations; a call on several such
// groups was bound by the host's launch rate: mixed small inverse roots (8 groups, 5 of them here) 5.4 -> 3.5 ms,
// one batch of 16 matrices of order 48 0.66 -> 0.21.
constexpr int RL = SN + 4;          // rows of X, R, E: 16 consecutive rows fall on different banks
constexpr int RM = SN + 16;         // rows of M: 128 bytes apart modulo 256
inline int small_root_lds_bytes(int ld, int nv) {
  const int chain = (nv + 1) * SN * ld, fac = 2 * SN * RL;
  return (2 * SN * RL + (chain > fac ? chain : fac)) * 4 + SN * RM * 8;
}
__global__ __launch_bounds__(NT) void small_root_kernel(SmallRootArgs a) {
  extern __shared__ __align__(16) float small_lds[];
  double* Ms = (double*)small_lds;                      // [64][RM]
  float* Xs = (float*)(Ms + SN * RM);
  float* Rs = Xs + SN * RL;
  float* Ts = Rs + SN * RL;                             // V_0 .. V_nv [64][ld] each, later two factors [64][RL]
  __shared__ double s_part[4];
  __shared__ double s_rho;
  __shared__ double s_coef[MAXC];
  __shared__ Ctrl s_ctl;             // the control block: in memory, every iteration would wait for it several times
  const int b = blockIdx.x, t = threadIdx.x;
  SolveArgs sv = a.sv;
  if (sv.ctrl[b].done) return;   // zero or non-finite input: reported by the prepare step
  if (t == 0) s_ctl = sv.ctrl[b];
  Ctrl* ctl = &s_ctl;
  const int lane = t & 63, wave = t >> 6, lr = lane & 15, lk = lane >> 4, ld = sv.ld;
  const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
  sv.V = Ts + SN * ld; sv.vstride = SN * ld; sv.bstride = 0;
  for (int idx = t; idx < SN * SN / 4; idx += NT) {
    const int r = idx >> 4, c = (idx & 15) * 4;
    const long long o = (long long)b * SN * SN + r * SN + c;
    *(f32x4*)&Xs[r * RL + c] = *(const f32x4*)(a.X[0] + o);
    *(f32x4*)&Rs[r * RL + c] = *(const f32x4*)(a.R + o);
#pragma unroll
    for (int e = 0; e < 4; ++e) Ms[r * RM + c + e] = a.M[o + e];
  }
  if (t == 0) s_rho = (double)sv.rho_part[b];           // residual of M_0, from the prepare step
  __syncthreads();
  f32x4 acc[2][2];
  for (int k = 0; k <= sv.max_iters; ++k) {
    if (k == sv.max_iters && sv.tol <= 0.0) break;
    if (a.p_s > 0 && k >= a.first_fit && k < sv.max_iters) {   // sketch chain V_j = R V_{j-1}
      const float* v0 = a.V0 + (long long)(k - a.first_fit) * SN * ld;
      for (int idx = t; idx < SN * ld / 4; idx += NT) *(f32x4*)&Ts[idx * 4] = *(const f32x4*)&v0[idx * 4];
      __syncthreads();
      for (int j = 1; j <= a.nv; ++j) {
        const float* vin = Ts + (j - 1) * SN * ld;
        float* vout = Ts + j * SN * ld;
        for (int c0 = 0; c0 < ld; c0 += 16) {             // wave w: rows 16 w .. 16 w + 15
          f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int k0 = 0; k0 < SN; k0 += 4)
            v = __builtin_amdgcn_mfma_f32_16x16x4f32(Rs[(16 * wave + lr) * RL + k0 + lk], vin[(k0 + lk) * ld + c0 + lr], v, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r) vout[(16 * wave + 4 * lk + r) * ld + c0 + lr] = v[r];
        }
        __syncthreads();
      }
    }
    sv.k = k;
    sv.mode = k < a.sched_len ? 3 : (a.p_s == 0 ? 1 : (k < a.warm ? 2 : 0));
    sv.sched_alpha = k < a.sched_len ? a.sched[k] : 0.0f;
    solve_body(sv, b, &s_rho, s_coef, ctl);
    __syncthreads();
    if (ctl->done || k == sv.max_iters) break;
    const float alpha = ctl->alpha;
    float* E1 = Ts;
    float* E2 = Ts + SN * RL;
    // dst = w1 * C1 + w2 * C2 + wa * A B for this wave's quadrant (C2 may be null)
    auto product = [&](const float* A, const float* B, float wa, const float* C1, float w1, const float* C2, float w2, float* dst) {
      small_mma(A, 1, RL, B, RL, wm0, wn0, acc);
      if (dst == A || dst == B) __syncthreads();          // in place: all reads end first
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int o = (wm0 + i * 16 + 4 * lk + r) * RL + wn0 + j * 16 + lr;
            float v = w1 * C1[o] + wa * acc[i][j][r];
            if (C2) v += w2 * C2[o];
            dst[o] = v;
          }
    };
    const float* E;                                       // E_p: (I + alpha R)^p = I + E_p
    if (sv.p == 1) {
      for (int idx = t; idx < SN * SN; idx += NT) { const int o = (idx >> 6) * RL + (idx & 63); E1[o] = alpha * Rs[o]; }
      E = E1;
    } else {
      product(Rs, Rs, alpha * alpha, Rs, 2.0f * alpha, nullptr, 0.0f, E1);
      E = E1;
      if (sv.p == 3) {
        __syncthreads();
        product(E1, Rs, alpha, E1, 1.0f, Rs, alpha, E2);
        E = E2;
      } else if (sv.p == 4) {
        __syncthreads();
        product(E1, E1, 1.0f, E1, 2.0f, nullptr, 0.0f, E2);
        E = E2;
      }
    }
    product(Xs, Rs, alpha, Xs, 1.0f, nullptr, 0.0f, Xs);  // X <- X (I + alpha R)
    __syncthreads();
    // M <- M + E_p M in fp64, R = I - M
    f64x4 m[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) m[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k0 = 0; k0 < SN; k0 += 4) {
      double av[2], bv[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) av[i] = (double)E[(wm0 + i * 16 + lr) * RL + k0 + lk];
#pragma unroll
      for (int j = 0; j < 2; ++j) bv[j] = Ms[(k0 + lk) * RM + wn0 + j * 16 + lr];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) m[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv[j], m[i][j], 0, 0, 0);
    }
    __syncthreads();
    double part = 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {                     // register r of lane (lr, lk): row 4 r + lk, column lr
          const int row = wm0 + i * 16 + 4 * r + lk, col = wn0 + j * 16 + lr;
          const bool in = row < sv.n && col < sv.n;
          const double v = in ? Ms[row * RM + col] + m[i][j][r] : 0.0;
          const double res = in ? ((row == col ? 1.0 : 0.0) - v) : 0.0;
          Ms[row * RM + col] = v;
          Rs[row * RL + col] = (float)res;
          part += res * res;
        }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
    if (lane == 0) s_part[wave] = part;
    __syncthreads();
    if (t == 0) s_rho = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
    __syncthreads();
  }
  if (t == 0) sv.ctrl[b] = s_ctl;
  float* Xg = a.X[ctl->iters & 1] + (long long)b * SN * SN;
  for (int idx = t; idx < SN * SN / 4; idx += NT) {
    const int r = idx >> 4, c = (idx & 15) * 4;
    *(f32x4*)&Xg[r * SN + c] = *(const f32x4*)&Xs[r * RL + c];
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
typedef unsigned long long u64;
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
  for (int s = 0; s < NC; ++s) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c[s] += __shfl_down(c[s], off, 64);
  }
  if (lane == 0) {
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

// KW waves, each with every KW-th chunk of 64 k, NCH chunks at most (n <= 64 KW NCH)
template <bool B16, int LD, int RB, int NCH, int KW>
__global__ __launch_bounds__(64 * KW, !B16 && RB * NCH * LD >= 256 ? 1 : 2) void fit_kernel(FitArgs a) {
  constexpr int NBLK = LD / 16, NQ = RB * NBLK, ROWS = 16 * RB;
  constexpr int NACC = NBLK == 1 ? 4 : (NBLK == 2 && KW == 4 ? 2 : 1);   // independent accumulators (the same for every RB)
  constexpr int CG = NBLK == 1 && RB == 1 ? 2 : 1;            // chunks whose operands are requested together
  extern __shared__ __align__(16) float fit_lds[];
  f32x4 (*red)[NQ][64] = (f32x4 (*)[NQ][64])fit_lds;          // [KW] partial sums
  float* own = fit_lds + KW * NQ * 256;                       // [nv][ROWS][LD]: this workgroup's rows of V_1 .. V_nv
  __shared__ float dfix[ROWS];
  __shared__ int s_next;
  const SolveArgs& sv = a.sv;
  const int b = blockIdx.y, G = gridDim.x, n = sv.rows, mine = blockIdx.x;
  if (sv.ctrl[b].done) return;
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
    const float* Vin = j == 1 ? a.V0 : a.V + ((long long)(j - 2) * gridDim.y + b) * n * LD;        // V_{j-1}
    float* Vout = a.V + ((long long)(j - 1) * gridDim.y + b) * n * LD;
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
  if (!s_next) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the partials of the others
  solve_body(sv, b);
}

template <bool B16, int LD, int RB, int NCH, int KW>
int launch_fit_t(const FitArgs& a, int batch, hipStream_t s) {
  const int rows = 16 * RB;
  if (a.sv.rows % rows || a.sv.rows / rows > FIT_MAX_CLUSTER || a.sv.rows > 64 * KW * NCH) return PRISM_EINVAL;
  const size_t lds = ((size_t)RB * (LD / 16) * KW * 256 + (size_t)a.nv * rows * LD) * sizeof(float);
  const auto kern = fit_kernel<B16, LD, RB, NCH, KW>;
  if (lds > 48 * 1024) {
    const int rc = allow_dynamic_lds((const void*)kern, (int)lds);
    if (rc != PRISM_OK) return rc;
  }
  hipLaunchKernelGGL(kern, dim3(a.sv.rows / rows, batch), dim3(64 * KW), lds, s, a);
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
}
// Rows per workgroup: 16 while those are at most two workgroups per CU, then 32 (two row blocks share the operands of
// V): 16 x 768 (bf16 R, 768 blocks) 72 / 55 us with 16 / 32 rows, 16 x 1024 (1024 blocks) 137 / 76, 4 x 1024 (256) 43 / 52,
// 1 x 768 (48) 31 / 38.  Order 64: one workgroup has all rows and hands nothing over.
template <bool B16, int LD>
int launch_fit_ld(const FitArgs& a, int batch, hipStream_t s) {
  const int n = a.sv.rows;
  const long long blocks = (long long)(n / 16) * batch;
  if constexpr (LD == 64) {
    return n <= 512 ? launch_fit_t<B16, LD, 1, 2, 4>(a, batch, s) : launch_fit_t<B16, LD, 1, 4, 4>(a, batch, s);
  } else {
    if (n > 1024) return launch_fit_t<B16, LD, 2, 4, 8>(a, batch, s);
    if (n == 64) return launch_fit_t<B16, LD, 4, 1, 4>(a, batch, s);
    if (blocks >= 512) return n <= 512 ? launch_fit_t<B16, LD, 2, 2, 4>(a, batch, s) : launch_fit_t<B16, LD, 2, 4, 4>(a, batch, s);
    return n <= 512 ? launch_fit_t<B16, LD, 1, 2, 4>(a, batch, s) : launch_fit_t<B16, LD, 1, 4, 4>(a, batch, s);
  }
}

}  // namespace

// Where the launches are short the fit in one launch is ahead of chain kernels, moments and solve; where they are full its
// workgroups, which sit through hand-overs and solve, are behind.  The line is drawn by 64-row blocks of the caller's
// batch.  Time of a call (sign, inverse root, bf16 polar, four or five updates) without / with the fused fit at orders
// 128, 256, 512, 1024:
//   sketch 64        128 blocks 1.18-1.27, 1.21-1.38, 1.14-1.43, 1.11-1.42;  256 blocks 0.85-0.88, 0.96-1.00, 0.94-0.98, 0.96-1.00
//   sketch 16, fp32  256 blocks 1.00-1.11, 1.01-1.04, 1.07, 1.05;  512 blocks 0.86-0.95, 0.96-0.99, 1.03-1.05, 1.01-1.03
//   sketch 16, bf16  256 blocks 1.10, 1.14, 1.18, 1.16;  512 blocks 0.93, 0.93, 0.98-1.14, 1.00; 1024 blocks 0.88, 0.98, 1.03, 0.93
//   sketch 32, fp32  256 blocks 0.97-1.06, 1.10, 1.07, 1.05;  512 blocks 0.87-0.98, 1.00, 1.03, 1.01
//   sketch 32, bf16  256 blocks 1.00, 1.29, 1.16, 1.08;  512 blocks 0.90, 1.01, 0.96, 0.94
// Above order 1024 the workgroups (32 rows, one per CU with bf16 R) have to fit the chip at a time; the streaming
// kernels also leave more of the chip to the products of the other half.  bf16 polar, eight
// updates, ms fused / streaming: 1 x 2048 1.30 / 1.41, 4 x 2048 (256 workgroups) 2.20 / 2.33, 6 x 1536 (288) 1.82 / 1.70,
// 7 x 1300 (280) 2.48 / 2.29; in halves 8 x 1536 (192 each) 2.11 / 2.25, 12 x 1300 (240) 3.25 / 3.07,
// 8 x 2048 (256) 3.52 / 3.73 with a sketch of 16 and 3.92 / 3.82 with 32, 16 x 1536 (384) 3.83 / 3.56.  fp32, where the
// products weigh more: sign 4 x 2048 6.12 / 6.25, 6 x 1536 4.25 / 4.30, 8 x 2048 12.05 / 12.20, 16 x 1536 11.28 / 11.07.
bool fit_fused_supported(int rows, int ld, int batch, bool b16, bool halves) {
  if (rows % 64) return false;
  const long long blocks = (long long)(rows / 64) * batch;
  if (rows <= 1024) {
    if (ld == 64) return blocks <= 128;
    if (rows <= 192) return blocks <= 256;
    if (rows <= 320) return blocks <= 384;
    if (b16 && rows > 512) return blocks <= 256;
    return ld == 16 || blocks <= 512;
  }
  const long long wgs = 2 * (halves ? blocks / 2 : blocks);
  return rows <= 2048 && ld <= 32 && wgs <= (b16 ? (halves ? 192 : 256) : 384);
}

int launch_fit(const FitArgs& a, int batch, hipStream_t s) {
  if (a.sv.rows % 64 || a.sv.rows > (a.sv.ld <= 32 ? 2048 : 1024) || a.sv.ngroups != a.sv.rows / 16 || a.nv < 2 || a.nv > PRISM_MAX_ROOT + 1 || a.polls < 0 ||
      batch <= 0 || a.ldr % 4 || (a.b16 && a.sv.ld > 32))
    return PRISM_EINVAL;
  if (a.b16) return a.sv.ld == 16 ? launch_fit_ld<true, 16>(a, batch, s) : launch_fit_ld<true, 32>(a, batch, s);
  if (a.sv.ld == 16) return launch_fit_ld<false, 16>(a, batch, s);
  if (a.sv.ld == 32) return launch_fit_ld<false, 32>(a, batch, s);
  return launch_fit_ld<false, 64>(a, batch, s);
}

int launch_small_polar(const SmallPolarArgs& a, int batch, hipStream_t s) {
  if (a.sv.rows != SN || (a.sv.ld != 16 && a.sv.ld != 32 && a.sv.ld != 64) || a.sv.ngroups != 1 || a.sv.nparts != 1 ||
      a.nv < 1 || a.nv > 5 || batch <= 0)
    return PRISM_EINVAL;
  const size_t lds = (size_t)small_lds_floats(a.sv.ld) * sizeof(float);
  const int rc = allow_dynamic_lds((const void*)small_polar_kernel, (int)(small_lds_floats(64) * sizeof(float)));
  if (rc != PRISM_OK) return rc;
  hipLaunchKernelGGL(small_polar_kernel, dim3(batch), dim3(NT), lds, s, a);
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
}

int launch_small_root(const SmallRootArgs& a, int batch, hipStream_t s) {
  if (a.sv.rows != SN || (a.sv.ld != 16 && a.sv.ld != 32) || a.sv.p < 1 || a.sv.p > 4 || a.nv != a.sv.p + 1 || batch <= 0) return PRISM_EINVAL;
  const int lds = small_root_lds_bytes(a.sv.ld, a.nv);
  const int rc = allow_dynamic_lds((const void*)small_root_kernel, lds);
  if (rc != PRISM_OK) return rc;
  hipLaunchKernelGGL(small_root_kernel, dim3(batch), dim3(NT), lds, s, a);
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
}

void launch_moments(const SolveArgs& a, int batch, hipStream_t s) {
  hipLaunchKernelGGL(moments_kernel, dim3(a.ngroups, batch), dim3(NT), 0, s, a);
}

void launch_solve(const SolveArgs& a, int batch, hipStream_t s) {
  hipLaunchKernelGGL(solve_kernel, dim3(batch), dim3(NT), 0, s, a);
}

}  // namespace prism
