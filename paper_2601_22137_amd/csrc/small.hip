// Whole calls on matrices of padded order 64 in one workgroup per matrix and one launch: norm, scaling, every iteration and
// the copy-out of the fp32 polar factor (both sides up to 64) and of the coupled inverse Newton iteration (p <= 4).
//
// What bounds them: latency of one workgroup, with many matrices the matrix pipe.  One 64 x 32 polar factor (nine updates) 143 -> 54 us, of which
// norm and copies were three launches of 3 to 7 us each; with six updates 64 x 32 101 -> 44, 64 x 64 103 -> 68, 16384 of 64 x 32 3.40 -> 0.81 ms,
// 16384 of 64 x 64 3.60 -> 2.34.  Inverse fourth roots: one of order 64 172 -> 93 us, 16 of order 48 173 -> 69, 8192 of order 64
// 5.3 -> 2.8 ms, of order 32 4.9 -> 0.67.
//
// NB: 16-row blocks of the order (template): a matrix of order 27 or 32 has no products with the padding.  Products on
// v_mfma_f32_16x16x4_f32 (A operand: lane (lr, lk) = (l % 16, l / 16) holds A[m = lr][k = lk], B operand B[k = lk][n = lr], register r
// of a result D[4 lk + r][lr]).  The k of an instruction are numbered 4 lk + s at step s of a block of 16: the four registers
// of a result block are then the four operands of the next product's steps, and an operand is read from LDS as one
// 16-byte vector along its row.  Between barriers only the LDS has to be complete; global memory is read ahead and
// written at the end.
#include "fit_device.h"

namespace prism {
namespace {

constexpr int SN = 64;
constexpr int SR = SN + 4;        // row stride of an LDS matrix: 16 rows start 4 banks apart, 4 rows 16
constexpr int NCMAX = 9;          // coefficients of m for p = 4

__device__ inline void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// What other lanes of the wave stored to LDS is there (a wave's LDS operations run in order; this keeps the compiler's too)
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
template <int NB> __device__ inline void block_of(int blk, int& i, int& j) {   // number -> block of the upper triangle
  i = 0;
  while (blk >= NB - i) { blk -= NB - i; ++i; }
  j = i + blk;
}
__device__ inline f32x4 mma16(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
  for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], c, 0, 0, 0);
  return c;
}

// State of the stop rule and the report, in LDS until the end
struct Report {
  float residual[PRISM_MAX_ITERS + 1], alpha[PRISM_MAX_ITERS];
  int iters, status, stop;
  float coef;
  float res0, res1, res2;
};
__device__ inline void report_init(Report& rep) {
  const int t = threadIdx.x;
  if (t <= PRISM_MAX_ITERS) rep.residual[t] = -1.0f;
  if (t < PRISM_MAX_ITERS) rep.alpha[t] = 0.0f;
  if (t == 0) { rep.iters = 0; rep.status = PRISM_INFO_BUDGET; rep.stop = 0; rep.coef = 0.0f; rep.res0 = rep.res1 = rep.res2 = 0.0f; }
}
__device__ inline void report_write(const Report& rep, prism_info* info) {
  const int t = threadIdx.x;
  if (t <= PRISM_MAX_ITERS) info->residual[t] = rep.residual[t];
  if (t < PRISM_MAX_ITERS) info->alpha[t] = rep.alpha[t];
  if (t == 0) { info->iters = rep.iters; info->status = rep.status; }
}
// The stop rule of solve_body, by one thread
__device__ inline void stop_test(Report& rep, const SolveArgs& sv, int k, double rho) {
  const double res = sqrt(rho / (double)sv.n);
  rep.residual[k] = (float)res;
  int status = -1;
  if (!(res == res) || res > 1.0e300) status = PRISM_INFO_DIVERGED;
  else if (sv.tol > 0.0 && res <= sv.tol) status = PRISM_INFO_CONVERGED;
  else if (k == sv.max_iters) status = PRISM_INFO_BUDGET;
  else if (sv.tol > 0.0 && k >= 2 && res > (double)rep.res1 && rep.res1 > rep.res2 && res > (double)rep.res0) status = PRISM_INFO_DIVERGED;
  if (status >= 0) { rep.status = status; rep.iters = k; rep.stop = 1; return; }
  if (k == 0) rep.res0 = (float)res;
  rep.res2 = rep.res1;
  rep.res1 = (float)res;
  rep.iters = k + 1;
}

// Chain V_j = R V_{j-1}, j = 1 .. NV, of CB column blocks of 16, and this thread's share of the moments.  R: [16 NB][SR] in LDS.
// Waves own row blocks (NB <= 2: of one column block each, else of all); what a wave hands to the others goes through
// Vb ([NV][CB][NB][64] vectors).  v0: S_k^T in blocks, this wave's part already in registers.
template <int NB, int CB> struct Chain {
  static constexpr int CPW = NB <= 2 ? 1 : CB;              // column blocks of a wave
  f32x4 v0[CPW][NB];
  int rb, c0;
  bool mine;
  __device__ void init(int wave) {
    rb = NB <= 2 ? wave % NB : wave;
    c0 = NB <= 2 ? wave / NB : 0;
    mine = NB <= 2 ? c0 < CB : wave < NB;
  }
  // request column blocks first .. first + CB - 1 of the ncb of S_k^T
  __device__ void request(const float* s, int ncb, int first) {
    if (!mine) return;
#pragma unroll
    for (int c = 0; c < CPW; ++c)
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) v0[c][kb] = *(const f32x4*)(s + ((kb * ncb + first + c0 + c) * 64 + (threadIdx.x & 63)) * 4);
  }
  __device__ void run(const float* Rs, f32x4* Vb, int nv) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    f32x4 ra[NB];
    if (mine) {
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) ra[kb] = *(const f32x4*)&Rs[(16 * rb + lr) * SR + 16 * kb + 4 * lk];
    }
#pragma unroll 1
    for (int j = 0; j < nv; ++j) {
      if (mine) {
        f32x4 acc[CPW];
#pragma unroll
        for (int c = 0; c < CPW; ++c) acc[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < CPW; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[kb][s], v0[c][kb][s], acc[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
          Vb[((j * CB + c0 + c) * NB + rb) * 64 + lane] = acc[c];
          if constexpr (NB == 1) v0[c][0] = acc[c];
        }
      }
      if (NB > 1 || j + 1 == nv) lds_barrier();
      if constexpr (NB > 1) {
        if (mine && j + 1 < nv) {
#pragma unroll
          for (int c = 0; c < CPW; ++c)
#pragma unroll
            for (int kb = 0; kb < NB; ++kb) v0[c][kb] = Vb[((j * CB + c0 + c) * NB + kb) * 64 + lane];
        }
      }
    }
  }
};
// c[s] += the moments of this thread's entries of V_1 .. V_nv (Vb as above)
template <class BL, int NB, int CB> __device__ inline void add_moments(const float* Vb, double* c) {
  constexpr int PER = NB * CB * 256;
#pragma unroll 1
  for (int e = threadIdx.x; e < PER; e += NT) {
    double v[BL::NV], w[BL::NW];
#pragma unroll
    for (int j = 0; j < BL::NV; ++j) v[j] = (double)Vb[j * PER + e];
    BL::make(v, w);
#pragma unroll
    for (int i = 0; i < BL::NW; ++i)
#pragma unroll
      for (int l = 0; l < BL::NW; ++l) c[i + l] += w[i] * w[l];
  }
}
template <class BL> __device__ inline void sum_moments(double* c, double (*out)[NCMAX]) {
  constexpr int NC = 2 * BL::NW - 1;
#pragma unroll
  for (int s = 0; s < NC; ++s) {
    const double x = wave_sum(c[s]);
    if ((threadIdx.x & 63) == 63) out[threadIdx.x >> 6][s] = x;
  }
}
// All column blocks of S_k^T in rounds of CB, then the moments of the four waves
template <class BL, int NB, int CB>
__device__ inline void chain_and_moments(Chain<NB, CB>& ch, const float* Rs, float* Vb, const float* s_k, int ncb, double (*out)[NCMAX]) {
  double c[2 * BL::NW - 1];
#pragma unroll
  for (int s = 0; s < 2 * BL::NW - 1; ++s) c[s] = 0.0;
#pragma unroll 1
  for (int first = 0; first < ncb; first += CB) {
    if (first) { lds_barrier(); ch.request(s_k, ncb, first); }
    ch.run(Rs, (f32x4*)Vb, BL::NV);
    add_moments<BL, NB, CB>(Vb, c);
  }
  sum_moments<BL>(c, out);
}
// Coefficient of iteration k into rep, by wave 0: fitted (moments in `mom`) or as the mode has it
__device__ inline void coefficient(Report& rep, const SolveArgs& sv, int k, bool fitted, int mode, float sched, const double (*mom)[NCMAX],
                                   double* s_c, int nc) {
  const int t = threadIdx.x;
  double lo, hi;
  fit_interval(sv.fn, sv.p, sv.d, lo, hi);
  double best = mode == 3 ? (double)sched : (mode == 1 ? lo : hi);
  if (fitted) {
    if (t < nc) s_c[t] = (mom[0][t] + mom[1][t]) + (mom[2][t] + mom[3][t]);
    wave_lds_sync();
    if (!minimise(s_c, nc, lo, hi, best)) best = lo;
  }
  if (t == 0) rep.coef = (float)best;
}

// ---- fp32 polar factor, both sides up to 64 ----
// Wave w holds rows 16 w .. 16 w + 15 of X in registers, xr[kb][s] = X[16 w + lr][16 kb + 4 lk + s]: operand and result of the
// update, as (X + X Q)^T = X^T + Q X^T.  X^T X is the sum of the waves' own parts (through LDS); R^2 and the stop test
// run on waves 1 to 3 beside the minimiser on wave 0.
// 64 x 32: 4 us per iteration; with full 64 x 64 products, operands read singly and the solve through LDS and barriers 13 (gram 2.4,
// chain 2.7, solve 4.5, R^2 and update 3.3).
template <int NB, int CB>
__global__ __launch_bounds__(NT, 2) void small_polar_kernel(SmallPolarArgs a) {
  constexpr int NBT = NB * (NB + 1) / 2, OWN = (NBT + 3) / 4, SQ = (NBT + 2) / 3;
  constexpr int SLOT = NB == 1 ? 2 : NBT;                   // KiB per wave for its part of X^T X; before, its rows of X
  constexpr int AREA = 4 * SLOT > 5 * CB * NB ? 4 * SLOT : 5 * CB * NB;
  constexpr int SXW = 16 * NB + 4;
  __shared__ __align__(16) float Rs[16 * NB * SR];          // R, later Q
  __shared__ __align__(16) float area[AREA * 256];          // parts of X^T X, then V_1 .. V_nv
  __shared__ double s_part[4], s_mom[4][NCMAX], s_c[NCMAX];
  __shared__ Report rep;
  const SolveArgs& sv = a.sv;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, lr = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = sv.n, mb = (a.L + 15) / 16, ncb = sv.ld / 16;
  float* src = a.x + (long long)b * a.m * a.n;
  auto at = [&](int row, int col) { return a.transpose ? col * a.n + row : row * a.n + col; };   // row < L, col < S of the iterate
  Chain<NB, CB> ch;
  ch.init(wave);
  const float* s_k = a.V0;
  if (a.first_fit == 0 && a.p_s > 0 && sv.max_iters > 0) ch.request(s_k, ncb, 0);

  f32x4 xr[NB];
  double ss = 0.0;
#pragma unroll
  for (int kb = 0; kb < NB; ++kb)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int row = 16 * wave + lr, col = 16 * kb + 4 * lk + s;
      xr[kb][s] = row < a.L && col < n ? src[at(row, col)] : 0.0f;
    }
  report_init(rep);
#pragma unroll
  for (int kb = 0; kb < NB; ++kb)
#pragma unroll
    for (int s = 0; s < 4; ++s) ss += (double)xr[kb][s] * (double)xr[kb][s];
  ss = wave_sum(ss);
  if (lane == 63) s_part[wave] = ss;
  lds_barrier();
  ss = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  const bool finite = (ss == ss) && ss < 1.0e300;
  if (!finite || ss == 0.0) {
    if (t == 0) rep.status = finite ? PRISM_INFO_ZERO : PRISM_INFO_NONFINITE;
    lds_barrier();
    report_write(rep, sv.info + b);
    return;
  }
  const double scale = 1.0 / sqrt(ss);
#pragma unroll
  for (int kb = 0; kb < NB; ++kb)
#pragma unroll
    for (int s = 0; s < 4; ++s) xr[kb][s] = (float)((double)xr[kb][s] * scale);

#pragma unroll 1
  for (int k = 0; k <= sv.max_iters; ++k) {
    if (k == sv.max_iters && sv.tol <= 0.0) break;
    const bool fitted = a.p_s > 0 && k >= a.first_fit && k < sv.max_iters;
    // this wave's part of X^T X, upper triangle of blocks: its rows as operands with k along the rows
    f32x4* slot = (f32x4*)area + wave * SLOT * 64;
    if (wave < mb) {
      float* own = (float*)slot;
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) *(f32x4*)&own[lr * SXW + 16 * kb + 4 * lk] = xr[kb];
      wave_lds_sync();
      f32x4 xa[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int s = 0; s < 4; ++s) xa[i][s] = own[(4 * lk + s) * SXW + 16 * i + lr];
      wave_lds_sync();
      f32x4 g[NBT];
#pragma unroll
      for (int q = 0; q < NBT; ++q) g[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        int q = 0;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = i; j < NB; ++j, ++q) g[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[i][s], xa[j][s], g[q], 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < NBT; ++q) slot[q * 64 + lane] = g[q];
    }
    lds_barrier();
    // R = I - X^T X, zero outside the leading n x n block; rho = ||R||_F^2
    double part = 0.0;
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
      const int blk = wave + 4 * o;
      if (blk < NBT) {
        int i, j;
        block_of<NB>(blk, i, j);
        f32x4 g = ((f32x4*)area)[blk * 64 + lane];
        for (int w = 1; w < mb; ++w) g += ((f32x4*)area)[(w * SLOT + blk) * 64 + lane];
        const int col = 16 * j + lr;
        double p = 0.0;
        f32x4 rv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + 4 * lk + r;
          rv[r] = (row < n && col < n) ? ((row == col ? 1.0f : 0.0f) - g[r]) : 0.0f;
          p += (double)rv[r] * (double)rv[r];
          Rs[row * SR + col] = rv[r];
        }
        if (i != j) { *(f32x4*)&Rs[col * SR + 16 * i + 4 * lk] = rv; p += p; }
        part += p;
      }
    }
    part = wave_sum(part);
    if (lane == 63) s_part[wave] = part;
    lds_barrier();
    if (fitted) {
      if (sv.d == 2) chain_and_moments<Blocks<2>, NB, CB>(ch, Rs, area, s_k, ncb, s_mom);
      else chain_and_moments<Blocks<1>, NB, CB>(ch, Rs, area, s_k, ncb, s_mom);
      s_k += SN * sv.ld;
    }
    if (k + 1 >= a.first_fit && a.p_s > 0 && k + 1 < sv.max_iters) ch.request(s_k, ncb, 0);   // for the next iteration
    lds_barrier();
    f32x4 sq[SQ];
    if (wave == 0) {
      const int mode = k < a.sched_len ? 3 : (a.p_s == 0 ? 1 : (k < a.warm ? 2 : 0));
      if (k < sv.max_iters) coefficient(rep, sv, k, fitted, mode, k < a.sched_len ? a.sched[k] : 0.0f, s_mom, s_c, 5);
    } else {
      if (t == NT - 1) stop_test(rep, sv, k, (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]));
      if (sv.d == 2) {
#pragma unroll
        for (int o = 0; o < SQ; ++o) {
          const int blk = wave - 1 + 3 * o;
          if (blk < NBT) {
            int i, j;
            block_of<NB>(blk, i, j);
            sq[o] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kb = 0; kb < NB; ++kb)
              sq[o] = mma16(*(const f32x4*)&Rs[(16 * i + lr) * SR + 16 * kb + 4 * lk], *(const f32x4*)&Rs[(16 * j + lr) * SR + 16 * kb + 4 * lk], sq[o]);
          }
        }
      }
    }
    lds_barrier();
    if (rep.stop) break;
    const float alpha = rep.coef;
    if (t == 0) rep.alpha[k] = alpha;
    if (sv.d == 2) {   // Q = R / 2 + alpha R^2, in the place of R
      if (wave > 0) {
#pragma unroll
        for (int o = 0; o < SQ; ++o) {
          const int blk = wave - 1 + 3 * o;
          if (blk < NBT) {
            int i, j;
            block_of<NB>(blk, i, j);
            const int col = 16 * j + lr;
            f32x4 q;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float* e = &Rs[(16 * i + 4 * lk + r) * SR + col];
              q[r] = 0.5f * *e + alpha * sq[o][r];
              *e = q[r];
            }
            if (i != j) *(f32x4*)&Rs[col * SR + 16 * i + 4 * lk] = q;
          }
        }
      }
      lds_barrier();
    }
    // X <- X + wa X B, B = Q or R
    const float wa = sv.d == 2 ? 1.0f : alpha;
    if (wave < mb) {
      f32x4 u[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        u[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) u[j] = mma16(*(const f32x4*)&Rs[(16 * j + lr) * SR + 16 * kb + 4 * lk], xr[kb], u[j]);
      }
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) xr[j][r] += wa * u[j][r];
    }
  }
  lds_barrier();
  report_write(rep, sv.info + b);
#pragma unroll
  for (int kb = 0; kb < NB; ++kb)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int row = 16 * wave + lr, col = 16 * kb + 4 * lk + s;
      if (row < a.L && col < n) src[at(row, col)] = xr[kb][s];
    }
}

// ---- coupled inverse Newton iteration (p <= 4), order up to 64 ----
// The launches of the general path (fit, update of X, one or two factor products, M) by one workgroup that keeps X, R, the
// factors E (fp32) and M (fp64) in LDS, all operands and roundings as there.  The first factor product and the stop test run
// on waves 1 to 3 beside the minimiser.  16 matrices of order 48 0.66 ms with launches.
constexpr int RM = SN + 16;         // rows of M: 128 bytes apart modulo 256
template <int NB, int CB, int P>
__global__ __launch_bounds__(NT) void small_root_kernel(SmallRootArgs a) {
  constexpr int N = 16 * NB, NBB = NB * NB, OWN = (NBB + 3) / 4, SQ = (NBB + 2) / 3;
  constexpr int VA = (P + 1) * CB * NB * 256, EA = 2 * N * SR;
  __shared__ __align__(16) double Ms[N * RM];
  __shared__ __align__(16) float Xs[N * SR], Rs[N * SR];
  __shared__ __align__(16) float area[VA > EA ? VA : EA];   // V_1 .. V_nv, then two factors
  __shared__ double s_part[4], s_mom[4][NCMAX], s_c[NCMAX];
  __shared__ Report rep;
  const SolveArgs& sv = a.sv;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, lr = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = sv.n, ncb = sv.ld / 16;
  float* src = a.x + (long long)b * n * n;
  Chain<NB, CB> ch;
  ch.init(wave);
  const float* s_k = a.V0;
  if (a.first_fit == 0 && a.p_s > 0 && sv.max_iters > 0) ch.request(s_k, ncb, 0);

  // c = (2 ||A||_F / (p + 1))^(1/p): X_0 = I / c, M_0 = A / c^p
  float in[N * N / NT];
  double ss = 0.0;
#pragma unroll
  for (int i = 0; i < N * N / NT; ++i) {
    const int e = t + i * NT, r = e / N, c = e % N;
    in[i] = r < n && c < n ? src[r * n + c] : 0.0f;
  }
  report_init(rep);
#pragma unroll
  for (int i = 0; i < N * N / NT; ++i) ss += (double)in[i] * (double)in[i];
  ss = wave_sum(ss);
  if (lane == 63) s_part[wave] = ss;
  lds_barrier();
  ss = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  const bool finite = (ss == ss) && ss < 1.0e300;
  if (!finite || ss == 0.0) {
    if (t == 0) rep.status = finite ? PRISM_INFO_ZERO : PRISM_INFO_NONFINITE;
    lds_barrier();
    report_write(rep, sv.info + b);
    return;
  }
  const double cp = 2.0 * sqrt(ss) / (double)(P + 1), scale = 1.0 / cp;
  const float cinv = (float)pow(cp, -1.0 / (double)P);
  double part = 0.0;
#pragma unroll
  for (int i = 0; i < N * N / NT; ++i) {
    const int e = t + i * NT, r = e / N, c = e % N;
    const bool inside = r < n && c < n;
    const double v = (double)in[i] * scale, res = inside ? (r == c ? 1.0 : 0.0) - v : 0.0;
    Ms[r * RM + c] = v;
    Rs[r * SR + c] = (float)res;
    Xs[r * SR + c] = r == c && inside ? cinv : 0.0f;
    part += res * res;
  }
  lds_barrier();                                            // s_part has been read
  part = wave_sum(part);
  if (lane == 63) s_part[wave] = part;
  lds_barrier();

  // one block (i, j) of A B: rows of A along k, B by its columns
  auto product = [&](const float* A, const float* B, int blk) {
    const int i = blk / NB, j = blk % NB;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) {
      f32x4 bv;
#pragma unroll
      for (int s = 0; s < 4; ++s) bv[s] = B[(16 * kb + 4 * lk + s) * SR + 16 * j + lr];
      acc = mma16(*(const f32x4*)&A[(16 * i + lr) * SR + 16 * kb + 4 * lk], bv, acc);
    }
    return acc;
  };
  auto each = [&](int blk, auto f) {                        // f(offset, r) for the entries that this lane holds of block blk
#pragma unroll
    for (int r = 0; r < 4; ++r) f((16 * (blk / NB) + 4 * lk + r) * SR + 16 * (blk % NB) + lr, r);
  };
  float* E1 = area;
  float* E2 = area + N * SR;
#pragma unroll 1
  for (int k = 0; k <= sv.max_iters; ++k) {
    if (k == sv.max_iters && sv.tol <= 0.0) break;
    const bool fitted = a.p_s > 0 && k >= a.first_fit && k < sv.max_iters;
    if (fitted) {
      chain_and_moments<BlocksInv<P>, NB, CB>(ch, Rs, area, s_k, ncb, s_mom);
      s_k += SN * sv.ld;
    }
    if (k + 1 >= a.first_fit && a.p_s > 0 && k + 1 < sv.max_iters) ch.request(s_k, ncb, 0);   // for the next iteration
    lds_barrier();
    f32x4 sq[SQ];
    if (wave == 0) {
      const int mode = k < a.sched_len ? 3 : (a.p_s == 0 ? 1 : (k < a.warm ? 2 : 0));
      if (k < sv.max_iters) coefficient(rep, sv, k, fitted, mode, k < a.sched_len ? a.sched[k] : 0.0f, s_mom, s_c, 2 * P + 1);
    } else {
      if (t == NT - 1) stop_test(rep, sv, k, (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]));
      if constexpr (P >= 2) {
#pragma unroll
        for (int o = 0; o < SQ; ++o)
          if (wave - 1 + 3 * o < NBB) sq[o] = product(Rs, Rs, wave - 1 + 3 * o);
      }
    }
    lds_barrier();
    if (rep.stop || k == sv.max_iters) break;
    const float alpha = rep.coef;
    if (t == 0) rep.alpha[k] = alpha;
    // E_p: (I + alpha R)^p = I + E_p;  X <- X (I + alpha R)
    if constexpr (P == 1) {
#pragma unroll
      for (int o = 0; o < OWN; ++o)
        if (wave + 4 * o < NBB) each(wave + 4 * o, [&](int off, int) { E1[off] = alpha * Rs[off]; });
    } else if (wave > 0) {
#pragma unroll
      for (int o = 0; o < SQ; ++o)
        if (wave - 1 + 3 * o < NBB)
          each(wave - 1 + 3 * o, [&](int off, int r) { E1[off] = (2.0f * alpha) * Rs[off] + (alpha * alpha) * sq[o][r]; });
    }
    f32x4 xu[OWN];
#pragma unroll
    for (int o = 0; o < OWN; ++o)
      if (wave + 4 * o < NBB) xu[o] = product(Xs, Rs, wave + 4 * o);
    lds_barrier();
    const float* E = E1;
#pragma unroll
    for (int o = 0; o < OWN; ++o)
      if (wave + 4 * o < NBB) {
        each(wave + 4 * o, [&](int off, int r) { Xs[off] += alpha * xu[o][r]; });
        if constexpr (P == 3) {
          const f32x4 v = product(E1, Rs, wave + 4 * o);
          each(wave + 4 * o, [&](int off, int r) { E2[off] = (E1[off] + alpha * v[r]) + alpha * Rs[off]; });
        } else if constexpr (P == 4) {
          const f32x4 v = product(E1, E1, wave + 4 * o);
          each(wave + 4 * o, [&](int off, int r) { E2[off] = 2.0f * E1[off] + v[r]; });
        }
      }
    if constexpr (P >= 3) { E = E2; lds_barrier(); }
    // M <- M + E_p M in fp64, R = I - M
    f64x4 m[OWN];
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
      const int blk = wave + 4 * o, i = blk / NB, j = blk % NB;
      m[o] = f64x4{0.0, 0.0, 0.0, 0.0};
      if (blk < NBB) {
#pragma unroll
        for (int k0 = 0; k0 < N; k0 += 4)
          m[o] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)E[(16 * i + lr) * SR + k0 + lk], Ms[(k0 + lk) * RM + 16 * j + lr], m[o], 0, 0, 0);
      }
    }
    lds_barrier();
    double part = 0.0;
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
      const int blk = wave + 4 * o;
      if (blk < NBB) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {                     // register r of lane (lr, lk): row 4 r + lk, column lr
          const int row = 16 * (blk / NB) + 4 * r + lk, col = 16 * (blk % NB) + lr;
          const bool inside = row < n && col < n;
          const double v = inside ? Ms[row * RM + col] + m[o][r] : 0.0;
          const double res = inside ? ((row == col ? 1.0 : 0.0) - v) : 0.0;
          Ms[row * RM + col] = v;
          Rs[row * SR + col] = (float)res;
          part += res * res;
        }
      }
    }
    part = wave_sum(part);
    if (lane == 63) s_part[wave] = part;
    lds_barrier();
  }
  lds_barrier();
  report_write(rep, sv.info + b);
#pragma unroll
  for (int i = 0; i < N * N / NT; ++i) {
    const int e = t + i * NT, r = e / N, c = e % N;
    if (r < n && c < n) src[r * n + c] = Xs[r * SR + c];
  }
}

}  // namespace

int launch_small_polar(const SmallPolarArgs& a, int batch, hipStream_t s) {
  const SolveArgs& sv = a.sv;
  if (sv.n < 1 || sv.n > SN || a.L < sv.n || a.L > SN || (sv.ld != 16 && sv.ld != 32 && sv.ld != 64) || (sv.d != 1 && sv.d != 2) || batch <= 0) return PRISM_EINVAL;
  const int nb = (sv.n + 15) / 16;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(batch), dim3(NT), 0, s, a);
    return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
  };
  if (sv.ld == 16) return nb == 1 ? go(small_polar_kernel<1, 1>) : (nb == 2 ? go(small_polar_kernel<2, 1>) : (nb == 3 ? go(small_polar_kernel<3, 1>) : go(small_polar_kernel<4, 1>)));
  return nb == 1 ? go(small_polar_kernel<1, 2>) : (nb == 2 ? go(small_polar_kernel<2, 2>) : (nb == 3 ? go(small_polar_kernel<3, 2>) : go(small_polar_kernel<4, 2>)));
}

template <int NB, int CB> static int launch_small_root_t(const SmallRootArgs& a, int batch, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(batch), dim3(NT), 0, s, a);
    return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
  };
  return a.sv.p == 1 ? go(small_root_kernel<NB, CB, 1>) : (a.sv.p == 2 ? go(small_root_kernel<NB, CB, 2>) : (a.sv.p == 3 ? go(small_root_kernel<NB, CB, 3>) : go(small_root_kernel<NB, CB, 4>)));
}
int launch_small_root(const SmallRootArgs& a, int batch, hipStream_t s) {
  const SolveArgs& sv = a.sv;
  if (sv.n < 1 || sv.n > SN || (sv.ld != 16 && sv.ld != 32) || sv.p < 1 || sv.p > 4 || batch <= 0) return PRISM_EINVAL;
  const int nb = (sv.n + 15) / 16;
  if (sv.ld == 16) return nb == 1 ? launch_small_root_t<1, 1>(a, batch, s) : (nb == 2 ? launch_small_root_t<2, 1>(a, batch, s) : (nb == 3 ? launch_small_root_t<3, 1>(a, batch, s) : launch_small_root_t<4, 1>(a, batch, s)));
  return nb == 1 ? launch_small_root_t<1, 2>(a, batch, s) : (nb == 2 ? launch_small_root_t<2, 2>(a, batch, s) : (nb == 3 ? launch_small_root_t<3, 2>(a, batch, s) : launch_small_root_t<4, 2>(a, batch, s)));
}

}  // namespace prism
