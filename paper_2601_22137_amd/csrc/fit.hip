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
#include "fit_device.h"

namespace prism {
namespace {

// grid (groups, batch): partial coefficient sums of one matrix, groups interleaved over the elements
__global__ __launch_bounds__(NT) void moments_kernel(SolveArgs a) {
  const int b = blockIdx.y, grp = blockIdx.x, ngrp = gridDim.x;
  if (a.ctrl[b].done) return;
  accumulate_for(a, b, grp, ngrp, a.cpart + ((long long)b * ngrp + grp) * MAXC);
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

// ---- chain, moments and solve of one iteration in one launch (fit_device.h) ----
template <bool B16, int LD, int RB, int NCH, int KW>
__global__ __launch_bounds__(64 * KW, !B16 && RB * NCH * LD >= 256 ? 1 : 2) void fit_kernel(FitArgs a) {
  extern __shared__ __align__(16) float fit_lds[];
  const int b = blockIdx.y;
  if (a.sv.ctrl[b].done) return;
  if (!fit_rows<B16, LD, RB, NCH, KW>(a, b, gridDim.y, blockIdx.x, gridDim.x, fit_lds)) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the partials of the others
  solve_body(a.sv, b);
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
