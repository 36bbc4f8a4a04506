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
//   (Matrices of padded order 64: small.hip.)
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
  solve_body(a, blockIdx.x, a.ngroups == 1 && a.fn != PRISM_FN_SQRT_NEWTON ? coef : nullptr);
}

// ---- chain, moments and solve of one iteration in one launch (fit_device.h) ----
template <bool B16, int LD, int RB, int NCH, int KW>
__global__ __launch_bounds__(64 * KW, !B16 && RB * NCH * LD >= 256 ? 1 : 2) void fit_kernel(FitArgs a) {
  extern __shared__ __align__(16) float fit_lds[];
  const int b = blockIdx.y;
  if (a.sv.ctrl[b].done) return;
  if (!fit_rows<B16, LD, RB, NCH, KW>(a, b, gridDim.y, blockIdx.x, gridDim.x, fit_lds)) return;
  solve_body<true>(a.sv, b);
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

void launch_moments(const SolveArgs& a, int batch, hipStream_t s) {
  hipLaunchKernelGGL(moments_kernel, dim3(a.ngroups, batch), dim3(NT), 0, s, a);
}

void launch_solve(const SolveArgs& a, int batch, hipStream_t s) {
  hipLaunchKernelGGL(solve_kernel, dim3(batch), dim3(NT), 0, s, a);
}

}  // namespace prism
