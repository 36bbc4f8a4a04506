// bf16 polar, where the fit is one launch (fit_kernel) and R^2 runs in 128 x 128 tiles: both in one launch, the tiles beside the
// fit.  What bounds it: the fit, 28 us at order 768, under which the 15 us of R^2 disappear.
// One 768 x 3072 matrix, five updates, 381 -> 335 us, 50257 x 768 1055 -> 1012; where the launches are full (16 matrices of order 768 per
// part of a grouped call) equal.
#include "fit_device.h"
#include "gemm_bf16_tile.h"

namespace prism {
namespace {

template <int LD, int RB, int NCH>
__global__ __launch_bounds__(NT, 2) void fit_square_kernel(FitArgs f, Bf16Desc q, int batch) {
  extern __shared__ __align__(1024) unsigned char smem[];
  const int nt = q.M / 128, tiles = nt * (nt + 1) / 2;
  fit_and_tiles<true, LD, RB, NCH>(f, batch, tiles, smem, [&](int b, int rem, auto alpha_of) {
    int tm = 0, left = rem;
    while (left >= nt - tm) { left -= nt - tm; ++tm; }
    gemm_bf16_tile<128, 128, BEPI_POLYQ, true, true, true, 4>(q, b, rem, tiles, tm, tm + left, smem, alpha_of);
  });
}

template <int LD, int RB, int NCH>
int launch_fit_square_t(const FitArgs& f, const Bf16Desc& q, int batch, hipStream_t s) {
  const size_t ring = (size_t)stages_of(128, 128) * (128 + 128) * 64;
  const size_t fit = ((size_t)RB * (LD / 16) * 4 * 256 + (size_t)f.nv * 16 * RB * LD) * sizeof(float);
  const size_t lds = ring > fit ? ring : fit;
  const auto kern = fit_square_kernel<LD, RB, NCH>;
  const int rc = allow_dynamic_lds((const void*)kern, (int)lds);
  if (rc != PRISM_OK) return rc;
  const long long nt = q.M / 128, wgs = (nt * (nt + 1) / 2 + f.sv.rows / (16 * RB)) * batch;
  if (wgs > 0x7fffffff) return PRISM_EUNSUPPORTED;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(NT), lds, s, f, q, batch);
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
}
template <int LD>
int launch_fit_square_ld(const FitArgs& f, const Bf16Desc& q, int batch, hipStream_t s) {
  const int n = f.sv.rows;
  if ((long long)(n / 16) * batch >= 512) return n <= 512 ? launch_fit_square_t<LD, 2, 2>(f, q, batch, s) : launch_fit_square_t<LD, 2, 4>(f, q, batch, s);
  return n <= 512 ? launch_fit_square_t<LD, 1, 2>(f, q, batch, s) : launch_fit_square_t<LD, 1, 4>(f, q, batch, s);
}

}  // namespace

bool fit_square_supported(const FitArgs& f) {
  return f.b16 && f.sv.rows >= 128 && f.sv.rows % 128 == 0 && f.sv.rows <= 1024 && (f.sv.ld == 16 || f.sv.ld == 32);
}

int launch_fit_square(const FitArgs& f, const Bf16Desc& q, int batch, hipStream_t s) {
  if (!fit_square_supported(f) || f.sv.ngroups != f.sv.rows / 16 || f.nv < 2 || f.nv > PRISM_MAX_ROOT + 1 || f.polls < 0 || batch <= 0 || f.ldr % 4) return PRISM_EINVAL;
  if (q.epi != BEPI_POLYQ || !q.sym || q.km != 3 || q.A != q.B || q.M != f.sv.rows || q.N != q.M || q.K != q.M || q.batch != batch || q.lda % 8 || q.ldb % 8 ||
      (!q.C32 && !q.Cin16) || q.ctrl_parts)
    return PRISM_EINVAL;
  return f.sv.ld == 16 ? launch_fit_square_ld<16>(f, q, batch, s) : launch_fit_square_ld<32>(f, q, batch, s);
}

}  // namespace prism
