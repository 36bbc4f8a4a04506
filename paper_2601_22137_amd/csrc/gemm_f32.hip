// fp32 / fp64 GEMMs on the CDNA4 matrix cores (v_mfma_f32_16x16x4_f32, v_mfma_f64_16x16x4_f64)
// with the epilogues of the PRISM iterations fused in (Table 1 of the paper: residual
// R = I - G, polynomial Q = R/2 + alpha R^2, update X + X Q, inverse-Newton factors).
// The tile itself is in gemm_f32_tile.h.
#include <cstdlib>
#include <initializer_list>

#include "gemm_f32_tile.h"

namespace prism {
namespace {

// ST: slabs in the ring.  Two workgroups per CU with 128 x 128 tiles (register bound), more with small ones.
// PAIR: two products in a launch (a variant of its own: choosing the descriptor costs every launch 1 to 2 us).
template <bool PAIR> struct GemmArg { typedef GemmDesc type; };
template <> struct GemmArg<true> { typedef GemmPair type; };
// WIDE: offsets within the tile of an operand beyond 32 bits (a variant of its own: they cost registers in the loop).
template <typename TC, typename TB, int TM, int TN, int WGM, int WGN, int ST, int EPI, bool A_KM, bool SYM, bool PAIR, bool WIDE>
__global__ __launch_bounds__(GEMM_NT, (TM * TN >= 128 * 128 ? 2 : 3)) void gemm_kernel(typename GemmArg<PAIR>::type arg) {
  int wg0 = 0, which = 0;
  if constexpr (PAIR) {
    which = (int)blockIdx.x >= arg.first;   // uniform
    wg0 = which ? arg.first : 0;
  }
  const GemmDesc& g = [&]() -> const GemmDesc& { if constexpr (PAIR) return arg.d[which]; else return arg; }();
  static_assert(WGM * WGN == 4, "four wavefronts");
  extern __shared__ __align__(1024) unsigned char smem[];

  // sym (square fp32 products whose exact result is symmetric): only the tiles on and above the
  // diagonal are computed; every off-diagonal tile is also stored mirrored.  Of a pair, the first alone may be (PAIR
  // without SYM).
  const bool sym = SYM || (PAIR && g.sym);
  const int tiles_m = g.M / TM, tiles_n = g.N / TN;
  const int per_mat = sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int total = per_mat * g.batch;
  int wg = (int)blockIdx.x - wg0;
  if ((total & 7) == 0) wg = (wg & 7) * (total >> 3) + (wg >> 3);  // one XCD = one contiguous tile range
  const int b = wg / per_mat;
  const int rem = wg - b * per_mat;
  int tm, tn;
  if (sym) {
    int left = rem;
    tm = 0;
    while (left >= tiles_m - tm) { left -= tiles_m - tm; ++tm; }
    tn = tm + left;
  } else if (g.tile_blocks) {
    // blocks of 8 x 8 tiles in sequence: the 64 tiles an XCD works on at a time (32 CUs, two workgroups
    // each) share 8 row panels and 8 column panels; row by row they are one row panel and 64 column panels
    const int blk = rem >> 6, w = rem & 63, nbn = tiles_n >> 3;
    tm = (blk / nbn) * 8 + (w >> 3);
    tn = (blk % nbn) * 8 + (w & 7);
  } else {
    tm = rem / tiles_n;
    tn = rem - tm * tiles_n;
  }
  const int cb = g.ctrl_parts ? b / g.ctrl_parts : b;   // split-K launches: the batch entries are parts of matrices
  if (g.ctrl && g.ctrl[cb].done) return;
  // block Gauss-Jordan: the pivot row / column block has launches of its own
  if ((tm * TM >= g.skip_m0 && tm * TM < g.skip_m1) || (tn * TN >= g.skip_n0 && tn * TN < g.skip_n1)) return;
  const float alpha = g.ctrl ? g.ctrl[cb].alpha : 1.0f;

  gemm_tile<TC, TB, TM, TN, WGM, WGN, ST, EPI, A_KM, SYM, WIDE, false>(g, sym, b, rem, per_mat, tm, tn, smem, [&](float& out) { out = alpha; return true; });
}

// One product, or two of the same shape and kind (GemmPair::d[1].batch > 0)
template <typename TC, typename TB, int TM, int TN, int WGM, int WGN, int EPI, bool A_KM, bool SYM>
int launch_one(const GemmPair& g, int total, hipStream_t s) {   // total: workgroups of the launch
  constexpr int ST = 4;
  const size_t lds = (size_t)ST * (TM * 64 + KMajor<TB, TN>::BYTES);
  auto launch = [&](auto kern, int wgs, const auto& arg) -> int {
    if (lds > 32 * 1024) {
      const int rc = allow_dynamic_lds((const void*)kern, (int)lds);
      if (rc != PRISM_OK) return rc;
    }
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(GEMM_NT), lds, s, arg);
    return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
  };
  const GemmDesc& d = g.d[0];
  const unsigned long long span_a = A_KM ? 16ull * d.lda + TM : (unsigned long long)TM * d.lda, span_b = 16ull * d.ldb + TN;
  const bool wide = span_a * 4 > 0xffffffffull || span_b * sizeof(TB) > 0xffffffffull;
  if (wide) {   // plain products only: the operands of the iterations are far smaller
    if constexpr (EPI == EPI_STORE)
      if (g.d[1].batch == 0) return launch(gemm_kernel<TC, TB, TM, TN, WGM, WGN, ST, EPI, A_KM, SYM, false, true>, total, d);
    return PRISM_EINVAL;
  }
  if (g.d[1].batch == 0) return launch(gemm_kernel<TC, TB, TM, TN, WGM, WGN, ST, EPI, A_KM, SYM, false, false>, total, d);
  if constexpr (sizeof(TC) == 4 && EPI == EPI_AXPY && !A_KM)
    return launch(gemm_kernel<TC, TB, TM, TN, WGM, WGN, ST, EPI, A_KM, SYM, true, false>, total, g);
  return PRISM_EINVAL;
}

template <typename TC, typename TB, int TM, int TN, int WGM, int WGN, int EPI>
int launch_epi(const GemmPair& g, int total, hipStream_t s) {
  if constexpr (sizeof(TC) == 8) {
    return launch_one<TC, TB, TM, TN, WGM, WGN, EPI, false, false>(g, total, s);
  } else {
    if constexpr (TM == TN) {
      if (g.d[0].sym && (g.d[1].batch == 0 || g.d[1].sym)) {
        return g.d[0].a_km ? launch_one<TC, TB, TM, TN, WGM, WGN, EPI, true, true>(g, total, s)
                      : launch_one<TC, TB, TM, TN, WGM, WGN, EPI, false, true>(g, total, s);
      }
    }
    return g.d[0].a_km ? launch_one<TC, TB, TM, TN, WGM, WGN, EPI, true, false>(g, total, s)
                  : launch_one<TC, TB, TM, TN, WGM, WGN, EPI, false, false>(g, total, s);
  }
}

template <typename TC, typename TB, int TM, int TN, int WGM, int WGN>
int launch_cfg(const GemmDesc& g, hipStream_t s, const GemmDesc* g2 = nullptr) {
  for (const GemmDesc* q : {&g, g2}) {
    if (!q) continue;
    if (q->M % TM || q->N % TN || q->K % BK || q->K < BK || q->lda % 4 || q->ldb % 4 || q->ldc % 4) return PRISM_EINVAL;
    if ((q->epi == EPI_POLYQ || q->epi == EPI_AXPY || q->epi == EPI_MNEXT) && (!q->Cin || q->ldcin % 4)) return PRISM_EINVAL;
  }
  if (g2 && (g2->M != g.M || g2->N != g.N || g2->batch != g.batch || g2->epi != g.epi || g2->a_km != g.a_km || (g2->sym && !g.sym))) return PRISM_EINVAL;
  const int tm = g.M / TM, tn = g.N / TN;
  GemmPair gb = {};
  gb.d[0] = g;
  if (g2) gb.d[1] = *g2;
  long long total = 0;
  static const int no_blocks = ab_switch("PRISM_F32_NO_TILE_BLOCKS");
  for (GemmDesc& d : gb.d) {
    if (d.batch == 0) continue;
    gb.first = (int)total;             // where the last one begins
    if (d.sym) {
      if (TM != TN || sizeof(TC) == 8 || d.M != d.N) return PRISM_EINVAL;
      total += (long long)tm * (tm + 1) / 2 * d.batch;
    } else {
      d.tile_blocks = !no_blocks && tm % 8 == 0 && tn % 8 == 0 && tm * tn > 64;
      total += (long long)tm * tn * d.batch;
    }
    if (total > 0x3fffffff) return PRISM_EINVAL;
  }
  if (total <= 0) return PRISM_EINVAL;
  if constexpr (sizeof(TC) == 8) {
    if (g.epi == EPI_STORE) return launch_epi<TC, TB, TM, TN, WGM, WGN, EPI_STORE>(gb, (int)total, s);
    if (g.epi == EPI_MNEXT) return launch_epi<TC, TB, TM, TN, WGM, WGN, EPI_MNEXT>(gb, (int)total, s);
  } else {
    if (g.epi == EPI_STORE) return launch_epi<TC, TB, TM, TN, WGM, WGN, EPI_STORE>(gb, (int)total, s);
    if constexpr (TM == TN) {
      if (g.epi == EPI_RESIDUAL) return launch_epi<TC, TB, TM, TN, WGM, WGN, EPI_RESIDUAL>(gb, (int)total, s);
      if (g.epi == EPI_POLYQ) return launch_epi<TC, TB, TM, TN, WGM, WGN, EPI_POLYQ>(gb, (int)total, s);
      if (g.epi == EPI_AXPY) return launch_epi<TC, TB, TM, TN, WGM, WGN, EPI_AXPY>(gb, (int)total, s);
    }
  }
  return PRISM_EINVAL;
}

}  // namespace

int launch_gemm_f32(const GemmDesc& g, int tile_m, int tile_n, hipStream_t s) {
  if (tile_m == 128 && tile_n == 128) return launch_cfg<float, float, 128, 128, 2, 2>(g, s);
  if (tile_m == 64 && tile_n == 64) return launch_cfg<float, float, 64, 64, 2, 2>(g, s);
  if (tile_m == 128 && tile_n == 64) return launch_cfg<float, float, 128, 64, 4, 1>(g, s);
  if (tile_m == 128 && tile_n == 32) return launch_cfg<float, float, 128, 32, 4, 1>(g, s);
  if (tile_m == 128 && tile_n == 16) return launch_cfg<float, float, 128, 16, 4, 1>(g, s);
  if (tile_m == 64 && tile_n == 32) return launch_cfg<float, float, 64, 32, 4, 1>(g, s);
  if (tile_m == 64 && tile_n == 16) return launch_cfg<float, float, 64, 16, 4, 1>(g, s);
  return PRISM_EINVAL;
}

// Square tile of a product: 128 x 128 tiles move half the bytes per flop, but a CU holds two of them at a
// time, so a launch runs in rounds of 512; 64 x 64 ones (four to five per CU) fill the chip from 256
// tiles on and lose little in the last round.  Measured, TFLOP/s with 128 / 64: 8192^3 147 / 143,
// 16 x 1024^3 (1024 large tiles) 138 / 135, 8 x 1024^3 (512) 133 / 133, 32 x 512^3 (512) 122 / 127, 1024^3
// (64) 33 / 99, 4 x 512^3 (64) 30 / 82; symmetric, large tiles: 32 x 1024^2 (1152 = 2.25 rounds) 112 / 129,
// 4096^2 (528) 96 / 122, 8192^2 (2080) equal.  So: large ones from two rounds on, when the last is
// nearly full.
int f32_tile(int M, int N, int batch, int sym) {
  if (M % 128 || N % 128) return 64;
  const long long tm = M / 128, tn = N / 128, t = (sym ? tm * (tm + 1) / 2 : tm * tn) * batch;
  const long long rounds = (t + 511) / 512;
  return (t >= 1024 && rounds * 512 * 20 <= t * 21) ? 128 : 64;
}

int f32_tiles(int M, int N, int batch, int sym) {   // tiles per matrix, i.e. residual partial sums
  const int T = f32_tile(M, N, batch, sym), tm = M / T, tn = N / T;
  return sym ? tm * (tm + 1) / 2 : tm * tn;
}

int launch_gemm_f32(const GemmDesc& g, hipStream_t s) {
  const int T = f32_tile(g.M, g.N, g.sel_batch ? g.sel_batch : g.batch, g.sym);
  return launch_gemm_f32(g, T, T, s);
}

int launch_gemm_f32_pair(const GemmDesc& a, const GemmDesc& b, hipStream_t s) {
  const int T = f32_tile(a.M, a.N, 2 * (a.sel_batch ? a.sel_batch : a.batch), a.sym && b.sym);
  return T == 128 ? launch_cfg<float, float, 128, 128, 2, 2>(a, s, &b) : launch_cfg<float, float, 64, 64, 2, 2>(a, s, &b);
}

int launch_gemm_f64a(const GemmDesc& g, int tile_m, int tile_n, hipStream_t s) {
  if (g.a_km) return PRISM_EINVAL;
  if (tile_m == 64 && tile_n == 64) return launch_cfg<double, double, 64, 64, 2, 2>(g, s);
  return PRISM_EINVAL;
}

}  // namespace prism
