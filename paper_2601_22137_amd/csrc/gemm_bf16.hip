// bf16 GEMMs C = A * B^T on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16, fp32
// accumulate) with the epilogues of the PRISM polar iteration fused in (Table 1, rows
// "Newton-Schulz, U V^T": Gram/residual R = I - X^T X, Q = R/2 + alpha R^2, update X + X Q).
//
// The instruction consumes operands with K contiguous (each lane feeds 8 consecutive k of one row).
// An operand may be stored that way ([M][K] / [N][K]) or with K as the slow index ([K][M] / [K][N]);
// the latter is read from LDS with transposing reads.  The polar iteration keeps one copy of the
// iterate, X[L][S]: the Gram product X^T X reads it as [K][M] for both operands, the update X Q reads
// it as [M][K]; R and Q are symmetric and are read as [K][N], which fetches whole cache lines per
// request where the K-contiguous form fetches 64 bytes per row and slab.
//
// One workgroup = 4 wavefronts (2 x 2) computes a TM x TN tile for one matrix; K runs in slabs of
// 32 moved straight from global memory into an LDS ring (no register staging; loads run
// STAGES - 1 slabs ahead to cover the memory latency), in a swizzled layout that keeps the
// 16-byte fragment reads free of bank conflicts.  Three tile shapes:
//   256 x 256  one workgroup per CU, four-deep ring (128 KiB): fewest bytes per flop
//   256 x 128  two workgroups per CU, three-deep rings (2 x 72 KiB): two wavefronts per SIMD, so the
//              matrix pipe has a second wave to issue from whenever one waits at a barrier or for
//              LDS, and the HBM-bound epilogue of one workgroup runs under the main loop of the other
//   128 x 128  three workgroups per CU (3 x 48 KiB), for products too small to fill the chip otherwise
// A launch may cover several shape groups (a descriptor per group): the workgroup index runs over
// the tiles of all groups.
#include "gemm_bf16_tile.h"

namespace prism {
namespace {

template <int TM, int TN, int EPI, bool SYM, bool KMA, bool KMB, int NW, bool LONG>
__global__ __launch_bounds__(64 * NW, (NW == 8 ? 1 : (LONG ? 2 : wgs_per_cu(TM, TN)))) void gemm_bf16_kernel(Bf16Multi mg) {
  constexpr int RT = TM / TN;                    // SYM: tile columns per tile row height
  static_assert(RT == 1 || RT == 2, "tile shape");
  extern __shared__ __align__(1024) unsigned char smem[];
  // Workgroup -> (group, tile).  The hardware deals consecutive workgroups round-robin to the 8
  // XCDs, each with its own L2.  xcd_private (set by the launcher for small matrices, or when all
  // operands of the launch fit the Infinity Cache together): every XCD gets a contiguous range of the
  // tiles of each group, i.e. whole matrices, so that the tiles sharing a panel share an L2 (without this the
  // 768-sized Gram fetched 7x its algorithmic bytes).  Of each group, not of the launch: the groups differ in K, and
  // four XCDs of eight had all of the long ones (small launches: of the launch, see launch_tw).  Otherwise workgroup i runs tile i: all XCDs
  // sweep the same matrix and share its panels through the Infinity Cache (private ranges measured
  // 20 % slower at 8 x 4096^2, where eight matrices at once overflow that cache).
  int wg = blockIdx.x;
  if (mg.xcd_private == XCD_LAUNCH) wg = (wg & 7) * (mg.tile_start[mg.ngroups] >> 3) + (wg >> 3);
  int gi = 0;
  while (gi + 1 < mg.ngroups && wg >= mg.tile_start[gi + 1]) ++gi;
  wg -= mg.tile_start[gi];
  if (mg.xcd_private == XCD_GROUPS) wg = (wg & 7) * ((mg.tile_start[gi + 1] - mg.tile_start[gi]) >> 3) + (wg >> 3);   // starts are multiples of 8
  const Bf16Desc& g = mg.d[gi];

  // SYM: A == B and the result is symmetric (Gram matrix, R^2): only the tiles that reach the
  // diagonal or lie above it are computed; a tile wholly above the diagonal blocks is also written
  // mirrored.
  const int tiles_m = g.M / TM, tiles_n = g.N / TN;
  const int per_mat = SYM ? RT * tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int b = wg / per_mat;
  if (b >= g.batch) return;   // the group's tiles are rounded up to whole rounds of the XCDs
  const int rem = wg - b * per_mat;
  int tm, tn;
  if (SYM) {       // row tm of the upper triangle holds tiles_n - RT * tm tiles
    int left = rem;
    tm = 0;
    while (left >= tiles_n - RT * tm) { left -= tiles_n - RT * tm; ++tm; }
    tn = RT * tm + left;
  } else if (g.xcd_blocks && !mg.xcd_private) {
    // Every XCD sweeps blocks of 4 x 8 tiles of its own (its 32 CUs run one block at a time): the
    // tiles that meet in an L2 share 4 row panels and 8 column panels, where the plain order gives an
    // XCD two tile columns of every row, i.e. 16 row panels and 2 column panels per 32 tiles.
    const int x = rem & 7, q = rem >> 3;
    const int blk = (q >> 5) * 8 + x, w = q & 31, nbn = tiles_n >> 3;
    tm = (blk / nbn) * 4 + (w >> 3);
    tn = (blk % nbn) * 8 + (w & 7);
  } else {
    tm = rem / tiles_n;
    tn = rem - tm * tiles_n;
  }
  const int cb = g.ctrl_parts ? b / g.ctrl_parts : b;   // split-K launches: the batch entries are parts of matrices
  if (g.ctrl && g.ctrl[cb].done) return;
  const float alpha = g.ctrl ? g.ctrl[cb].alpha : 1.0f;
  gemm_bf16_tile<TM, TN, EPI, SYM, KMA, KMB, NW, LONG>(g, b, rem, per_mat, tm, tn, smem, [&](float& out) { out = alpha; return true; });
}

// tiles of one matrix
template <int TM, int TN, bool SYM>
long long tiles_per_matrix(const Bf16Desc& g) {
  const long long tm = g.M / TM, tn = g.N / TN;
  return SYM ? (TM / TN) * tm * (tm + 1) / 2 : tm * tn;
}

// Slabs of 64 k or of 32 for an update of `tiles` tiles with K = k: two workgroups per CU against three.  From K = 512 on up to one round of the longer ones (512 tiles), and
// from K = 768 on beyond one of the shorter (768).  Us, slabs of 32 / 64: K = 512, 512 tiles 17.7 / 16.8, 640 22.5 / 23.6, 4096 105 / 110; K = 768, 576 tiles 31.3 / 34.0, 720
// 35.8 / 38.3, 2304 71.6 / 68.9; K = 1024, 640 38.0 / 40.2, 1024 43.9 / 40.2.  Below K = 512 a single launch gains 0.3 us, but beside the launches of another part of a
// grouped call, whose workgroups find less room, it loses more: 14 layers of width 151 (K = 256) 633 / 656, 8 of 384 719 / 747, 10 of 300 760 / 791, 16 of 256 697 / 713.
bool slabs_of_64(long long tiles, int k) { return k >= 512 && (tiles <= 512 || (k >= 768 && tiles > 768)); }

template <int TM, int TN, int EPI, bool SYM, bool KMA, bool KMB, int NW>
int launch_tw(Bf16Multi& mg, hipStream_t s) {
  long long total = 0;
  bool lines = true;   // K in whole slabs of 64
  // A launch whose tiles are no multiple of eight is rounded up where the operands are large enough for their fetches past the L2s to be what
  // it waits for (Gram product of 50257 x 768 in 12 parts, 252 tiles of 77 MB: 64 -> 52 us); small ones are faster in plain order (one
  // 768 x 3072 in 6 parts, 126 tiles of 5 MB: 10.2 against 11.6).  One-pass Gram products in plain order / rounded up, us: 12 x 3072 x 768 (252 tiles, 54 MB) 53 / 39,
  // 2 x 6144 x 1536 (156, 36 MB) 67 / 64, 3 x 5120 x 1280 (165, 38 MB) 58 / 55; of several rounds 20 x 768 x 768 (420, 22 MB) 31 / 23, 6 x 1280 x 1280 (330, 19 MB) 34 / 27.
  double operand_bytes = 0.0;
  for (int i = 0; i < mg.ngroups; ++i) {
    const Bf16Desc& g = mg.d[i];
    total += tiles_per_matrix<TM, TN, SYM>(g) * g.batch;
    operand_bytes += 2.0 * g.batch * ((double)g.M * g.K + (g.A == g.B ? 0.0 : (double)g.N * g.K));
    lines = lines && g.K % 64 == 0;
  }
  const bool wide = lines && slabs_of_64(total, mg.d[0].K);
  // Launches of several rounds are rounded up too, small ones keep whole ranges of the launch (three updates of five layers of width 320, update of 465 tiles
  // and Gram product of 120: 182 us with plain order and groups, 168 with groups and the launch).
  if (mg.xcd_private) mg.xcd_private = operand_bytes >= 32.0 * 1024 * 1024 || total > 256 ? XCD_GROUPS : (total % 8 == 0 ? XCD_LAUNCH : 0);
  total = 0;
  for (int i = 0; i < mg.ngroups; ++i) {
    mg.tile_start[i] = (int)total;
    total += tiles_per_matrix<TM, TN, SYM>(mg.d[i]) * mg.d[i].batch;
    if (mg.xcd_private == XCD_GROUPS) total = (total + 7) & ~7ll;
    if (total > 0x7fffffff) return PRISM_EUNSUPPORTED;
  }
  mg.tile_start[mg.ngroups] = (int)total;
  auto launch = [&](auto kern, int lds) -> int {
    const int rc = allow_dynamic_lds((const void*)kern, lds);
    if (rc != PRISM_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64 * NW), lds, s, mg);
    return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
  };
  if constexpr (long_slabs(TM, TN, EPI, KMA)) {
    if (wide) return launch(gemm_bf16_kernel<TM, TN, EPI, SYM, KMA, KMB, NW, true>, ring_bytes(TM, TN, true));
  }
  return launch(gemm_bf16_kernel<TM, TN, EPI, SYM, KMA, KMB, NW, false>, ring_bytes(TM, TN, false));
}

// 256 x 256 tiles run with eight wavefronts (mg.waves8), every other shape with four
template <int TM, int TN, int EPI, bool SYM, bool KMA = false, bool KMB = false>
int launch_te(Bf16Multi& mg, hipStream_t s) {
  if constexpr (TM == 256 && TN == 256) {
    if (mg.waves8) return launch_tw<TM, TN, EPI, SYM, KMA, KMB, 8>(mg, s);
  }
  return launch_tw<TM, TN, EPI, SYM, KMA, KMB, 4>(mg, s);
}

template <int TM, int TN>
int launch_t(Bf16Multi& mg, hipStream_t s) {
  const int epi = mg.d[0].epi, sym = mg.d[0].sym, km = mg.d[0].km;
  for (int i = 0; i < mg.ngroups; ++i) {
    const Bf16Desc& g = mg.d[i];
    if (g.epi != epi || g.sym != sym || g.km != km) return PRISM_EINVAL;
    if (g.M % TM || g.N % TN || g.K % BF_BK || g.K < BF_BK || g.lda % 8 || g.ldb % 8) return PRISM_EINVAL;
    if ((long long)(g.M / TM) * (g.N / TN) * g.batch <= 0) return PRISM_EINVAL;
    if (g.sym && (g.M != g.N || g.A != g.B)) return PRISM_EINVAL;
    if ((g.epi == BEPI_GRAM || g.epi == BEPI_POLYQ) && !g.sym) return PRISM_EINVAL;   // symmetric products only
    if (g.epi == BEPI_STORE && (!g.C32 || (g.sym && km != 3))) return PRISM_EINVAL;
    // without the fp32 matrix: GRAM with a diagonal array, POLYQ with R in bf16
    if (g.epi == BEPI_GRAM && ((!g.C32 && !g.diag) || g.rho_stride < tiles_per_matrix<TM, TN, true>(g))) return PRISM_EINVAL;
    if (g.epi == BEPI_POLYQ && !g.C32 && !g.Cin16) return PRISM_EINVAL;
  }
  // operand layouts (km: bit 0 = A stored [K][M], bit 1 = B stored [K][N]) per kind of product
  switch (epi) {
    case BEPI_STORE:
      if (sym) return launch_te<TM, TN, BEPI_STORE, true, true, true>(mg, s);
      if (km == 3) return launch_te<TM, TN, BEPI_STORE, false, true, true>(mg, s);
      if (km == 2) return launch_te<TM, TN, BEPI_STORE, false, false, true>(mg, s);
      if (km == 0) return launch_te<TM, TN, BEPI_STORE, false>(mg, s);
      return PRISM_EINVAL;
    case BEPI_GRAM:
      if (km == 3) return launch_te<TM, TN, BEPI_GRAM, true, true, true>(mg, s);
      if (km == 0) return launch_te<TM, TN, BEPI_GRAM, true>(mg, s);
      return PRISM_EINVAL;
    case BEPI_POLYQ:
      if (km == 3) return launch_te<TM, TN, BEPI_POLYQ, true, true, true>(mg, s);
      if (km == 0) return launch_te<TM, TN, BEPI_POLYQ, true>(mg, s);
      return PRISM_EINVAL;
    case BEPI_APPLY:
      if (km == 2) return launch_te<TM, TN, BEPI_APPLY, false, false, true>(mg, s);
      if (km == 0) return launch_te<TM, TN, BEPI_APPLY, false>(mg, s);
      return PRISM_EINVAL;
  }
  return PRISM_EINVAL;
}

}  // namespace

int launch_gemm_bf16_multi(const Bf16Desc* groups, int ngroups, int tile_m, int tile_n, hipStream_t s) {
  if (ngroups < 1 || ngroups > BF16_MAX_GROUPS) return PRISM_EINVAL;
  Bf16Multi mg = {};
  mg.ngroups = ngroups;
  // bytes of all operands of the launch against half the 256 MiB Infinity Cache
  double operand_bytes = 0.0;
  bool small = true;
  static const int no_blocks = ab_switch("PRISM_BF16_NO_XCD_BLOCKS");
  for (int i = 0; i < ngroups; ++i) {
    Bf16Desc& g = mg.d[i];
    g = groups[i];
    operand_bytes += 2.0 * g.batch * ((double)g.M * g.K + (g.A == g.B ? 0.0 : (double)g.N * g.K));
    const long long tm = g.M / tile_m, tn = g.N / tile_n;
    const long long per_mat = g.sym ? (tile_m / tile_n) * tm * (tm + 1) / 2 : tm * tn;
    if (per_mat > 64) small = false;
    g.xcd_blocks = !no_blocks && !g.sym && per_mat % 256 == 0 && tm % 4 == 0 && tn % 8 == 0;
  }
  mg.xcd_private = small || operand_bytes <= 128.0 * 1024 * 1024;
  static const int waves4 = ab_switch("PRISM_BF16_WAVES4");
  mg.waves8 = !waves4;
  if (tile_m == 256 && tile_n == 256) return launch_t<256, 256>(mg, s);
  if (tile_m == 256 && tile_n == 128) return launch_t<256, 128>(mg, s);
  if (tile_m == 128 && tile_n == 128) return launch_t<128, 128>(mg, s);
  return PRISM_EINVAL;
}

int launch_gemm_bf16(const Bf16Desc& g, int tile_m, int tile_n, hipStream_t s) {
  return launch_gemm_bf16_multi(&g, 1, tile_m, tile_n, s);
}

}  // namespace prism
