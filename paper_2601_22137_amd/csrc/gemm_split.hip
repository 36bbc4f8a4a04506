// fp32 products on the bf16 matrix cores.  Each operand comes as three bf16 planes h + m + l that add up to it exactly (split3.h; |m| up to 2^-8 of it, |l| up to
// 2^-17); of the nine products of planes the six largest are formed.  The two m l and l l are left out: together up to 2^-24 of a term, of either
// sign, 2^-27.6 rms (5e-9).  Products of two bf16 numbers are exact in fp32, so that only the accumulation rounds.  It is closed every 256 k into a second set of
// registers, as in gemm_f32_tile.h; the error against 64 bits is then below that of the fp32 matrix cores with the same
// windows: relative Frobenius error at K = 256, 1024, 4096, 8192, Gaussian operands 2.4, 2.4, 2.6, 2.7e-7 (fp32 cores 2.9, 2.9, 3.0, 3.1), positive
// ones 2.0, 1.1, 0.83, 0.97e-7 (2.5, 1.3, 0.90, 1.0), identity plus 1 % 1.9, 2.1, 2.3, 2.5e-7 (2.7, 3.1, 3.2, 3.4), over six decades 0.51, 1.2, 2.0, 2.2e-7 (0.84, 1.6,
// 2.5, 2.7).  Sums of one term (diagonal operands) round once per plane product: 3.1e-8 (2.5).
//
// Within a sum entry (i, j) of X^T X meets m_i h_j before h_i m_j and entry (j, i) the other way round, so a symmetric product is symmetric to rounding only (1e-8 of its
// norm) unless one half is stored as the mirror image of the other: whole 64 x 64 blocks below the diagonal are, the blocks on it are not.  Its skew part is
// less than the rounding of the product, so a square of it taken as R^T R is within rounding of R R.
//
// What bounds it: the matrix pipe at the clock the power limit leaves (1.6 GHz; 1.3 to 1.4 PFLOP/s of bf16 work, a sixth of
// that in fp32 flops).  8192^3 220 TFLOP/s, 32 x 1024^3 203, 4 x 1024^3 190, against 147, 138 and 115 on the fp32 cores.
//
// One workgroup of eight wavefronts computes a 128 x 256 tile (2 x 4 wavefronts of 64 x 64) or a 128 x 128 one (64 x 32 each), one of four a
// 64 x 64 one (2 x 2 of 32 x 32), where there are too few of the others.  K runs in slabs of 32 moved straight into an LDS ring of two (144 KiB) or three slabs; a fragment of a plane serves two or three of the six
// products, so per MFMA the LDS and the loads have half the traffic of a plain bf16 product.  B is stored [K][N] and read with transposing
// reads, A as [M][K] or [K][M].  Splitting fp32 into three bf16 numbers is a published method (Henry, Tang, Heinecke, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", 2019).
#include <type_traits>

#include "split3.h"

namespace prism {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef const void __attribute__((address_space(1)))* gptr_t;
typedef void __attribute__((address_space(3)))* lptr_t;

constexpr int SLAB = 32, WINDOW = 8;   // k per slab; slabs per partial sum (256 k)

template <int N> __device__ inline void wait_vmcnt() { __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70); }
template <int N> __device__ inline void wait_lgkm() {   // the counter has four bits
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(N < 15 ? N : 15) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

__device__ inline float apow(float a, int e) { return e == 0 ? 1.0f : (e == 1 ? a : a * a); }

constexpr int plane_bytes(int T) { return T * SLAB * 2; }
constexpr int slab_bytes(int TM, int TN) { return 3 * (plane_bytes(TM) + plane_bytes(TN)); }
constexpr int ring_of(int TM, int TN) { return TM * TN > 128 * 128 ? 2 : 3; }

// 16-byte unit c of row k of a K-major slab of T columns lies at c ^ turn(k): the four rows of a transposing read fall on different banks
template <int T> __device__ inline int turn(int k) { return T == 64 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); }

template <bool PAIR> struct SplitArg { typedef GemmDesc type; };
template <> struct SplitArg<true> { typedef GemmPair type; };

template <int TM, int TN, int WR, int WC, int EPI, bool A_KM, bool SYM, bool PAIR>
__global__ __launch_bounds__(64 * WR * WC, TM == 64 ? 2 : 1) void gemm_split_kernel(typename SplitArg<PAIR>::type arg) {
  constexpr int NW = WR * WC;
  constexpr int ST = ring_of(TM, TN);
  constexpr int WTM = TM / WR, WTN = TN / WC, NBM = WTM / 32, NBN = WTN / 32, NB = NBM * NBN;
  constexpr int PA = plane_bytes(TM), PB = plane_bytes(TN), BUF = slab_bytes(TM, TN);
  constexpr int IA = PA / 1024 / NW, IB = PB / 1024 / NW, NL = 3 * (IA + IB);   // load instructions per wave: plane of A, of B, slab
  static_assert(IA * NW * 1024 == PA && IB * NW * 1024 == PB, "whole instructions");
  extern __shared__ __align__(1024) unsigned char smem[];
  int wg = blockIdx.x, which = 0;
  if constexpr (PAIR) {
    which = wg >= arg.first;   // uniform
    wg -= which ? arg.first : 0;
  }
  const GemmDesc& g = [&]() -> const GemmDesc& { if constexpr (PAIR) return arg.d[which]; else return arg; }();

  // Tile: one XCD has a contiguous range of the product's tiles, here in blocks of 8 x 4 (32 CUs, one workgroup each).  Launches are rounded up to
  // multiples of eight for that: in plain order, which products of another number of tiles had, the panels come past the L2s (us in plain order / so: 64 x 64 tiles,
  // order 448 x 10 28 / 20, both updates of a square root in one launch 60 / 34, 704 x 20 139 / 102; 128 x 128 tiles, 640 x 10 46 / 37, 896 x 20 212 / 174).
  const bool sym = SYM || (PAIR && TM == TN && g.sym);
  const int tiles_m = g.M / TM, tiles_n = g.N / TN;
  const int per_mat = sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int total = per_mat * g.batch;
  if ((total & 7) == 0) {   // without the test for surplus workgroups: 40 ns a launch, also of those behind convergence
    wg = (wg & 7) * (total >> 3) + (wg >> 3);
  } else {
    wg = (wg & 7) * ((total >> 3) + 1) + (wg >> 3);
    if (wg >= total) return;
  }
  const int b = wg / per_mat, rem = wg - b * per_mat;
  int tm, tn;
  if (sym) {
    int left = rem;
    tm = 0;
    while (left >= tiles_m - tm) { left -= tiles_m - tm; ++tm; }
    tn = tm + left;
  } else if (g.tile_blocks) {
    const int blk = rem >> 5, w = rem & 31, nbn = tiles_n >> 2;
    tm = (blk / nbn) * 8 + (w >> 2);
    tn = (blk % nbn) * 4 + (w & 3);
  } else {
    tm = rem / tiles_n;
    tn = rem - tm * tiles_n;
  }
  if (g.ctrl && g.ctrl[b].done) return;
  const float alpha = g.ctrl ? g.ctrl[b].alpha : 1.0f;

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm0 = (wave / WC) * WTM, wn0 = (wave % WC) * WTN;
  const int m0 = tm * TM, n0 = tn * TN;
  const int lda = g.lda, ldb = g.ldb, KT = g.K / SLAB;
  const long long psA = 2 * g.psA, psB = 2 * g.psB;
  const char* A = (const char*)(g.A3 + (long long)b * g.strideA + (A_KM ? (long long)m0 : (long long)m0 * lda));
  const char* B = (const char*)(g.B3 + (long long)b * g.strideB + n0);

  // Slabs in LDS as in gemm_bf16_tile.h: [k][row] with the 16-byte units of row k turned for an operand stored
  // K-major, 64-byte rows, four to a 256-byte line, chunks xor-ed with the line for a K-contiguous one.
  unsigned offA[IA], offB[IB];
#pragma unroll
  for (int u = 0; u < IA; ++u) {
    if constexpr (A_KM) {
      constexpr int U = TM / 8;
      const int k = (u * NW + wave) * (64 / U) + lane / U, c = (lane % U) ^ turn<TM>(k);
      offA[u] = (unsigned)(k * lda + c * 8) * 2u;
    } else {
      const int lq = lane >> 4, lu = (lane & 15) ^ ((wave * 4 + lq) & 15);
      offA[u] = (unsigned)(((u * NW + wave) * 16 + 4 * lq + (lu >> 2)) * lda + (lu & 3) * 8) * 2u;
    }
  }
#pragma unroll
  for (int u = 0; u < IB; ++u) {
    constexpr int U = TN / 8;
    const int k = (u * NW + wave) * (64 / U) + lane / U, c = (lane % U) ^ turn<TN>(k);
    offB[u] = (unsigned)(k * ldb + c * 8) * 2u;
  }
  const long long stepA = A_KM ? (long long)SLAB * lda * 2 : SLAB * 2, stepB = (long long)SLAB * ldb * 2;
  auto issue = [&](int kt, int slot, int u) {   // load instruction u of NL: the planes of A, those of B
    if (u < 3 * IA) {
      const int p = u / IA, v = u % IA;
      __builtin_amdgcn_global_load_lds((gptr_t)(A + p * psA + kt * stepA + offA[v]), (lptr_t)(smem + slot * BUF + p * PA + (v * NW + wave) * 1024), 16, 0, 0);
    } else {
      const int p = (u - 3 * IA) / IB, v = (u - 3 * IA) % IB;
      __builtin_amdgcn_global_load_lds((gptr_t)(B + p * psB + kt * stepB + offB[v]), (lptr_t)(smem + slot * BUF + 3 * PA + p * PB + (v * NW + wave) * 1024), 16, 0, 0);
    }
  };

  f32x16 acc[NB], sum[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[i][r] = 0.0f; sum[i][r] = 0.0f; }

  const int lr = lane & 31, lh = lane >> 5;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  unsigned fra[A_KM ? NBM : 4], frb[NBN];
  {
    const int i = lane & 15, mb = (lane >> 4) & 1, kg = lane >> 5;
    if constexpr (A_KM) {
#pragma unroll
      for (int f = 0; f < NBM; ++f) {
        const int c = wm0 / 8 + 4 * f + 2 * mb + ((i & 3) >> 1);
        fra[f] = lds0 + (8 * kg + (i >> 2)) * (TM * 2) + ((c ^ turn<TM>(i >> 2)) * 16) + 8 * (i & 1);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)   // [16-k half][parity of the row block]
        fra[q] = lds0 + wm0 * 64 + (lr >> 2) * 256 + (((((lr & 3) << 2) + (q >> 1) * 2 + lh) ^ ((lr >> 2) + 8 * ((q ^ (wm0 >> 5)) & 1))) << 4);
    }
#pragma unroll
    for (int f = 0; f < NBN; ++f) {
      const int c = wn0 / 8 + 4 * f + 2 * mb + ((i & 3) >> 1);
      frb[f] = lds0 + 3 * PA + (8 * kg + (i >> 2)) * (TN * 2) + ((c ^ turn<TN>(i >> 2)) * 16) + 8 * (i & 1);
    }
  }
  // Fragment reads in inline assembly, waited for by hand: as builtins they would wait for every load into the ring.
  auto read_tr = [&](unsigned a, auto otag) {
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(a), "i"(decltype(otag)::value));
    return r;
  };
  u32x4 a0[2][NBM], b0[2][NBN], a1[NBM], b1[NBN], a2[NBM], b2[NBN];
  constexpr int READS = NBM * (A_KM ? 2 : 1) + 2 * NBN;   // LDS reads of the fragments of one plane
  // plane P of both operands, 16-k half KK of the slab in `slot`
  auto read_plane = [&](int slot, auto kktag, auto ptag, int set) {
    constexpr int KK = decltype(kktag)::value, P = decltype(ptag)::value;
    const unsigned o = (unsigned)slot * BUF;
#pragma unroll
    for (int f = 0; f < NBM; ++f) {
      u32x4 v;
      if constexpr (A_KM) {
        const u32x2 h0 = read_tr(fra[f] + o, std::integral_constant<int, P * PA + KK * 32 * TM>{});
        const u32x2 h1 = read_tr(fra[f] + o, std::integral_constant<int, P * PA + KK * 32 * TM + 8 * TM>{});
        v = (u32x4){h0[0], h0[1], h1[0], h1[1]};
      } else {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(fra[KK * 2 + (f & 1)] + o), "i"(P * PA + f * 2048));
      }
      if constexpr (P == 0) a0[set][f] = v;
      else if constexpr (P == 1) a1[f] = v;
      else a2[f] = v;
    }
#pragma unroll
    for (int f = 0; f < NBN; ++f) {
      const u32x2 h0 = read_tr(frb[f] + o, std::integral_constant<int, P * PB + KK * 32 * TN>{});
      const u32x2 h1 = read_tr(frb[f] + o, std::integral_constant<int, P * PB + KK * 32 * TN + 8 * TN>{});
      const u32x4 v = {h0[0], h0[1], h1[0], h1[1]};
      if constexpr (P == 0) b0[set][f] = v;
      else if constexpr (P == 1) b1[f] = v;
      else b2[f] = v;
    }
  };
  auto mma = [&](const u32x4 (&x)[NBM], const u32x4 (&y)[NBN]) {
#pragma unroll
    for (int m = 0; m < NB; ++m)
      acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[m / NBN]), __builtin_bit_cast(bf16x8, y[m % NBN]), acc[m], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  std::integral_constant<int, 0> I0;
  std::integral_constant<int, 1> I1;
  std::integral_constant<int, 2> I2;
  // The six products of 16 k, smallest first.  The fragments of the lesser planes have one set of registers, refilled for the
  // next 16 k (of `slot`) as soon as their MFMAs have been issued; plane 0, needed to the end, has two.
  auto step = [&](int set, int slot, auto kktag, auto moretag, auto loads) {
    constexpr bool MORE = decltype(moretag)::value;
    wait_lgkm<READS>();   // planes 2 and 0 have arrived; plane 1 was requested last
    mma(a2, b0[set]);
    mma(a0[set], b2);
    if constexpr (MORE) {
      read_plane(slot, kktag, I2, 0);
      read_plane(slot, kktag, I0, set ^ 1);
    }
    loads(0);
    __builtin_amdgcn_sched_barrier(0);
    wait_lgkm<MORE ? 2 * READS : 0>();
    mma(a1, b1);
    mma(a1, b0[set]);
    loads(1);
    __builtin_amdgcn_sched_barrier(0);
    mma(a0[set], b1);
    if constexpr (MORE) read_plane(slot, kktag, I1, 0);
    __builtin_amdgcn_sched_barrier(0);
    mma(a0[set], b0[set]);
    loads(2);
    __builtin_amdgcn_sched_barrier(0);
  };
  // every read of the slab at hand has arrived, and this wave's share of the next one has landed
  auto slab_barrier = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto close = [&](int kt) {
    if ((kt + 1) % WINDOW == 0) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) { sum[i][r] += acc[i][r]; acc[i][r] = 0.0f; }
    }
  };
  auto none = [](int) {};
#pragma unroll
  for (int q = 0; q < ST; ++q)
#pragma unroll
    for (int u = 0; u < NL; ++u) issue(q, q, u);   // K of ST slabs at least
  wait_vmcnt<(ST - 1) * NL>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  read_plane(0, I0, I2, 0);
  read_plane(0, I0, I0, 0);
  read_plane(0, I0, I1, 0);
  int slot = 0, kt = 0;
  for (; kt < KT - ST; ++kt) {
    const int next = slot == ST - 1 ? 0 : slot + 1;
    step(0, slot, I1, std::true_type{}, none);
    wait_vmcnt<(ST - 2) * NL>();
    slab_barrier();
    step(1, next, I0, std::true_type{}, [&](int w) {   // slab kt + ST takes the place of slab kt
#pragma unroll
      for (int u = w * NL / 3; u < (w + 1) * NL / 3; ++u) issue(kt + ST, slot, u);
    });
    slot = next;
    close(kt);
  }
  for (; kt < KT - 1; ++kt) {
    const int next = slot == ST - 1 ? 0 : slot + 1;
    step(0, slot, I1, std::true_type{}, none);
    wait_vmcnt<0>();
    slab_barrier();
    step(1, next, I0, std::true_type{}, none);
    slot = next;
    close(kt);
  }
  step(0, slot, I1, std::true_type{}, none);
  step(1, 0, I0, std::false_type{}, none);
  __syncthreads();   // the ring becomes strips

  // ---- epilogue: 32 rows of the wave at a time through a strip of its own, rows read back in runs of eight columns ----
  constexpr int SW = WTN + 4;
  static_assert(NW * 32 * SW * 4 <= ST * BUF, "strips in the ring");
  float* strip = (float*)smem + wave * 32 * SW;
  constexpr int LPR = WTN / 8, RPI = 64 / LPR, ITS = 32 / RPI;
  const int rr = lane / LPR, cc = (lane % LPR) * 8;
  // sym: what lies below the diagonal by whole 64 x 64 blocks is the mirror image, within a tile too
  const bool lower = sym && tm == tn && wm0 / 64 > wn0 / 64;
  const bool mirror = sym && (tm != tn || wm0 / 64 < wn0 / 64);
  float* C = g.C ? (float*)g.C + (long long)b * g.strideC : nullptr;
  uint16_t* C3 = g.C3 ? g.C3 + (long long)b * g.strideC : nullptr;
  constexpr bool ADDENDS = EPI != EPI_RESIDUAL;
  const float* cin = (const float*)g.Cin + (long long)b * g.strideCin;
  const float* cin2 = g.Cin2 + (long long)b * g.strideCin;
  const float wc = EPI == EPI_POLYQ ? g.c1 : g.c_in * apow(alpha, g.cin_alpha_pow);
  const float wa = EPI == EPI_POLYQ ? alpha : apow(alpha, g.coef_is_alpha);
  const float wc2 = apow(alpha, g.cin2_alpha_pow);
  float part = 0.0f;
  if (lower && EPI != EPI_RESIDUAL) return;
  auto put = [&](const float (&v)[8], int row, int col) {
    const long long o = (long long)row * g.ldc + col;
    if (C) {
      *(f32x4*)(C + o) = (f32x4){v[0], v[1], v[2], v[3]};
      *(f32x4*)(C + o + 4) = (f32x4){v[4], v[5], v[6], v[7]};
    }
    if (C3) {
      s3_u32x4 p[3];
      split3(v, p);
#pragma unroll
      for (int q = 0; q < 3; ++q) *(s3_u32x4*)(C3 + q * g.psC + o) = p[q];
    }
  };
#pragma unroll
  for (int i = 0; i < NBM && !lower; ++i) {
    f32x4 in[ADDENDS ? ITS : 1][2];
    if constexpr (ADDENDS) {
#pragma unroll
      for (int it = 0; it < ITS; ++it) {
        const float* p = cin + (long long)(m0 + wm0 + i * 32 + it * RPI + rr) * g.ldcin + n0 + wn0 + cc;
        in[it][0] = *(const f32x4*)p;
        in[it][1] = *(const f32x4*)(p + 4);
      }
    }
    // register r of lane l: row (r / 4) 8 + (l / 32) 4 + r % 4, column l % 32 of a block
#pragma unroll
    for (int j = 0; j < NBN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) strip[((r >> 2) * 8 + lh * 4 + (r & 3)) * SW + j * 32 + lr] = sum[i * NBN + j][r] + acc[i * NBN + j][r];
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int row = it * RPI + rr, gi = m0 + wm0 + i * 32 + row, gj = n0 + wn0 + cc;
      float* sp = strip + row * SW + cc;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = sp[e];
      if constexpr (EPI == EPI_RESIDUAL) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = (gi < g.n_true && gj + e < g.n_true) ? ((gi == gj + e ? 1.0f : 0.0f) - v[e]) : 0.0f;
          part = __builtin_fmaf(v[e], v[e], part);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = __builtin_fmaf(wa, v[e], wc * in[ADDENDS ? it : 0][e >> 2][e & 3]);
        if (EPI == EPI_AXPY && g.Cin2) {
          const float* p = cin2 + (long long)gi * g.ldcin + gj;
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = __builtin_fmaf(wc2, p[e], v[e]);
        }
      }
      put(v, gi, gj);
      if (mirror) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sp[e] = v[e];
      }
    }
    if (mirror) {   // eight rows of a column are eight entries of a row of the mirror image
#pragma unroll
      for (int it = 0; it < WTN / 16; ++it) {
        const int col = it * 16 + (lane >> 2), rq = (lane & 3) * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = strip[(rq + e) * SW + col];
        put(v, n0 + wn0 + col, m0 + wm0 + i * 32 + rq);
      }
    }
  }
  if (EPI == EPI_RESIDUAL) {
    if (mirror) part *= 2.0f;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
    __syncthreads();
    float* red = (float*)smem;
    if (lane == 0) red[wave] = part;
    __syncthreads();
    if (t == 0) {
      float r = (red[0] + red[1]) + (red[2] + red[3]);
      if (NW == 8) r += (red[4] + red[5]) + (red[6] + red[7]);
      g.rho_part[(long long)b * per_mat + rem] = r;
    }
  }
}

__global__ __launch_bounds__(256) void split3_kernel(const float* x, uint16_t* p, long long groups, long long ps) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < groups; i += (long long)gridDim.x * 256) {
    const f32x4 lo = *(const f32x4*)(x + i * 8), hi = *(const f32x4*)(x + i * 8 + 4);
    const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    s3_u32x4 q[3];
    split3(v, q);
#pragma unroll
    for (int k = 0; k < 3; ++k) *(s3_u32x4*)(p + k * ps + i * 8) = q[k];
  }
}

// Tile of a launch, from the rounds it takes.  A round is 256 workgroups of the larger tiles, one per CU, and 512 of the smallest, two per CU, in
// 0.6 of the time of 256 of 128 x 128; one of 128 x 256 takes 1.9 of it.  Sign of n = 1000 (1024), us, tiles of 64 / 128 / 256 x 128 (128 x 256 is 2 % faster): one matrix 841 / 1301 / 1978,
// two 1192 / 1374 / 1996, four 1967 / 1693 / 2122, eight 3382 / 3034 / 2853; of 2048, one 3419 / 2896 / 3623, two 6190 / 5182 / 4884.
struct SplitTile { int m, n; };
SplitTile split_tile(int M, int N, int batch, int sym) {
  static const int sw = ab_switch("PRISM_SPLIT_TILE");   // 64, 128, 256 (128 x 256)
  if (sw == 64 || M % 128 || N % 128) return {64, 64};
  if (sw == 128 || (sw == 256 && (sym || N % 256))) return {128, 128};
  if (sw == 256) return {128, 256};
  const long long tm = M / 128, tn = N / 128;
  const long long t = (sym ? tm * (tm + 1) / 2 : tm * tn) * batch, fine = (sym ? tm * (2 * tm + 1) : 4 * tm * tn) * batch;
  const long long rounds = (t + 255) / 256;
  if (3 * ((fine + 511) / 512) < 5 * rounds) return {64, 64};
  if (!sym && N % 256 == 0 && 19 * ((t / 2 + 255) / 256) <= 10 * rounds) return {128, 256};
  return {128, 128};
}

template <int TM, int TN, int WR, int WC>
int launch_cfg(GemmPair& g, hipStream_t s) {
  long long total = 0;
  for (GemmDesc& d : g.d) {
    if (d.batch == 0) continue;
    if (d.M % TM || d.N % TN || d.K % SLAB || d.K / SLAB < ring_of(TM, TN) || d.lda % 8 || d.ldb % 8 || d.ldc % 8 || !d.A3 || !d.B3 || (!d.C && !d.C3)) return PRISM_EINVAL;
    if ((d.epi == EPI_POLYQ || d.epi == EPI_AXPY) && (!d.Cin || d.ldcin % 4)) return PRISM_EINVAL;
    if (d.sym && (TM != TN || d.M != d.N)) return PRISM_EINVAL;
    if (d.ctrl_parts || d.skip_m1 || d.skip_n1 || d.sym_skew_bound || d.acc_neg || d.cin_one_minus_alpha) return PRISM_EINVAL;
    if ((unsigned long long)(d.a_km ? 32ull * d.lda + TM : (unsigned long long)TM * d.lda) * 2 > 0xffffffffull || (32ull * d.ldb + TN) * 2 > 0xffffffffull) return PRISM_EINVAL;
    const int tm = d.M / TM, tn = d.N / TN;
    g.first = (int)total;
    d.tile_blocks = !d.sym && tm % 8 == 0 && tn % 4 == 0 && tm * tn > 32;
    total += ((d.sym ? (long long)tm * (tm + 1) / 2 : (long long)tm * tn) * d.batch + 7) & ~7ll;
    if (total > 0x3fffffff) return PRISM_EINVAL;
  }
  if (total <= 0) return PRISM_EINVAL;
  const GemmDesc& d = g.d[0];
  auto launch = [&](auto kern, const auto& arg) -> int {
    constexpr int lds = ring_of(TM, TN) * slab_bytes(TM, TN);
    const int rc = allow_dynamic_lds((const void*)kern, lds);
    if (rc != PRISM_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64 * WR * WC), lds, s, arg);
    return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
  };
  // the products there are: symmetric ones (the polar iteration) of an operand stored [K][M], others of one stored [M][K], updates of one stored [M][K]
  const bool pair = g.d[1].batch != 0;
  auto residual_or_square = [&](auto e) -> int {
    constexpr int E = decltype(e)::value;
    if constexpr (TM == TN) {
      if (d.a_km && d.sym && !pair) return launch(gemm_split_kernel<TM, TN, WR, WC, E, true, true, false>, d);
    }
    if (d.a_km || d.sym || pair) return PRISM_EINVAL;
    return launch(gemm_split_kernel<TM, TN, WR, WC, E, false, false, false>, d);
  };
  switch (d.epi) {
    case EPI_RESIDUAL: return residual_or_square(std::integral_constant<int, EPI_RESIDUAL>{});
    case EPI_POLYQ: return residual_or_square(std::integral_constant<int, EPI_POLYQ>{});
    case EPI_AXPY:
      if (d.a_km) return PRISM_EINVAL;
      if (pair) return launch(gemm_split_kernel<TM, TN, WR, WC, EPI_AXPY, false, false, true>, g);
      if constexpr (TM == TN) {
        if (d.sym) return launch(gemm_split_kernel<TM, TN, WR, WC, EPI_AXPY, false, true, false>, d);
      }
      return d.sym ? PRISM_EINVAL : launch(gemm_split_kernel<TM, TN, WR, WC, EPI_AXPY, false, false, false>, d);
  }
  return PRISM_EINVAL;
}

}  // namespace

int split_tiles(int M, int N, int batch, int sym) {
  const SplitTile T = split_tile(M, N, batch, sym);
  const int tm = M / T.m, tn = N / T.n;
  return sym ? tm * (tm + 1) / 2 : tm * tn;
}

int launch_gemm_split(const GemmDesc& a, const GemmDesc* b, hipStream_t s) {
  if (b && (b->M != a.M || b->N != a.N || b->K != a.K || b->batch != a.batch || b->epi != a.epi || b->a_km != a.a_km || b->sym)) return PRISM_EINVAL;
  GemmPair g = {};
  g.d[0] = a;
  if (b) g.d[1] = *b;
  const SplitTile T = split_tile(a.M, a.N, (a.sel_batch ? a.sel_batch : a.batch) * (b ? 2 : 1), a.sym);
  if (T.m == 64) return launch_cfg<64, 64, 2, 2>(g, s);
  return T.n == 256 ? launch_cfg<128, 256, 2, 4>(g, s) : launch_cfg<128, 128, 2, 4>(g, s);
}

void launch_split3(const float* x, uint16_t* p, long long count, long long ps, hipStream_t s) {
  const long long groups = count / 8, wgs = (groups + 255) / 256;
  hipLaunchKernelGGL(split3_kernel, dim3((unsigned)(wgs < 4096 ? wgs : 4096)), dim3(256), 0, s, x, p, groups, ps);
}

}  // namespace prism
