// fp32 / fp64 GEMMs on the CDNA4 matrix cores (v_mfma_f32_16x16x4_f32, v_mfma_f64_16x16x4_f64)
// with the epilogues of the PRISM iterations fused in (Table 1 of the paper: residual
// R = I - G, polynomial Q = R/2 + alpha R^2, update X + X Q, inverse-Newton factors).
//
// One workgroup = 256 threads = 4 wavefronts computes one TM x TN tile of C for one matrix of
// the batch.  K is consumed in slabs of BK = 16 that go from global memory straight into an LDS ring of
// ST slabs (no staging registers, loads run ST slabs ahead of the MFMAs).  The fragments of slab t + 1
// are read into a second register set while the MFMAs of slab t run, and the one barrier of a slab
// sits behind them, so that neither the LDS latency nor the load latency is on the path of the
// matrix pipe.  All operand sizes are padded to tile multiples by the caller, so the main loop has no
// bounds checks; masks are applied in the epilogue only.
//
// What bounds it: the fp32 (fp64) matrix pipe, 157 (79) TFLOP/s nominal.  Measured: 8192^3 147 TFLOP/s,
// 32 x 1024^3 140, fp64 32 x 1024^3 70.  (Slabs staged through registers, with the LDS writes, the barrier
// and the first fragment reads of a slab between its MFMAs and those of the next: 135, 120 and 60.)
//
// k order: MFMA step e of a slab takes k = 4 q + e from lane group q = lane / 16 (any order serves, as
// long as both operands agree): a K-contiguous A is then read with one 16-byte LDS read per row block
// and slab.
#include <type_traits>

#include <cstdlib>
#include <initializer_list>

#include "common.h"

namespace prism {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int BK = 16;
constexpr int NT = 256;

typedef const void __attribute__((address_space(1)))* gptr_t;
typedef void __attribute__((address_space(3)))* lptr_t;

__device__ inline f32x4 mfma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline f64x4 mfma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename T> struct Acc;
template <> struct Acc<float> { typedef f32x4 type; };
template <> struct Acc<double> { typedef f64x4 type; };

__device__ inline float apow(float alpha, int p) { return p == 0 ? 1.0f : (p == 1 ? alpha : alpha * alpha); }

template <int D, typename F>
__device__ inline void unrolled(F&& f) {
  if constexpr (D > 0) {
    unrolled<D - 1>(f);
    f(std::integral_constant<int, D - 1>{});
  }
}

// s_waitcnt vmcnt(N) with the other counters left alone (gfx9 encoding)
template <int N> __device__ inline void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// LDS reads as inline assembly: the compiler would otherwise treat them as possible readers of the
// slabs still on their way into LDS and wait for every outstanding load.  It does not know when their
// results arrive either: slab_barrier() below waits for them before anything may use them.
template <typename T> __device__ inline void keep(T v) { asm volatile("" ::"v"(v)); }   // v is in use up to here
template <int OFF> __device__ inline f32x4 lds_b128(unsigned a) {
  f32x4 r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(a), "n"(OFF));
  return r;
}
template <int OFF> __device__ inline float lds_b32(unsigned a) {
  float r;
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(a), "n"(OFF));
  return r;
}
template <int O0, int O1> __device__ inline f32x2 lds_2st64_b32(unsigned a) {   // offsets in units of 256 bytes
  f32x2 r;
  asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(r) : "v"(a), "n"(O0), "n"(O1));
  return r;
}
template <int O0, int O1> __device__ inline f64x2 lds_2st64_b64(unsigned a) {   // offsets in units of 512 bytes
  f64x2 r;
  asm volatile("ds_read2st64_b64 %0, %1 offset0:%2 offset1:%3" : "=v"(r) : "v"(a), "n"(O0), "n"(O1));
  return r;
}

// A slab of an operand stored with K as the slow index, [16 k][T columns]: rows of T * sizeof(E) bytes.
// A fragment read takes 16 consecutive columns of the four rows 4 q + e; the 16-column pieces of row k
// are stored xor-ed with (k / 4) & MASK so that the four lane groups (fp64: the two groups served at
// once) fall on different banks.
template <typename E, int T> struct KMajor {
  static constexpr int EB = (int)sizeof(E);
  static constexpr int ROW = T * EB;
  static constexpr int PIECES = T / 16;                        // 16-column pieces per row
  static constexpr int MASK = EB == 8 ? 1 : (PIECES >= 4 ? 3 : PIECES - 1);
  static constexpr int BYTES = BK * ROW;
  static constexpr int UNITS = ROW / 16;                       // 16-byte units per row
  static constexpr int UPP = EB;                               // ... per piece: 16 * EB / 16
};

// ST: slabs in the ring.  Two workgroups per CU with 128 x 128 tiles (register bound), more with small ones.
// PAIR: two products in a launch (a variant of its own: choosing the descriptor costs every launch 1 to 2 us).
template <bool PAIR> struct GemmArg { typedef GemmDesc type; };
template <> struct GemmArg<true> { typedef GemmPair type; };
// WIDE: offsets within the tile of an operand beyond 32 bits (a variant of its own: they cost registers in the loop).
template <typename TC, typename TB, int TM, int TN, int WGM, int WGN, int ST, int EPI, bool A_KM, bool SYM, bool PAIR, bool WIDE>
__global__ __launch_bounds__(NT, (TM * TN >= 128 * 128 ? 2 : 3)) void gemm_kernel(typename GemmArg<PAIR>::type arg) {
  int wg0 = 0, which = 0;
  if constexpr (PAIR) {
    which = (int)blockIdx.x >= arg.first;   // uniform
    wg0 = which ? arg.first : 0;
  }
  const GemmDesc& g = [&]() -> const GemmDesc& { if constexpr (PAIR) return arg.d[which]; else return arg; }();
  constexpr int WTM = TM / WGM, WTN = TN / WGN;  // wave tile
  constexpr int BM = WTM / 16, BN = WTN / 16;    // 16x16 blocks per wave
  static_assert(WGM * WGN == 4 && BM >= 1 && BN >= 1 && TM >= 64, "bad tiling");
  typedef KMajor<float, TM> AL;
  typedef KMajor<TB, TN> BL;
  constexpr int A_BYTES = TM * 64, B_BYTES = BL::BYTES, STAGE = A_BYTES + B_BYTES;
  constexpr int LDA = A_BYTES / 4096;                         // load instructions per wave and slab
  constexpr int LDB = B_BYTES >= 4096 ? B_BYTES / 4096 : 1;
  constexpr int B_LANES = B_BYTES >= 4096 ? 64 : B_BYTES / 64;   // active lanes (skinny B: a wave moves less than 1 KiB)
  constexpr int NL = LDA + LDB;
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

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);   // uniform: LDS destinations stay scalar
  const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;
  const int m0 = tm * TM, n0 = tn * TN;
  const int lr = lane & 15, lq = lane >> 4;
  const char* Ab = (const char*)((const float*)g.A + (long long)b * g.strideA + (A_KM ? (long long)m0 : (long long)m0 * g.lda));
  const char* Bb = (const char*)((const TB*)g.B + (long long)b * g.strideB + n0);
  const long long astep = A_KM ? (long long)BK * g.lda * 4 : (long long)BK * 4;   // bytes from slab to slab
  const long long bstep = (long long)BK * g.ldb * (int)sizeof(TB);

  // Global -> LDS (global_load_lds_dwordx4): a wave instruction fills 64 consecutive 16-byte units of LDS;
  // every lane fetches the unit that belongs at its place.
  // K-contiguous A: rows of 64 bytes (16 k), four to a 256-byte line, unit (row & 3, c) at slot
  // ((row & 3) * 4 + c) ^ (line & 15), conflict free for 16 consecutive rows reading the same c.
  typedef std::conditional_t<WIDE, unsigned long long, unsigned> off_t;
  off_t aoff[LDA], boff[LDB];
  if constexpr (A_KM) {
#pragma unroll
    for (int it = 0; it < LDA; ++it) {
      const int unit = (it * 4 + wave) * 64 + lane, k = unit / AL::UNITS, u = (unit % AL::UNITS) ^ (AL::UPP * ((k >> 2) & AL::MASK));
      aoff[it] = ((off_t)k * (unsigned)g.lda + u * 4) * 4u;
    }
  } else {
    const int lu = (lane & 15) ^ ((wave * 4 + lq) & 15);
#pragma unroll
    for (int it = 0; it < LDA; ++it) aoff[it] = ((off_t)((it * 4 + wave) * 16 + 4 * lq + (lu >> 2)) * (unsigned)g.lda + (lu & 3) * 4) * 4u;
  }
#pragma unroll
  for (int it = 0; it < LDB; ++it) {
    const int unit = (it * 4 + wave) * B_LANES + lane, k = unit / BL::UNITS, u = (unit % BL::UNITS) ^ (BL::UPP * ((k >> 2) & BL::MASK));
    boff[it] = (off_t)k * (unsigned)g.ldb * (unsigned)sizeof(TB) + (unsigned)u * 16u;
  }
  // Requests are unconditional, so that the number of younger ones in flight is a constant at every wait.
  // Past the end the offsets collapse to zero: the whole wave then fetches the same 16 bytes of the
  // first slab (and nobody reads the result).
  const int KT = g.K / BK;
  auto issue_load = [&](int kt, int slot, int u) {   // u in [0, NL): first the LDA of A, then the LDB of B
    const off_t keep = kt < KT ? ~(off_t)0 : 0;      // uniform
    if (kt >= KT) kt = 0;
    if (u < LDA) {
      unsigned char* dst = smem + slot * STAGE + wave * 1024 + u * 4096;
      __builtin_amdgcn_global_load_lds((gptr_t)(Ab + kt * astep + (aoff[u] & keep)), (lptr_t)dst, 16, 0, 0);
    } else if (B_LANES == 64 || lane < B_LANES) {
      unsigned char* dst = smem + slot * STAGE + A_BYTES + wave * (B_LANES * 16) + (u - LDA) * 4096;
      __builtin_amdgcn_global_load_lds((gptr_t)(Bb + kt * bstep + (boff[u - LDA] & keep)), (lptr_t)dst, 16, 0, 0);
    }
  };

  // fragment addresses within slot 0
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  unsigned fra[BM], frb[BN];
#pragma unroll
  for (int i = 0; i < BM; ++i) {
    const int row = wm0 + 16 * i + lr;
    if (A_KM) fra[i] = lds0 + (unsigned)(4 * lq * AL::ROW + (((wm0 / 16 + i) ^ (lq & AL::MASK)) * 16 + lr) * 4);
    else fra[i] = lds0 + (unsigned)((row >> 2) * 256 + ((((row & 3) << 2) + lq) ^ ((row >> 2) & 15)) * 16);
  }
#pragma unroll
  for (int j = 0; j < BN; ++j)
    frb[j] = lds0 + (unsigned)(A_BYTES + 4 * lq * BL::ROW + (((wn0 / 16 + j) ^ (lq & BL::MASK)) * 16 + lr) * BL::EB);

  float fa[2][BM][4];      // fragments: [set][block][MFMA step]
  TB fb[2][BN][4];
  constexpr bool A2 = AL::ROW % 256 == 0, B2 = BL::ROW % (BL::EB == 8 ? 512 : 256) == 0;   // two rows per read instruction
  constexpr int NRA = A_KM ? BM * (A2 ? 2 : 4) : BM, NRB = BN * (B2 ? 2 : 4), NR = NRA + NRB;   // read instructions per slab
  auto read_frag = [&](auto stag, auto slottag, auto rtag) {   // read instruction r of the slab in `slot` into set s
    constexpr int s = decltype(stag)::value, r = decltype(rtag)::value;
    constexpr int O = decltype(slottag)::value * STAGE;
    if constexpr (r < NRA) {
      if constexpr (!A_KM) {
        const f32x4 v = lds_b128<O>(fra[r]);
#pragma unroll
        for (int e = 0; e < 4; ++e) fa[s][r][e] = v[e];
      } else if constexpr (A2) {
        constexpr int i = r / 2, e = (r % 2) * 2;
        const f32x2 v = lds_2st64_b32<(O + e * AL::ROW) / 256, (O + (e + 1) * AL::ROW) / 256>(fra[i]);
        fa[s][i][e] = v[0]; fa[s][i][e + 1] = v[1];
      } else {
        fa[s][r / 4][r % 4] = lds_b32<O + (r % 4) * AL::ROW>(fra[r / 4]);
      }
    } else {
      constexpr int q = r - NRA;
      if constexpr (sizeof(TB) == 8) {
        constexpr int j = q / 2, e = (q % 2) * 2;
        const f64x2 v = lds_2st64_b64<(O + e * BL::ROW) / 512, (O + (e + 1) * BL::ROW) / 512>(frb[j]);
        fb[s][j][e] = v[0]; fb[s][j][e + 1] = v[1];
      } else if constexpr (B2) {
        constexpr int j = q / 2, e = (q % 2) * 2;
        const f32x2 v = lds_2st64_b32<(O + e * BL::ROW) / 256, (O + (e + 1) * BL::ROW) / 256>(frb[j]);
        fb[s][j][e] = v[0]; fb[s][j][e + 1] = v[1];
      } else {
        fb[s][q / 4][q % 4] = lds_b32<O + (q % 4) * BL::ROW>(frb[q / 4]);
      }
    }
  };

  typename Acc<TC>::type acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j) acc[i][j] = (typename Acc<TC>::type){0, 0, 0, 0};

  // Long fp32 sums are accumulated in two levels (partial sums of 256 terms inside the matrix
  // core accumulator, then added up in registers): the rounding error then grows like the square
  // root of the chunk length instead of that of K, which the 1e-5 parity bar needs at K = 8192.
  constexpr bool FLUSH = sizeof(TC) == 4;
  constexpr int CHUNK = 16;                        // slabs per partial sum (256 k)
  static_assert(CHUNK % ST == 0 && ST % 2 == 0, "the ring turns a whole number of times per partial sum");
  typename Acc<TC>::type ksum[FLUSH ? BM : 1][FLUSH ? BN : 1];
  if (FLUSH) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j) ksum[i][j] = (typename Acc<TC>::type){0, 0, 0, 0};
  }
  auto flush = [&]() {
    if constexpr (FLUSH) {
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) {
          ksum[i][j] += acc[i][j];
          acc[i][j] = (typename Acc<TC>::type){0, 0, 0, 0};
        }
    }
  };
  // fp32: operands swapped, so that a lane ends up with four consecutive columns of one row of C
  auto mma = [&](int s, int e, int i, int j) {
    if constexpr (sizeof(TC) == 4) acc[i][j] = mfma(fb[s][j][e], fa[s][i][e], acc[i][j]);
    else acc[i][j] = mfma((TC)fa[s][i][e], (TC)fb[s][j][e], acc[i][j]);
  };

  // Barrier of a slab: this wave's fragments have arrived and its share of the slab after the next one has
  // landed (`younger` slabs may still be in flight); behind it every wave may read that slab and the slot
  // whose fragments are all in registers may be refilled.
  auto slab_barrier = [&](auto ytag) {
    wait_vmcnt<decltype(ytag)::value * NL>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int d = 0; d < ST; ++d)
#pragma unroll
    for (int u = 0; u < NL; ++u) issue_load(d, d, u);
  slab_barrier(std::integral_constant<int, ST - 1>{});
  unrolled<NR>([&](auto r) { read_frag(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, r); });
  slab_barrier(std::integral_constant<int, ST - 2>{});

  constexpr int NM = 4 * BM * BN;              // MFMAs per slab
  constexpr int NO = NR + NL;                  // other instructions to place among them
  // slab kt = d (mod ST): its fragments are in set d & 1; slab kt + 1 is in slot d + 1
  auto step = [&](auto dtag, int kt) {
    constexpr int d = decltype(dtag)::value;
    constexpr int EVERY = NM / NO > 0 ? NM / NO : 1;
    unrolled<(NM > NO ? NM : NO)>([&](auto utag) {
      constexpr int u = decltype(utag)::value;
      if constexpr (u < NM) {
        mma(d & 1, u / (BM * BN), (u / BN) % BM, u % BN);
        __builtin_amdgcn_sched_barrier(0);
      }
      // reads first (their results are wanted at the end of the slab), then the loads
      constexpr int o = (u % EVERY == 0) ? u / EVERY : NO;
      if constexpr (o < NR) {
        read_frag(std::integral_constant<int, (d + 1) & 1>{}, std::integral_constant<int, (d + 1) % ST>{}, std::integral_constant<int, o>{});
        __builtin_amdgcn_sched_barrier(0);
      } else if constexpr (o < NO) {
        issue_load(kt + ST, d, o - NR);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    slab_barrier(std::integral_constant<int, ST - 2>{});
    // the registers of a read stay its own until it has returned, also where nobody uses the result
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int i = 0; i < BM; ++i) keep(fa[(d + 1) & 1][i][e]);
#pragma unroll
      for (int j = 0; j < BN; ++j) keep(fb[(d + 1) & 1][j][e]);
    }
  };
  // Two nested loops, so that inside the inner one the accumulators are touched by MFMAs only; the
  // partial sums are closed between inner loops.
  const int KR = KT / ST * ST;
  for (int kt0 = 0; kt0 < KR; kt0 += CHUNK) {
    const int kt1 = kt0 + CHUNK < KR ? kt0 + CHUNK : KR;
    for (int kt = kt0; kt < kt1; kt += ST)
      unrolled<ST>([&](auto dt) { step(dt, kt + decltype(dt)::value); });
    flush();
  }
  if (KR < KT) {   // K no multiple of ST slabs
    step(std::integral_constant<int, 0>{}, KR);
    if (KR + 1 < KT) step(std::integral_constant<int, 1>{}, KR + 1);
    if (KR + 2 < KT) step(std::integral_constant<int, 2>{}, KR + 2);
  }
  static_assert(ST == 4, "the remainder lists the steps of a four-slab ring");
  wait_vmcnt<0>();   // the requests past the end write into this workgroup's LDS: none may outlive it
  __syncthreads();   // ... nor the reuse of the ring below
  if constexpr (FLUSH) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j) acc[i][j] += ksum[i][j];
  }

  // ---- epilogue ----
  TC part = 0;
  if constexpr (sizeof(TC) == 4) {
    // register r of lane l: row lr of the block, column 4 lq + r: one 16-byte access per block and operand
    const float wc = g.cin_one_minus_alpha ? (1.0f - alpha) : g.c_in * apow(alpha, g.cin_alpha_pow);
    const float wa = g.acc_neg ? -apow(alpha, g.coef_is_alpha) : apow(alpha, g.coef_is_alpha);
    const float wc2 = apow(alpha, g.cin2_alpha_pow);
    const bool skew = SYM && g.sym_skew_bound > 0 && ((m0 < g.sym_skew_bound) != (n0 < g.sym_skew_bound));
#pragma unroll
    for (int i = 0; i < BM; ++i) {
      const int gi = m0 + wm0 + i * 16 + lr;
      f32x4 cin[BN], cin2[BN];
      if constexpr (EPI == EPI_POLYQ || EPI == EPI_AXPY) {
#pragma unroll
        for (int j = 0; j < BN; ++j) {
          const long long oi = (long long)b * g.strideCin + (long long)gi * g.ldcin + n0 + wn0 + j * 16 + 4 * lq;
          cin[j] = *(const f32x4*)((const float*)g.Cin + oi);
          cin2[j] = (f32x4){0, 0, 0, 0};
          if (EPI == EPI_AXPY && g.Cin2) cin2[j] = *(const f32x4*)(g.Cin2 + oi);
        }
      }
#pragma unroll
      for (int j = 0; j < BN; ++j) {
        const int gj = n0 + wn0 + j * 16 + 4 * lq;
        f32x4 v = acc[i][j];
        if constexpr (EPI == EPI_STORE) {
          if (g.acc_neg) v = -v;
        } else if constexpr (EPI == EPI_RESIDUAL) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = (gi < g.n_true && gj + r < g.n_true) ? ((gi == gj + r ? 1.0f : 0.0f) - v[r]) : 0.0f;
            part += v[r] * v[r];
          }
        } else if constexpr (EPI == EPI_POLYQ) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = g.c1 * cin[j][r] + alpha * v[r];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = wc * cin[j][r] + wa * v[r];
          if (g.Cin2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] += wc2 * cin2[j][r];
          }
        }
        *(f32x4*)((float*)g.C + (long long)b * g.strideC + (long long)gi * g.ldc + gj) = v;
        if (sym && tm != tn) {
          if (skew) v = -v;
#pragma unroll
          for (int r = 0; r < 4; ++r) ((float*)g.C)[(long long)b * g.strideC + (long long)(gj + r) * g.ldc + gi] = v[r];
        }
      }
    }
    if (sym && tm != tn) part *= 2.0f;
  } else {
    // register r of lane l: row 4 r + lq of the block, column lr
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gi = m0 + wm0 + i * 16 + 4 * r + lq, gj = n0 + wn0 + j * 16 + lr;
          TC v = acc[i][j][r];
          const long long oc = (long long)b * g.strideC + (long long)gi * g.ldc + gj;
          if constexpr (EPI == EPI_STORE) {
            ((TC*)g.C)[oc] = g.acc_neg ? -v : v;
          } else {
            const bool in = (gi < g.n_true && gj < g.n_true);
            if (g.Cin) v += ((const TC*)g.Cin)[(long long)b * g.strideCin + (long long)gi * g.ldcin + gj];
            ((TC*)g.C)[oc] = in ? v : (TC)0;
            const TC res = in ? ((gi == gj ? (TC)1 : (TC)0) - v) : (TC)0;
            g.R32out[(long long)b * g.strideR + (long long)gi * g.ldr + gj] = (float)res;
            part += res * res;
          }
        }
  }
  if (EPI == EPI_RESIDUAL || EPI == EPI_MNEXT) {
    TC* red = (TC*)smem;                 // the ring is free behind the last barrier
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    if (t == 0) g.rho_part[(long long)b * per_mat + rem] = (float)(red[0] + red[1] + red[2] + red[3]);
  }
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
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(NT), lds, s, arg);
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
    if ((q->epi == EPI_POLYQ || q->epi == EPI_AXPY) && (!q->Cin || q->ldcin % 4)) return PRISM_EINVAL;
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
