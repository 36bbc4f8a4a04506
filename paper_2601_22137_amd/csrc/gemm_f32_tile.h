// One tile of an fp32 / fp64 product on the CDNA4 matrix cores, with the epilogues of the PRISM iterations: the device
// code of gemm_f32.hip (a launch per product) and flow.hip (all iterations of a call in one launch).
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
#pragma once
#include <type_traits>

#include "split3.h"

namespace prism {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int BK = 16;
constexpr int GEMM_NT = 256;

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Cache policy of stores that other workgroups of the launch read (sc1), and a buffer over them: 32-bit byte offsets, less
// than 2 GiB
constexpr int COH_AUX = 16;
__device__ inline __amdgpu_buffer_rsrc_t coherent_buffer(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7ffffff0, 0x00027000);
}

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
template <int OFF> __device__ inline double lds_b64(unsigned a) {
  double r;
  asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(r) : "v"(a), "n"(OFF));
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

// COH: other workgroups of the launch read the result.  It is written past the caches that are not coherent between XCDs
// (sc1, as agent-scope atomics have it), with 32-bit offsets within a matrix.
template <bool COH> __device__ inline void store_f32x4(float* base, long long at, f32x4 v) {
  if constexpr (!COH) *(f32x4*)(base + at) = v;
  else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), coherent_buffer(base), (int)at * 4, 0, COH_AUX);
}
template <bool COH> __device__ inline void store_f32(float* base, long long at, float v) {
  if constexpr (!COH) base[at] = v;
  else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), coherent_buffer(base), (int)at * 4, 0, COH_AUX);
}
template <bool COH> __device__ inline void store_f64(double* base, long long at, double v) {
  if constexpr (!COH) base[at] = v;
  else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), coherent_buffer(base), (int)at * 8, 0, COH_AUX);
}

// Tile (tm, tn) of matrix b; rem: its number within the matrix.  alpha_of(alpha), called by all threads behind the main loop,
// gives the coefficient; false (for all): the result is not wanted, nothing is stored.
// ST: slabs in the ring.  WIDE: offsets within the tile of an operand beyond 32 bits (a variant of its own: they cost
// registers in the loop).
template <typename TC, typename TB, int TM, int TN, int WGM, int WGN, int ST, int EPI, bool A_KM, bool SYM, bool WIDE, bool COH, class AlphaOf>
__device__ inline void gemm_tile(const GemmDesc& g, bool sym, int b, int rem, int per_mat, int tm, int tn, unsigned char* smem,
                                 AlphaOf alpha_of) {
  constexpr int WTM = TM / WGM, WTN = TN / WGN;  // wave tile
  constexpr int BM = WTM / 16, BN = WTN / 16;    // 16x16 blocks per wave
  static_assert(WGM * WGN == 4 && BM >= 1 && BN >= 1 && TM >= 32, "bad tiling");
  typedef KMajor<float, TM> AL;
  typedef KMajor<TB, TN> BL;
  constexpr int A_BYTES = TM * 64, B_BYTES = BL::BYTES, STAGE = A_BYTES + B_BYTES;
  constexpr int LDA = A_BYTES >= 4096 ? A_BYTES / 4096 : 1;   // load instructions per wave and slab
  constexpr int A_LANES = A_BYTES >= 4096 ? 64 : A_BYTES / 64;
  constexpr int LDB = B_BYTES >= 4096 ? B_BYTES / 4096 : 1;
  constexpr int B_LANES = B_BYTES >= 4096 ? 64 : B_BYTES / 64;   // active lanes (skinny B: a wave moves less than 1 KiB)
  constexpr int NL = LDA + LDB;

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
      const int unit = (it * 4 + wave) * A_LANES + lane, k = unit / AL::UNITS, u = (unit % AL::UNITS) ^ (AL::UPP * ((k >> 2) & AL::MASK));
      aoff[it] = ((off_t)k * (unsigned)g.lda + u * 4) * 4u;
    }
  } else {
    const int lu = (lane & 15) ^ ((wave * (A_LANES / 16) + lq) & 15);
#pragma unroll
    for (int it = 0; it < LDA; ++it) aoff[it] = ((off_t)((it * 4 + wave) * (A_LANES / 4) + 4 * lq + (lu >> 2)) * (unsigned)g.lda + (lu & 3) * 4) * 4u;
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
      unsigned char* dst = smem + slot * STAGE + wave * (A_LANES * 16) + u * 4096;
      if (A_LANES == 64 || lane < A_LANES) __builtin_amdgcn_global_load_lds((gptr_t)(Ab + kt * astep + (aoff[u] & keep)), (lptr_t)dst, 16, 0, 0);
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
      if constexpr (sizeof(TB) == 8 && !B2) {
        fb[s][q / 4][q % 4] = lds_b64<O + (q % 4) * BL::ROW>(frb[q / 4]);
      } else if constexpr (sizeof(TB) == 8) {
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
    if (ST == 4 || kt1 % CHUNK == 0) flush();   // longer rings: what remains behind KR belongs to the last partial sum
  }
  if (KR < KT) {   // K no multiple of ST slabs
    unrolled<ST - 1>([&](auto dt) { if (KR + decltype(dt)::value < KT) step(dt, KR + decltype(dt)::value); });
  }
  wait_vmcnt<0>();   // the requests past the end write into this workgroup's LDS: none may outlive it
  __syncthreads();   // ... nor the reuse of the ring below
  if constexpr (FLUSH) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j) acc[i][j] += ksum[i][j];
  }

  // ---- epilogue ----
  // Addends (COH; fp64, whose accesses the compiler keeps in order with the stores: 16 round trips) are requested at once,
  // ahead of the wait for alpha.
  constexpr bool ADDENDS = EPI == EPI_POLYQ || EPI == EPI_AXPY, AHEAD = COH && ADDENDS;
  f32x4 far[AHEAD ? BM : 1][AHEAD ? BN : 1], far2[AHEAD ? BM : 1][AHEAD ? BN : 1];
  const float* cin_b = (const float*)g.Cin + (long long)b * g.strideCin;
  const float* cin2_b = g.Cin2 + (long long)b * g.strideCin;
  if constexpr (AHEAD) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j) {
        const long long oi = (long long)(m0 + wm0 + i * 16 + lr) * g.ldcin + n0 + wn0 + j * 16 + 4 * lq;
        far[i][j] = *(const f32x4*)(cin_b + oi);
        if (EPI == EPI_AXPY && g.Cin2) far2[i][j] = *(const f32x4*)(cin2_b + oi);
      }
  }
  double min[EPI == EPI_MNEXT ? BM : 1][EPI == EPI_MNEXT ? BN : 1][4];
  if constexpr (EPI == EPI_MNEXT) {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          min[i][j][r] = ((const double*)g.Cin + (long long)b * g.strideCin)[(long long)(m0 + wm0 + i * 16 + 4 * r + lq) * g.ldcin + n0 + wn0 + j * 16 + lr];
  }
  float alpha = 1.0f;
  if (!alpha_of(alpha)) return;
  TC part = 0;
  // (the contractions below are spelled out: the same bits from every kernel that has this tile)
  if constexpr (sizeof(TC) == 4) {
    // register r of lane l: row lr of the block, column 4 lq + r: one 16-byte access per block and operand
    const float wc = g.cin_one_minus_alpha ? (1.0f - alpha) : g.c_in * apow(alpha, g.cin_alpha_pow);
    const float wa = g.acc_neg ? -apow(alpha, g.coef_is_alpha) : apow(alpha, g.coef_is_alpha);
    const float wc2 = apow(alpha, g.cin2_alpha_pow);
    float* Cb = (float*)g.C + (long long)b * g.strideC;
    const bool skew = SYM && g.sym_skew_bound > 0 && ((m0 < g.sym_skew_bound) != (n0 < g.sym_skew_bound));
#pragma unroll
    for (int i = 0; i < BM; ++i) {
      const int gi = m0 + wm0 + i * 16 + lr;
      f32x4 cin[BN], cin2[BN];
      if constexpr (ADDENDS) {
#pragma unroll
        for (int j = 0; j < BN; ++j) {
          const long long oi = (long long)gi * g.ldcin + n0 + wn0 + j * 16 + 4 * lq;
          cin2[j] = (f32x4){0, 0, 0, 0};
          if constexpr (AHEAD) {
            cin[j] = far[i][j];
            if (EPI == EPI_AXPY && g.Cin2) cin2[j] = far2[i][j];
          } else {
            cin[j] = *(const f32x4*)(cin_b + oi);
            if (EPI == EPI_AXPY && g.Cin2) cin2[j] = *(const f32x4*)(cin2_b + oi);
          }
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
            part = __builtin_fmaf(v[r], v[r], part);
          }
        } else if constexpr (EPI == EPI_POLYQ) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = __builtin_fmaf(alpha, v[r], g.c1 * cin[j][r]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = __builtin_fmaf(wa, v[r], wc * cin[j][r]);
          if (g.Cin2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = __builtin_fmaf(wc2, cin2[j][r], v[r]);
          }
        }
        store_f32x4<COH>(Cb, (long long)gi * g.ldc + gj, v);
        if (sym && tm != tn) {
          if (skew) v = -v;
#pragma unroll
          for (int r = 0; r < 4; ++r) store_f32<COH>(Cb, (long long)(gj + r) * g.ldc + gi, v[r]);
        }
      }
    }
    if (sym && tm != tn) part *= 2.0f;
  } else {
    // register r of lane l: row 4 r + lq of the block, column lr
    // With planes of the residual, the wave passes it through a strip of its own (the ring is free), for rows in runs of eight columns.
    constexpr int WTM = TM / WGM, WTN = TN / WGN, SW = WTN + 4;
    const bool planes = !COH && EPI == EPI_MNEXT && g.C3;
    float* strip = (float*)smem + wave * WTM * SW;
    static_assert(EPI != EPI_MNEXT || WGM * WGN * WTM * SW * 4 <= ST * STAGE, "strips in the ring");
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gi = m0 + wm0 + i * 16 + 4 * r + lq, gj = n0 + wn0 + j * 16 + lr;
          TC v = acc[i][j][r];
          const long long oc = (long long)gi * g.ldc + gj;
          TC* Cb = (TC*)g.C + (long long)b * g.strideC;
          if constexpr (EPI == EPI_STORE) {
            store_f64<COH>(Cb, oc, g.acc_neg ? -v : v);
          } else {
            const bool in = (gi < g.n_true && gj < g.n_true);
            v += min[i][j][r];
            store_f64<COH>(Cb, oc, in ? v : (TC)0);
            const TC res = in ? ((gi == gj ? (TC)1 : (TC)0) - v) : (TC)0;
            if (planes) strip[(i * 16 + 4 * r + lq) * SW + j * 16 + lr] = (float)res;
            else store_f32<COH>(g.R32out + (long long)b * g.strideR, (long long)gi * g.ldr + gj, (float)res);
            part = __builtin_fma(res, res, part);
          }
        }
    if (planes) {
      constexpr int LPR = WTN / 8, RPI = 64 / LPR;
#pragma unroll
      for (int it = 0; it < WTM / RPI; ++it) {
        const int row = it * RPI + lane / LPR, col = (lane % LPR) * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = strip[row * SW + col + e];
        const long long o = (long long)b * g.strideR + (long long)(m0 + wm0 + row) * g.ldr + n0 + wn0 + col;
        *(f32x4*)(g.R32out + o) = (f32x4){v[0], v[1], v[2], v[3]};
        *(f32x4*)(g.R32out + o + 4) = (f32x4){v[4], v[5], v[6], v[7]};
        s3_u32x4 q[3];
        split3(v, q);
#pragma unroll
        for (int k = 0; k < 3; ++k) *(s3_u32x4*)(g.C3 + k * g.psC + o) = q[k];
      }
      __syncthreads();   // the partial sums take the place of the strips
    }
  }
  if (EPI == EPI_RESIDUAL || EPI == EPI_MNEXT) {
    TC* red = (TC*)smem;                 // the ring is free behind the last barrier
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    if (t == 0) store_f32<COH>(g.rho_part + (long long)b * per_mat, rem, (float)(red[0] + red[1] + red[2] + red[3]));
  }
}

}  // namespace
}  // namespace prism
