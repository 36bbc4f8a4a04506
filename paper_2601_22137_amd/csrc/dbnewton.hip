// Pieces of the PRISM DB Newton iteration in product form (paper App. A.2):
//   N_k = M_k^{-1} for symmetric positive definite M_k   (the paper factors M_k; here: in-place
//         block Gauss-Jordan elimination without pivoting, which is stable for SPD matrices)
//   g00 = <D0,D0>, g02 = <D0,D2>, g22 = <D2,D2>,  D0 = M - I, D2 = M + N - 2I
//         (the O(n^2) quantities behind the quartic m(alpha) = ||I - M_{k+1}||_F^2; the printed
//         trace combinations expand these inner products and cancel badly near convergence)
//   M_{k+1} = 2a(1-a) I + (1-a)^2 M_k + a^2 N_k
// Block Gauss-Jordan: for every pivot block k
//   P = A_kk^{-1},  A_kj <- P A_kj  (j != k),  A_ij <- A_ij - A_ik A_kj  (i, j != k),  A_ik <- -A_ik P  (i != k),  A_kk <- P
// Two levels: outer pivot blocks of 512 or 256, whose rank updates are launches of the fp32 GEMM kernel (>= 64 flop per
// byte of the matrix they sweep; with blocks of 64 the sweep is HBM bound), each inverted by the same
// elimination with pivots of 64, which one workgroup inverts in fp64 (larger ones would be fewer steps, but an
// inverse of order 128 rounded to fp32 costs the ill-conditioned cases accuracy: 2.9e-4 against 2e-4 at cond 1e4).
// The new row panel of an outer block goes to scratch; from there the row and, transposed, the column are written.
#include "common.h"

namespace prism {
namespace {

constexpr int NT = 256;

__global__ __launch_bounds__(NT) void copy_kernel(const float* __restrict__ src, float* __restrict__ dst, long long per_mat,
                                                  const Ctrl* __restrict__ ctrl) {
  const int b = blockIdx.y;
  if (ctrl && ctrl[b].done) return;
  const long long i = ((long long)blockIdx.x * NT + threadIdx.x) * 4;
  if (i < per_mat) *(float4*)(dst + (long long)b * per_mat + i) = *(const float4*)(src + (long long)b * per_mat + i);
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int BS = 64;   // pivots of the elimination

// value of lane P of every group of 16 lanes, to all lanes of the group
template <int P> __device__ inline double bcast16(double v) {
  const long long w = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)w, 0x150 + P, 0xF, 0xF, false);           // row_newbcast:P
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(w >> 32), 0x150 + P, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
template <int L> __device__ inline double from_lane(double v) {   // uniform
  const long long w = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)w, L), hi = __builtin_amdgcn_readlane((int)(w >> 32), L);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// 1 / x: the hardware's approximation (2^-24) and two Newton steps, to an ulp; the last instruction puts 0 and infinity where a division
// has them (an infinite pivot, one that has vanished), which the Newton steps leave as not-a-number.  (By division behind a
// test of the exponent: 2 x 2048^2 6.00 ms, not 5.72.)
__device__ inline double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-x, r, 1.0), r, r), x, 1.0);
}
// One elimination step of the 16 x 16 inverse below: pivot P.  A chain of latencies, 16 of them in each of the four steps of a 64 x 64
// inverse: with an exact division 2 x 512^2 160 us, not 152.  (The pivot column by exchanges of lane halves and rows instead of the
// shuffle: 164.)
template <int P> __device__ inline void invert16_step(double (&e)[4], int lr, int lq) {
  constexpr int G = P >> 2, C = P & 3;           // the pivot column sits in lane group G, register C
  const double inv = reciprocal(from_lane<G * 16 + P>(e[C]));
  const double f = __shfl(e[C], G * 16 + lr, 64);
  double rw[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) rw[s] = bcast16<P>(e[s]) * inv;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const bool pc = s == C && lq == G;
    if (lr == P) e[s] = pc ? inv : rw[s];
    else e[s] = pc ? -f * inv : e[s] - f * rw[s];
  }
}
// Inverse of a 16 x 16 matrix held by one wave: lane (lr = l % 16, lq = l / 16), register s: entry [lr][4 lq + s].
template <int P = 0> __device__ inline void invert16(double (&e)[4], int lr, int lq) {
  invert16_step<P>(e, lr, lq);
  if constexpr (P + 1 < 16) invert16<P + 1>(e, lr, lq);
}

// LDS written and read by the same wave: the operations of a wave complete in order, only the
// compiler has to keep them so
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inverse of a 64 x 64 matrix by one workgroup (four wavefronts) in fp64.  Wave w holds rows 16 w .. 16 w + 15 as
// the accumulators of v_mfma_f64_16x16x4_f64 (acc[j], register r of lane (lr, lq): row 4 r + lq, column 16 j + lr).
// Block Gauss-Jordan with 16 x 16 pivots D, one barrier per pivot: the owner of the pivot row shares it through
// LDS; every wave inverts D by itself (handing the inverse round would cost a second barrier); wave i forms
// B = A_ik D^-1 and takes A_ij -= B A_kj (j != k), A_ik = -B; the owner takes A_kj = D^-1 A_kj, A_kk = D^-1.
// B is formed as its transpose, whose accumulator layout is the operand layout of the update.
constexpr int RSD = BS + 16;               // rows 128 bytes apart modulo 256: two lane groups fall on different banks
struct Inv64Lds {
  double row[2][16][RSD];                  // pivot row, double buffered
  double scr[4][16][17];                   // per wave: transposes
};
__device__ inline void invert64(f64x4 (&acc)[4], Inv64Lds& m) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double (*scr)[17] = m.scr[w];
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {
    double (*pr)[RSD] = m.row[k & 1];      // the other buffer may still be read from the step before
    if (w == k) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) pr[4 * r + lq][16 * j + lr] = acc[j][r];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j == k) {
#pragma unroll
          for (int r = 0; r < 4; ++r) scr[4 * r + lq][lr] = acc[j][r];
        }
    }
    __syncthreads();
    double e[4];                           // the owner inverts D, the others D^T (symmetric up to rounding only)
#pragma unroll
    for (int s = 0; s < 4; ++s) e[s] = w == k ? pr[lr][16 * k + 4 * lq + s] : pr[4 * lq + s][16 * k + lr];
    invert16(e, lr, lq);
    f64x4 own;                             // new block k of this wave
    if (w == k) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f64x4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(e[s], pr[4 * lq + s][16 * j + lr], c, 0, 0, 0);
        acc[j] = c;
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) scr[lr][4 * lq + s] = e[s];
    } else {
      f64x4 bt = {0.0, 0.0, 0.0, 0.0};     // register r: B[lr][4 r + lq]
#pragma unroll
      for (int s = 0; s < 4; ++s) bt = __builtin_amdgcn_mfma_f64_16x16x4f64(e[s], scr[lr][4 * lq + s], bt, 0, 0, 0);
      wave_lds_fence();
      bt = -bt;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(bt[s], pr[4 * s + lq][16 * j + lr], acc[j], 0, 0, 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) scr[lr][4 * s + lq] = bt[s];
    }
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) own[r] = scr[4 * r + lq][lr];
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j == k) acc[j] = own;
  }
}

// P = inverse of the leading 64 x 64 block of every matrix (the first pivot of an elimination); sync (may be null) is zeroed
__global__ __launch_bounds__(NT) void first_pivot_kernel(const float* __restrict__ S, long long stride, int ld,
                                                         float* __restrict__ P, unsigned* __restrict__ sync, const Ctrl* __restrict__ ctrl) {
  const int b = blockIdx.x;
  if (ctrl && ctrl[b].done) return;
  __shared__ Inv64Lds m;
  if (sync && threadIdx.x < FIT_SYNC_WORDS) sync[(long long)b * FIT_SYNC_WORDS + threadIdx.x] = 0u;
  static_assert(FIT_SYNC_WORDS <= NT, "one pass");
  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4, w = threadIdx.x >> 6;
  const float* blk = S + (long long)b * stride + (long long)(16 * w + lq) * ld + lr;
  f64x4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[j][r] = (double)blk[(long long)(4 * r) * ld + 16 * j];
  invert64(acc, m);
  float* out = P + (long long)b * 2 * BS * BS;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(16 * w + 4 * r + lq) * BS + 16 * j + lr] = (float)acc[j][r];
}

// 32 x 32 quadrant of a 64 x 64 x 64 product: acc[i][j] = A B, both operands in LDS, rows of SL floats.
// k order: lane group lq takes k = 16 c + 4 lq + e at step e, so that A comes as one 16-byte read per row and
// chunk; with SL = 68 the four rows of a B read lie 64 bytes apart modulo 256.
constexpr int SL = BS + 4;
__device__ inline void mma64(const float* As, const float* Bs, int m0, int n0, f32x4 (&acc)[2][2]) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    f32x4 a[2];
    float bv[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = *(const f32x4*)(As + (m0 + 16 * i + lr) * SL + 16 * c + 4 * lq);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[j][e] = Bs[(16 * c + 4 * lq + e) * SL + n0 + 16 * j + lr];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], bv[j][e], acc[i][j], 0, 0, 0);
  }
}

// One elimination step with the 64 x 64 pivot k of an n x n matrix, from S to D (a tile is read by many
// workgroups, so not in place), tile (ti, tj):
//   D_kk = P, D_kj = P S_kj, D_ik = -S_ik P, D_ij = S_ij - S_ik (P S_kj),
// P = S_kk^-1 from the step before.  `pivot` (tile (k + 1, k + 1)): inverts its result, P of the next step.
// Every tile forms P S_kj for itself, twice the products of the update alone, instead of a launch of its own for the pivot row and
// one for the column.  COH: the other tiles are done by workgroups of the same launch: past the caches that are not coherent
// between XCDs (sc1, as agent-scope atomics have it), in rows of 16 bytes per lane through LDS; otherwise straight from the
// registers of the product (through LDS a launch of 400 tiles took 3 % longer: order 1280 391 -> 402 us).
union JordanLds {
  float t[3][BS * SL];                       // P, S_kj (later P S_kj), S_ik (later the result)
  Inv64Lds inv;                              // over the first two
};
static_assert(sizeof(Inv64Lds) <= 2 * BS * SL * sizeof(float), "the inverse leaves the third array alone");
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ inline __amdgpu_buffer_rsrc_t past_caches(const void* base) { return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7ffffff0, 0x00027000); }
// Entry (row, col) of a matrix with leading dimension ld.  A matrix may have more than 2^31 entries where a step is a launch; one that is swept in one
// launch has 512 tiles at most, and offsets below 2^29.
template <bool COH> using offset_t = std::conditional_t<COH, int, long long>;
template <bool COH> __host__ __device__ constexpr offset_t<COH> offset_of(int row, int ld, int col) { return (offset_t<COH>)row * ld + col; }
static_assert(offset_of<false>(46399, 46400, 46336) == 46399ll * 46400 + 46336, "in 64 bits");
template <bool COH> __device__ inline f32x4 get4(const float* base, offset_t<COH> at) {
  if constexpr (COH) return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(past_caches(base), at * 4, 0, 16));
  else return *(const f32x4*)(base + at);
}
template <bool COH> __device__ inline void put4(float* base, offset_t<COH> at, f32x4 v) {
  if constexpr (COH) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), past_caches(base), at * 4, 0, 16);
  else *(f32x4*)(base + at) = v;
}
template <bool COH>
__device__ inline void jordan_tile(const float* S, int sld, float* D, int dld, const float* P, float* Pnext, int k, int ti, int tj, bool pivot, JordanLds& m) {
  const int t = threadIdx.x, lane = t & 63, lr = lane & 15, lq = lane >> 4, w = t >> 6;
  const bool prow = ti == k, pcol = tj == k;
  const int r0 = t >> 4, c0 = (t & 15) * 4;   // copies: 16 rows of 16 bytes per thread and pass
  const int m0 = (w >> 1) * 32, n0 = (w & 1) * 32;
  f32x4 vp[4], vb[4], va[4], old[4];          // old: rows, or blocks (i, j) of the product at 2 i + j
  auto entry = [&](int i, int j, int r, int ld) { return offset_of<COH>(ti * BS + m0 + 16 * i + 4 * lq + r, ld, tj * BS + n0 + 16 * j + lr); };
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + 16 * q;
    vp[q] = get4<COH>(P, r * BS + c0);
    vb[q] = pcol ? vp[q] : get4<COH>(S, offset_of<COH>(k * BS + r, sld, tj * BS + c0));
    va[q] = prow ? vp[q] : get4<COH>(S, offset_of<COH>(ti * BS + r, sld, k * BS + c0));
    old[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if (COH && !prow && !pcol) old[q] = get4<COH>(S, offset_of<COH>(ti * BS + r, sld, tj * BS + c0));
  }
  if (prow && pcol) {
#pragma unroll
    for (int q = 0; q < 4; ++q) put4<COH>(D, offset_of<COH>(ti * BS + r0 + 16 * q, dld, tj * BS + c0), vp[q]);
    return;
  }
  if (!COH && !prow && !pcol) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) old[q][r] = S[entry(q >> 1, q & 1, r, sld)];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int o = (r0 + 16 * q) * SL + c0;
    *(f32x4*)&m.t[0][o] = vp[q]; *(f32x4*)&m.t[1][o] = vb[q]; *(f32x4*)&m.t[2][o] = va[q];
  }
  __syncthreads();
  f32x4 acc[2][2];
  auto into = [&](float* x) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[(m0 + 16 * i + 4 * lq + r) * SL + n0 + 16 * j + lr] = acc[i][j][r];
  };
  if (!pcol) {                               // T = P S_kj
    mma64(m.t[0], m.t[1], m0, n0, acc);
    if (!prow) {
      __syncthreads();
      into(m.t[1]);
      __syncthreads();
    }
  }
  if (!prow) mma64(m.t[2], m.t[1], m0, n0, acc);   // S_ik T, or S_ik P
  if constexpr (COH) {
    __syncthreads();
    into(m.t[2]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float* p = &m.t[2][(r0 + 16 * q) * SL + c0];
      f32x4 v = *(const f32x4*)p;
      if (!prow) v = old[q] - v;
      put4<COH>(D, offset_of<COH>(ti * BS + r0 + 16 * q, dld, tj * BS + c0), v);
      if (pivot) *(f32x4*)p = v;
    }
    if (!pivot) return;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4& a = acc[q >> 1][q & 1];
      if (!prow) a = old[q] - a;
#pragma unroll
      for (int r = 0; r < 4; ++r) D[entry(q >> 1, q & 1, r, dld)] = a[r];
    }
    if (!pivot) return;
    __syncthreads();
    into(m.t[2]);
  }
  __syncthreads();
  f64x4 v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[j][r] = (double)m.t[2][(16 * w + 4 * r + lq) * SL + 16 * j + lr];
  invert64(v, m.inv);
  if constexpr (!COH) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) Pnext[(16 * w + 4 * r + lq) * BS + 16 * j + lr] = (float)v[j][r];
    return;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) m.t[2][(16 * w + 4 * r + lq) * SL + 16 * j + lr] = (float)v[j][r];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) put4<COH>(Pnext, (r0 + 16 * q) * BS + c0, *(const f32x4*)&m.t[2][(r0 + 16 * q) * SL + c0]);
}

// A step for all tiles of every matrix: one workgroup each, the pivot the first of its matrix.  What bounds it: on small matrices that
// inverse (a serial chain; the other tiles finish meanwhile), on large ones the sweep of S and D.
// 2 x 2048^2, a block of 512: 8 steps of 17 us; the pivot kernel of one barrier per row (87 us) and the three products
// that this replaces took 8 times 105 us.
struct StepArgs {
  const float* S; long long sstride; int sld;
  float* D; long long dstride; int dld;
  float* P;                                  // [batch][2][64][64]: slot k & 1 is read, the other written
  int nt, k;
  const Ctrl* ctrl;
};
__global__ __launch_bounds__(NT) void jordan_step_kernel(StepArgs g) {
  const int b = blockIdx.y;
  if (g.ctrl && g.ctrl[b].done) return;
  __shared__ __align__(16) JordanLds m;
  const bool more = g.k + 1 < g.nt;
  const int next = more ? (g.k + 1) * (g.nt + 1) : 0;
  const int idx = blockIdx.x == 0 ? next : ((int)blockIdx.x == next ? 0 : (int)blockIdx.x);
  float* P = g.P + (long long)b * 2 * BS * BS;
  jordan_tile<false>(g.S + (long long)b * g.sstride, g.sld, g.D + (long long)b * g.dstride, g.dld, P + (g.k & 1) * BS * BS, P + (~g.k & 1) * BS * BS, g.k,
                     idx / g.nt, idx % g.nt, more && blockIdx.x == 0, m);
}

// All steps in one launch: between steps a hand-over instead of a launch, and one launch instead of nt for every iteration enqueued past convergence.
// One workgroup of a matrix does the pivot tiles, one after the other, and waits for nothing but the tiles of the step before; the others take
// tiles by number.  What bounds it: the inverse of a pivot, 10 of 15 us per step.  2 x 512^2 (8 steps) 144 -> 135 us, 768 x 2 231 -> 211; in calls of DB
// Newton, whose budget is mostly past convergence, 2 x 2048^2 5.71 -> 5.22 ms, 2 x 512^2 0.995 -> 0.882.
// Waits end wherever the workgroups are: who waits holds a tile of step k and waits for steps before k, whose tiles have lower numbers and
// were taken by workgroups that run; the pivot workgroup, before it waits, takes what nobody has taken yet.
struct SweepArgs {
  const float* S; long long sstride; int sld;   // step k reads S (k = 0) or what k - 1 wrote, and writes tmp and out in turn, the last one out
  float* out; long long ostride; int old;
  float* tmp; long long tstride; int tld;
  float* P;                                  // as above
  unsigned* sync;                            // [batch][FIT_SYNC_WORDS], zeroed by the launch before: tiles taken, tiles done
  int nt;                                    // two at least
  const Ctrl* ctrl;
};
__global__ __launch_bounds__(NT, 3) void jordan_sweep_kernel(SweepArgs g) {
  const int b = blockIdx.y, t = threadIdx.x, nt = g.nt, all = nt * nt;
  if (g.ctrl && g.ctrl[b].done) return;
  __shared__ __align__(16) JordanLds m;
  __shared__ int s_job;
  constexpr int PIVOT = -1, LEAVE = -2;
  unsigned* taken = g.sync + (long long)b * FIT_SYNC_WORDS;
  unsigned* done = taken + 32;
  auto load = [](unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto take = [&]() { return (int)__hip_atomic_fetch_add(taken, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - 1; };
  // tiles by number: all - 1 in a step (without the next pivot), all in the last one
  const int total = nt * (all - 1) + 1;
  auto step_of = [&](int id) { const int k = id / (all - 1); return k < nt ? k : nt - 1; };
  auto wait = [&](int id) {                  // one thread: until all steps before that of tile id are done
    const unsigned need = (unsigned)(step_of(id) * all);
    while (load(done) < need) __builtin_amdgcn_s_sleep(1);
  };
  if (t == 0) s_job = take();
  __syncthreads();
  int id = __builtin_amdgcn_readfirstlane(s_job), kp = 0;
  bool chain = id < 0;                       // the first of its matrix: pivots, step kp next
  __syncthreads();
  float* P = g.P + (long long)b * 2 * BS * BS;
  for (;;) {
    if (t == 0) {
      if (chain) {
        for (;;) {
          if (load(done) >= (unsigned)(kp * all)) { s_job = PIVOT; break; }
          unsigned n = load(taken);          // one more than the tiles taken
          if ((int)n - 1 < kp * (all - 1)) {
            if (__hip_atomic_compare_exchange_strong(taken, &n, n + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
              wait((int)n - 1);
              s_job = (int)n - 1;
              break;
            }
          } else {
            __builtin_amdgcn_s_sleep(1);
          }
        }
      } else {
        if (id < 0) id = take();
        if (id >= total) s_job = LEAVE;
        else { wait(id); s_job = id; }
      }
    }
    __syncthreads();
    const int job = __builtin_amdgcn_readfirstlane(s_job);
    if (job == LEAVE) return;
    int k, idx;
    if (job == PIVOT) {
      k = kp;
      idx = (k + 1) * (nt + 1);
    } else {
      k = step_of(job);
      idx = job - k * (all - 1);
      if (k + 1 < nt && idx >= (k + 1) * (nt + 1)) ++idx;
    }
    const bool to_tmp = (nt - 1 - k) & 1;
    const float* S = k == 0 ? g.S + (long long)b * g.sstride : (to_tmp ? g.out + (long long)b * g.ostride : g.tmp + (long long)b * g.tstride);
    const int sld = k == 0 ? g.sld : (to_tmp ? g.old : g.tld);
    float* D = to_tmp ? g.tmp + (long long)b * g.tstride : g.out + (long long)b * g.ostride;
    jordan_tile<true>(S, sld, D, to_tmp ? g.tld : g.old, P + (k & 1) * BS * BS, P + (~k & 1) * BS * BS, k, idx / nt, idx % nt, job == PIVOT, m);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the tile has reached memory
    __syncthreads();
    if (t == 0) __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (job == PIVOT && ++kp == nt - 1) chain = false;
    id = -1;
  }
}

// grid (groups, batch): partial sums of the three inner products over the true n x n part; the
// five coefficient partials are written where the solve kernel adds them up.
__global__ __launch_bounds__(NT) void db_moments_kernel(const float* __restrict__ M, const float* __restrict__ N, int np,
                                                        int n_true, const Ctrl* __restrict__ ctrl, double* __restrict__ cpart) {
  const int b = blockIdx.y, grp = blockIdx.x, ngrp = gridDim.x;
  if (ctrl[b].done) return;
  const long long total = (long long)np * np;
  const float* Mb = M + (long long)b * total;
  const float* Nb = N + (long long)b * total;
  double g00 = 0.0, g02 = 0.0, g22 = 0.0;
  for (long long idx = ((long long)grp * NT + threadIdx.x) * 4; idx < total; idx += (long long)ngrp * NT * 4) {
    const int r = (int)(idx / np), c = (int)(idx % np);
    if (r >= n_true) break;
    const float4 m4 = *(const float4*)(Mb + idx), n4 = *(const float4*)(Nb + idx);
    const float mv[4] = {m4.x, m4.y, m4.z, m4.w}, nv[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (c + e < n_true) {
        const double eye = (r == c + e) ? 1.0 : 0.0;
        const double d0 = (double)mv[e] - eye, d2 = (double)mv[e] + (double)nv[e] - 2.0 * eye;
        g00 += d0 * d0; g02 += d0 * d2; g22 += d2 * d2;
      }
    }
  }
  __shared__ double red[4][3];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    g00 += __shfl_down(g00, off, 64); g02 += __shfl_down(g02, off, 64); g22 += __shfl_down(g22, off, 64);
  }
  if (lane == 0) { red[wave][0] = g00; red[wave][1] = g02; red[wave][2] = g22; }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double a = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
    const double c = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
    const double d = (red[0][2] + red[1][2]) + (red[2][2] + red[3][2]);
    double* out = cpart + ((long long)b * ngrp + grp) * 17;
    out[0] = a; out[1] = -4.0 * a; out[2] = 4.0 * a + 2.0 * c; out[3] = -4.0 * c; out[4] = d;
    for (int s = 5; s < 16; ++s) out[s] = 0.0;   // slot 16 belongs to the check of the inverse (db_probe_kernel)
  }
}

// Check of the inverse with one probe vector v of +-1 entries: ||M (N v) - v||^2 estimates
// ||M N - I||_F^2 (its expectation over such v), i.e. the error of N measured against the smallest
// entries of its spectrum, which is what the large components of X = A^(1/2) inherit.  Pass 0: w = N v.
// Pass 1: partial sums of (M w - v)^2 into slot 16 of the coefficient partials, which the solve
// kernel adds up.
// grid (groups, batch); a wave takes 4 rows at a time, four columns of loads (16 bytes a lane) in flight.  HBM or Infinity Cache bound once the
// chip has a workgroup per CU: 2 x 2048^2 39 us with 16 rows per wave (64 workgroups).  The
// padding needs no mask: M and N are the identity there, so padded rows reproduce v exactly.
__device__ inline float probe_entry(int c) { return ((unsigned)c * 2654435761u >> 16) & 1u ? 1.0f : -1.0f; }
constexpr int PR = 4;   // rows per wave and sweep
__global__ __launch_bounds__(NT) void db_probe_kernel(const float* __restrict__ A, int np, const Ctrl* __restrict__ ctrl,
                                                      float* __restrict__ w, double* __restrict__ cpart, int pass) {
  const int b = blockIdx.y, grp = blockIdx.x, ngrp = gridDim.x;
  if (ctrl[b].done) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* Ab = A + (long long)b * np * np;
  float* wb = w + (long long)b * np;
  double err = 0.0;
  for (int r0 = PR * (4 * grp + wave); r0 < np; r0 += 4 * PR * ngrp) {
    double dot[PR];
#pragma unroll
    for (int k = 0; k < PR; ++k) dot[k] = 0.0;
#pragma unroll 4
    for (int c = lane * 4; c < np; c += 256) {
      float4 x;
      if (pass == 0) x = make_float4(probe_entry(c), probe_entry(c + 1), probe_entry(c + 2), probe_entry(c + 3));
      else x = *(const float4*)(wb + c);
#pragma unroll
      for (int k = 0; k < PR; ++k) {
        const float4 a = *(const float4*)(Ab + (long long)(r0 + k) * np + c);
        dot[k] += ((double)a.x * (double)x.x + (double)a.y * (double)x.y) + ((double)a.z * (double)x.z + (double)a.w * (double)x.w);
      }
    }
#pragma unroll
    for (int k = 0; k < PR; ++k) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) dot[k] += __shfl_down(dot[k], off, 64);
    }
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < PR; ++k) {
        if (pass == 0) wb[r0 + k] = (float)dot[k];
        else { const double d = dot[k] - (double)probe_entry(r0 + k); err += d * d; }
      }
    }
  }
  if (pass == 1) {
    __shared__ double red[4];
    if (lane == 0) red[wave] = err;
    __syncthreads();
    if (threadIdx.x == 0) cpart[((long long)b * ngrp + grp) * 17 + 16] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

// grid (parts, batch)
__global__ __launch_bounds__(NT) void db_update_m_kernel(float* __restrict__ M, const float* __restrict__ N, int np, int n_true,
                                                         const Ctrl* __restrict__ ctrl, float* __restrict__ rho_part) {
  const int b = blockIdx.y;
  if (ctrl[b].done) return;
  const double a = (double)ctrl[b].alpha;
  const double wi = 2.0 * a * (1.0 - a), wm = (1.0 - a) * (1.0 - a), wn = a * a;
  const long long total = (long long)np * np;
  float* Mb = M + (long long)b * total;
  const float* Nb = N + (long long)b * total;
  double rho = 0.0;
  for (long long idx = ((long long)blockIdx.x * NT + threadIdx.x) * 4; idx < total; idx += (long long)gridDim.x * NT * 4) {
    const int r = (int)(idx / np), c = (int)(idx % np);
    if (r >= n_true) break;
    float4 m4 = *(const float4*)(Mb + idx);
    const float4 n4 = *(const float4*)(Nb + idx);
    float mv[4] = {m4.x, m4.y, m4.z, m4.w};
    const float nv[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (c + e < n_true) {
        const double eye = (r == c + e) ? 1.0 : 0.0;
        const double mn = wi * eye + wm * (double)mv[e] + wn * (double)nv[e];
        mv[e] = (float)mn;
        const double d = eye - (double)mv[e];
        rho += d * d;
      }
    }
    *(float4*)(Mb + idx) = make_float4(mv[0], mv[1], mv[2], mv[3]);
  }
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) rho += __shfl_down(rho, off, 64);
  if (lane == 0) red[wave] = rho;
  __syncthreads();
  if (threadIdx.x == 0) rho_part[(long long)b * gridDim.x + blockIdx.x] = (float)((red[0] + red[1]) + (red[2] + red[3]));
}

// The new row panel T = P A_k,: ([nr][np], nr rows from row k0 on) into the matrix, and the new column panel -A_:,k P from it: A_ik is the
// transpose of A_ki, with the other sign where i has been swept and k has not, so -A_ik P is T_i^T for i < k and -T_i^T beyond.
// One workgroup per 64 x 64 tile.  (A product of its own for the column panel and a copy of each: 2 x 2048^2, 16 outer blocks in a call,
// 2 x 22 + 2 x 6 us per block, now 22 + 9.)
__global__ __launch_bounds__(NT) void panels_kernel(const float* __restrict__ T, float* __restrict__ N, int np, int nr, int k0,
                                                    const Ctrl* __restrict__ ctrl) {
  const int b = blockIdx.y;
  if (ctrl && ctrl[b].done) return;
  __shared__ float tile[BS][BS + 1];
  const int tiles_c = np / BS, tr = blockIdx.x / tiles_c, c0 = (blockIdx.x % tiles_c) * BS;
  if (c0 >= k0 && c0 < k0 + nr) return;          // the pivot block itself is already in place
  const float sign = c0 < k0 ? 1.0f : -1.0f;
  const float* src = T + ((long long)b * nr + tr * BS) * np + c0;
  float* M = N + (long long)b * np * np;
  const int r = threadIdx.x >> 4, c = (threadIdx.x & 15) * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = *(const f32x4*)(src + (long long)(r + 16 * q) * np + c);
    *(f32x4*)(M + (long long)(k0 + tr * BS + r + 16 * q) * np + c0 + c) = v;
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[r + 16 * q][c + e] = sign * v[e];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = tile[c + e][r + 16 * q];
    *(f32x4*)(M + (long long)(c0 + r + 16 * q) * np + k0 + tr * BS + c) = v;
  }
}

// Inverse of n x n SPD matrices by block Gauss-Jordan with pivots of 64, n a multiple of 64: from src to out, through
// tmp (each with its leading dimension and batch stride).  src may be out if n / 64 is even, tmp if it is odd.
struct Mat { float* p; long long stride; int ld; };
// Where all steps are one launch, by the workgroups of the whole group's batch.  Up to one per CU (256) it is ahead: us by steps / in one launch, order 1024 287 / 271,
// 704 x 2 196 / 188, 448 x 5 132 / 123, 192 x 28 61 / 58.  With two per CU the reads past the L2s cost more than the launches (not the polling: longer sleeps
// change nothing), most where one matrix has them all: 1408 (484) 436 / 856, 1280 (400) 391 / 589, 1152 (324) 349 / 380, 960 x 2 297 / 345, 768 x 3 245 / 261, 320 x 12
// 105 / 115.  Orders of a power of two are still ahead (steps of theirs fall off there: 1024 x 2 422 / 374, 512 x 5 207 / 173, 512 x 8 213 / 191, 256 x 32 111 / 97).
// In an iteration that may end before its budget many launches come behind its end, and an empty one instead of nt is worth more than that up to 324 workgroups
// per matrix: budget of 12 to 1e-5, 384 x 10 796 / 730, 640 x 4 1111 / 986, 768 x 3 1276 / 1167, 1152 1681 / 1547, but 1280 1859 / 2187, 1408 2027 / 2924 (five
// updates whatever the residual: 768 x 3 1615 / 1733, 1152 2157 / 2352).
bool sweeps_in_one_launch(int nt, int batch, bool may_end) {
  const long long wgs = (long long)nt * nt * batch;
  return nt > 1 && (wgs <= 256 || (wgs <= 512 && ((nt & (nt - 1)) == 0 || (may_end && nt <= 18))));
}
void gauss_jordan_64(Mat src, Mat out, Mat tmp, float* P, unsigned* sync, int n, int batch, int sel_batch, const Ctrl* ctrl, bool may_end, hipStream_t s) {
  const int nt = n / BS;
  const bool one = sweeps_in_one_launch(nt, sel_batch, may_end);
  hipLaunchKernelGGL(first_pivot_kernel, dim3(batch), dim3(NT), 0, s, src.p, src.stride, src.ld, P, one ? sync : nullptr, ctrl);
  if (one) {
    SweepArgs a = {};
    a.S = src.p; a.sstride = src.stride; a.sld = src.ld; a.out = out.p; a.ostride = out.stride; a.old = out.ld;
    a.tmp = tmp.p; a.tstride = tmp.stride; a.tld = tmp.ld; a.P = P; a.sync = sync; a.nt = nt; a.ctrl = ctrl;
    hipLaunchKernelGGL(jordan_sweep_kernel, dim3(nt * nt, batch), dim3(NT), 0, s, a);
    return;
  }
  for (int k = 0; k < nt; ++k) {
    const Mat dst = ((nt - 1 - k) & 1) ? tmp : out;
    StepArgs a = {};
    a.S = src.p; a.sstride = src.stride; a.sld = src.ld; a.D = dst.p; a.dstride = dst.stride; a.dld = dst.ld;
    a.P = P; a.nt = nt; a.k = k; a.ctrl = ctrl;
    hipLaunchKernelGGL(jordan_step_kernel, dim3(nt * nt, batch), dim3(NT), 0, s, a);
    src = dst;
  }
}

// Outer pivot block: 512 or 256 when it divides the order; 0: pivots of 64 all the way, as long as the tiles of a
// sweep run in one round (three workgroups per CU), where a sweep costs little more than its pivot.  Measured,
// direct / with outer blocks: 768 x 2 (288 tiles) 243 / 320 us, 1024 x 1 (256) 300 / 387, 512 x 8 (512) 226 / 219,
// 1024 x 4 (1024) 604 / 454, 2048 x 2 (2048) 1074 / 979, 4096 x 1 (4096) 3204 / 2213.
int outer_block(int np, int batch) {
  if ((long long)(np / BS) * (np / BS) * batch <= 768) return 0;
  return (np > 512 && np % 512 == 0) ? 512 : ((np > 256 && np % 256 == 0) ? 256 : 0);
}

}  // namespace

// pivot inverses, the second buffer of the elimination and, with outer blocks, the new row panel
long long spd_inverse_scratch_floats(int np, int batch, int sel_batch) {
  const long long OB = outer_block(np, sel_batch), n = OB ? OB : np;
  return (2ll * BS * BS + n * n + OB * np) * batch;
}

int launch_spd_inverse(const float* M, float* N, int np, int batch, int sel_batch, const Ctrl* ctrl, bool may_end, float* scratch, unsigned* sync,
                       hipStream_t s) {
  if (np % BS || batch <= 0 || !scratch || !sync) return PRISM_EINVAL;
  const long long per_mat = (long long)np * np;
  const int OB = outer_block(np, sel_batch);
  float* P = scratch;
  const long long tn = OB ? OB : np;
  const Mat tmp = {P + 2ll * BS * BS * batch, tn * tn, (int)tn};
  auto copy = [&](const float* from, float* to) {
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((per_mat / 4 + NT - 1) / NT), batch), dim3(NT), 0, s, from, to, per_mat, ctrl);
  };
  if (OB == 0) {
    const Mat out = {N, per_mat, np};
    Mat src = {const_cast<float*>(M), per_mat, np};
    if (M == N && ((np / BS) & 1)) { copy(M, tmp.p); src = tmp; }
    gauss_jordan_64(src, out, tmp, P, sync, np, batch, sel_batch, ctrl, may_end, s);
    return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
  }
  if (M != N) copy(M, N);
  float* Trow = tmp.p + tn * tn * batch;                  // [batch][OB][np]: P A_k,:
  const long long tstride = (long long)OB * np;
  for (int k = 0; k < np / OB; ++k) {
    float* Pk = N + (long long)k * OB * np + k * OB;
    float* rowk = N + (long long)k * OB * np;
    float* colk = N + k * OB;
    const Mat piv = {Pk, per_mat, np};
    gauss_jordan_64(piv, piv, tmp, P, sync, OB, batch, sel_batch, ctrl, may_end, s);   // P = A_kk^{-1}, in place: 8 or 4 pivots
    GemmDesc g = {};
    g.batch = batch; g.sel_batch = sel_batch; g.ctrl = ctrl; g.K = OB; g.epi = EPI_STORE; g.c_in = 1.0f;
    GemmDesc r = g;                                      // T = P A_k,:
    r.A = Pk; r.strideA = per_mat; r.lda = np; r.B = rowk; r.strideB = per_mat; r.ldb = np;
    r.C = Trow; r.strideC = tstride; r.ldc = np; r.M = OB; r.N = np; r.skip_n0 = k * OB; r.skip_n1 = (k + 1) * OB;
    int rc = launch_gemm_f32(r, s);
    if (rc != PRISM_OK) return rc;
    GemmDesc u = g;                                      // A_ij <- A_ij - A_ik T_j, i, j outside the pivot block
    u.A = colk; u.strideA = per_mat; u.lda = np; u.B = Trow; u.strideB = tstride; u.ldb = np;
    u.C = N; u.strideC = per_mat; u.ldc = np; u.Cin = N; u.strideCin = per_mat; u.ldcin = np;
    u.M = np; u.N = np; u.epi = EPI_AXPY; u.acc_neg = 1;
    u.skip_m0 = u.skip_n0 = k * OB; u.skip_m1 = u.skip_n1 = (k + 1) * OB;
    // A half-swept symmetric matrix is symmetric within the swept and within the unswept blocks and
    // antisymmetric between them, and the update keeps that: upper triangle of tiles only
    u.sym = 1; u.sym_skew_bound = k * OB;
    rc = launch_gemm_f32(u, s);
    if (rc != PRISM_OK) return rc;
    hipLaunchKernelGGL(panels_kernel, dim3((unsigned)((OB / BS) * (np / BS)), batch), dim3(NT), 0, s, Trow, N, np, OB, k * OB, ctrl);
  }
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
}

void launch_db_moments(const float* M, const float* N, int np, int n_true, int batch, const Ctrl* ctrl, double* cpart,
                       int ngroups, hipStream_t s) {
  hipLaunchKernelGGL(db_moments_kernel, dim3(ngroups, batch), dim3(NT), 0, s, M, N, np, n_true, ctrl, cpart);
}

void launch_db_probe(const float* M, const float* N, int np, int n_true, int batch, const Ctrl* ctrl, float* w, double* cpart,
                     int ngroups, hipStream_t s) {
  (void)n_true;
  hipLaunchKernelGGL(db_probe_kernel, dim3(ngroups, batch), dim3(NT), 0, s, N, np, ctrl, w, cpart, 0);
  hipLaunchKernelGGL(db_probe_kernel, dim3(ngroups, batch), dim3(NT), 0, s, M, np, ctrl, w, cpart, 1);
}

void launch_db_update_m(float* M, const float* N, int np, int n_true, int batch, const Ctrl* ctrl, float* rho_part,
                        int nparts, hipStream_t s) {
  hipLaunchKernelGGL(db_update_m_kernel, dim3(nparts, batch), dim3(NT), 0, s, M, N, np, n_true, ctrl, rho_part);
}

}  // namespace prism
