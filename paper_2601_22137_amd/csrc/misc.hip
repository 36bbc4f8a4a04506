// Entry and exit of the PRISM iterations: Frobenius norm of the input, initial iterates
// (paper Section 3: X_0 = A / ||A||_F; App. A.3: X_0 = I / c, M_0 = A / c^p with
// c = (2 ||A||_F / (p+1))^(1/p)), copy into the padded internal layouts, and the final
// un-scaling / copy-out (A^{1/2} = sqrt(s) X, A^{-1/2} = Y / sqrt(s)).  Matrix sign (Section 4)
// starts like the polar factor; the Chebyshev inverse (App. A.4) keeps A_s = A / ||A||_F, starts
// from X_0 = A_s^T and returns X / ||A||_F.
#include <cstdint>

#include "common.h"

namespace prism {
namespace {

constexpr int NT = 256;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline unsigned short f2bf(float x) {
  unsigned int u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ inline float bf2f(unsigned short h) { return __uint_as_float(((unsigned int)h) << 16); }

// Sum of a matrix's partials, on every lane: a strided share per lane, then a fixed tree (as one serial loop per thread
// it was a latency chain of nsum loads in front of every tile).
__device__ inline double total_sumsq(const double* part, int nsum) {
  double v = 0.0;
  for (int i = threadIdx.x & 63; i < nsum; i += 64) v += part[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// sumsq_part[b][blockIdx.x] = sum of squares of a strided share of matrix b (fp64).
// An inf or nan entry makes its partial non-finite, which the prepare step reports.
// bx in [0, gx): the share of the matrix, b: the matrix (the launch geometry of a single group, which
// the launches over several groups reproduce so that every matrix gets the same partial sums)
// src: the matrix
__device__ inline void sumsq_body(const PrepArgs& a, const void* src, int bx, int b, int gx) {
  const long long total = (long long)a.m * a.n;
  double acc = 0.0;
  const long long first = (long long)bx * NT + threadIdx.x, step = (long long)gx * NT;
  // 16-byte loads, four in flight, from wherever the matrix starts: which thread adds up which entry follows from the
  // shape, not from the address.  The entries behind the last whole vector go to the first workgroup.
  auto sweep = [&](auto* x, auto add16, auto add1) {
    constexpr int PER = 16 / (int)sizeof(*x);
    const long long nv = total / PER;
    auto load = [&](long long i) {
      u32x4 w;
      __builtin_memcpy(&w, x + i * PER, 16);   // aligned to the element only
      return w;
    };
    long long i = first;
    for (; i + 3 * step < nv; i += 4 * step) {
      const u32x4 w0 = load(i), w1 = load(i + step), w2 = load(i + 2 * step), w3 = load(i + 3 * step);
      add16(w0); add16(w1); add16(w2); add16(w3);
    }
    for (; i < nv; i += step) add16(load(i));
    if (bx == 0 && nv * PER + threadIdx.x < total) add1(x[nv * PER + threadIdx.x]);
  };
  if (a.dt == PRISM_BF16) {
    sweep((const unsigned short*)src,
          [&](const u32x4& w) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double x0 = (double)__uint_as_float(w[e] << 16), x1 = (double)__uint_as_float(w[e] & 0xFFFF0000u);
              acc += x0 * x0 + x1 * x1;
            }
          },
          [&](unsigned short h) { acc += (double)bf2f(h) * (double)bf2f(h); });
  } else {
    sweep((const float*)src,
          [&](const u32x4& w) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc += (double)__uint_as_float(w[e]) * (double)__uint_as_float(w[e]);
          },
          [&](float x) { acc += (double)x * (double)x; });
  }
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) a.sumsq_part[(long long)b * a.nsum + bx] = red[0] + red[1] + red[2] + red[3];
}
__device__ inline const void* source(const PrepArgs& a, int b) {
  return (const char*)a.src + (long long)b * a.m * a.n * (a.dt == PRISM_BF16 ? 2 : 4);
}
__global__ __launch_bounds__(NT) void sumsq_kernel(PrepArgs a) { sumsq_body(a, source(a, blockIdx.y), blockIdx.x, blockIdx.y, gridDim.x); }
// several shape groups in one launch: workgroup -> (group, matrix, share)
__global__ __launch_bounds__(NT) void sumsq_multi_kernel(PrepMulti m) {
  int w = blockIdx.x, gi = 0;
  while (gi + 1 < m.ngroups && w >= m.start[gi + 1]) ++gi;
  w -= m.start[gi];
  const PrepArgs& a = m.d[gi];
  const int b = w / a.nsum, first = m.from.first[gi];
  sumsq_body(a, first < 0 ? source(a, b) : m.from.p[first + b], w % a.nsum, b, a.nsum);
}

// fp32: one workgroup per 64 x 64 tile of the padded internal iterate [Lp][Sp].
__global__ __launch_bounds__(NT) void prepare_kernel(PrepArgs a) {
  const int b = blockIdx.y;
  const int tiles_c = a.Sp / 64;
  const int tr = blockIdx.x / tiles_c, tc = blockIdx.x % tiles_c;
  const double ss = total_sumsq(a.sumsq_part + (long long)b * a.nsum, a.nsum);
  const bool finite = (ss == ss) && ss < 1.0e300;
  const bool zero = finite && ss == 0.0;
  const double norm = sqrt(ss);
  double scale = 0.0, cinv = 0.0;
  if (finite && !zero) {
    if (a.fn == PRISM_FN_SQRT_NEWTON) {
      scale = 1.0;                                             // App. A.2 starts from A itself
    } else if (a.fn == PRISM_FN_INV_ROOT) {
      const double cp = 2.0 * norm / (double)(a.root_p + 1);   // c^p
      scale = 1.0 / cp;
      cinv = pow(cp, -1.0 / (double)a.root_p);                 // 1 / c
    } else {
      scale = 1.0 / norm;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Ctrl c;
    c.done = (finite && !zero) ? 0 : 1;
    c.iters = 0;
    c.status = !finite ? PRISM_INFO_NONFINITE : (zero ? PRISM_INFO_ZERO : PRISM_INFO_BUDGET);
    c.plain = 0;
    c.alpha = 0.0f; c.res0 = 0.0f; c.res1 = 0.0f; c.res2 = 0.0f;
    c.norm = norm; c.scale = scale;
    a.ctrl[b] = c;
    a.info[b].iters = 0;
    a.info[b].status = c.status;
  }
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i <= PRISM_MAX_ITERS; i += NT) a.info[b].residual[i] = -1.0f;
    for (int i = threadIdx.x; i < PRISM_MAX_ITERS; i += NT) a.info[b].alpha[i] = 0.0f;
    for (int i = threadIdx.x; i < FIT_SYNC_WORDS; i += NT) a.sync[(long long)b * FIT_SYNC_WORDS + i] = 0u;
  }

  float rho = 0.0f;
  const long long mat = (long long)a.m * a.n;
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int lr = e >> 6, lc = e & 63;
    const int r = tr * 64 + lr, c = tc * 64 + lc;   // position in the internal [Lp][Sp] iterate
    double v = 0.0;
    if (r < a.L && c < a.S) {
      const long long si = a.transpose ? ((long long)c * a.n + r) : ((long long)r * a.n + c);
      v = (double)((const float*)a.src)[(long long)b * mat + si] * scale;
    }
    const long long o = (long long)b * a.Lp * a.Sp + (long long)r * a.Sp + c;
    if (a.fn == PRISM_FN_SIGN) {
      a.X32[o] = (float)v;
    } else if (a.fn == PRISM_FN_SQRT_NEWTON) {   // X_0 = M_0 = A, Y_0 = I; the padding of M is the identity
      const bool in = (r < a.S && c < a.S);
      const float eye = (r == c) ? 1.0f : 0.0f;
      a.X32[o] = (float)v;
      a.Y32[o] = in ? eye : 0.0f;
      a.R32[o] = in ? (float)v : eye;
      const double res = in ? ((double)eye - v) : 0.0;
      rho += (float)(res * res);
    } else if (a.fn == PRISM_FN_INVERSE) {
      a.Y32[o] = (float)v;                                                                    // A_s
      a.X32[(long long)b * a.Lp * a.Sp + (long long)c * a.Sp + r] = (float)v;                 // X_0 = A_s^T
    } else if (a.fn == PRISM_FN_POLAR) {
      a.X32[o] = (float)v;
    } else if (a.fn == PRISM_FN_SQRT) {
      a.X32[o] = (float)v;
      a.Y32[o] = (r == c && r < a.S) ? 1.0f : 0.0f;
    } else {  // inverse root: v = M_0 entry
      const bool in = (r < a.S && c < a.S);
      const double eye = (r == c && in) ? 1.0 : 0.0;
      a.M64[o] = v;
      a.X32[o] = (float)(eye * cinv);
      const double res = in ? (eye - v) : 0.0;
      a.R32[o] = (float)res;
      rho += (float)(res * res);
    }
  }
  if (a.fn == PRISM_FN_INV_ROOT || a.fn == PRISM_FN_SQRT_NEWTON) {
    __shared__ float red[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rho += __shfl_down(rho, off, 64);
    if (lane == 0) red[wave] = rho;
    __syncthreads();
    if (threadIdx.x == 0)
      a.rho_part[(long long)b * gridDim.x + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
  }
}

// bf16 polar: one workgroup per 64 x 128 tile of the CALLER's matrix (padded).  The tile is read with 16-byte loads along
// the caller's rows (VEC; entry by entry where the rows are no multiples of 16 bytes), scaled and split into high and
// low halves; a tall or square matrix goes straight into the internal [Lp][Sp] iterate, a wide one (the iterate is its
// transpose) through an LDS transpose, everything as 16-byte vectors.  HBM bound (50257 x 768: norm and copy-in
// 73 + 98 us as entry-wise passes, now 14 + 36).
constexpr int PC = 128;                    // columns per tile
// Entry (row, i) of a transposed tile of `units` 16-byte units per row: the units are rotated by row / 8, so that the
// 2-byte writes of a wave (rows 8 apart) spread over the banks.
__device__ inline int rotated(int row, int i, int units) { return (((i >> 3) + (row >> 3)) & (units - 1)) * 8 + (i & 7); }
// 8 consecutive entries of the caller's matrix from column c of a row on (zeros from column n on)
template <bool VEC> __device__ inline u32x4 load8(const unsigned short* row, int c, int n) {
  if constexpr (VEC) return *(const u32x4*)(row + c);
  u32x4 w;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned lo = c + 2 * e < n ? row[c + 2 * e] : 0u, hi = c + 2 * e + 1 < n ? row[c + 2 * e + 1] : 0u;
    w[e] = lo | (hi << 16);
  }
  return w;
}
template <bool VEC>
__device__ inline void prepare_bf16_body(const PrepArgs& a, const unsigned short* src, int bx, int b) {
  const int tiles_c = (a.transpose ? a.Lp : a.Sp) / PC;             // tiles over the padded, caller-oriented matrix
  const int tr = bx / tiles_c, tc = bx % tiles_c;
  u32x4 in[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {              // 1024 vectors of 8 per tile, requested ahead of the norm
    const int v = threadIdx.x + it * NT;
    const int r = tr * 64 + (v >> 4), c = tc * PC + (v & 15) * 8;
    in[it] = u32x4{0u, 0u, 0u, 0u};
    if (r < a.m && c < a.n) in[it] = load8<VEC>(src + (long long)r * a.n, c, a.n);
  }
  const double ss = total_sumsq(a.sumsq_part + (long long)b * a.nsum, a.nsum);
  const bool finite = (ss == ss) && ss < 1.0e300;
  const bool zero = finite && ss == 0.0;
  const double norm = sqrt(ss);
  const float scale = (finite && !zero) ? (float)(1.0 / norm) : 0.0f;
  if (bx == 0 && threadIdx.x == 0) {
    Ctrl c;
    c.done = (finite && !zero) ? 0 : 1;
    c.iters = 0;
    c.status = !finite ? PRISM_INFO_NONFINITE : (zero ? PRISM_INFO_ZERO : PRISM_INFO_BUDGET);
    c.plain = 0;
    c.alpha = 0.0f; c.res0 = 0.0f; c.res1 = 0.0f; c.res2 = 0.0f;
    c.norm = norm; c.scale = scale;
    a.ctrl[b] = c;
    a.info[b].iters = 0;
    a.info[b].status = c.status;
  }
  if (bx == 0) {
    for (int i = threadIdx.x; i <= PRISM_MAX_ITERS; i += NT) a.info[b].residual[i] = -1.0f;
    for (int i = threadIdx.x; i < PRISM_MAX_ITERS; i += NT) a.info[b].alpha[i] = 0.0f;
    for (int i = threadIdx.x; i < FIT_SYNC_WORDS; i += NT) a.sync[(long long)b * FIT_SYNC_WORDS + i] = 0u;
  }
  const long long mat_int = (long long)a.Lp * a.Sp;
  __shared__ __align__(16) unsigned short tile_hi[PC][72], tile_lo[PC][72];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int v = threadIdx.x + it * NT;
    const int lr = v >> 4, lc = (v & 15) * 8;
    u32x4 hi, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned w = in[it][e];
      const float x0 = __uint_as_float(w << 16) * scale, x1 = __uint_as_float(w & 0xFFFF0000u) * scale;
      const unsigned short h0 = f2bf(x0), h1 = f2bf(x1);
      hi[e] = (unsigned)h0 | ((unsigned)h1 << 16);
      if (a.Xa_lo) lo[e] = (unsigned)f2bf(x0 - bf2f(h0)) | ((unsigned)f2bf(x1 - bf2f(h1)) << 16);
      if (a.transpose) {
        const int p = rotated(lc, lr, 8);
        tile_hi[lc + 2 * e][p] = h0; tile_hi[lc + 2 * e + 1][p] = h1;
        if (a.Xa_lo) { tile_lo[lc + 2 * e][p] = (unsigned short)lo[e]; tile_lo[lc + 2 * e + 1][p] = (unsigned short)(lo[e] >> 16); }
      }
    }
    if (!a.transpose) {  // rows / columns beyond the caller's matrix but inside the padded array are written as zeros
      const long long o = (long long)b * mat_int + (long long)(tr * 64 + lr) * a.Sp + tc * PC + lc;
      *(u32x4*)(a.Xa_hi + o) = hi;
      if (a.Xa_lo) *(u32x4*)(a.Xa_lo + o) = lo;
    }
  }
  if (!a.transpose) return;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int v = threadIdx.x + it * NT;
    const int lc = v >> 3, lr = (v & 7) * 8;      // row lc of the transposed tile, 8 consecutive source rows
    const long long o = (long long)b * mat_int + (long long)(tc * PC + lc) * a.Sp + tr * 64 + lr;   // internal row = caller's column
    *(u32x4*)(a.Xa_hi + o) = *(const u32x4*)&tile_hi[lc][rotated(lc, lr, 8)];
    if (a.Xa_lo) *(u32x4*)(a.Xa_lo + o) = *(const u32x4*)&tile_lo[lc][rotated(lc, lr, 8)];
  }
}
template <bool VEC> __global__ __launch_bounds__(NT) void prepare_bf16_kernel(PrepArgs a) {
  prepare_bf16_body<VEC>(a, (const unsigned short*)source(a, blockIdx.y), blockIdx.x, blockIdx.y);
}
__global__ __launch_bounds__(NT) void prepare_bf16_multi_kernel(PrepMulti m) {
  int w = blockIdx.x, gi = 0;
  while (gi + 1 < m.ngroups && w >= m.start[gi + 1]) ++gi;
  w -= m.start[gi];
  const PrepArgs& a = m.d[gi];
  const int tiles = (a.Lp / 64) * (a.Sp / PC);
  const int b = w / tiles, first = m.from.first[gi];
  prepare_bf16_body<true>(a, (const unsigned short*)(first < 0 ? source(a, b) : m.from.p[first + b]), w % tiles, b);
}

// bf16 polar, rows of the caller's matrix in 16-byte vectors (VEC; entry by entry otherwise): the result is the high half of
// the iterate.  One workgroup per 64 x 128 tile of the caller's matrix: a tall or
// square one is copied, a wide one (the iterate is its transpose) goes through an LDS transpose.  HBM bound
// (50257 x 768: 88 us entry by entry, now 24).
template <bool VEC> __device__ inline void store8(unsigned short* row, int c, int n, const u32x4& w) {
  if constexpr (VEC) {
    *(u32x4*)(row + c) = w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (c + 2 * e < n) row[c + 2 * e] = (unsigned short)w[e];
      if (c + 2 * e + 1 < n) row[c + 2 * e + 1] = (unsigned short)(w[e] >> 16);
    }
  }
}
template <bool VEC>
__device__ inline void finalize_bf16_body(const FinalArgs& a, const unsigned short* src, int bx, int b) {   // src: the input, where it is not at dst
  const Ctrl c = a.ctrl[b];
  if (c.status == PRISM_INFO_NONFINITE || c.status == PRISM_INFO_ZERO) {
    if (!src) return;
    const int across = (a.n + PC - 1) / PC, row0 = bx / across * 64, col0 = bx % across * PC;
    for (int v = threadIdx.x; v < 1024; v += NT) {
      const int r = row0 + (v >> 4), col = col0 + (v & 15) * 8;
      if (r < a.m && col < a.n)
        store8<VEC>((unsigned short*)a.dst + ((long long)b * a.m + r) * a.n, col, a.n, load8<VEC>(src + (long long)r * a.n, col, a.n));
    }
    return;
  }
  const int par = c.iters & 1;
  const long long mat_int = (long long)b * a.Lp * a.Sp;
  const unsigned short* hi = a.Xa_hi[par] + mat_int;
  unsigned short* dst = (unsigned short*)a.dst + (long long)b * a.m * a.n;
  if (!a.transpose && a.Xa_hi[par] == (const unsigned short*)a.dst) return;   // the caller's array was that iterate buffer: in place
  const int tiles_c = (a.n + PC - 1) / PC;
  const int tr = bx / tiles_c, tc = bx % tiles_c;
  if (!a.transpose) {
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int v = threadIdx.x + it * NT;
      const int r = tr * 64 + (v >> 4), col = tc * PC + (v & 15) * 8;
      const long long o = (long long)r * a.Sp + col;
      if (r < a.m && col < a.n) store8<VEC>(dst + (long long)r * a.n, col, a.n, *(const u32x4*)(hi + o));
    }
    return;
  }
  // caller's tile (64 rows tr, 128 columns tc) = transpose of the internal tile (128 rows tc, 64 columns tr)
  __shared__ __align__(16) unsigned short tile[64][PC + 8];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int v = threadIdx.x + it * NT;
    const int lr = v >> 3, lc = (v & 7) * 8;                 // internal row (caller's column), 8 internal columns
    const int ri = tc * PC + lr, ci = tr * 64 + lc;
    u32x4 w = {0u, 0u, 0u, 0u};
    const long long o = (long long)ri * a.Sp + ci;
    if (ri < a.Lp && ci < a.Sp) w = *(const u32x4*)(hi + o);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile[lc + 2 * e][rotated(lc, lr, 16)] = (unsigned short)(w[e] & 0xFFFFu);
      tile[lc + 2 * e + 1][rotated(lc, lr, 16)] = (unsigned short)(w[e] >> 16);
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int v = threadIdx.x + it * NT;
    const int lr = v >> 4, lc = (v & 15) * 8;                // caller's row within the tile, 8 caller's columns
    const int r = tr * 64 + lr, col = tc * PC + lc;
    if (r < a.m && col < a.n) store8<VEC>(dst + (long long)r * a.n, col, a.n, *(const u32x4*)&tile[lr][rotated(lr, lc, 16)]);
  }
}
template <bool VEC> __global__ __launch_bounds__(NT) void finalize_bf16_kernel(FinalArgs a) { finalize_bf16_body<VEC>(a, nullptr, blockIdx.x, blockIdx.y); }
__global__ __launch_bounds__(NT) void finalize_bf16_multi_kernel(FinalMulti m) {
  int w = blockIdx.x, gi = 0;
  while (gi + 1 < m.ngroups && w >= m.start[gi + 1]) ++gi;
  w -= m.start[gi];
  const FinalArgs& a = m.d[gi];
  const int tiles = ((a.m + 63) / 64) * ((a.n + PC - 1) / PC);
  const int b = w / tiles, first = m.from.first[gi];
  finalize_bf16_body<true>(a, first < 0 ? nullptr : (const unsigned short*)m.from.p[first + b], w % tiles, b);
}

// fp32: one thread per element of the caller's array.
__global__ __launch_bounds__(NT) void finalize_kernel(FinalArgs a) {
  const int b = blockIdx.y;
  const Ctrl c = a.ctrl[b];
  if (c.status == PRISM_INFO_NONFINITE || c.status == PRISM_INFO_ZERO) return;
  const int par = c.iters & 1;
  const long long set = a.ring ? (long long)(c.iters % a.ring) * a.ring_bytes : 0;
  const float* X = (const float*)((const char*)a.X32[a.ring ? 0 : par] + set);
  const float* Y = (const float*)((const char*)a.Y32[a.ring ? 0 : par] + set);
  const long long mat = (long long)a.m * a.n;
  const long long i = (long long)blockIdx.x * NT + threadIdx.x;
  if (i >= mat) return;
  const int r = (int)(i / a.n), col = (int)(i % a.n);
  const long long o = (long long)b * a.Lp * a.Sp +
                      (a.transpose ? ((long long)col * a.Sp + r) : ((long long)r * a.Sp + col));
  if (a.fn == PRISM_FN_INVERSE) {
    ((float*)a.dst)[(long long)b * mat + i] = (float)((double)X[o] / c.norm);
  } else if (a.fn == PRISM_FN_POLAR) {
    ((float*)a.dst)[(long long)b * mat + i] = X[o];
  } else if (a.fn == PRISM_FN_SQRT_NEWTON) {
    ((float*)a.dst)[(long long)b * mat + i] = X[o];
    ((float*)a.dst2)[(long long)b * mat + i] = Y[o];
  } else if (a.fn == PRISM_FN_SQRT) {
    const double rs = sqrt(c.norm);
    ((float*)a.dst)[(long long)b * mat + i] = (float)((double)X[o] * rs);
    ((float*)a.dst2)[(long long)b * mat + i] = (float)((double)Y[o] / rs);
  } else {
    ((float*)a.dst)[(long long)b * mat + i] = X[o];
  }
}

__global__ __launch_bounds__(NT) void make_e_kernel(float* E, const float* R, const Ctrl* ctrl, int np) {
  const int b = blockIdx.y;
  if (ctrl[b].done) return;
  const float alpha = ctrl[b].alpha;
  const long long total = (long long)np * np;
  const long long i = (long long)blockIdx.x * NT + threadIdx.x;
  if (i >= total) return;
  E[(long long)b * total + i] = alpha * R[(long long)b * total + i];
}

// One workgroup per 64 x 64 tile on or above the diagonal; thread t: row t / 4, 16 consecutive columns.
__global__ __launch_bounds__(NT) void gram_reduce_kernel(GramReduceArgs a) {
  int gi = 0;
  while (gi + 1 < a.ngroups && (int)blockIdx.y >= a.first[gi + 1]) ++gi;
  const int bl = blockIdx.y - a.first[gi], b = a.boff[gi] + bl;
  if (a.ctrl[b].done) return;
  const int nt = a.np / 64;
  int left = blockIdx.x, tm = 0;
  while (left >= nt - tm) { left -= nt - tm; ++tm; }
  const int tn = tm + left;
  const int m0 = tm * 64, n0 = tn * 64;
  const long long SS = (long long)a.np * a.np;
  const int r = threadIdx.x >> 2, c0 = (threadIdx.x & 3) * 16;
  __shared__ float tile[64][65];
  {
    f32x4 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int parts = a.parts[gi];
    const float* src = a.part[gi] + (long long)bl * parts * SS + (long long)(m0 + r) * a.np + n0 + c0;
    int p = 0;
    for (; p + 4 <= parts; p += 4) {   // four parts requested at a time, added in order
      f32x4 v[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) v[u][q] = *(const f32x4*)(src + (long long)(p + u) * SS + 4 * q);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += v[u][q];
    }
    for (; p < parts; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] += *(const f32x4*)(src + (long long)p * SS + 4 * q);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + r, n = n0 + c0 + 4 * q + e;
        tile[r][c0 + 4 * q + e] = (m < a.n_true && n < a.n_true) ? ((m == n ? 1.0f : 0.0f) - acc[q][e]) : 0.0f;
      }
  }
  __syncthreads();
  const bool diag_tile = tm == tn;
  float part = 0.0f;
  auto emit = [&](int row0, int col0, bool transposed) {   // this thread's 16 entries of the tile at (row0, col0)
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int c = c0 + e;
      v[e] = transposed ? tile[c][r] : ((diag_tile && c < r) ? tile[c][r] : tile[r][c]);
    }
    const long long o = (long long)b * SS + (long long)(row0 + r) * a.np + col0 + c0;
    if (a.R32) {
#pragma unroll
      for (int q = 0; q < 4; ++q) *(f32x4*)(a.R32 + o + 4 * q) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    }
    if (a.Rb) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u32x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (unsigned)f2bf(v[8 * h + 2 * e]) | ((unsigned)f2bf(v[8 * h + 2 * e + 1]) << 16);
        *(u32x4*)(a.Rb + o + 8 * h) = pk;
      }
    }
    if (!transposed) {
#pragma unroll
      for (int e = 0; e < 16; ++e) part += v[e] * v[e];
      if (a.diag && diag_tile && r >= c0 && r < c0 + 16) a.diag[(long long)b * a.np + m0 + r] = tile[r][r];
    }
  };
  emit(m0, n0, false);
  if (!diag_tile) { emit(n0, m0, true); part *= 2.0f; }
  __shared__ float red[4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
  __syncthreads();
  if (threadIdx.x == 0) a.rho_part[(long long)b * a.rho_stride + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  if (blockIdx.x == 0)
    for (int i = gridDim.x + threadIdx.x; i < a.rho_stride; i += NT) a.rho_part[(long long)b * a.rho_stride + i] = 0.0f;
}

}  // namespace

int gram_reduce_parts(int np) { return (np / 64) * (np / 64 + 1) / 2; }

void launch_gram_reduce(const GramReduceArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(gram_reduce_parts(a.np), a.first[a.ngroups]), dim3(NT), 0, s, a);
}

void launch_make_e(float* E, const float* R, const Ctrl* ctrl, int batch, int np, hipStream_t s) {
  const long long total = (long long)np * np;
  hipLaunchKernelGGL(make_e_kernel, dim3((unsigned)((total + NT - 1) / NT), batch), dim3(NT), 0, s, E, R, ctrl, np);
}

void launch_sumsq(const PrepArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(sumsq_kernel, dim3(a.nsum, a.batch), dim3(NT), 0, s, a);
}

// rows of the caller's matrices are whole 16-byte vectors
static bool bf16_vector_rows(int n, const void* user) { return n % 8 == 0 && ((uintptr_t)user & 15) == 0; }

void launch_prepare(const PrepArgs& a, hipStream_t s) {
  if (a.dt == PRISM_BF16) {
    const dim3 grid((unsigned)((a.Lp / 64) * (a.Sp / PC)), a.batch);   // the padding is written too
    if (bf16_vector_rows(a.n, a.src)) hipLaunchKernelGGL(prepare_bf16_kernel<true>, grid, dim3(NT), 0, s, a);
    else hipLaunchKernelGGL(prepare_bf16_kernel<false>, grid, dim3(NT), 0, s, a);
    return;
  }
  const int tiles = (a.Lp / 64) * (a.Sp / 64);
  hipLaunchKernelGGL(prepare_kernel, dim3(tiles, a.batch), dim3(NT), 0, s, a);
}

// The pre-scaling and copy-out steps of several shape groups in one launch each (bf16 polar, every group
// on the 16-byte vector path); false: the caller launches them group by group.
static void set_sources(Sources& to, const Sources* from) {
  if (from) { to = *from; return; }
  for (int& f : to.first) f = -1;
}
bool launch_prep_multi(const PrepArgs* groups, int ngroups, const Sources* from, hipStream_t s) {
  if (ngroups < 2 || ngroups > BF16_MAX_GROUPS) return false;
  PrepMulti ms = {}, mp = {};
  set_sources(ms.from, from);
  set_sources(mp.from, from);
  ms.ngroups = mp.ngroups = ngroups;
  long long ts = 0, tp = 0;
  for (int i = 0; i < ngroups; ++i) {
    const PrepArgs& a = groups[i];
    if (a.dt != PRISM_BF16 || !bf16_vector_rows(a.n, from ? nullptr : a.src)) return false;   // sources: their caller has looked
    ms.d[i] = mp.d[i] = a;
    ms.start[i] = (int)ts; mp.start[i] = (int)tp;
    ts += (long long)a.nsum * a.batch;
    tp += (long long)(a.Lp / 64) * (a.Sp / PC) * a.batch;
    if (ts > 0x7fffffff || tp > 0x7fffffff) return false;
  }
  ms.start[ngroups] = (int)ts; mp.start[ngroups] = (int)tp;
  hipLaunchKernelGGL(sumsq_multi_kernel, dim3((unsigned)ts), dim3(NT), 0, s, ms);
  hipLaunchKernelGGL(prepare_bf16_multi_kernel, dim3((unsigned)tp), dim3(NT), 0, s, mp);
  return true;
}

bool launch_finalize_multi(const FinalArgs* groups, int ngroups, const Sources* from, hipStream_t s) {
  if (ngroups < 2 || ngroups > BF16_MAX_GROUPS) return false;
  FinalMulti mf = {};
  set_sources(mf.from, from);
  mf.ngroups = ngroups;
  long long t = 0;
  for (int i = 0; i < ngroups; ++i) {
    const FinalArgs& a = groups[i];
    if (a.dt != PRISM_BF16 || !bf16_vector_rows(a.n, a.dst)) return false;
    mf.d[i] = a;
    mf.start[i] = (int)t;
    t += (long long)((a.m + 63) / 64) * ((a.n + PC - 1) / PC) * a.batch;
    if (t > 0x7fffffff) return false;
  }
  mf.start[ngroups] = (int)t;
  hipLaunchKernelGGL(finalize_bf16_multi_kernel, dim3((unsigned)t), dim3(NT), 0, s, mf);
  return true;
}

void launch_finalize(const FinalArgs& a, hipStream_t s) {
  if (a.dt == PRISM_BF16) {
    const dim3 grid((unsigned)(((a.m + 63) / 64) * ((a.n + PC - 1) / PC)), a.batch);
    if (bf16_vector_rows(a.n, a.dst)) hipLaunchKernelGGL(finalize_bf16_kernel<true>, grid, dim3(NT), 0, s, a);
    else hipLaunchKernelGGL(finalize_bf16_kernel<false>, grid, dim3(NT), 0, s, a);
    return;
  }
  const long long mat = (long long)a.m * a.n;
  hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)((mat + NT - 1) / NT), a.batch), dim3(NT), 0, s, a);
}

namespace {
__global__ __launch_bounds__(256) void scatter_info_kernel(InfoScatter a) {
  const int words = (int)(sizeof(prism_info) / 4);
  for (int g = 0; g < a.ngroups; ++g) {
    if (!a.dst[g]) continue;
    const unsigned* src = (const unsigned*)(a.src + a.first[g]);
    unsigned* dst = (unsigned*)a.dst[g];
    const int n = (a.first[g + 1] - a.first[g]) * words;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) dst[i] = src[i];
  }
}
}  // namespace

namespace {
constexpr int GATHER = 64;
struct GatherArgs { const char* from[GATHER]; char* dst; long long bytes; };
// one matrix per blockIdx.y, whatever its alignment
__global__ __launch_bounds__(256) void gather_kernel(GatherArgs a) {
  const char* src = a.from[blockIdx.y];
  char* dst = a.dst + (long long)blockIdx.y * a.bytes;
  const long long first = (long long)blockIdx.x * 256 + threadIdx.x, step = (long long)gridDim.x * 256;
  if ((((uintptr_t)src | (uintptr_t)dst | (uintptr_t)a.bytes) & 15) == 0)
    for (long long i = first; i < a.bytes / 16; i += step) ((u32x4*)dst)[i] = ((const u32x4*)src)[i];
  else
    for (long long i = first; i < a.bytes / 2; i += step) ((unsigned short*)dst)[i] = ((const unsigned short*)src)[i];
}
}  // namespace

void launch_gather(void* dst, const void* const* from, int count, size_t bytes, hipStream_t s) {
  if (bytes == 0) return;
  for (int b0 = 0; b0 < count; b0 += GATHER) {
    GatherArgs a = {};
    const int n = count - b0 < GATHER ? count - b0 : GATHER;
    for (int i = 0; i < n; ++i) a.from[i] = (const char*)from[b0 + i];
    a.dst = (char*)dst + (size_t)b0 * bytes;
    a.bytes = (long long)bytes;
    const size_t blocks = (bytes + 16383) / 16384;
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)(blocks > 512 ? 512 : blocks), n), dim3(256), 0, s, a);
  }
}

void launch_scatter_info(const InfoScatter& a, hipStream_t s) {
  static_assert(sizeof(prism_info) % 4 == 0, "reports are copied word by word");
  hipLaunchKernelGGL(scatter_info_kernel, dim3(8), dim3(256), 0, s, a);
}

}  // namespace prism
