// All iterations of an fp32 call in one launch, for matrices whose products take a few microseconds each: there a launch per
// step is bound by launch gaps, by the host's launch rate, and by the launches that follow convergence (2.6 us each for
// nothing).
//
// A cluster of workgroups works on each matrix.  The steps of its iterations - tiles of products, row blocks of the fit - are
// numbered in order; a workgroup takes the next number from a counter of the matrix, waits until the steps it depends on are
// complete (a second counter, in units of steps), does it and counts it.  Nobody depends on workgroups being resident
// together: a step waits for lower numbers only, and those were taken by workgroups that run.  (The row blocks of one fit do wait
// for each other, bounded: see fit_rows.)  Nobody waits for a launch either: a workgroup leaves when its matrix stops.
//
// What changes hands is written past the caches that are not coherent between XCDs (sc1) and read through them: every iteration
// writes to memory that no workgroup has read before (a ring of sets of arrays), so nothing stale can be found there; when
// the ring comes round, each workgroup first invalidates its caches (agent-scope acquire, 8 to 10 us with 256 workgroups).
// (Read past the caches as well, every tile gets its panels from the Infinity Cache: inverse roots 4 x 256 0.38 ms, not 0.32;
// 8 x 512 1.21, not 1.10.)
// The sums are those of the launches it replaces (gemm_f32_tile.h, fit_device.h), bit for bit.
#include "fit_device.h"
#include "gemm_f32_tile.h"

namespace prism {
namespace {

constexpr int FLOW_RING = 8;                        // slabs in flight per tile: the panels come from far away
// words of a matrix's counters (FitArgs::sync)
constexpr int FLOW_TICKET = FIT_MAX_CLUSTER + 32;   // next step
constexpr int FLOW_STATE = FIT_MAX_CLUSTER + 64;    // steps complete; behind it the bits of alpha, or FLOW_STOPPED
constexpr unsigned FLOW_STOPPED = 0xFFFFD09Eu;      // (a NaN; a caller's coefficient with these bits is replaced by another)

// which kinds of products a kernel has: polar factor (X^T X, symmetric), sign / square root / inverse (all tiles), inverse root
enum { FLOW_GRAM, FLOW_FULL, FLOW_ROOT };

template <int FAM, int LD, int NCH>
__global__ __launch_bounds__(NT, 2) void flow_kernel(FlowArgs a) {
  extern __shared__ __align__(1024) unsigned char smem[];
  __shared__ int s_ticket;
  __shared__ u64 s_state;
  __shared__ Ctrl s_ctl;
  constexpr int CTL_WORDS = (int)(sizeof(Ctrl) / 4);
  const int b = blockIdx.x / a.cluster, batch = gridDim.x / a.cluster, t = threadIdx.x;
  unsigned* sync = a.fit.sync + (long long)b * FIT_SYNC_WORDS;
  unsigned* count = sync + FLOW_STATE;
  const int max_iters = a.fit.sv.max_iters, G = a.fit.sv.rows / 16;
  const int nres = a.residual ? a.items[0] : 0;
  int rest = 0;
  for (int i = a.residual; i < a.nops; ++i) rest += a.items[i];
  const int na = nres + 1 + rest, nb = nres + G + rest;     // steps of an iteration without and with a chain
  const int t1 = a.first_fit * na;

  float alpha = 0.0f;
  int turn = 0;                 // of the ring
  bool stale = false;           // caches may hold what lay in its sets a turn ago
  // Until `need` steps of this matrix are complete; false: it has stopped.
  auto wait_for = [&](int need) -> bool {
    if (t == 0) {
      u64 v;
      for (;;) {
        v = __hip_atomic_load((u64*)count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((unsigned)v >= (unsigned)need || (unsigned)(v >> 32) == FLOW_STOPPED) break;
        __builtin_amdgcn_s_sleep(1);
      }
      s_state = v;
    }
    if (stale && t < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    stale = false;
    __syncthreads();
    const unsigned bits = __builtin_amdgcn_readfirstlane((unsigned)(s_state >> 32));
    alpha = __uint_as_float(bits);
    return bits != FLOW_STOPPED;
  };
  auto take = [&]() { return (int)__hip_atomic_fetch_add(sync + FLOW_TICKET, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  // The step is complete: its stores have reached memory.
  auto finish = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };

  // Whether the matrix is done (never begun: zero or not finite; or stopped while this workgroup had no place on the chip) is one
  // thread's to see, for the whole workgroup: whoever solves sets it in this launch, and waves that look for themselves could part
  // ways.  The number is taken in the same breath: nobody counts on those of a matrix that is done.
  if (t == 0) {
    const int first = take();
    s_ticket = coh_load<true>(&a.fit.sv.ctrl[b].done) ? -1 : first;
  }
  __syncthreads();
  for (;;) {
    const int ticket = __builtin_amdgcn_readfirstlane(s_ticket);
    if (ticket < 0) return;
    int k, base;
    if (ticket < t1) { k = ticket / na; base = k * na; }
    else { k = (ticket - t1) / nb; base = t1 + k * nb; k += a.first_fit; }
    if (k > max_iters || (k == max_iters && a.fit.sv.tol <= 0.0)) return;
    const long long cur = (long long)(k % a.ring) * a.ring_bytes, next = (long long)((k + 1) % a.ring) * a.ring_bytes;
    stale = k / a.ring != turn;
    turn = k / a.ring;
    const bool fitted = a.p_s > 0 && k >= a.first_fit && k < max_iters;
    const int nfit = fitted ? G : 1;
    int r = ticket - base;
    const int known = base + nres + nfit;                     // alpha is there
    if (k == max_iters && r >= nres + nfit) return;

    if (r >= nres && r < nres + nfit) {                       // fit
      if (!wait_for(base + nres)) return;
      FitArgs f = a.fit;
      f.V0 += (long long)(k - a.first_fit) * f.sv.rows * LD;
      f.epoch = FIT_EPOCH * (unsigned)k;
      f.R = (const char*)f.R + cur;
      bool solver = !fitted;
      if (fitted) solver = fit_rows<false, LD, 1, NCH, 4>(f, b, batch, r - nres, G, (float*)smem);
      if (solver) {
        if (t < CTL_WORDS) ((unsigned*)&s_ctl)[t] = coh_load<true>((const unsigned*)(f.sv.ctrl + b) + t);
        __syncthreads();
        f.sv.k = k;
        if (k == 0 && !a.residual) { f.sv.rho_part = a.rho0; f.sv.nparts = a.nparts0; }
        f.sv.last = k == max_iters;
        f.sv.mode = k < a.sched_len ? 3 : (a.p_s == 0 ? 1 : (k < a.warm ? 2 : 0));
        f.sv.sched_alpha = k < a.sched_len ? a.sched[k] : 0.0f;
        solve_body<true>(f.sv, b, nullptr, &s_ctl);
        __syncthreads();
        if (t < CTL_WORDS) coh_store<true>((unsigned*)(f.sv.ctrl + b) + t, ((const unsigned*)&s_ctl)[t]);
        if (t == 0) {
          unsigned bits = __float_as_uint(s_ctl.alpha);
          if (bits == FLOW_STOPPED) bits ^= 1u;
          coh_store<true>(count + 1, s_ctl.done ? FLOW_STOPPED : bits);
        }
      }
      finish();
      if (t == 0) s_ticket = take();
      __syncthreads();
      continue;
    }

    int op = 0;
    if (r >= nres) {
      r -= nres + nfit;
      op = a.residual;
      while (r >= a.items[op]) { r -= a.items[op]; ++op; }
    }
    GemmDesc g = a.op[op];
    auto in_set = [](auto*& p, long long offset) { p = (std::remove_reference_t<decltype(p)>)((const char*)p + offset); };
    if (!a.fixed_a[op]) in_set(g.A, cur);
    in_set(g.B, cur);
    in_set(g.Cin, cur);
    if (g.Cin2) in_set(g.Cin2, cur);
    g.C = (char*)g.C + (a.next_c[op] ? next : cur);
    g.R32out = (float*)((char*)g.R32out + next);
    const bool beside = op >= a.residual && a.start[op] < 0;
    if (!wait_for(op < a.residual ? base : (beside ? base + nres : known + a.start[op]))) return;
    int upcoming = 0;
    if (t == 0) upcoming = take();                                // on its way while this tile is computed
    const int tile = a.tile[op], tiles_m = g.M / tile, tiles_n = g.N / tile;
    int tm, tn, per_mat;
    if (g.sym) {
      int left = r;
      tm = 0;
      while (left >= tiles_m - tm) { left -= tiles_m - tm; ++tm; }
      tn = tm + left;
      per_mat = tiles_m * (tiles_m + 1) / 2;
    } else {
      tm = r / tiles_n;
      tn = r - tm * tiles_n;
      per_mat = tiles_m * tiles_n;
    }
    bool go = true;
    auto alpha_of = [&](float& out) {
      if (beside) go = wait_for(known);
      out = alpha;
      return go;
    };
    auto product = [&](auto epi, auto km, auto symmetric) {
      if (tile == 32)
        gemm_tile<float, float, 32, 32, 2, 2, FLOW_RING, decltype(epi)::value, decltype(km)::value, decltype(symmetric)::value, false, true>(
            g, g.sym, b, r, per_mat, tm, tn, smem, alpha_of);
      else
        gemm_tile<float, float, 64, 64, 2, 2, FLOW_RING, decltype(epi)::value, decltype(km)::value, decltype(symmetric)::value, false, true>(
            g, g.sym, b, r, per_mat, tm, tn, smem, alpha_of);
    };
    typedef std::bool_constant<FAM == FLOW_GRAM> gram_t;
    if constexpr (FAM == FLOW_ROOT) {
      if (g.epi == EPI_AXPY) product(std::integral_constant<int, EPI_AXPY>{}, std::false_type{}, std::false_type{});
      else if (tile == 32) gemm_tile<double, double, 32, 32, 2, 2, FLOW_RING, EPI_MNEXT, false, false, false, true>(g, false, b, r, per_mat, tm, tn, smem, alpha_of);
      else gemm_tile<double, double, 64, 64, 2, 2, 4, EPI_MNEXT, false, false, false, true>(g, false, b, r, per_mat, tm, tn, smem, alpha_of);
    } else {
      if (g.epi == EPI_RESIDUAL) product(std::integral_constant<int, EPI_RESIDUAL>{}, gram_t{}, gram_t{});
      else if (g.epi == EPI_POLYQ) product(std::integral_constant<int, EPI_POLYQ>{}, gram_t{}, gram_t{});
      else product(std::integral_constant<int, EPI_AXPY>{}, std::false_type{}, std::false_type{});
    }
    if (!go) return;
    if (t == 0) s_ticket = upcoming;
    finish();
  }
}

template <int FAM, int LD, int NCH>
int launch_flow_t(const FlowArgs& a, int batch, hipStream_t s) {
  const size_t ring = (size_t)FLOW_RING * 2 * 64 * 64;      // 64 x 64 fp32 tiles; the fp64 ones (ring of four, or 32 x 32) take less
  const size_t fit = ((size_t)(LD / 16) * 4 * 256 + (size_t)a.fit.nv * 16 * LD) * sizeof(float);
  const size_t lds = ring > fit ? ring : fit;
  const auto kern = flow_kernel<FAM, LD, NCH>;
  const int rc = allow_dynamic_lds((const void*)kern, (int)lds);
  if (rc != PRISM_OK) return rc;
  hipLaunchKernelGGL(kern, dim3(a.cluster * batch), dim3(NT), lds, s, a);
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_EHIP;
}
template <int FAM, int LD>
int launch_flow_ld(const FlowArgs& a, int batch, hipStream_t s) {
  if (a.fit.sv.rows <= 512) return launch_flow_t<FAM, LD, 2>(a, batch, s);
  if constexpr (LD <= 32) return launch_flow_t<FAM, LD, 4>(a, batch, s);
  return PRISM_EINVAL;
}

}  // namespace

int flow_tiles(const GemmDesc& g, int tile) {
  const int tm = g.M / tile, tn = g.N / tile;
  return g.sym ? tm * (tm + 1) / 2 : tm * tn;
}

int launch_flow(const FlowArgs& a, int batch, hipStream_t s) {
  const SolveArgs& sv = a.fit.sv;
  if (batch <= 0 || a.cluster < 1 || (long long)a.cluster * batch > 0x3fffffff || sv.rows % 64 || sv.rows > 1024 || sv.ngroups != sv.rows / 16 ||
      a.nops < 1 || a.ring < 2 || a.nops > FLOW_MAX_OPS || a.fit.nv < 2 || a.fit.nv > PRISM_MAX_ROOT + 1 || a.fit.ldr % 4)
    return PRISM_EINVAL;
  for (int i = 0; i < a.nops; ++i)
    {
      const GemmDesc& g = a.op[i];
      if (g.M % 64 || g.N % 64 || g.K % BK || g.K < BK || g.lda % 4 || g.ldb % 4 || g.ldc % 4 || g.batch != batch || (g.sym && g.M != g.N) ||
          (a.tile[i] != 32 && a.tile[i] != 64) || a.items[i] != flow_tiles(g, a.tile[i]) || (long long)g.M * g.ldc * (g.epi == EPI_MNEXT ? 8 : 4) > 0x7ffffff0ll)
        return PRISM_EINVAL;
      if ((g.epi == EPI_POLYQ || g.epi == EPI_AXPY) && !g.Cin) return PRISM_EINVAL;
      if ((g.epi == EPI_RESIDUAL || g.epi == EPI_MNEXT) && (g.rho_part != sv.rho_part || a.items[i] != sv.nparts)) return PRISM_EINVAL;
    }
  auto by_ld = [&](auto f) -> int {
    constexpr int FAM = decltype(f)::value;
    if (sv.ld == 16) return launch_flow_ld<FAM, 16>(a, batch, s);
    if (sv.ld == 32) return launch_flow_ld<FAM, 32>(a, batch, s);
    return launch_flow_ld<FAM, 64>(a, batch, s);
  };
  if (sv.fn == PRISM_FN_POLAR) return by_ld(std::integral_constant<int, FLOW_GRAM>{});
  if (sv.fn == PRISM_FN_INV_ROOT) return by_ld(std::integral_constant<int, FLOW_ROOT>{});
  return by_ld(std::integral_constant<int, FLOW_FULL>{});
}

}  // namespace prism
