// Host side of libprism: argument checks, workspace layout and the launch sequences of the
// PRISM iterations (paper Table 1; Section 4; App. A.1, A.3, A.4).  Every call only enqueues kernels on
// the caller's stream: the whole budget of iterations is enqueued up front and each kernel
// skips matrices whose `done` flag the on-device solve step has set, so there is no host
// round trip per iteration.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>
#include <vector>
#include <utility>

#include "common.h"
#include "workspace_cache.h"

namespace prism {

static thread_local std::string g_last_error;
void set_last_error(const char* msg) { g_last_error = msg ? msg : ""; }

#ifdef PRISM_AB_SWITCHES
int ab_switch(const char* name) {
  const char* v = getenv(name);
  return v ? atoi(v) : 0;
}
#endif

int allow_dynamic_lds(const void* kernel, int bytes) {
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, int> granted;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { set_last_error("hipGetDevice failed"); return PRISM_EHIP; }
  std::lock_guard<std::mutex> lock(mu);
  int& have = granted[std::make_pair(dev, kernel)];
  if (have >= bytes) return PRISM_OK;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) {
    (void)hipGetLastError();
    set_last_error("hipFuncSetAttribute(MaxDynamicSharedMemorySize) failed");
    return PRISM_EHIP;
  }
  have = bytes;
  return PRISM_OK;
}

// ---------------------------------------------------------------- event profiling
static_assert(PK_COUNT == PRISM_PROFILE_KINDS, "prism.h must size the profile arrays for every kernel kind");
namespace {
struct ProfRec { int kind; hipEvent_t a, b; };
bool g_prof_on = false;
thread_local bool t_prof_off = false;   // set while an entry point that must not create HIP objects runs on this thread
std::vector<ProfRec> g_prof;
std::mutex g_prof_mu;   // calls from several host threads may record while profiling is on
}  // namespace

ProfScope::ProfScope(int kind, hipStream_t s) : slot(-1), stream(s) {
  std::lock_guard<std::mutex> lock(g_prof_mu);
  if (!g_prof_on || t_prof_off) return;
  ProfRec r;
  r.kind = kind;
  if (hipEventCreate(&r.a) != hipSuccess || hipEventCreate(&r.b) != hipSuccess) return;
  (void)hipEventRecord(r.a, s);
  g_prof.push_back(r);
  slot = (int)g_prof.size() - 1;
}
ProfScope::~ProfScope() {
  if (slot < 0) return;
  std::lock_guard<std::mutex> lock(g_prof_mu);
  if (slot < (int)g_prof.size()) (void)hipEventRecord(g_prof[slot].b, stream);
}

namespace {

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Plan {
  int fn, dt, batch, m, n;
  int S, L, Sp, Lp, transpose;
  int d, p, p_s, ld, nv;
  int tile;        // GEMM tile of the main products
  bool split;      // bf16: iterate carried as high + low part
  int nsum;        // partial sums of the Frobenius norm per matrix
  int max_parts;   // residual partials per matrix
  // byte offsets into the workspace
  size_t o_ctrl, o_info, o_sync, o_sumsq, o_rho, o_v0, o_v, o_cpart, o_fit_cpart;
  size_t o_vp0, o_vp;                             // bf16 polar: bf16 planes of the sketches and of V_1 .. V_{nv-1}
  bool has_planes;
  int ngroups;     // workgroups per matrix of the moments kernel
  bool shared_gpu; // PRISM_FLAG_SHARED_GPU
  size_t o_x[2], o_y[2], o_r, o_q, o_t[3];        // fp32 paths (o_y doubles as M64 for inverse root)
  size_t o_xhi[2], o_xlo[2], o_rb, o_qb;          // bf16 polar
  bool x3;                                        // fp32: products from bf16 planes (gemm_split.hip)
  size_t o_x3[2], o_y3[2], o_r3, o_t3;            // ... of the arrays above (Q: planes only, at o_q; t: T_1 of the inverse root)
  int ring; long long ring_bytes;                 // fp32: all iterations in one launch (flow.hip), sets of arrays from o_x[0] on
  int ksplit;      // polar: parts of the K loop of X^T X (0 = one pass); partial products at o_gpart
  size_t o_gpart;
  size_t total;
};

// Internal flag of make_plan: no split-K Gram product.  Its partial products need scratch of their own; a call whose
// workspace is large enough without them only takes the one-pass product.
constexpr unsigned FLAG_NO_SPLIT_K = 1u << 31;
// ... and no flow kernel (whose ring of arrays takes more than the two iterates)
constexpr unsigned FLAG_NO_FLOW = 1u << 30;
// ... and no planes of fp32 operands
constexpr unsigned FLAG_NO_PLANES = 1u << 29;
constexpr long long MAX_ENTRIES = (1ll << 31) - 1;   // of a matrix, sides padded

// Batches that run as two halves unless the caller asks otherwise (run_auto)
bool in_halves(int batch, int S) { return batch >= 8 && batch % 2 == 0 && S >= 1024; }
// inverse root of padded order 64: small_root_kernel (one workgroup per CU above order 48, and still ahead of the general path when
// the launches of that are full: order 64, p = 4, to a tolerance 1024 matrices 0.40 against 1.36 ms, 8192 2.8 against 7.0; with a fixed
// budget of four updates 8192 2.0 against 3.7)
bool takes_small_root(const Plan& P) { return P.fn == PRISM_FN_INV_ROOT && P.Sp == 64 && P.p <= 4 && P.ld <= 32; }
// fp32 polar factor of a 64 x 64 padded iterate: small_polar_kernel
bool takes_small_polar(const Plan& P) {
  static const int off = ab_switch("PRISM_NO_SMALL_KERNEL");
  return !off && P.fn == PRISM_FN_POLAR && P.dt == PRISM_F32 && P.Sp == 64 && P.Lp == 64 && P.ngroups == 1;
}
bool takes_fused_fit(const Plan& P, int sel_batch) {
  return fit_fused_supported(P.Sp, P.ld, sel_batch, P.dt == PRISM_BF16, in_halves(sel_batch, P.S)) && !takes_small_polar(P) && !takes_small_root(P);
}
// All iterations in one launch (flow.hip): sets of arrays in its ring, 0: a launch per step.  bytes: of one set.
// A workgroup for every row block of a fit has to be there (launch_flow's cluster), and the tiles must not be those of a
// launch that fills the chip.  (The first line - batch times order / 16 within the slots - is that of one 16-row block per
// workgroup, not one where both sides are equal: at 16 matrices of order 256 the flow kernel is still far ahead, below.)  Time with launches / with the flow kernel, budget of 40 to 1e-5 (9 to 13 updates), by 64 x 64 tiles
// of the update over the batch:
//   sign          order 256: 16 tiles 2.2, 128 2.0, 256 1.6;  512: 64 1.5, 256 1.5, 512 1.2;  768: 144 1.3, 288 1.1, 576 1.0;  1024: 256 1.0
//   inverse root  order 256: 16 tiles 2.6, 128 1.7, 256 1.9;  512: 64 1.7, 256 1.5, 512 1.1;  768: 144 1.2, 288 1.2, 576 1.1;  1024: 256 1.2
//   polar         order 256: 32 tiles 1.7, 256 1.6, 512 1.4;  512: 128 1.6, 512 1.1, 1024 1.0;  768: 288 1.2, 576 1.2;  1024: 512 1.1
//   square root   order 256: 16 tiles 2.6, 128 2.7, 256 2.0;  512: 64 2.0, 256 1.5, 512 1.2;  768: 144 1.5, 288 1.3;  1024: 256 1.1
int flow_tiles_of(const Plan& P, int sel_batch) { return (P.Sp / 64) * (P.Lp / 64) * sel_batch; }
int flow_ring(const Plan& P, int sel_batch, size_t bytes) {
  static const int off = ab_switch("PRISM_NO_FLOW");
  if (off || P.dt != PRISM_F32 || P.fn == PRISM_FN_SQRT_NEWTON || (P.fn == PRISM_FN_INV_ROOT && (P.p < 2 || P.p > 4)) || P.ksplit) return 0;
  if (P.Sp > 768 || (P.ld == 64 && P.Sp > 512) || !takes_fused_fit(P, sel_batch)) return 0;
  if (flow_tiles_of(P, sel_batch) > (P.Sp <= 512 ? 512 : 320) || FLOW_SLOTS / sel_batch < P.Sp / 16) return 0;
  return bytes <= (16u << 20) ? 8 : 4;
}

// fp32 products from bf16 planes (gemm_split.hip), where the calls are not a launch of their own (flow_ring).  Padding: whole tiles of 128 where
// they cost less than the smaller tiles do (about a fifth per product).  us from fp32 operands / from planes, tolerance 1e-5:
//   sign          24 x 384 1059 / 911, 16 x 512 1340 / 1125, 64 x 512 4082 / 3455, 768: 4 1361 / 1154, 16 3722 / 3334, 1000: 1 961 / 856, 4 2256 / 1676, 2 x 1900
//                 6837 / 4558, 4096 25082 / 16976; padded to 64: 10 x 448 824 / 756, 6 x 576 1002 / 890, 2 x 832 1180 / 986
//   square root   24 x 384 981 / 879, 16 x 512 1174 / 951, 1000: 1 778 / 697, 4 1916 / 1370, 2 x 1900 5608 / 3929, 4096 21024 / 14124; padded to 64: 10 x 448 752 / 706,
//                 6 x 576 826 / 753
//   inverse       24 x 384 1335 / 1129, 16 x 512 1620 / 1332, 1000: 1 1125 / 987, 4 2902 / 2113
//   polar         24 x 576 x 384 1061 / 997, 64 x 768 x 512 3924 / 3734, 1500 x 1000: 1 1011 / 859, 4 2178 / 1784, 6144 x 4096 24706 / 18894
//   inverse root  p = 4, 4 x 896 2059 / 1813, 1000: 1 978 / 924, 4 2457 / 2202, 8 4308 / 3916, 2 x 1900 7167 / 6002, 4096 32383 / 28820; p = 2, 12 x 896 4436 / 4302,
//                 4 x 1000 2200 / 2010; 512 and 768 equal
// Inverse roots: by the order alone, so that a matrix has the same bits alone and in any batch; its fp64 product pays for the padding and gains nothing (order 1088
// would be 1152).  Not for p = 1, where the iterate has the scale of the input, nor for polar factors of more than 8064 rows: the Gram products of up to
// eight such matrices run in parts (P.ksplit), which have no planes; of others (larger batches, orders above 1152) only the products were compared, not the calls.
// The others go by the caller's batch too, so that their bits may depend on it (sign of order 512: one launch on fp32 operands for 8 matrices, planes for 9).
int planes_unit(const Plan& P, int sel_batch) {
  const double s = round_up(P.S, 128) / (double)round_up(P.S, 64), l = round_up(P.L, 128) / (double)round_up(P.L, 64), grown = s * s * l;
  if (P.fn == PRISM_FN_INV_ROOT) return grown < 1.1 ? 128 : 0;
  // Order 384: the products are all epilogue, and full launches are behind (both updates of 64 square roots 119 / 148, of 40 87 / 85)
  if (P.Sp < 512 && (long long)(P.Sp / 64) * (P.Lp / 64) * sel_batch > 1536) return 0;
  if (grown < 1.19) return 128;
  // 64 x 64 tiles: one round (512).  A product of 10 x 448 23 / 20 us, 6 x 576 26 / 24, 3 x 832 34 / 29.  Beyond a round they are ahead too (4 x 832 46 / 38), but there
  // the calls have not been compared.
  return (long long)((P.S + 63) / 64) * ((P.L + 63) / 64) * sel_batch <= 512 ? 64 : 0;
}
bool takes_planes(const Plan& P, int sel_batch) {
  static const int off = ab_switch("PRISM_NO_F32_PLANES") || ab_switch("PRISM_F32_NO_SYM");   // (no such kernel)
  if (off || P.dt != PRISM_F32 || P.ksplit || P.fn == PRISM_FN_SQRT_NEWTON || (P.fn == PRISM_FN_POLAR && P.L > 8192 - 128)) return false;
  if (P.fn == PRISM_FN_INV_ROOT ? P.p < 2 || P.Sp <= 768 : P.Sp < 384) return false;
  return planes_unit(P, sel_batch) && !flow_ring(P, sel_batch, 0);
}

// shared_shapes: the plan of a launch sequence over several shape groups with the same short side;
// the iterate buffers are then laid out per group by the caller (offsets o_x* stay 0).  sel_batch: the batch of the
// whole group where `batch` is a part of it (0: the same)
int make_plan(Plan& P, int fn, int batch, int m, int n, int dt, int degree, int sketch_dim, int root_p,
              unsigned flags, bool shared_shapes = false, int sel_batch = 0) {
  if (batch <= 0 || m <= 0 || n <= 0) return PRISM_EINVAL;
  if (degree != 3 && degree != 5) return PRISM_EINVAL;
  if (sketch_dim < 0 || sketch_dim > PRISM_MAX_SKETCH) return PRISM_EINVAL;
  if (dt != PRISM_F32 && dt != PRISM_BF16) return PRISM_EINVAL;
  if (fn < PRISM_FN_POLAR || fn > PRISM_FN_SQRT_NEWTON) return PRISM_EINVAL;
  if (fn != PRISM_FN_POLAR && m != n) return PRISM_EINVAL;
  if (fn == PRISM_FN_INV_ROOT && (root_p < 1 || root_p > PRISM_MAX_ROOT || degree != 3)) return PRISM_EINVAL;
  if (fn != PRISM_FN_POLAR && dt == PRISM_BF16) return PRISM_EUNSUPPORTED;
  if ((long long)m * n > MAX_ENTRIES) { set_last_error("a matrix may hold at most 2^31 - 1 entries"); return PRISM_EUNSUPPORTED; }
  if (batch > PRISM_MAX_BATCH) { set_last_error("more than PRISM_MAX_BATCH matrices in one group"); return PRISM_EUNSUPPORTED; }
  P = Plan();
  P.fn = fn; P.dt = dt; P.batch = batch; P.m = m; P.n = n;
  P.transpose = (fn == PRISM_FN_POLAR && m < n) ? 1 : 0;
  P.S = m < n ? m : n;
  P.L = m < n ? n : m;
  P.d = degree == 3 ? 1 : 2;
  P.p = fn == PRISM_FN_INV_ROOT ? root_p : 0;
  P.p_s = sketch_dim;
  P.ld = sketch_dim <= 16 ? 16 : (sketch_dim <= 32 ? 32 : 64);
  P.nv = fn == PRISM_FN_INV_ROOT ? root_p + 1 : (fn == PRISM_FN_INVERSE ? 3 : 2 * P.d + 1);
  P.split = (dt == PRISM_BF16) && !(flags & PRISM_FLAG_BF16_PLAIN_ITERATE);
  P.shared_gpu = (flags & PRISM_FLAG_SHARED_GPU) != 0;
  if (dt == PRISM_BF16) {
    P.tile = P.S >= 512 ? 256 : 128;   // padding granularity; the tile is chosen per launch
  } else {
    // Newton: the block elimination wants large pivot blocks.  Others: the padding costs more than 64 x 64
    // tiles do (n = 300: 320 against 384) until the sides are large
    P.tile = P.S <= 256 || (P.S < 4096 && fn != PRISM_FN_SQRT_NEWTON) ? 64 : 128;
  }
  P.Sp = round_up(P.S, P.tile);
  P.Lp = round_up(P.L, P.tile);
  // Polar factor of a few tall matrices: X^T X has few tiles and a long K loop, which would leave
  // most CUs idle; the loop is then cut into parts that run as separate workgroups and a second
  // pass adds the partial products up (in part order, so results stay run-to-run identical).
  P.ksplit = 0;
  static const int no_split_k = ab_switch("PRISM_NO_SPLIT_K");
  if (fn == PRISM_FN_POLAR && !no_split_k && !shared_shapes && !(flags & FLAG_NO_SPLIT_K) && P.Sp > 64) {
    const long long nt = (P.Sp + 127) / 128, gb = sel_batch ? sel_batch : batch, tri = nt * (nt + 1) / 2 * gb, full = nt * nt * gb;
    if (dt == PRISM_BF16 && tri <= 64 && (gb == 1 || (gb <= 8 && P.L >= 8192))) {
      // A single matrix, or up to eight long ones (with several matrices the launch, which a grouped call shares between
      // its shapes, is full enough: three layers of width 512, split 0.61 ms, not 0.54).  Parts by the time they are expected
      // to take, in us, from what was measured (order 768, 128 x 128 tiles): a slab of 32 k 0.37 while the CUs have one
      // workgroup each, the second pass 6, and per part 1.6e-6 per entry or the latency of its loads, the update 2.7e-9 per
      // row and squared order (the parts are of equal length and add up to whole tiles, so a number of parts that does
      // not suit L pads the iterate).  With more workgroups than CUs the slab time is taken to grow in proportion.  That was
      // not measured for this product and is probably too much (three fit a CU; a slab of other 128 x 128 products takes 0.65 to 0.75
      // where two or three do), and it is why 50257 x 768 stops at one each.  One 768 x 3072 matrix: Gram product
      // 35 -> 20 us; 50257 x 768: 88 -> 73 us; 768 x 768 stays one pass (9 us).  Gain per iteration expected / measured at
      // other orders: 128 x 1024 1.5 / 2.4 us, 256 x 2048 12.0 / 10.8, 512 x 1024 1.2 / 4.4, 512 x 4096 32.2 / 27.6, 1024 x 2048
      // 5.1 / 10.2, 1280 x 5120 28.1 / 27.5.
      const double s2 = (double)P.Sp * P.Sp;
      auto cost = [&](long long Kp, int parts) {
        const double load = (double)tri * parts / 256.0;
        return Kp * 0.0116 * (load > 1.0 ? load : 1.0) + (double)Kp * parts * s2 * 2.7e-9 + (parts > 1 ? 6.0 + parts * (s2 * 1.6e-6 > 0.35 ? s2 * 1.6e-6 : 0.35) : 0.0);
      };
      double best = cost(P.Lp, 1);
      const int Lp0 = P.Lp;
      for (int parts = 2; parts <= 64 && parts * tri <= 384 && parts * 256 <= Lp0; ++parts) {
        int unit = P.tile;                    // Kp parts has to be a multiple of the tile, Kp one of 32
        for (int q = parts; unit > 32 && q % 2 == 0; q /= 2) unit /= 2;
        const int Kp = round_up((P.L + parts - 1) / parts, unit);
        if ((long long)P.Sp * Kp * parts > MAX_ENTRIES) continue;   // the padding must not cost a matrix its place within the limit
        if (cost(Kp, parts) < best) { best = cost(Kp, parts); P.ksplit = parts; P.Lp = Kp * parts; }
      }
    } else if (dt == PRISM_F32 && batch <= 8 && P.L > 8192 - 128 && tri <= 48) {
      // as many parts of 1024 rows and more as there may be; they are of equal length and add up to multiples of 64
      // (L need not suit them: 58241 rows, 911 times 64 when rounded up by itself, get 32 parts of 1824)
      for (int parts = 32; parts >= 2; --parts) {
        const int Kp = round_up((P.L + parts - 1) / parts, parts % 2 ? 64 : 32);
        if (Kp >= 1024 && full * parts <= 4096 && (long long)P.Sp * Kp * parts <= MAX_ENTRIES) { P.ksplit = parts; P.Lp = Kp * parts; break; }
      }
    }
  }
  if (!(flags & FLAG_NO_PLANES) && takes_planes(P, sel_batch ? sel_batch : batch) &&
      (long long)round_up(P.S, 128) * round_up(P.L, 128) <= MAX_ENTRIES) {
    P.x3 = true;
    const int unit = planes_unit(P, sel_batch ? sel_batch : batch);
    P.Sp = round_up(P.S, unit);
    P.Lp = round_up(P.L, unit);
  }
  if ((long long)P.Sp * P.Lp > MAX_ENTRIES) {   // the kernels keep some offsets within a matrix in 32 bits
    set_last_error("a matrix may hold at most 2^31 - 1 entries after its sides are rounded up to tile multiples");
    return PRISM_EUNSUPPORTED;
  }
  // shares of the Frobenius norm: 32 to 64 KiB each, so that one large matrix fills the chip (64 shares of a 77 MB matrix
  // took 99 us) and a batch of small ones is not launched 64 times over
  P.nsum = (int)(((long long)m * n + 16383) / 16384);
  if (P.nsum > 512) P.nsum = 512;
  const int t0 = (P.Sp / 64) * (P.Lp / 64);   // prepare-step tiles (inverse root residual of M_0)
  P.max_parts = t0;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  const size_t SS = (size_t)P.Sp * P.Sp, LS = (size_t)P.Lp * P.Sp, B = (size_t)batch;
  P.o_ctrl = take(B * sizeof(Ctrl));
  P.o_info = take(B * sizeof(prism_info));
  P.o_rho = take(B * P.max_parts * sizeof(float));
  P.o_v0 = take((size_t)PRISM_MAX_ITERS * P.Sp * P.ld * sizeof(float));   // S_k^T for every k, generated once per call
  P.o_v = take((size_t)P.nv * B * P.Sp * P.ld * sizeof(float));
  // Room in V: until the fit begins the norm's partial sums lie at its head (4 KiB a matrix at most, in V_1 .. V_{nv-1}).
  // fit_kernel does not store V_nv, and has its counters and coefficient partials there (640 + 8.5 Sp bytes
  // a matrix, of 64 Sp and more; with the residual partials of flow_kernel 4 Sp^2 / 1024 more).
  P.o_sumsq = P.o_v;
  P.o_sync = P.o_v + (size_t)(P.nv - 1) * B * P.Sp * P.ld * sizeof(float);
  P.o_fit_cpart = P.o_sync + B * FIT_SYNC_WORDS * sizeof(unsigned);
  {
    const long long el = (long long)P.Sp * P.ld;
    P.ngroups = el <= 4096 ? 1 : (int)(el / 4096 > 64 ? 64 : el / 4096);   // 1: done inside the solve kernel
    if (fn == PRISM_FN_SQRT_NEWTON) {   // the moments run over the n x n matrices themselves
      const long long mm = (long long)P.Sp * P.Sp / 16384;   // 64 entries a thread (2 x 2048^2: 64 groups 39 us)
      P.ngroups = mm < 1 ? 1 : (mm > 256 ? 256 : (int)mm);
    }
  }
  P.o_cpart = take(B * P.ngroups * 17 * sizeof(double));
  if (dt == PRISM_BF16 && P.ld <= 32 && P.p_s > 0) {   // operands of the plane chain kernel: 3 x 2 bytes per entry
    P.o_vp0 = take((size_t)PRISM_MAX_ITERS * P.Sp * P.ld * 6);
    P.o_vp = take((size_t)(P.nv - 1) * B * P.Sp * P.ld * 6);
    P.has_planes = true;
  }
  if (dt == PRISM_BF16) {
    for (int i = 0; i < 2 && !shared_shapes; ++i) {
      P.o_xhi[i] = take(B * LS * 2);
      P.o_xlo[i] = P.split ? take(B * LS * 2) : 0;
    }
    P.o_r = take(B * SS * 4);
    P.o_rb = take(B * SS * 2);
    P.o_qb = P.d == 2 ? take(B * SS * 2) : 0;
  } else if (fn == PRISM_FN_SQRT_NEWTON) {
    for (int i = 0; i < 2; ++i) { P.o_x[i] = take(B * SS * 4); P.o_y[i] = take(B * SS * 4); }
    P.o_r = take(B * SS * 4);        // M_k
    P.o_q = take(B * SS * 4);        // N_k = M_k^{-1}
    P.o_t[0] = take((size_t)spd_inverse_scratch_floats(P.Sp, batch, sel_batch ? sel_batch : batch) * 4 + 256);   // pivot panels of the inverse
  } else {
    if (fn == PRISM_FN_INVERSE) P.o_y[0] = take(B * SS * 4);   // A / ||A||_F
    const size_t set0 = off;
    P.o_x[0] = take(B * (fn == PRISM_FN_POLAR ? LS : SS) * 4);
    if (fn == PRISM_FN_SQRT) P.o_y[0] = take(B * SS * 4);
    if (fn == PRISM_FN_INV_ROOT) P.o_y[0] = take(B * SS * 8);  // M
    const size_t iterate = off - set0;
    P.o_r = take(B * SS * 4);
    if (fn == PRISM_FN_INV_ROOT) for (int i = 0; i < 3; ++i) P.o_t[i] = take(B * SS * 4);
    else P.o_q = (P.d == 2 || fn == PRISM_FN_INVERSE) ? take(B * SS * (P.x3 ? 6 : 4)) : 0;
    P.ring = (flags & FLAG_NO_FLOW) || P.x3 ? 0 : flow_ring(P, sel_batch ? sel_batch : batch, off - set0);
    if (P.ring) {
      P.ring_bytes = (long long)(off - set0);
      off = set0 + (size_t)P.ring * P.ring_bytes;
      P.o_x[1] = P.o_x[0] + P.ring_bytes;
      P.o_y[1] = P.o_y[0] + P.ring_bytes;
    } else {
      P.o_x[1] = off;
      if (fn == PRISM_FN_SQRT || fn == PRISM_FN_INV_ROOT) P.o_y[1] = off + (P.o_y[0] - P.o_x[0]);
      off += iterate;
    }
    if (P.x3) {
      for (int i = 0; i < 2; ++i) {
        P.o_x3[i] = take(B * (fn == PRISM_FN_POLAR ? LS : SS) * 6);
        if (fn == PRISM_FN_SQRT || (fn == PRISM_FN_INVERSE && i == 0)) P.o_y3[i] = take(B * SS * 6);
      }
      P.o_r3 = take(B * SS * 6);
      if (P.p == 3 || P.p == 4) P.o_t3 = take(B * SS * 6);
    }
  }
  P.o_gpart = P.ksplit ? take(B * P.ksplit * SS * 4) : 0;
  P.total = off;
  return PRISM_OK;
}

std::mutex g_mu;
WorkspaceCache g_cache;

// optional: the caller takes a plan that needs less if there is no such memory
int get_workspace(size_t bytes, const void* owner, const prism_options* opt, char** out, bool optional = false) {
  if (opt && opt->workspace) {
    if (opt->workspace_bytes < bytes || ((uintptr_t)opt->workspace & 255)) return PRISM_ENOMEM;
    *out = (char*)opt->workspace;
    return PRISM_OK;
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { set_last_error("hipGetDevice failed"); return PRISM_EHIP; }
  std::lock_guard<std::mutex> lock(g_mu);
  void* p = g_cache.get(dev, owner, bytes, optional, [](size_t n) -> void* {
    void* fresh = nullptr;
    if (hipMalloc(&fresh, n) == hipSuccess) return fresh;
    (void)hipGetLastError();
    return nullptr;
  });
  if (!p) {
    if (!optional) set_last_error("hipMalloc of the workspace failed");
    return PRISM_ENOMEM;
  }
  *out = (char*)p;
  return PRISM_OK;
}

#define CHECK_LAUNCH(expr)                         \
  do {                                             \
    int rc_ = (expr);                              \
    if (rc_ != PRISM_OK) return rc_;               \
  } while (0)

int check_hip() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error(hipGetErrorString(e)); return PRISM_EHIP; }
  return PRISM_OK;
}

struct Run {
  Plan P;
  char* ws;
  hipStream_t s;
  Ctrl* ctrl;
  prism_info* info;
  float* rho;
  float* v0;
  float* v;
  uint16_t* vp0 = nullptr;             // bf16 planes of the sketches / of V_1 .. (bf16 polar, large launches)
  uint16_t* vp = nullptr;
  int max_iters, warm;
  int fit_polls = FIT_POLLS;
  const float* sched; int sched_len;   // caller's coefficients for the leading updates (host array)
  int first_fit;                       // first update whose coefficient is fitted
  double tol;
  uint64_t seed;
  // bf16 polar: the iterate buffers, per shape group (one group for a single-shape call).  All
  // groups share the short side, so R, Q, the chain vectors and the control blocks of all their
  // matrices form one batch (matrices [boff, boff + batch) belong to the group); only the Gram
  // product and the update see the long side, and take all groups in one launch each.
  // Plain iterate, no padding, tall or square input: the caller's array serves as the odd one of
  // the two iterate buffers (the input is consumed by the prepare step before the first update
  // writes there), so that after an odd number of updates the result is in place.
  struct XGroup {
    int batch, boff, m, n, L, Lp, transpose;
    void* x;                                   // caller's array
    uint16_t* Xhi[2]; uint16_t* Xlo[2];        // iterate [Lp][Sp], double buffered
    bool aliased;                              // buffer 1 is the caller's array
    double* sumsq; int nsum;                   // partial sums of the Frobenius norms (several groups)
    int ksplit; float* gpart;                  // parts of the K loop of X^T X (0: one pass) and their products
  };
  std::vector<XGroup> xg;
  // Kernels whose sums differ in order are chosen by the caller's batch of these matrices, however it is enqueued (whole,
  // as two halves, as a group of a grouped call), so that the results are the same bits.
  int sel_batch = 0;

  template <typename T> T* at(size_t off) const { return (T*)(ws + off); }

  // The planes of an fp32 array (P.x3)
  struct Planes { const float* x; uint16_t* p; long long ps; bool only; };   // only: there is no fp32 array, x is its name
  std::vector<Planes> split;
  const Planes* planes_of(const void* x) const {
    for (const Planes& q : split)
      if (q.x == x) return &q;
    return nullptr;
  }
  void list_planes() {
    if (!P.x3) return;
    const long long SS = (long long)P.batch * P.Sp * P.Sp, LS = (long long)P.batch * P.Lp * P.Sp;
    auto add = [&](size_t o, size_t o3, long long ps) { if (o3) split.push_back({at<float>(o), at<uint16_t>(o3), ps, o == o3}); };
    for (int i = 0; i < 2; ++i) {
      add(P.o_x[i], P.o_x3[i], P.fn == PRISM_FN_POLAR ? LS : SS);
      add(P.o_y[i], P.o_y3[i], SS);
    }
    add(P.o_r, P.o_r3, SS);
    add(P.o_q, P.o_q, SS);
    add(P.o_t[1], P.o_t3, SS);
  }
  // what the first products read, from the arrays that the prepare step has written
  void split_start() {
    for (const Planes& q : split) {
      const bool start = q.x == at<float>(P.o_x[0]) || (P.o_y3[0] && q.x == at<float>(P.o_y[0])) || (P.fn == PRISM_FN_INV_ROOT && q.x == at<float>(P.o_r));
      if (start) launch_split3(q.x, q.p, q.ps, q.ps, s);
    }
  }
  GemmDesc with_planes(GemmDesc g) const {
    const Planes *a = planes_of(g.A), *b = planes_of(g.B), *c = planes_of(g.C);
    if (!a || !b) return g;
    g.A3 = a->p; g.psA = a->ps; g.B3 = b->p; g.psB = b->ps;
    if (c) {
      g.C3 = c->p; g.psC = c->ps;
      if (c->only) g.C = nullptr;
    }
    return g;
  }
  int gemm(const GemmDesc& g) const {
    const GemmDesc q = with_planes(g);
    return q.A3 ? launch_gemm_split(q, nullptr, s) : launch_gemm_f32(g, s);
  }
  int gemm_pair(const GemmDesc& a, const GemmDesc& b) const {
    const GemmDesc qa = with_planes(a), qb = with_planes(b);
    return qa.A3 && qb.A3 ? launch_gemm_split(qa, &qb, s) : launch_gemm_f32_pair(a, b, s);
  }
  int tiles(int M, int N, int sym) const { return P.x3 ? split_tiles(M, N, sel_batch, sym) : f32_tiles(M, N, sel_batch, sym); }

  // sketch + chain V_j = R V_{j-1} (fp32 matrix cores, skinny N = padded sketch width)
  // Rb: bf16 copy of R (bf16 polar path): the products then read it instead of R, except the diagonal,
  // which comes from D (entry i of matrix b at D[b * strideD + i * ldd])
  int chain(const float* R, int k, const uint16_t* Rb = nullptr, const float* D = nullptr, long long strideD = 0,
            int ldd = 0) {
    const int Sp = P.Sp, ld = P.ld;
    const long long vs = (long long)P.batch * Sp * ld;
    if (Sp == 64 && !Rb) {   // whole chain in one launch
      ProfScope ps(PK_CHAIN, s);
      return launch_chain_tiny(R, (long long)Sp * Sp, Sp, v0 + (long long)(k - first_fit) * Sp * ld, 0, v, vs,
                               (long long)Sp * ld, P.nv, ld, P.batch, ctrl, s);
    }
    for (int j = 1; j <= P.nv; ++j) {
      const float* vin = (j == 1) ? v0 + (long long)(k - first_fit) * Sp * ld : v + (j - 2) * vs;
      const long long sin = (j == 1) ? 0 : (long long)Sp * ld;
      ProfScope ps(PK_CHAIN, s);
      if (Rb && planes()) {
        const long long pe = (long long)Sp * ld * 3;   // plane entries per matrix
        const uint16_t* pin = (j == 1) ? vp0 + (long long)(k - first_fit) * pe : vp + (long long)(j - 2) * P.batch * pe;
        uint16_t* pout = j < P.nv ? vp + (long long)(j - 1) * P.batch * pe : nullptr;
        CHECK_LAUNCH(launch_chain_planes(Rb, (long long)Sp * Sp, Sp, D, strideD, ldd, vin, sin, pin, j == 1 ? 0 : pe,
                                         v + (j - 1) * vs, (long long)Sp * ld, pout, pe, Sp, ld, P.batch, ctrl, s));
      } else if (Rb)
        CHECK_LAUNCH(launch_chain_bf16(Rb, (long long)Sp * Sp, Sp, D, strideD, ldd, vin, sin, v + (j - 1) * vs,
                                       (long long)Sp * ld, Sp, ld, P.batch, ctrl, s, sel_batch));
      else
        CHECK_LAUNCH(launch_chain(R, (long long)Sp * Sp, Sp, vin, sin, v + (j - 1) * vs, (long long)Sp * ld, Sp, ld,
                                  P.batch, ctrl, s, sel_batch));
    }
    return PRISM_OK;
  }

  // The coefficient of iteration k: chain, moments, solve.  One launch where fit_kernel takes the matrices (a rule on
  // order and batch of a call on one group, so that grouped and single calls agree); without a fit the solve only.
  int fit(int k, int nparts, const float* R, const uint16_t* Rb = nullptr, const float* D = nullptr, long long strideD = 0,
          int ldd = 0) {
    if (!fit_needed(k)) return solve(k, nparts);
    if (!fused()) {
      CHECK_LAUNCH(chain(R, k, Rb, D, strideD, ldd));
      return solve(k, nparts);
    }
    ProfScope ps(PK_CHAIN, s);
    return launch_fit(fit_args(k, nparts, R, Rb, D, strideD, ldd), P.batch, s);
  }
  FitArgs fit_args(int k, int nparts, const float* R, const uint16_t* Rb, const float* D, long long strideD, int ldd) const {
    FitArgs f = {};
    f.sv = solve_args(k, nparts, 0);
    f.sv.ngroups = P.Sp / 16; f.sv.cpart = at<double>(P.o_fit_cpart);
    f.b16 = Rb != nullptr; f.R = Rb ? (const void*)Rb : (const void*)R; f.strideR = (long long)P.Sp * P.Sp; f.ldr = P.Sp;
    f.D = D; f.strideD = strideD; f.ldd = ldd;
    f.V0 = v0 + (long long)(k - first_fit) * P.Sp * P.ld; f.V = v; f.nv = P.nv;
    f.sync = at<unsigned>(P.o_sync); f.epoch = FIT_EPOCH * (unsigned)k; f.polls = fit_polls;
    return f;
  }
  bool fused() const { return takes_fused_fit(P, sel_batch); }
  // Without a tolerance no launches follow convergence, and the line lies lower.  Eight updates, launches / flow kernel: sign order
  // 256, 128 tiles 1.2, 512 0.98; order 512, 128 tiles 1.2, 256 1.0, 512 0.88; inverse root 256 tiles 1.2 and 1.1; polar 256 tiles 1.1
  // and 1.1, 512 1.0 and 0.90; square root (two updates) 2 x 128 tiles 1.2 and 1.1, 2 x 256 0.93 and 0.89; order 768 0.96 to 1.04.
  bool flow() const {
    return P.ring && (tol > 0.0 || (P.Sp <= 512 && flow_tiles_of(P, sel_batch) * (P.fn == PRISM_FN_SQRT ? 2 : 1) <= 256));
  }
  bool small_root() const { return takes_small_root(P); }
  bool small_polar() const { return takes_small_polar(P); }

  SolveArgs solve_args(int k, int nparts, int phase) const {
    SolveArgs a = {};
    a.phase = phase;
    a.fn = P.fn; a.k = k; a.d = P.d; a.p = P.p; a.n = P.S; a.rows = P.Sp; a.ld = P.ld;
    a.V = v; a.vstride = (long long)P.batch * P.Sp * P.ld; a.bstride = (long long)P.Sp * P.ld;
    a.rho_part = rho; a.nparts = nparts;
    a.ctrl = ctrl; a.info = info; a.tol = tol; a.max_iters = max_iters;
    a.mode = k < sched_len ? 3 : (P.p_s == 0 ? 1 : (k < warm ? 2 : 0));
    a.sched_alpha = k < sched_len ? sched[k] : 0.0f;
    a.last = (k == max_iters);
    a.cpart = at<double>(P.o_cpart); a.ngroups = P.ngroups;
    return a;
  }
  int solve(int k, int nparts, int phase = 0) {
    const SolveArgs a = solve_args(k, nparts, phase);
    if (a.mode == 0 && !a.last && a.ngroups > 1 && P.fn != PRISM_FN_SQRT_NEWTON) {
      ProfScope ps(PK_MOMENTS, s);
      launch_moments(a, P.batch, s);
    }
    {
      ProfScope ps(PK_SOLVE, s);
      launch_solve(a, P.batch, s);
    }
    return check_hip();
  }
  bool fit_needed(int k) const { return P.p_s > 0 && k >= first_fit && k < max_iters; }
  // bf16 chain products too large for the 16-row kernel read V as bf16 planes
  bool planes() const {
    return vp0 && !fused() && chain_bf16_supported(P.Sp, P.ld, sel_batch, P.Sp) && !chain_takes_small_kernel(P.Sp, P.ld, sel_batch, true);
  }
};

GemmDesc f32_desc(const Run& r, const float* A, int lda, long long sa, const float* B, int ldb, long long sb,
                  int M, int N, int K, int a_km) {
  GemmDesc g = {};
  g.A = A; g.strideA = sa; g.lda = lda; g.B = B; g.strideB = sb; g.ldb = ldb;
  g.M = M; g.N = N; g.K = K; g.a_km = a_km; g.batch = r.P.batch; g.sel_batch = r.sel_batch; g.n_true = r.P.S; g.ctrl = r.ctrl;
  g.c_in = 1.0f;
  return g;
}

// Upper-triangle products with a mirrored lower half.  Taken only where the symmetry does not rest
// on iterates commuting: X^T X, the square of a matrix that was itself stored mirrored, and updates
// whose result never re-enters the residual (X of the inverse root, X and Y of DB Newton).  In the
// coupled square root, the sign and the Chebyshev inverse the iterates commute only up to kappa * eps;
// mirroring there turns that defect into a perturbation the iteration amplifies (divergence from
// kappa ~ 1e3 on), so those keep every tile.
int f32_sym() {
  static const int off = ab_switch("PRISM_F32_NO_SYM");
  return off ? 0 : 1;
}

// The products of an iteration for the flow kernel.  phase: -1 beside the fit (alpha enters at the end), then in order; products of
// the same phase read nothing of each other.
struct FlowOp { GemmDesc d; int phase; };

int run_flow(const Run& r, const FlowOp* ops, int nops, bool residual, const float* R, int nparts0) {
  const Plan& P = r.P;
  FlowArgs a = {};
  const int slots = FLOW_SLOTS / r.sel_batch;
  int widest = 0, nparts = 0;
  a.nops = nops; a.residual = residual;
  // phases: -2 the residual, -1 beside the fit, ...
  auto phase = [&](int i) { return i < (int)residual ? -2 : ops[i].phase; };
  for (int i = 0; i < nops; ++i) {
    // 32 x 32 tiles where the phase has workgroups for all of them
    int fine = 0;
    for (int j = 0; j < nops; ++j)
      if (phase(j) == phase(i)) fine += flow_tiles(ops[j].d, 32);
    static const int forced = ab_switch("PRISM_FLOW_TILE");
    a.tile[i] = forced ? forced : (fine <= slots && phase(i) != -1 ? 32 : 64);   // beside the fit nobody waits for them
    a.items[i] = flow_tiles(ops[i].d, a.tile[i]);
    if (ops[i].d.epi == EPI_RESIDUAL || ops[i].d.epi == EPI_MNEXT) nparts = a.items[i];
  }
  for (int i = 0; i < nops; ++i) {
    int together = phase(i) == -1 ? P.Sp / 16 : 0;
    a.start[i] = phase(i) == -1 ? -1 : 0;
    for (int j = residual; j < nops; ++j) {
      if (phase(i) >= 0 && phase(j) < phase(i)) a.start[i] += a.items[j];
      if (phase(j) == phase(i)) together += a.items[j];
    }
    if (i < (int)residual) together = a.items[i];
    if (together > widest) widest = together;
  }
  // beside other groups a quarter of the chip is left to them: their workgroups otherwise wait until this call is through.  Inverse
  // roots of 16 matrices of 8 orders from 10 to 576, workgroups of a group / us: 256 1170, 192 1070, 128 1245, 64 1670 (the one mix
  // that this was measured on)
  const int share = P.shared_gpu ? 3 * FLOW_SLOTS / 4 / r.sel_batch : slots, least = P.Sp / 16;
  const int most = share > least ? share : least;
  a.cluster = widest < most ? widest : most;
  a.fit = r.fit_args(0, nparts, R, nullptr, nullptr, 0, 0);
  a.rho0 = r.rho; a.nparts0 = nparts0;
  float* rho = (float*)(r.at<double>(P.o_fit_cpart) + (long long)P.batch * (P.Sp / 16) * 17);   // behind the coefficient partials
  a.fit.sv.rho_part = rho;
  a.fit.V0 = r.v0; a.fit.epoch = 0;
  a.ring = P.ring; a.ring_bytes = P.ring_bytes;
  const char* set0 = r.at<char>(P.o_x[0]);
  auto in_ring = [&](const void* p) { return (const char*)p >= set0 && (const char*)p < set0 + P.ring * P.ring_bytes; };
  for (int i = 0; i < nops; ++i) {
    a.op[i] = ops[i].d;
    a.op[i].rho_part = rho;
    a.fixed_a[i] = !in_ring(ops[i].d.A);
    // results that the next iteration starts from: the descriptor has them in the second set
    a.next_c[i] = (const char*)ops[i].d.C >= set0 + P.ring_bytes;
    if (a.next_c[i]) a.op[i].C = (char*)a.op[i].C - P.ring_bytes;
  }
  a.first_fit = P.p_s == 0 || r.first_fit > r.max_iters ? r.max_iters : r.first_fit;
  a.warm = r.warm; a.sched_len = r.sched_len; a.p_s = P.p_s;
  for (int i = 0; i < r.sched_len; ++i) a.sched[i] = r.sched[i];
  ProfScope ps(PK_FLOW, r.s);
  return launch_flow(a, P.batch, r.s);
}

// Matrices of padded order 64: the whole call from the caller's array to the caller's array (small.hip)
int run_small(const Run& r, float* x) {
  const Plan& P = r.P;
  auto fill = [&](auto& a) {
    a.sv = r.solve_args(0, 1, 0);
    a.x = x; a.V0 = r.v0;
    a.p_s = P.p_s; a.first_fit = r.first_fit; a.warm = r.warm; a.sched_len = r.sched_len;
    for (int i = 0; i < r.sched_len; ++i) a.sched[i] = r.sched[i];
  };
  if (P.fn == PRISM_FN_POLAR) {
    SmallPolarArgs a = {};
    fill(a);
    a.m = P.m; a.n = P.n; a.L = P.L; a.transpose = P.transpose;
    ProfScope ps(PK_F32_SMALL_POLAR, r.s);
    return launch_small_polar(a, P.batch, r.s);
  }
  SmallRootArgs a = {};
  fill(a);
  ProfScope ps(PK_SMALL_ROOT, r.s);
  return launch_small_root(a, P.batch, r.s);
}

int run_polar_f32(Run& r) {
  const Plan& P = r.P;
  const int Sp = P.Sp, Lp = P.Lp;
  const long long SS = (long long)Sp * Sp, LS = (long long)Lp * Sp;
  float* X[2] = {r.at<float>(P.o_x[0]), r.at<float>(P.o_x[1])};
  float* R = r.at<float>(P.o_r);
  float* Q = P.d == 2 ? r.at<float>(P.o_q) : nullptr;
  const bool polar = P.fn != PRISM_FN_SIGN;
  const int sym = polar ? f32_sym() : 0;
  const int nparts = r.tiles(Sp, Sp, sym);
  // G = X^T X; matrix sign: G = X X (any square input, all tiles)
  auto residual = [&](int cur) {
    GemmDesc g = f32_desc(r, X[cur], Sp, LS, X[cur], Sp, LS, Sp, Sp, Lp, polar ? 1 : 0);
    g.sym = sym;
    g.epi = EPI_RESIDUAL; g.C = R; g.strideC = SS; g.ldc = Sp; g.rho_part = r.rho;
    return g;
  };
  auto square = [&]() {
    GemmDesc q = f32_desc(r, R, Sp, SS, R, Sp, SS, Sp, Sp, Sp, polar ? 1 : 0);  // mirrored R: R^2 = R^T R (from planes: to rounding, see gemm_split.hip)
    q.sym = sym;
    q.epi = EPI_POLYQ; q.C = Q; q.strideC = SS; q.ldc = Sp; q.Cin = R; q.strideCin = SS; q.ldcin = Sp; q.c1 = 0.5f;
    return q;
  };
  auto update = [&](int cur) {
    GemmDesc a = f32_desc(r, X[cur], Sp, LS, P.d == 2 ? Q : R, Sp, SS, Lp, Sp, Sp, 0);      // X + X Q
    a.epi = EPI_AXPY; a.C = X[cur ^ 1]; a.strideC = LS; a.ldc = Sp; a.Cin = X[cur]; a.strideCin = LS; a.ldcin = Sp;
    a.coef_is_alpha = P.d == 1;
    return a;
  };
  if (r.flow()) {
    if (P.d == 1) {
      const FlowOp ops[] = {{residual(0), 0}, {update(0), -1}};
      return run_flow(r, ops, 2, true, R, nparts);
    }
    const FlowOp ops[] = {{residual(0), 0}, {square(), -1}, {update(0), 0}};
    return run_flow(r, ops, 3, true, R, nparts);
  }
  int cur = 0;
  for (int k = 0; k <= r.max_iters; ++k) {
    if (k == r.max_iters && r.tol <= 0.0) break;
    if (polar && P.ksplit) {
      ProfScope ps(PK_F32_RESID, r.s);
      const int Kp = Lp / P.ksplit;
      float* gpart = r.at<float>(P.o_gpart);
      for (int b = 0; b < P.batch; ++b) {   // the parts of one matrix are the batch of a plain product
        GemmDesc sp = f32_desc(r, X[cur] + (long long)b * LS, Sp, (long long)Kp * Sp, X[cur] + (long long)b * LS, Sp,
                               (long long)Kp * Sp, Sp, Sp, Kp, 1);
        sp.batch = P.ksplit; sp.sel_batch = 0; sp.epi = EPI_STORE; sp.C = gpart + (long long)b * P.ksplit * SS; sp.strideC = SS; sp.ldc = Sp;
        sp.ctrl = r.ctrl + b; sp.ctrl_parts = P.ksplit;
        CHECK_LAUNCH(launch_gemm_f32(sp, r.s));
      }
      GramReduceArgs ra = {};
      ra.ngroups = 1; ra.part[0] = gpart; ra.parts[0] = P.ksplit; ra.first[1] = P.batch; ra.np = Sp; ra.n_true = P.S;
      ra.R32 = R; ra.rho_part = r.rho; ra.rho_stride = gram_reduce_parts(Sp); ra.ctrl = r.ctrl;
      launch_gram_reduce(ra, r.s);
      CHECK_LAUNCH(check_hip());
    } else {
      ProfScope ps(PK_F32_RESID, r.s);
      CHECK_LAUNCH(r.gemm(residual(cur)));
    }
    CHECK_LAUNCH(r.fit(k, (polar && P.ksplit) ? gram_reduce_parts(Sp) : nparts, R));
    if (k == r.max_iters) break;
    if (P.d == 2) { ProfScope ps(PK_F32_POLYQ, r.s); CHECK_LAUNCH(r.gemm(square())); }
    { ProfScope ps(PK_F32_APPLY, r.s); CHECK_LAUNCH(r.gemm(update(cur))); }
    cur ^= 1;
  }
  return PRISM_OK;
}

// Tile shape of a bf16 product.  Large tiles move fewer bytes per flop but need enough tiles to give
// every CU work and a K long enough to amortise their epilogue: 128 x 128 (three workgroups per CU)
// below that.  (At K = 768 the bare product is faster with large tiles from 144 tiles on, the update
// GEMM with its three-output epilogue is not.)  Among the large shapes 256 x 128 runs two workgroups
// per CU, which overlap each other's epilogue and barrier waits; 256 x 256 runs one.
struct Tile { int m, n; };
int bf16_tile_forced() {
  static const int forced = ab_switch("PRISM_BF16_TILE");   // 128, 256, or 2561 for 256 x 128
  return forced;
}
Tile bf16_big_tile() {
  static const int big = ab_switch("PRISM_BF16_BIG");       // 2: 256 x 128
  return big == 2 ? Tile{256, 128} : Tile{256, 256};
}
Tile bf16_tile(const Plan& P, int M, int N, int K, bool symmetric) {
  const int forced = bf16_tile_forced();
  if (P.tile != 256) return Tile{128, 128};
  if (forced == 128) return Tile{128, 128};
  if (forced == 256) return Tile{256, 256};
  if (forced == 2561) return Tile{256, 128};
  const long long per_mat = symmetric ? (long long)(M / 256) * (M / 256 + 1) / 2 : (long long)(M / 256) * (N / 256);
  // (32 x 1536^2, five iterations: 3.58 ms with large tiles against 4.18; 64 x 768^2: 1.88 against 1.72)
  return (per_mat * P.batch >= 192 && K >= 1536) ? bf16_big_tile() : Tile{128, 128};
}

int run_polar_bf16(Run& r) {
  const Plan& P = r.P;
  const int Sp = P.Sp;
  const int sym = 1;   // X^T X and the square of the (mirrored, hence exactly symmetric) R: upper triangle of tiles
  const int ng = (int)r.xg.size();
  if (ng < 1 || ng > BF16_MAX_GROUPS) return PRISM_EINVAL;
  // Tile shapes.  One shape per launch: with several groups the Gram product and the update take the
  // large tiles when the launch as a whole has enough of them.
  long long gram256 = 0, upd256 = 0;
  for (const Run::XGroup& x : r.xg) {
    gram256 += (long long)(Sp / 256) * (Sp / 256 + 1) / 2 * x.batch;
    upd256 += (long long)(x.Lp / 256) * (Sp / 256) * x.batch;
  }
  Tile Tg, Ta;
  if (ng == 1) {
    // with other work beside this call, large Gram tiles also when they are few (measured on the
    // Muon-shaped batch of four groups on four streams: 3.96 -> 3.80 ms; alone on the GPU the same
    // choice costs 1.40 instead of 1.07 ms of Gram time per step)
    Tg = bf16_tile(P, Sp, Sp, r.xg[0].Lp, true);
    Ta = bf16_tile(P, r.xg[0].Lp, Sp, Sp, false);
    if (P.tile == 256 && P.shared_gpu && bf16_tile_forced() == 0) Tg = Tile{256, 256};
  } else {
    const bool pad256 = P.tile == 256;
    static const int multi_gram = ab_switch("PRISM_BF16_MULTI_GRAM");   // 1: 128 x 128, 2: 256 x 128, 3: 256 x 256
    static const int multi_upd = ab_switch("PRISM_BF16_MULTI_UPD");
    auto pick = [&](int sw, bool big) {
      if (!pad256 || sw == 1) return Tile{128, 128};
      if (sw == 2) return Tile{256, 128};
      if (sw == 3) return Tile{256, 256};
      return big ? bf16_big_tile() : Tile{128, 128};
    };
    // measured on the Muon-shaped groups (order 768, K from 768 to 3072): 256 x 256 tiles (eight
    // wavefronts) for the Gram products and the updates beat 128 x 128 ones from 96 matrices' worth of
    // tiles on (update: 2.90 against 2.96 ms per step with 256 x 128 tiles)
    Tg = multi_gram ? pick(multi_gram, false) : ((pad256 && gram256 >= 96) ? Tile{256, 256} : Tile{128, 128});
    Ta = multi_upd ? pick(multi_upd, false) : ((pad256 && upd256 >= 96) ? Tile{256, 256} : Tile{128, 128});
  }
  const Tile Tq = (ng == 1) ? Tg : bf16_tile(P, Sp, Sp, Sp, true);
  const long long SS = (long long)Sp * Sp;
  float* R = r.at<float>(P.o_r);
  uint16_t* Rb = r.at<uint16_t>(P.o_rb);
  uint16_t* Qb = P.d == 2 ? r.at<uint16_t>(P.o_qb) : nullptr;
  static const int chain_f32 = ab_switch("PRISM_BF16_CHAIN_F32");
  // The fit can read the bf16 copy of R (plus its exact diagonal) when the chain kernels take the
  // shape; with symmetric tiles the fp32 matrix is then not written at all: the Gram epilogue
  // stores the bf16 copy and the diagonal (at the head of the buffer of R), R^2 reads the copy.
  // Only with the plain bf16 iterate: with the split one the linear term of Q = R/2 + alpha R^2 keeps
  // the fp32 R (taking it from the bf16 copy raises the residual floor by a few 1e-4, which at
  // tol = 1e-2 cost the reduced config-3 case one more iteration than the oracle).
  const bool chain_b = !chain_f32 && (P.p_s == 0 || chain_bf16_supported(Sp, P.ld, r.sel_batch, Sp));
  const bool lean = chain_b && sym && !P.split;
  float* Dg = R;
  const int ntg = Sp / Tg.m;
  int nparts = (Tg.m / Tg.n) * ntg * (ntg + 1) / 2;   // residual partial sums per matrix: tiles of the Gram product
  for (const Run::XGroup& x : r.xg)
    if (x.ksplit && nparts < gram_reduce_parts(Sp)) nparts = gram_reduce_parts(Sp);   // ... or of its second pass
  // launch order of the groups: longest K first, so that the short tiles fill the last round
  int order[BF16_MAX_GROUPS];
  for (int i = 0; i < ng; ++i) order[i] = i;
  for (int i = 1; i < ng; ++i)
    for (int j = i; j > 0 && r.xg[order[j]].Lp > r.xg[order[j - 1]].Lp; --j) { const int t = order[j]; order[j] = order[j - 1]; order[j - 1] = t; }
  int cur = 0;
  for (int k = 0; k <= r.max_iters; ++k) {
    if (k == r.max_iters && r.tol <= 0.0) break;
    {
      Bf16Desc gd[BF16_MAX_GROUPS], sd[BF16_MAX_GROUPS];   // one pass, split
      int n1 = 0, n2 = 0;
      GramReduceArgs ra = {};
      for (int i = 0; i < ng; ++i) {
        const Run::XGroup& x = r.xg[order[i]];
        Bf16Desc& g = x.ksplit ? sd[n2] : gd[n1++];
        g = Bf16Desc{};
        g.sym = sym;
        // X^T X straight from the [Lp][Sp] iterate: both operands stored [K][M]
        g.A = x.Xhi[cur]; g.lda = Sp; g.B = x.Xhi[cur]; g.ldb = Sp; g.km = 3;
        g.M = Sp; g.N = Sp; g.ctrl = r.ctrl + x.boff;
        if (x.ksplit) {
          // part p of a matrix = rows [p Kp, (p + 1) Kp) of its iterate: the parts of all matrices are one batch, Kp Sp apart
          g.K = x.Lp / x.ksplit; g.batch = x.batch * x.ksplit; g.strideA = g.strideB = (long long)g.K * Sp;
          g.epi = BEPI_STORE; g.C32 = x.gpart; g.strideC32 = SS; g.ldc32 = Sp; g.ctrl_parts = x.ksplit;
          ra.part[n2] = x.gpart; ra.parts[n2] = x.ksplit; ra.boff[n2] = x.boff; ra.first[n2 + 1] = ra.first[n2] + x.batch;
          ++n2;
          continue;
        }
        g.K = x.Lp; g.batch = x.batch; g.strideA = g.strideB = (long long)x.Lp * Sp; g.epi = BEPI_GRAM; g.n_true = P.S;
        g.C32 = lean ? nullptr : R + x.boff * SS; g.strideC32 = SS; g.ldc32 = Sp;
        // with the bf16 chain only the R^2 epilogue and the chain's diagonal read the fp32 matrix: both stay
        // inside the tiles the Gram product computes when its tile rows are whole multiples of those of R^2
        g.upper32 = (chain_b && Tg.m % Tq.m == 0) ? 1 : 0;
        g.Cb = Rb + x.boff * SS; g.strideCb = SS; g.ldcb = Sp;
        g.diag = lean ? Dg + (long long)x.boff * Sp : nullptr; g.strideDiag = Sp;
        g.rho_part = r.rho + (long long)x.boff * nparts; g.rho_stride = nparts;
      }
      ProfScope ps(PK_BF16_GRAM, r.s);
      if (n1) CHECK_LAUNCH(launch_gemm_bf16_multi(gd, n1, Tg.m, Tg.n, r.s));
      if (n2) {
        CHECK_LAUNCH(launch_gemm_bf16_multi(sd, n2, 128, 128, r.s));
        ra.ngroups = n2; ra.np = Sp; ra.n_true = P.S;
        ra.R32 = lean ? nullptr : R; ra.Rb = Rb; ra.diag = lean ? Dg : nullptr; ra.rho_part = r.rho; ra.rho_stride = nparts;
        ra.ctrl = r.ctrl;
        launch_gram_reduce(ra, r.s);
        CHECK_LAUNCH(check_hip());
      }
    }
    // where the fit reads R: the bf16 copy with the exact diagonal, or the fp32 matrix
    const uint16_t* fit_b = chain_b ? Rb : nullptr;
    const float* fit_d = lean ? Dg : (chain_b ? R : nullptr);
    const long long fit_sd = lean ? Sp : (chain_b ? SS : 0);
    const int fit_ldd = lean ? 1 : (chain_b ? Sp + 1 : 0);
    Bf16Desc q = {};
    if (P.d == 2) {   // one launch over the matrices of all groups: R has the same order everywhere
      q.A = Rb; q.strideA = SS; q.lda = Sp; q.B = Rb; q.strideB = SS; q.ldb = Sp;
      q.km = 3;   // R is symmetric bit for bit: read as [K][M], whose whole-cache-line loads are the faster ones
      q.M = Sp; q.N = Sp; q.K = Sp; q.batch = P.batch; q.epi = BEPI_POLYQ; q.sym = sym;
      q.C32 = lean ? nullptr : R; q.strideC32 = SS; q.ldc32 = Sp; q.Cb = Qb; q.strideCb = SS; q.ldcb = Sp; q.c1 = 0.5f;
      q.Cin16 = lean ? Rb : nullptr;
      q.ctrl = r.ctrl;
    }
    const uint16_t* Bop = P.d == 2 ? Qb : Rb;
    static const int no_square = ab_switch("PRISM_NO_FIT_SQUARE");
    if (!no_square && P.d == 2 && Tq.m == 128 && Tq.n == 128 && chain_b && r.fit_needed(k) && r.fused() &&
        fit_square_supported(r.fit_args(k, nparts, R, fit_b, fit_d, fit_sd, fit_ldd))) {
      ProfScope ps(PK_FIT_SQUARE, r.s);
      CHECK_LAUNCH(launch_fit_square(r.fit_args(k, nparts, R, fit_b, fit_d, fit_sd, fit_ldd), q, P.batch, r.s));
    } else {
      CHECK_LAUNCH(r.fit(k, nparts, R, fit_b, fit_d, fit_sd, fit_ldd));
      if (k == r.max_iters) break;
      if (P.d == 2) { ProfScope ps(PK_BF16_POLYQ, r.s); CHECK_LAUNCH(launch_gemm_bf16(q, Tq.m, Tq.n, r.s)); }
    }
    // One pass: the product reads the high half of the iterate only; the epilogue adds the low
    // half's share elementwise (see the kernel) and splits the result again.
    Bf16Desc ad[BF16_MAX_GROUPS];
    for (int i = 0; i < ng; ++i) {
      const Run::XGroup& x = r.xg[order[i]];
      const long long LS = (long long)x.Lp * Sp;
      Bf16Desc& a = ad[i];
      a = Bf16Desc{};
      a.A = x.Xhi[cur]; a.strideA = LS; a.lda = Sp; a.B = Bop + x.boff * SS; a.strideB = SS; a.ldb = Sp;
      a.km = 2;   // Q (d = 1: R) is symmetric: read as [K][N]
      a.M = x.Lp; a.N = Sp; a.K = Sp; a.batch = x.batch; a.epi = BEPI_APPLY;
      a.Cb = x.Xhi[cur ^ 1]; a.Cb2 = x.Xlo[cur ^ 1]; a.strideCb = LS; a.ldcb = Sp;
      a.Xhi = x.Xhi[cur]; a.Xlo = x.Xlo[cur]; a.coef_is_alpha = P.d == 1; a.ctrl = r.ctrl + x.boff;
    }
    { ProfScope ps(PK_BF16_APPLY, r.s); CHECK_LAUNCH(launch_gemm_bf16_multi(ad, ng, Ta.m, Ta.n, r.s)); }
    cur ^= 1;
  }
  return PRISM_OK;
}

int run_sqrt_f32(Run& r) {
  const Plan& P = r.P;
  const int Sp = P.Sp;
  const long long SS = (long long)Sp * Sp;
  float* X[2] = {r.at<float>(P.o_x[0]), r.at<float>(P.o_x[1])};
  float* Y[2] = {r.at<float>(P.o_y[0]), r.at<float>(P.o_y[1])};
  float* R = r.at<float>(P.o_r);
  float* Q = P.d == 2 ? r.at<float>(P.o_q) : nullptr;
  // X_k and Y_k commute up to kappa * eps only: every product keeps all its tiles.  (Mirroring only
  // Y X and R^2 is stable but costs the root an order of magnitude of accuracy from kappa ~ 1e4 on.)
  const int sym = 0;
  const int nparts = r.tiles(Sp, Sp, sym);
  auto residual = [&](int cur) {
    GemmDesc g = f32_desc(r, Y[cur], Sp, SS, X[cur], Sp, SS, Sp, Sp, Sp, 0);    // G = Y X
    g.sym = sym;
    g.epi = EPI_RESIDUAL; g.C = R; g.strideC = SS; g.ldc = Sp; g.rho_part = r.rho;
    return g;
  };
  auto square = [&]() {
    GemmDesc q = f32_desc(r, R, Sp, SS, R, Sp, SS, Sp, Sp, Sp, 0);
    q.sym = sym;
    q.epi = EPI_POLYQ; q.C = Q; q.strideC = SS; q.ldc = Sp; q.Cin = R; q.strideCin = SS; q.ldcin = Sp; q.c1 = 0.5f;
    return q;
  };
  const float* Pm = P.d == 2 ? Q : R;
  auto update_x = [&](int cur) {
    GemmDesc ax = f32_desc(r, X[cur], Sp, SS, Pm, Sp, SS, Sp, Sp, Sp, 0);        // X + X Q
    ax.epi = EPI_AXPY; ax.C = X[cur ^ 1]; ax.strideC = SS; ax.ldc = Sp; ax.Cin = X[cur]; ax.strideCin = SS; ax.ldcin = Sp;
    ax.coef_is_alpha = P.d == 1;
    return ax;
  };
  auto update_y = [&](int cur) {
    GemmDesc ay = f32_desc(r, Pm, Sp, SS, Y[cur], Sp, SS, Sp, Sp, Sp, 0);        // Y + Q Y
    ay.epi = EPI_AXPY; ay.C = Y[cur ^ 1]; ay.strideC = SS; ay.ldc = Sp; ay.Cin = Y[cur]; ay.strideCin = SS; ay.ldcin = Sp;
    ay.coef_is_alpha = P.d == 1;
    return ay;
  };
  if (r.flow()) {
    if (P.d == 1) {
      const FlowOp ops[] = {{residual(0), 0}, {update_x(0), -1}, {update_y(0), -1}};
      return run_flow(r, ops, 3, true, R, nparts);
    }
    const FlowOp ops[] = {{residual(0), 0}, {square(), -1}, {update_x(0), 0}, {update_y(0), 0}};
    return run_flow(r, ops, 4, true, R, nparts);
  }
  int cur = 0;
  for (int k = 0; k <= r.max_iters; ++k) {
    if (k == r.max_iters && r.tol <= 0.0) break;
    { ProfScope ps(PK_F32_RESID, r.s); CHECK_LAUNCH(r.gemm(residual(cur))); }
    CHECK_LAUNCH(r.fit(k, nparts, R));
    if (k == r.max_iters) break;
    if (P.d == 2) { ProfScope ps(PK_F32_POLYQ, r.s); CHECK_LAUNCH(r.gemm(square())); }
    { ProfScope ps(PK_F32_APPLY, r.s); CHECK_LAUNCH(r.gemm_pair(update_x(cur), update_y(cur))); }
    cur ^= 1;
  }
  return PRISM_OK;
}

// Chebyshev inverse (App. A.4): R = I - A_s X, Q = R + alpha R^2, X <- X + X Q
int run_inverse_f32(Run& r) {
  const Plan& P = r.P;
  const int Sp = P.Sp;
  const long long SS = (long long)Sp * Sp;
  float* X[2] = {r.at<float>(P.o_x[0]), r.at<float>(P.o_x[1])};
  const float* As = r.at<float>(P.o_y[0]);
  float* R = r.at<float>(P.o_r);
  float* Q = r.at<float>(P.o_q);
  const int sym = 0;   // A_s X_k is symmetric up to kappa * eps only: all tiles
  const int nparts = r.tiles(Sp, Sp, sym);
  auto residual = [&](int cur) {
    GemmDesc g = f32_desc(r, As, Sp, SS, X[cur], Sp, SS, Sp, Sp, Sp, 0);
    g.sym = sym;
    g.epi = EPI_RESIDUAL; g.C = R; g.strideC = SS; g.ldc = Sp; g.rho_part = r.rho;
    return g;
  };
  auto square = [&]() {
    GemmDesc q = f32_desc(r, R, Sp, SS, R, Sp, SS, Sp, Sp, Sp, 0);
    q.sym = sym;
    q.epi = EPI_POLYQ; q.C = Q; q.strideC = SS; q.ldc = Sp; q.Cin = R; q.strideCin = SS; q.ldcin = Sp; q.c1 = 1.0f;
    return q;
  };
  auto update = [&](int cur) {
    GemmDesc ax = f32_desc(r, X[cur], Sp, SS, Q, Sp, SS, Sp, Sp, Sp, 0);
    ax.epi = EPI_AXPY; ax.C = X[cur ^ 1]; ax.strideC = SS; ax.ldc = Sp; ax.Cin = X[cur]; ax.strideCin = SS; ax.ldcin = Sp;
    return ax;
  };
  if (r.flow()) {
    const FlowOp ops[] = {{residual(0), 0}, {square(), -1}, {update(0), 0}};
    return run_flow(r, ops, 3, true, R, nparts);
  }
  int cur = 0;
  for (int k = 0; k <= r.max_iters; ++k) {
    if (k == r.max_iters && r.tol <= 0.0) break;
    { ProfScope ps(PK_F32_RESID, r.s); CHECK_LAUNCH(r.gemm(residual(cur))); }
    CHECK_LAUNCH(r.fit(k, nparts, R));
    if (k == r.max_iters) break;
    { ProfScope ps(PK_F32_POLYQ, r.s); CHECK_LAUNCH(r.gemm(square())); }
    { ProfScope ps(PK_F32_APPLY, r.s); CHECK_LAUNCH(r.gemm(update(cur))); }
    cur ^= 1;
  }
  return PRISM_OK;
}

// DB Newton in product form (App. A.2): N = M^{-1}, X <- (1-a) X + a X N, Y likewise,
// M <- 2a(1-a) I + (1-a)^2 M + a^2 N.  The stop test of iteration k runs before the inverse.
int run_sqrt_newton_f32(Run& r) {
  const Plan& P = r.P;
  const int Sp = P.Sp;
  const long long SS = (long long)Sp * Sp;
  float* X[2] = {r.at<float>(P.o_x[0]), r.at<float>(P.o_x[1])};
  float* Y[2] = {r.at<float>(P.o_y[0]), r.at<float>(P.o_y[1])};
  float* M = r.at<float>(P.o_r);
  float* N = r.at<float>(P.o_q);
  const int nparts0 = (Sp / 64) * (Sp / 64);               // prepare step: one partial per 64 x 64 tile
  const int nparts = nparts0 < 512 ? nparts0 : 512;        // later: the M update
  const int sym = f32_sym();                               // X, Y never re-enter M: mirrored halves are safe
  int cur = 0;
  for (int k = 0; k <= r.max_iters; ++k) {
    if (k == r.max_iters && r.tol <= 0.0) break;
    CHECK_LAUNCH(r.solve(k, k == 0 ? nparts0 : nparts, 1));
    if (k == r.max_iters) break;
    { ProfScope ps(PK_SPD_INVERSE, r.s); CHECK_LAUNCH(launch_spd_inverse(M, N, Sp, P.batch, r.sel_batch, r.ctrl, r.tol > 0.0, r.at<float>(P.o_t[0]), r.at<unsigned>(P.o_sync), r.s)); }
    {   // also without a fit: the probe of the inverse shares the partials with the moments
      ProfScope ps(PK_DB_MOMENTS, r.s);
      launch_db_moments(M, N, Sp, P.S, P.batch, r.ctrl, r.at<double>(P.o_cpart), P.ngroups, r.s);
      launch_db_probe(M, N, Sp, P.S, P.batch, r.ctrl, r.v, r.at<double>(P.o_cpart), P.ngroups, r.s);
    }
    CHECK_LAUNCH(r.solve(k, 0, 2));
    GemmDesc ax = f32_desc(r, X[cur], Sp, SS, N, Sp, SS, Sp, Sp, Sp, 0);
    ax.epi = EPI_AXPY; ax.C = X[cur ^ 1]; ax.strideC = SS; ax.ldc = Sp; ax.Cin = X[cur]; ax.strideCin = SS; ax.ldcin = Sp;
    ax.cin_one_minus_alpha = 1; ax.coef_is_alpha = 1; ax.sym = sym;
    GemmDesc ay = f32_desc(r, Y[cur], Sp, SS, N, Sp, SS, Sp, Sp, Sp, 0);
    ay.epi = EPI_AXPY; ay.C = Y[cur ^ 1]; ay.strideC = SS; ay.ldc = Sp; ay.Cin = Y[cur]; ay.strideCin = SS; ay.ldcin = Sp;
    ay.cin_one_minus_alpha = 1; ay.coef_is_alpha = 1; ay.sym = sym;
    { ProfScope ps(PK_F32_APPLY, r.s); CHECK_LAUNCH(launch_gemm_f32_pair(ax, ay, r.s)); }
    { ProfScope ps(PK_DB_UPDATE_M, r.s); launch_db_update_m(M, N, Sp, P.S, P.batch, r.ctrl, r.rho, nparts, r.s); }
    CHECK_LAUNCH(check_hip());
    cur ^= 1;
  }
  return PRISM_OK;
}

int run_inv_root_f32(Run& r) {
  const Plan& P = r.P;
  const int Sp = P.Sp, p = P.p;
  const long long SS = (long long)Sp * Sp;
  float* X[2] = {r.at<float>(P.o_x[0]), r.at<float>(P.o_x[1])};
  double* M[2] = {r.at<double>(P.o_y[0]), r.at<double>(P.o_y[1])};
  float* R = r.at<float>(P.o_r);
  float* Tm[3] = {r.at<float>(P.o_t[0]), r.at<float>(P.o_t[1]), r.at<float>(P.o_t[2])};
  const int nparts0 = (Sp / 64) * (Sp / 64);  // residual of M_0 comes from the prepare step (64 x 64 tiles)
  const int nparts = (Sp / 64) * (Sp / 64);   // later ones from the fp64 product (64 x 64 tiles)
  auto update = [&](int cur) {
    GemmDesc ax = f32_desc(r, X[cur], Sp, SS, R, Sp, SS, Sp, Sp, Sp, 0);         // X (I + alpha R)
    ax.epi = EPI_AXPY; ax.C = X[cur ^ 1]; ax.strideC = SS; ax.ldc = Sp; ax.Cin = X[cur]; ax.strideCin = SS; ax.ldcin = Sp;
    ax.coef_is_alpha = 1; ax.sym = f32_sym();   // X never re-enters M; the power chain below keeps all tiles
    return ax;
  };
  // (I + alpha R)^q = I + E_q, built on the part beyond the identity so that fp32 rounding acts
  // on the small quantity only: E_1 = alpha R, squaring E <- 2E + E E, times T: E <- E + E_1 + E E_1.
  // E_1 itself is never stored: wherever it is an operand R stands in and the epilogue supplies
  // the powers of alpha.
  auto square = [&](const float* E /* null: E_1 */, float* dst) {
    const float* Eop = E ? E : R;
    GemmDesc sq = f32_desc(r, Eop, Sp, SS, Eop, Sp, SS, Sp, Sp, Sp, 0);
    sq.epi = EPI_AXPY; sq.C = dst; sq.strideC = SS; sq.ldc = Sp; sq.Cin = Eop; sq.strideCin = SS; sq.ldcin = Sp; sq.c_in = 2.0f;
    if (!E) { sq.cin_alpha_pow = 1; sq.coef_is_alpha = 2; }
    return sq;
  };
  auto times_t = [&](const float* U, float* dst) {                             // U + alpha R + alpha U R
    GemmDesc mu = f32_desc(r, U, Sp, SS, R, Sp, SS, Sp, Sp, Sp, 0);
    mu.epi = EPI_AXPY; mu.C = dst; mu.strideC = SS; mu.ldc = Sp; mu.Cin = U; mu.strideCin = SS; mu.ldcin = Sp; mu.c_in = 1.0f;
    mu.Cin2 = R; mu.cin2_alpha_pow = 1; mu.coef_is_alpha = 1;
    return mu;
  };
  auto m_times = [&](const float* E, const double* Min, double* Mout, float* Rout) {   // Mout = Min + E Min in fp64
    GemmDesc mn = {};
    mn.A = E; mn.strideA = SS; mn.lda = Sp; mn.B = Min; mn.strideB = SS; mn.ldb = Sp;
    mn.M = Sp; mn.N = Sp; mn.K = Sp; mn.batch = P.batch; mn.n_true = P.S; mn.ctrl = r.ctrl;
    mn.epi = EPI_MNEXT; mn.C = Mout; mn.strideC = SS; mn.ldc = Sp;
    mn.Cin = Min; mn.strideCin = SS; mn.ldcin = Sp;
    mn.R32out = Rout; mn.strideR = SS; mn.ldr = Sp; mn.rho_part = r.rho;
    if (const Run::Planes* q = r.planes_of(Rout)) { mn.C3 = q->p; mn.psC = q->ps; }
    return mn;
  };
  if (r.flow()) {   // p = 2 .. 4
    FlowOp ops[FLOW_MAX_OPS];
    int n = 0;
    const float* E = Tm[1];
    auto put = [&](const GemmDesc& d, int phase) { ops[n].d = d; ops[n++].phase = phase; };
    put(update(0), -1);
    put(square(nullptr, Tm[1]), -1);
    if (p == 3) { put(times_t(Tm[1], Tm[2]), 0); E = Tm[2]; }
    if (p == 4) { put(square(Tm[1], Tm[2]), 0); E = Tm[2]; }
    put(m_times(E, M[0], M[1], R), 1);
    return run_flow(r, ops, n, false, R, nparts);
  }
  int cur = 0, mc = 0;   // current X and M buffers
  for (int k = 0; k <= r.max_iters; ++k) {
    if (k == r.max_iters && r.tol <= 0.0) break;
    CHECK_LAUNCH(r.fit(k, k == 0 ? nparts0 : nparts, R));
    if (k == r.max_iters) break;
    // The update of X and the first square of the chain below depend on R alone.  Where neither fills the chip they share a
    // launch.
    const bool paired = p >= 2 && 2ll * (Sp / 64) * (Sp / 64) * r.sel_batch <= 1024;
    if (!paired) {
      ProfScope ps(PK_F32_APPLY, r.s);
      CHECK_LAUNCH(r.gemm(update(cur)));
    }
    auto run_square = [&](const float* E, float* dst) -> int {
      ProfScope ps(PK_F32_STORE, r.s);
      return !E && paired ? r.gemm_pair(update(cur), square(E, dst)) : r.gemm(square(E, dst));
    };
    auto run_m_times = [&](const float* E, const double* Min, double* Mout, float* Rout) -> int {
      ProfScope ps(PK_F64_MNEXT, r.s);
      return launch_gemm_f64a(m_times(E, Min, Mout, Rout), 64, 64, r.s);
    };
    if (p <= 4) {
      const float* U = nullptr;   // null: E = E_1 = alpha R
      int hb = 0;
      while ((p >> (hb + 1)) != 0) ++hb;
      for (int bit = hb - 1; bit >= 0; --bit) {
        float* dst = (U == Tm[1]) ? Tm[2] : Tm[1];
        CHECK_LAUNCH(run_square(U, dst));
        U = dst;
        if ((p >> bit) & 1) {
          float* dst2 = (U == Tm[1]) ? Tm[2] : Tm[1];
          { ProfScope ps(PK_F32_STORE, r.s); CHECK_LAUNCH(r.gemm(times_t(U, dst2))); }
          U = dst2;
        }
      }
      if (!U) {   // p = 1: E_p = alpha R.  The product below overwrites R, so it cannot read R as an operand
        { ProfScope ps(PK_MAKE_T, r.s); launch_make_e(Tm[0], R, r.ctrl, P.batch, Sp, r.s); }
        CHECK_LAUNCH(check_hip());
        U = Tm[0];
      }
      CHECK_LAUNCH(run_m_times(U, M[mc], M[mc ^ 1], R));                               // M' = M + E_p M in fp64
      mc ^= 1;
    } else {
      // p = 5 .. 8: (I + alpha R)^p as p / 2 factors (I + E_2), and (I + E_1) for odd p, applied to M
      // one after the other in fp64.  Every squaring in fp32 doubles the rounding error of its operand
      // times (1 + E), and M must stay consistent with X^p A: with one fp32 chain up to E_8 the root of
      // a 1024 x 1024 matrix came out with a relative error of 2e-5, with two factors (I + E_4) 1.6e-5,
      // with factors of order <= 2 6e-6 (p = 8; 4e-6, 2e-6, 1e-6 for p = 7, 6, 5).
      float* E2 = Tm[1];
      CHECK_LAUNCH(run_square(nullptr, E2));
      int left = p / 2 + (p & 1);
      if (p & 1) {
        { ProfScope ps(PK_MAKE_T, r.s); launch_make_e(Tm[0], R, r.ctrl, P.batch, Sp, r.s); }
        CHECK_LAUNCH(check_hip());
        --left;
        CHECK_LAUNCH(run_m_times(Tm[0], M[mc], M[mc ^ 1], Tm[2]));   // the residual of an intermediate product goes to a spare array
        mc ^= 1;
      }
      for (; left > 0; --left) {
        CHECK_LAUNCH(run_m_times(E2, M[mc], M[mc ^ 1], left == 1 ? R : Tm[2]));
        mc ^= 1;
      }
    }
    cur ^= 1;
  }
  return PRISM_OK;
}

// bf16 polar, plain iterate, shapes that need no padding, array aligned like the workspace buffers:
// the caller's array takes the place of buffer 1 of its own orientation
void alias_output(const Plan& P, Run::XGroup& x) {
  static const int no_alias = ab_switch("PRISM_BF16_NO_OUTPUT_ALIAS");
  const int S = x.m < x.n ? x.m : x.n;
  x.aliased = false;
  if (P.split || x.transpose || P.Sp != S || x.Lp != x.L || no_alias || ((uintptr_t)x.x & 255)) return;
  x.Xhi[1] = (uint16_t*)x.x;
  x.aliased = true;
}
// iterate buffers of one shape group in the arguments of the pre-scaling and copy-out kernels
void bf16_prep_final(const Plan& P, const Run::XGroup& x, PrepArgs& pa, FinalArgs& fa) {
  pa.Xa_hi = x.Xhi[0]; pa.Xa_lo = x.Xlo[0];
  for (int i = 0; i < 2; ++i) { fa.Xa_hi[i] = x.Xhi[i]; fa.Xa_lo[i] = x.Xlo[i]; }
  (void)P;
}

// The arguments of a call on one array, but for those that make_plan looks at
int check_arguments(int fn, const void* a, const void* inv_out, int batch, int m, int n, int max_iters, double tol, const prism_options* opt) {
  if (batch < 0 || m < 0 || n < 0) return PRISM_EINVAL;
  const bool empty = batch == 0 || m == 0 || n == 0;
  if (!empty && !a) return PRISM_EINVAL;
  if (!empty && (fn == PRISM_FN_SQRT || fn == PRISM_FN_SQRT_NEWTON) && !inv_out) return PRISM_EINVAL;
  if (max_iters < 0 || max_iters > PRISM_MAX_ITERS) return PRISM_EINVAL;
  if (!(tol == tol)) return PRISM_EINVAL;
  if (opt && opt->warm_iters < 0) return PRISM_EINVAL;
  if (opt && (opt->schedule_len < 0 || opt->schedule_len > PRISM_MAX_ITERS || (opt->schedule_len > 0 && !opt->alpha_schedule)))
    return PRISM_EINVAL;
  return PRISM_OK;
}

int run(int fn, void* a, void* inv_out, int root_p, int batch, int m, int n, int dt, int degree, int max_iters,
        int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt, int sel_batch = 0, const void* owner = nullptr) {
  set_last_error("");
  const bool empty = batch == 0 || m == 0 || n == 0;   // nothing to compute; the arguments are still checked
  int rc = check_arguments(fn, a, inv_out, batch, m, n, max_iters, tol, opt);
  if (rc != PRISM_OK) return rc;
  Run r;
  if (empty) return make_plan(r.P, fn, 1, m ? m : 1, n ? n : 1, dt, degree, sketch_dim, root_p, opt ? opt->flags : 0u);
  if (sel_batch == 0) sel_batch = batch;
  rc = make_plan(r.P, fn, batch, m, n, dt, degree, sketch_dim, root_p, opt ? opt->flags : 0u, false, sel_batch);
  if (rc != PRISM_OK) return rc;
  const unsigned plain = FLAG_NO_SPLIT_K | FLAG_NO_FLOW | FLAG_NO_PLANES;
  if ((r.P.ksplit || r.P.ring || r.P.x3) && opt && opt->workspace && opt->workspace_bytes < r.P.total) {
    rc = make_plan(r.P, fn, batch, m, n, dt, degree, sketch_dim, root_p, opt->flags | plain, false, sel_batch);
    if (rc != PRISM_OK) return rc;
  }
  r.s = (hipStream_t)stream;
  rc = get_workspace(r.P.total, owner ? owner : stream, opt, &r.ws, r.P.x3);
  if (rc == PRISM_ENOMEM && r.P.x3) {   // the planes are what did not fit
    rc = make_plan(r.P, fn, batch, m, n, dt, degree, sketch_dim, root_p, (opt ? opt->flags : 0u) | plain, false, sel_batch);
    if (rc != PRISM_OK) return rc;
    rc = get_workspace(r.P.total, owner ? owner : stream, opt, &r.ws);
  }
  if (rc != PRISM_OK) return rc;
  r.list_planes();
  const Plan& P = r.P;
  r.ctrl = r.at<Ctrl>(P.o_ctrl);
  r.info = (opt && opt->info) ? opt->info : r.at<prism_info>(P.o_info);
  r.rho = r.at<float>(P.o_rho);
  r.v0 = r.at<float>(P.o_v0);
  r.v = r.at<float>(P.o_v);
  if (P.has_planes) { r.vp0 = r.at<uint16_t>(P.o_vp0); r.vp = r.at<uint16_t>(P.o_vp); }
  r.max_iters = max_iters; r.tol = tol; r.seed = seed; r.warm = opt ? opt->warm_iters : 0;
  if (opt && (opt->flags & PRISM_FLAG_FIT_NO_WAIT)) r.fit_polls = 0;
  r.sched = opt ? opt->alpha_schedule : nullptr;
  r.sched_len = opt ? opt->schedule_len : 0;
  if (fn == PRISM_FN_SQRT_NEWTON) r.warm = 0;   // no upper end to start from: the coefficient is not clamped to a fit interval
  r.first_fit = r.warm > r.sched_len ? r.warm : r.sched_len;
  r.sel_batch = sel_batch;

  PrepArgs pa = {};
  pa.fn = fn; pa.dt = dt; pa.batch = batch; pa.m = m; pa.n = n; pa.S = P.S; pa.L = P.L; pa.Sp = P.Sp; pa.Lp = P.Lp;
  pa.transpose = P.transpose; pa.root_p = root_p; pa.src = a;
  pa.sumsq_part = r.at<double>(P.o_sumsq); pa.nsum = P.nsum; pa.ctrl = r.ctrl; pa.info = r.info;
  pa.sync = r.at<unsigned>(P.o_sync);
  pa.rho_part = r.rho; pa.tile = P.tile;
  FinalArgs fa = {};
  fa.fn = fn; fa.dt = dt; fa.batch = batch; fa.m = m; fa.n = n; fa.S = P.S; fa.L = P.L; fa.Sp = P.Sp; fa.Lp = P.Lp;
  fa.transpose = P.transpose; fa.dst = a; fa.dst2 = inv_out; fa.ctrl = r.ctrl;
  if (dt == PRISM_BF16) {
    Run::XGroup x = {};
    x.batch = batch; x.boff = 0; x.m = m; x.n = n; x.L = P.L; x.Lp = P.Lp; x.transpose = P.transpose; x.x = a;
    for (int i = 0; i < 2; ++i) {
      x.Xhi[i] = r.at<uint16_t>(P.o_xhi[i]);
      x.Xlo[i] = P.split ? r.at<uint16_t>(P.o_xlo[i]) : nullptr;
    }
    x.ksplit = P.ksplit; x.gpart = r.at<float>(P.o_gpart);
    alias_output(P, x);
    r.xg.push_back(x);
    bf16_prep_final(P, x, pa, fa);
  } else {
    pa.X32 = r.at<float>(P.o_x[0]);
    if (fn == PRISM_FN_SQRT || fn == PRISM_FN_INVERSE || fn == PRISM_FN_SQRT_NEWTON) pa.Y32 = r.at<float>(P.o_y[0]);
    if (fn == PRISM_FN_SQRT_NEWTON) pa.R32 = r.at<float>(P.o_r);
    if (fn == PRISM_FN_INV_ROOT) { pa.M64 = r.at<double>(P.o_y[0]); pa.R32 = r.at<float>(P.o_r); }
    for (int i = 0; i < 2; ++i) {
      fa.X32[i] = r.at<float>(P.o_x[i]);
      fa.Y32[i] = (fn == PRISM_FN_SQRT || fn == PRISM_FN_SQRT_NEWTON) ? r.at<float>(P.o_y[i]) : nullptr;
    }
    fa.ring = r.flow() ? P.ring : 0; fa.ring_bytes = P.ring_bytes;
  }
  const bool small = r.small_polar() || r.small_root();
  if (!small) { ProfScope ps(PK_PREP, r.s); launch_sumsq(pa, r.s); launch_prepare(pa, r.s); r.split_start(); }
  if (P.p_s > 0 && max_iters > r.first_fit && fn != PRISM_FN_SQRT_NEWTON) {
    ProfScope ps(PK_SKETCH, r.s);
    launch_sketch(r.v0, P.Sp, P.S, P.ld, P.p_s, seed, r.first_fit, max_iters - r.first_fit, P.fn, r.s, r.fused() || small);
    if (r.planes()) CHECK_LAUNCH(launch_split_planes(r.v0, r.vp0, P.Sp, P.ld, max_iters - r.first_fit, r.s));
  }
  rc = check_hip();
  if (rc != PRISM_OK) return rc;
  if (small) return run_small(r, (float*)a);
  if (dt == PRISM_BF16) rc = run_polar_bf16(r);
  else if (fn == PRISM_FN_POLAR || fn == PRISM_FN_SIGN) rc = run_polar_f32(r);
  else if (fn == PRISM_FN_INVERSE) rc = run_inverse_f32(r);
  else if (fn == PRISM_FN_SQRT_NEWTON) rc = run_sqrt_newton_f32(r);
  else if (fn == PRISM_FN_SQRT) rc = run_sqrt_f32(r);
  else rc = run_inv_root_f32(r);
  if (rc != PRISM_OK) return rc;
  { ProfScope ps(PK_FINAL, r.s); launch_finalize(fa, r.s); }
  return check_hip();
}

// bf16 polar factors of several shape groups that share the short side (the weight gradients of a
// layer stack: 768 x 768, 768 x 3072, 3072 x 768, 768 x 2304): one launch sequence for all of them
// on the caller's stream.  R, Q, the chain vectors and the control blocks of all matrices form one
// batch, so R^2, the chain products, the moments and the solve are single launches over every
// matrix of the call; the Gram product and the update take one descriptor per group in one launch
// each (the kernel maps its workgroup index to group, matrix and tile).  Every matrix goes through
// the kernels its own single-group call would pick.  Returns PRISM_EUNSUPPORTED (nothing enqueued)
// when the groups do not fit this form; the caller then takes the per-group path.
int run_polar_bf16_shapes(const prism_group* groups, int ngroups, int degree, int max_iters, int sketch_dim, uint64_t seed,
                          double tol, void* stream, const prism_options* opt, int batch_scale = 1, const void* const* const* from = nullptr,
                          const void* owner = nullptr) {
  static const int off = ab_switch("PRISM_NO_SHARED_SHAPES");
  if (off || ngroups < 2 || ngroups > BF16_MAX_GROUPS) return PRISM_EUNSUPPORTED;
  if (max_iters < 0 || max_iters > PRISM_MAX_ITERS || !(tol == tol)) return PRISM_EINVAL;
  if (opt && (opt->warm_iters < 0 || opt->schedule_len < 0 || opt->schedule_len > PRISM_MAX_ITERS ||
              (opt->schedule_len > 0 && !opt->alpha_schedule)))
    return PRISM_EINVAL;
  const unsigned flags = opt ? opt->flags : 0u;
  Plan Pg[BF16_MAX_GROUPS];
  long long btot = 0;
  for (int g = 0; g < ngroups; ++g) {
    if (groups[g].batch <= 0 || groups[g].m <= 0 || groups[g].n <= 0 || !groups[g].x) return PRISM_EUNSUPPORTED;   // empty or invalid: per-group path
    const int rc = make_plan(Pg[g], PRISM_FN_POLAR, groups[g].batch, groups[g].m, groups[g].n, PRISM_BF16, degree, sketch_dim, 0, flags, false,
                             groups[g].batch * batch_scale);
    if (rc != PRISM_OK) return rc;
    if (Pg[g].S != Pg[0].S || Pg[g].Sp != Pg[0].Sp || Pg[g].tile != Pg[0].tile) return PRISM_EUNSUPPORTED;
    // every group must get the chain kernels of its own call (batch_scale: the groups passed in are
    // 1 / batch_scale of the caller's groups each)
    const int bg = groups[g].batch * batch_scale, b0 = groups[0].batch * batch_scale;
    if (chain_takes_small_kernel(Pg[g].Sp, Pg[g].ld, bg, true) != chain_takes_small_kernel(Pg[0].Sp, Pg[0].ld, b0, true) ||
        chain_takes_small_kernel(Pg[g].Sp, Pg[g].ld, bg, false) != chain_takes_small_kernel(Pg[0].Sp, Pg[0].ld, b0, false) ||
        fit_fused_supported(Pg[g].Sp, Pg[g].ld, bg, true, in_halves(bg, Pg[g].S)) != fit_fused_supported(Pg[0].Sp, Pg[0].ld, b0, true, in_halves(b0, Pg[0].S)) ||
        chain_bf16_supported(Pg[g].Sp, Pg[g].ld, bg, Pg[g].Sp) != chain_bf16_supported(Pg[0].Sp, Pg[0].ld, b0, Pg[0].Sp))
      return PRISM_EUNSUPPORTED;
    btot += groups[g].batch;
  }
  if (btot > PRISM_MAX_BATCH) return PRISM_EUNSUPPORTED;
  Sources sources = {};
  if (from) {   // (the caller has looked at their number and alignment)
    if (btot > MAX_SOURCES) return PRISM_EUNSUPPORTED;
    int at = 0;
    for (int g = 0; g < ngroups; ++g) {
      if ((uintptr_t)groups[g].x & 15) return PRISM_EUNSUPPORTED;
      sources.first[g] = at;
      for (int b = 0; b < groups[g].batch; ++b) sources.p[at++] = from[g][b];
    }
  }
  // Beside split Gram products the few other ones go with them, as products of one part (same R): two launches instead of
  // three.  One layer (four shapes), three updates without a fit, us: width 256 170 -> 142 (no split: 143), 512 200 -> 166 (193),
  // 768 286 -> 250 (284), 1280 622 -> 579 (583).
  bool any_split = false;
  for (int g = 0; g < ngroups; ++g) any_split = any_split || Pg[g].ksplit;
  for (int g = 0; g < ngroups && any_split; ++g) {
    const long long nt = (Pg[g].Sp + 127) / 128;
    if (!Pg[g].ksplit && nt * (nt + 1) / 2 * groups[g].batch <= 64) Pg[g].ksplit = 1;
  }
  Run r;
  int rc = make_plan(r.P, PRISM_FN_POLAR, (int)btot, Pg[0].S, Pg[0].S, PRISM_BF16, degree, sketch_dim, 0, flags, true);
  if (rc != PRISM_OK) return rc;
  Plan& P = r.P;
  // iterate buffers per group behind the shared part
  size_t off_bytes = P.total;
  auto take = [&](size_t bytes) { size_t o = off_bytes; off_bytes = align256(off_bytes + bytes); return o; };
  size_t o_xhi[BF16_MAX_GROUPS][2], o_xlo[BF16_MAX_GROUPS][2], o_gpart[BF16_MAX_GROUPS], o_sumsq[BF16_MAX_GROUPS];
  for (int g = 0; g < ngroups; ++g) {
    const size_t bytes = (size_t)groups[g].batch * Pg[g].Lp * Pg[g].Sp * 2;
    for (int i = 0; i < 2; ++i) {
      o_xhi[g][i] = take(bytes);
      o_xlo[g][i] = P.split ? take(bytes) : 0;
    }
    o_sumsq[g] = take((size_t)groups[g].batch * Pg[g].nsum * sizeof(double));
    o_gpart[g] = Pg[g].ksplit ? take((size_t)groups[g].batch * Pg[g].ksplit * P.Sp * P.Sp * 4) : 0;
  }
  P.total = off_bytes;
  r.s = (hipStream_t)stream;
  rc = get_workspace(P.total, owner ? owner : stream, nullptr, &r.ws);
  if (rc != PRISM_OK) return rc;
  r.ctrl = r.at<Ctrl>(P.o_ctrl);
  r.info = r.at<prism_info>(P.o_info);
  r.rho = r.at<float>(P.o_rho);
  r.v0 = r.at<float>(P.o_v0);
  r.v = r.at<float>(P.o_v);
  if (P.has_planes) { r.vp0 = r.at<uint16_t>(P.o_vp0); r.vp = r.at<uint16_t>(P.o_vp); }
  r.max_iters = max_iters; r.tol = tol; r.seed = seed; r.warm = opt ? opt->warm_iters : 0;
  if (opt && (opt->flags & PRISM_FLAG_FIT_NO_WAIT)) r.fit_polls = 0;
  r.sched = opt ? opt->alpha_schedule : nullptr;
  r.sched_len = opt ? opt->schedule_len : 0;
  r.first_fit = r.warm > r.sched_len ? r.warm : r.sched_len;
  r.sel_batch = groups[0].batch * batch_scale;
  int boff = 0;
  for (int g = 0; g < ngroups; ++g) {
    Run::XGroup x = {};
    x.batch = groups[g].batch; x.boff = boff; x.m = groups[g].m; x.n = groups[g].n;
    x.L = Pg[g].L; x.Lp = Pg[g].Lp; x.transpose = Pg[g].transpose; x.x = groups[g].x;
    for (int i = 0; i < 2; ++i) {
      x.Xhi[i] = r.at<uint16_t>(o_xhi[g][i]);
      x.Xlo[i] = P.split ? r.at<uint16_t>(o_xlo[g][i]) : nullptr;
    }
    x.ksplit = Pg[g].ksplit; x.gpart = r.at<float>(o_gpart[g]);
    x.sumsq = r.at<double>(o_sumsq[g]); x.nsum = Pg[g].nsum;
    alias_output(P, x);
    r.xg.push_back(x);
    boff += x.batch;
  }
  auto group_args = [&](const Run::XGroup& x, PrepArgs& pa, FinalArgs& fa) {
    pa = PrepArgs{}; fa = FinalArgs{};
    pa.fn = PRISM_FN_POLAR; pa.dt = PRISM_BF16; pa.batch = x.batch; pa.m = x.m; pa.n = x.n;
    pa.S = P.S; pa.L = x.L; pa.Sp = P.Sp; pa.Lp = x.Lp; pa.transpose = x.transpose; pa.root_p = 0; pa.src = x.x;
    pa.sumsq_part = x.sumsq; pa.nsum = x.nsum;
    pa.ctrl = r.ctrl + x.boff; pa.info = r.info + x.boff; pa.rho_part = r.rho; pa.tile = P.tile;
    pa.sync = r.at<unsigned>(P.o_sync) + (long long)x.boff * FIT_SYNC_WORDS;
    fa.fn = PRISM_FN_POLAR; fa.dt = PRISM_BF16; fa.batch = x.batch; fa.m = x.m; fa.n = x.n;
    fa.S = P.S; fa.L = x.L; fa.Sp = P.Sp; fa.Lp = x.Lp; fa.transpose = x.transpose; fa.dst = x.x; fa.dst2 = nullptr;
    fa.ctrl = r.ctrl + x.boff;
    bf16_prep_final(P, x, pa, fa);
  };
  PrepArgs pa; FinalArgs fa;
  {
    ProfScope ps(PK_PREP, r.s);
    PrepArgs pas[BF16_MAX_GROUPS];
    int np = 0;
    for (const Run::XGroup& x : r.xg) { group_args(x, pa, fa); pas[np++] = pa; }
    if (!launch_prep_multi(pas, np, from ? &sources : nullptr, r.s)) {
      if (from) return PRISM_EUNSUPPORTED;
      for (int i = 0; i < np; ++i) { launch_sumsq(pas[i], r.s); launch_prepare(pas[i], r.s); }
    }
  }
  if (P.p_s > 0 && max_iters > r.first_fit) {
    ProfScope ps(PK_SKETCH, r.s);
    launch_sketch(r.v0, P.Sp, P.S, P.ld, P.p_s, seed, r.first_fit, max_iters - r.first_fit, P.fn, r.s, r.fused());
    if (r.planes()) CHECK_LAUNCH(launch_split_planes(r.v0, r.vp0, P.Sp, P.ld, max_iters - r.first_fit, r.s));
  }
  rc = check_hip();
  if (rc != PRISM_OK) return rc;
  rc = run_polar_bf16(r);
  if (rc != PRISM_OK) return rc;
  {
    ProfScope ps(PK_FINAL, r.s);
    FinalArgs fas[BF16_MAX_GROUPS];
    int nf = 0;
    for (const Run::XGroup& x : r.xg) { group_args(x, pa, fa); fas[nf++] = fa; }
    if (!launch_finalize_multi(fas, nf, from ? &sources : nullptr, r.s))
      for (int i = 0; i < nf; ++i) launch_finalize(fas[i], r.s);
  }
  rc = check_hip();
  if (rc != PRISM_OK) return rc;
  // the reports were written into one array over all matrices: hand each group its part
  InfoScatter sc = {};
  sc.src = r.info; sc.ngroups = ngroups;
  bool wanted = false;
  boff = 0;
  for (int g = 0; g < ngroups; ++g) {
    sc.dst[g] = groups[g].info; sc.first[g] = (int)boff;
    wanted = wanted || groups[g].info;
    boff += groups[g].batch;
  }
  sc.first[ngroups] = (int)boff;
  if (wanted) launch_scatter_info(sc, r.s);
  return check_hip();
}

// Streams of the grouped call: the caller's and three of the library's own, per device, created on first use (default
// priority).  A process has four hardware queues by default; with four streams of its own beside the caller's, which then only
// waits, two of them shared a queue and ran one after the other.
// The part on the caller's stream has a workspace of its own too (its owner is the Fork), so that a call from another stream allocates
// nothing; such parts are ordered after one another by an event, as the others are by their streams.
constexpr int GROUP_STREAMS = 4;
struct Fork {
  hipStream_t streams[GROUP_STREAMS - 1] = {};
  hipEvent_t forked = nullptr, joined[GROUP_STREAMS - 1] = {};
  hipEvent_t own_part = nullptr;   // end of the latest eager part on a caller's stream
  bool own_recorded = false;
  bool ready = false;

  // Before and after the part on the caller's stream.  A call under capture leaves the event alone: what it waits for would lie
  // outside the graph (graphs share the workspaces and are the caller's to order).
  static bool capturing(hipStream_t user) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(user, &status) != hipSuccess) (void)hipGetLastError();
    return status != hipStreamCaptureStatusNone;
  }
  bool begin_own(hipStream_t user) { return !own_recorded || capturing(user) || hipStreamWaitEvent(user, own_part, 0) == hipSuccess; }
  bool end_own(hipStream_t user) {
    if (capturing(user)) return true;
    own_recorded = hipEventRecord(own_part, user) == hipSuccess;
    return own_recorded;
  }
};
std::mutex g_fork_mu;
std::map<int, Fork> g_forks;

int get_fork(Fork** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { set_last_error("hipGetDevice failed"); return PRISM_EHIP; }
  std::lock_guard<std::mutex> lock(g_fork_mu);
  Fork& f = g_forks[dev];
  if (!f.ready) {
    if (hipEventCreateWithFlags(&f.forked, hipEventDisableTiming) != hipSuccess) return PRISM_EHIP;
    if (hipEventCreateWithFlags(&f.own_part, hipEventDisableTiming) != hipSuccess) return PRISM_EHIP;
    for (int i = 0; i < GROUP_STREAMS - 1; ++i) {
      if (hipStreamCreateWithFlags(&f.streams[i], hipStreamNonBlocking) != hipSuccess) return PRISM_EHIP;
      if (hipEventCreateWithFlags(&f.joined[i], hipEventDisableTiming) != hipSuccess) return PRISM_EHIP;
    }
    f.ready = true;
  }
  *out = &f;
  return PRISM_OK;
}

int run_grouped(int fn, const prism_group* groups, int ngroups, int root_p, int dt, int degree, int max_iters,
                int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt, bool from_auto_split = false,
                const void* const* const* from = nullptr) {
  set_last_error("");
  if (ngroups == 0) return PRISM_OK;
  if (!groups || ngroups < 0) return PRISM_EINVAL;
  for (int g = 0; from && g < ngroups; ++g) {
    if (groups[g].batch > 0 && !from[g]) return PRISM_EINVAL;
    for (int b = 0; b < groups[g].batch; ++b)
      if (!from[g][b] && groups[g].m > 0 && groups[g].n > 0) return PRISM_EINVAL;
  }
  // matrices with addresses of their own, for a path that takes them one behind the other only.  A call that will be refused,
  // for whichever group, copies nothing.
  auto gather = [&]() -> int {
    if (!from) return PRISM_OK;
    for (int g = 0; g < ngroups; ++g) {
      const prism_group& q = groups[g];
      const bool empty = q.batch == 0 || q.m == 0 || q.n == 0;
      Plan P;
      CHECK_LAUNCH(check_arguments(fn, q.x, q.inv_out, q.batch, q.m, q.n, max_iters, tol, opt));
      CHECK_LAUNCH(make_plan(P, fn, empty ? 1 : q.batch, q.m ? q.m : 1, q.n ? q.n : 1, dt, degree, sketch_dim, root_p, opt ? opt->flags : 0u));
    }
    for (int g = 0; g < ngroups; ++g) {
      const prism_group& q = groups[g];
      if (q.batch > 0 && q.m > 0 && q.n > 0)
        launch_gather(q.x, from[g], q.batch, (size_t)q.m * q.n * (dt == PRISM_BF16 ? 2 : 4), (hipStream_t)stream);
    }
    from = nullptr;
    return check_hip();
  };
  if (opt && (opt->workspace || opt->info)) return PRISM_EINVAL;
  if (fn == PRISM_FN_INVERSE) degree = 5;                     // fixed polynomial
  if (fn == PRISM_FN_SQRT_NEWTON) { degree = 3; sketch_dim = sketch_dim ? 1 : 0; seed = 0; }
  static std::mutex enqueue_mu;      // the internal streams and events are shared by all callers on a device
  std::lock_guard<std::mutex> enqueue_lock(enqueue_mu);
  if (ngroups == 1) {
    prism_options o = opt ? *opt : prism_options{};
    o.info = groups[0].info;
    CHECK_LAUNCH(gather());
    return run(fn, groups[0].x, groups[0].inv_out, root_p, groups[0].batch, groups[0].m, groups[0].n, dt, degree,
               max_iters, sketch_dim, seed, tol, stream, &o);
  }
  int rc;
  Fork* f = nullptr;
  hipStream_t user = (hipStream_t)stream;
  const bool single_stream = opt && (opt->flags & PRISM_FLAG_SINGLE_STREAM);
  if (fn == PRISM_FN_POLAR && dt == PRISM_BF16 && !from_auto_split) {
    // Groups that share the short side run as one launch sequence over all their matrices.  With
    // many matrices the sequence is issued for four quarters (or two halves) of every group on
    // streams of their own: the latency-bound steps of one part (chain, moments, solve, prologues and
    // epilogues of short products) then run beside the products of another.  Measured on the
    // Muon-shaped batch of 64 (replayed from a HIP graph / eager): one sequence 4.00 / 3.93 ms, two
    // halves 3.80 / 3.82, four quarters 3.39 / 4.07, one call per group on four streams 3.40 / 4.09.
    static const int no_halves = ab_switch("PRISM_SHARED_SHAPES_NO_HALVES");
    static const int parts_sw = ab_switch("PRISM_SHARED_SHAPES_PARTS");
    long long btot = 0;
    int common = 4;   // parts every group's batch divides into: 4, else 2, else 1
    for (int gi = 0; gi < ngroups; ++gi) {
      btot += groups[gi].batch;
      while (common > 1 && (groups[gi].batch <= 0 || groups[gi].batch % common)) common >>= 1;
    }
    const int NP = (parts_sw == 2 || parts_sw == 4) ? (common >= parts_sw ? parts_sw : common) : common;
    const bool even = ngroups <= BF16_MAX_GROUPS && NP >= 2 && !single_stream;
    // sources that the launches over several groups read where they are: aligned to vectors, with a place in their arguments
    bool direct = btot / (even && btot >= 32 && !no_halves ? NP : 1) <= MAX_SOURCES;
    for (int gi = 0; from && direct && gi < ngroups; ++gi) {
      direct = groups[gi].n % 8 == 0;
      for (int b = 0; b < groups[gi].batch; ++b) direct = direct && ((uintptr_t)from[gi][b] & 15) == 0;
    }
    if (!direct) CHECK_LAUNCH(gather());
    if (!even || btot < 32 || no_halves) {
      rc = run_polar_bf16_shapes(groups, ngroups, degree, max_iters, sketch_dim, seed, tol, stream, opt, 1, from);
      if (rc != PRISM_EUNSUPPORTED) return rc;
    } else {
      prism_group half[4][BF16_MAX_GROUPS];   // NP <= 4 parts
      const void* const* half_from[4][BF16_MAX_GROUPS];
      for (int gi = 0; gi < ngroups; ++gi) {
        const size_t bytes = (size_t)(groups[gi].batch / NP) * groups[gi].m * groups[gi].n * 2;
        for (int h = 0; h < NP; ++h) {
          half[h][gi] = groups[gi];
          half[h][gi].batch = groups[gi].batch / NP;
          half[h][gi].x = (char*)groups[gi].x + h * bytes;
          half_from[h][gi] = from ? from[gi] + h * (groups[gi].batch / NP) : nullptr;
          half[h][gi].info = groups[gi].info ? groups[gi].info + h * (groups[gi].batch / NP) : nullptr;
        }
      }
      rc = get_fork(&f);
      if (rc != PRISM_OK) return rc;
      if (!f->begin_own(user) || hipEventRecord(f->forked, user) != hipSuccess) {
        (void)hipGetLastError();
        set_last_error("hipEventRecord failed");
        return PRISM_EHIP;
      }
      int forked = 0, first_error = PRISM_OK;
      for (; forked < NP - 1; ++forked)
        if (hipStreamWaitEvent(f->streams[forked], f->forked, 0) != hipSuccess) { first_error = PRISM_EHIP; break; }
      bool unsupported = false;
      for (int h = 0; h < NP && first_error == PRISM_OK; ++h) {
        first_error = run_polar_bf16_shapes(half[h], ngroups, degree, max_iters, sketch_dim, seed, tol, h ? f->streams[h - 1] : user, opt, NP,
                                            from ? half_from[h] : nullptr, h ? nullptr : f);
        if (h == 0 && first_error == PRISM_EUNSUPPORTED) { unsupported = true; first_error = PRISM_OK; break; }   // nothing was enqueued
      }
      if (!f->end_own(user)) {
        (void)hipGetLastError();
        if (first_error == PRISM_OK) { set_last_error("hipEventRecord failed"); first_error = PRISM_EHIP; }
      }
      for (int i = 0; i < forked; ++i) {
        if (hipEventRecord(f->joined[i], f->streams[i]) != hipSuccess || hipStreamWaitEvent(user, f->joined[i], 0) != hipSuccess) {
          (void)hipGetLastError();
          if (first_error == PRISM_OK) { set_last_error("joining an internal stream failed"); first_error = PRISM_EHIP; }
        }
      }
      if (!unsupported) return first_error;
    }
    set_last_error("");
  }
  CHECK_LAUNCH(gather());
  if (single_stream) {
    for (int gi = 0; gi < ngroups; ++gi) {
      prism_options o = opt ? *opt : prism_options{};
      o.info = groups[gi].info;
      rc = run(fn, groups[gi].x, groups[gi].inv_out, root_p, groups[gi].batch, groups[gi].m, groups[gi].n, dt, degree,
               max_iters, sketch_dim, seed, tol, stream, &o);
      if (rc != PRISM_OK) return rc;
    }
    return PRISM_OK;
  }
  rc = get_fork(&f);
  if (rc != PRISM_OK) return rc;
  const int used = ngroups < GROUP_STREAMS ? ngroups : GROUP_STREAMS;
  // Longest group first, each to the stream with the least to do: what a group takes is latency per iteration (one workgroup
  // per matrix up to order 64, then growing with the order) and the work of its products, roughly: the ranking is what counts.
  std::vector<std::pair<double, int>> order;
  for (int gi = 0; gi < ngroups; ++gi) {
    const prism_group& g = groups[gi];
    const double s = g.m < g.n ? g.m : g.n, l = g.m < g.n ? g.n : g.m;
    order.emplace_back((s <= 64 ? 25.0 : 45.0 + 0.07 * s) + 8.0 * g.batch * l * s * s * 1e-8, gi);
  }
  std::stable_sort(order.begin(), order.end(), [](const std::pair<double, int>& x, const std::pair<double, int>& y) { return x.first > y.first; });
  // nothing is forked before this record succeeds
  if (!f->begin_own(user) || hipEventRecord(f->forked, user) != hipSuccess) { (void)hipGetLastError(); set_last_error("hipEventRecord failed"); return PRISM_EHIP; }
  int first_error = PRISM_OK;
  int forked = 0;   // internal streams that wait for the caller's stream: exactly these are joined again below
  for (; forked < used - 1; ++forked)
    if (hipStreamWaitEvent(f->streams[forked], f->forked, 0) != hipSuccess) { first_error = PRISM_EHIP; break; }
  double load[GROUP_STREAMS] = {};
  for (int i = 0; i < ngroups && first_error == PRISM_OK; ++i) {
    const int gi = order[i].second;
    int at = 0;
    for (int q = 1; q < used; ++q)
      if (load[q] < load[at]) at = q;
    load[at] += order[i].first;
    prism_options o = opt ? *opt : prism_options{};
    o.info = groups[gi].info;
    o.flags |= PRISM_FLAG_SHARED_GPU;
    first_error = run(fn, groups[gi].x, groups[gi].inv_out, root_p, groups[gi].batch, groups[gi].m, groups[gi].n, dt,
                      degree, max_iters, sketch_dim, seed, tol, at ? f->streams[at - 1] : user, &o,
                      from_auto_split ? ngroups * groups[gi].batch : 0, at ? nullptr : f);
  }
  if (!f->end_own(user)) {
    (void)hipGetLastError();
    if (first_error == PRISM_OK) { set_last_error("hipEventRecord failed"); first_error = PRISM_EHIP; }
  }
  // Join every forked stream back into the caller's, on every exit: after an error too, and past a
  // failing record or wait of one stream (the others are still joined, so that no forked work is
  // left unordered and a stream capture of the caller is not left with dangling branches).
  for (int i = 0; i < forked; ++i) {
    if (hipEventRecord(f->joined[i], f->streams[i]) != hipSuccess || hipStreamWaitEvent(user, f->joined[i], 0) != hipSuccess) {
      (void)hipGetLastError();
      if (first_error == PRISM_OK) { set_last_error("joining an internal stream failed"); first_error = PRISM_EHIP; }
    }
  }
  return first_error;
}

// Single-shape entry points: a large batch of large matrices is enqueued as two half batches on
// the internal streams, so that the partial last wave of tiles and the latency-bound kernels of one
// half run beside the GEMMs of the other (+3 % on 8 x 4096^2 and 32 x 1024^2).  Every matrix is
// computed exactly as in an unsplit call; an explicit workspace keeps the call on one stream.
int run_auto(int fn, void* a, void* inv_out, int root_p, int batch, int m, int n, int dt, int degree, int max_iters,
             int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt) {
  static const int no_split = ab_switch("PRISM_NO_BATCH_SPLIT");
  const int S = m < n ? m : n;
  if (no_split || !a || !in_halves(batch, S) || (opt && opt->workspace) || (opt && (opt->flags & PRISM_FLAG_SINGLE_STREAM)) || g_prof_on)
    return run(fn, a, inv_out, root_p, batch, m, n, dt, degree, max_iters, sketch_dim, seed, tol, stream, opt);
  const size_t esz = dt == PRISM_BF16 ? 2 : 4;
  const size_t half = (size_t)(batch / 2) * m * n * esz;
  prism_group gr[2];
  for (int h = 0; h < 2; ++h) {
    gr[h].x = (char*)a + h * half;
    gr[h].inv_out = inv_out ? (char*)inv_out + h * half : nullptr;
    gr[h].info = (opt && opt->info) ? opt->info + h * (batch / 2) : nullptr;
    gr[h].batch = batch / 2; gr[h].m = m; gr[h].n = n;
  }
  prism_options o = opt ? *opt : prism_options{};
  o.info = nullptr;
  return run_grouped(fn, gr, 2, root_p, dt, degree, max_iters, sketch_dim, seed, tol, stream, &o, true);
}

}  // namespace
}  // namespace prism

// Device memory of the entry point that allocates nothing: one array per GPU, part of the loaded
// code object, alive until the process ends.  In host code this name only stands for the symbol;
// the device address is looked up once per device and that pointer is what the kernels get.
// (No `used` attribute: the compiler gives a static device variable that host code refers to a
// global symbol in the code object by itself, which is what the runtime's lookup by name needs;
// with the attribute the symbol stays local and the lookup fails.)
static __device__ __align__(256) unsigned char scratch[PRISM_STATIC_SCRATCH_BYTES];

namespace prism {
namespace {
std::mutex g_scratch_mu;
std::map<int, void*> g_scratch_ptr;   // device ordinal -> address of that device's copy of `scratch`

int static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); set_last_error("hipGetDevice failed"); return PRISM_EHIP; }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  auto it = g_scratch_ptr.find(dev);
  if (it == g_scratch_ptr.end()) {
    void* ptr = nullptr;   // the current device is `dev`: the address returned is that of its copy
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      (void)hipGetLastError();
      set_last_error("hipGetSymbolAddress of the static scratch array failed");
      return PRISM_EHIP;
    }
    if ((uintptr_t)ptr & 255) { set_last_error("static scratch array is not 256-byte aligned"); return PRISM_EHIP; }
    it = g_scratch_ptr.emplace(dev, ptr).first;
  }
  *out = it->second;
  return PRISM_OK;
}
}  // namespace
}  // namespace prism

using namespace prism;

extern "C" {

const char* prism_last_error(void) { return g_last_error.c_str(); }

int prism_release_workspaces(void) {
  set_last_error("");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = PRISM_OK, current = 0;
  const bool have_current = hipGetDevice(&current) == hipSuccess;
  for (auto& kv : g_cache.blocks) {
    if (hipSetDevice(kv.first.first) != hipSuccess) { rc = PRISM_EHIP; continue; }
    for (void* p : kv.second.retired)
      if (hipFree(p) != hipSuccess) rc = PRISM_EHIP;
    if (kv.second.ptr && hipFree(kv.second.ptr) != hipSuccess) rc = PRISM_EHIP;
  }
  g_cache.blocks.clear();
  if (have_current) (void)hipSetDevice(current);
  if (rc != PRISM_OK) { (void)hipGetLastError(); set_last_error("hipFree of a cached workspace failed"); }
  return rc;
}

int prism_profile_enable(int on) {
  std::lock_guard<std::mutex> lock(g_prof_mu);
  for (auto& r : g_prof) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
  g_prof.clear();
  g_prof_on = on != 0;
  return PRISM_OK;
}

int prism_profile_collect(double* ms_by_kind, long long* launches_by_kind, int nkinds) {
  if (!ms_by_kind || !launches_by_kind || (nkinds < PK_COUNT && nkinds != PK_FIT_SQUARE)) return PRISM_EINVAL;   // (that many: see prism.h)
  std::lock_guard<std::mutex> lock(g_prof_mu);
  for (int i = 0; i < nkinds; ++i) { ms_by_kind[i] = 0.0; launches_by_kind[i] = 0; }
  for (auto& r : g_prof) {
    if (hipEventSynchronize(r.b) != hipSuccess) return PRISM_EHIP;
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, r.a, r.b) != hipSuccess) return PRISM_EHIP;
    if (r.kind >= nkinds) continue;
    ms_by_kind[r.kind] += ms;
    launches_by_kind[r.kind] += 1;
  }
  return PRISM_OK;
}

int prism_workspace_bytes(int fn, int batch, int m, int n, prism_dtype dt, int degree, int sketch_dim,
                          int root_p, size_t* out_bytes) {
  if (!out_bytes || batch < 0 || m < 0 || n < 0) return PRISM_EINVAL;
  const bool empty = batch == 0 || m == 0 || n == 0;
  Plan P;
  int rc = empty ? make_plan(P, fn, 1, m ? m : 1, n ? n : 1, (int)dt, degree, sketch_dim, root_p, 0u)
                 : make_plan(P, fn, batch, m, n, (int)dt, degree, sketch_dim, root_p, 0u);
  if (rc != PRISM_OK) return rc;
  *out_bytes = empty ? 0 : P.total;
  return PRISM_OK;
}

int prism_polar(void* x, int batch, int m, int n, prism_dtype dt, int degree, int max_iters, int sketch_dim,
                uint64_t seed, double tol, void* stream) {
  return run_auto(PRISM_FN_POLAR, x, nullptr, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, nullptr);
}
int prism_polar_ex(void* x, int batch, int m, int n, prism_dtype dt, int degree, int max_iters, int sketch_dim,
                   uint64_t seed, double tol, void* stream, const prism_options* opt) {
  return run_auto(PRISM_FN_POLAR, x, nullptr, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, opt);
}
int prism_polar_static(void* x, int batch, int m, int n, prism_dtype dt, int degree, int max_iters, int sketch_dim,
                       uint64_t seed, double tol, void* stream, const prism_options* opt) {
  set_last_error("");
  if (opt && opt->workspace) { set_last_error("prism_polar_static takes no workspace: it uses the static array"); return PRISM_EINVAL; }
  if (batch < 0 || m < 0 || n < 0) return PRISM_EINVAL;
  prism_options o = opt ? *opt : prism_options{};
  if (batch > 0 && m > 0 && n > 0) {
    Plan P;
    const int rc = make_plan(P, PRISM_FN_POLAR, batch, m, n, (int)dt, degree, sketch_dim, 0, o.flags);
    if (rc != PRISM_OK) return rc;
    if ((P.ksplit || P.ring || P.x3) && P.total > (size_t)PRISM_STATIC_SCRATCH_BYTES)   // as the driver does with a workspace of this size
      (void)make_plan(P, PRISM_FN_POLAR, batch, m, n, (int)dt, degree, sketch_dim, 0, o.flags | FLAG_NO_SPLIT_K | FLAG_NO_FLOW | FLAG_NO_PLANES);
    if (P.total > (size_t)PRISM_STATIC_SCRATCH_BYTES) {
      set_last_error("prism_polar_static: this call needs more than PRISM_STATIC_SCRATCH_BYTES of scratch; use prism_polar_ex");
      return PRISM_EUNSUPPORTED;
    }
    void* ptr = nullptr;
    const int rs = static_scratch(&ptr);
    if (rs != PRISM_OK) return rs;
    o.workspace = ptr;
    o.workspace_bytes = (size_t)PRISM_STATIC_SCRATCH_BYTES;
  }
  // straight to the single-stream driver: no internal streams, no cached workspace, no timing events
  t_prof_off = true;
  const int rc = run(PRISM_FN_POLAR, x, nullptr, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, &o);
  t_prof_off = false;
  return rc;
}

int prism_sqrt(void* a, void* inv_out, int batch, int m, int n, prism_dtype dt, int degree, int max_iters,
               int sketch_dim, uint64_t seed, double tol, void* stream) {
  return run_auto(PRISM_FN_SQRT, a, inv_out, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, nullptr);
}
int prism_sqrt_ex(void* a, void* inv_out, int batch, int m, int n, prism_dtype dt, int degree, int max_iters,
                  int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt) {
  return run_auto(PRISM_FN_SQRT, a, inv_out, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, opt);
}
int prism_inv_root(void* a, int root_p, int batch, int m, int n, prism_dtype dt, int degree, int max_iters,
                   int sketch_dim, uint64_t seed, double tol, void* stream) {
  return run_auto(PRISM_FN_INV_ROOT, a, nullptr, root_p, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, nullptr);
}
int prism_inv_root_ex(void* a, int root_p, int batch, int m, int n, prism_dtype dt, int degree, int max_iters,
                      int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt) {
  return run_auto(PRISM_FN_INV_ROOT, a, nullptr, root_p, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, opt);
}

int prism_sign(void* x, int batch, int m, int n, prism_dtype dt, int degree, int max_iters, int sketch_dim,
               uint64_t seed, double tol, void* stream) {
  return run_auto(PRISM_FN_SIGN, x, nullptr, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, nullptr);
}
int prism_sign_ex(void* x, int batch, int m, int n, prism_dtype dt, int degree, int max_iters, int sketch_dim,
                  uint64_t seed, double tol, void* stream, const prism_options* opt) {
  return run_auto(PRISM_FN_SIGN, x, nullptr, 0, batch, m, n, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, opt);
}
int prism_inverse(void* a, int batch, int m, int n, prism_dtype dt, int max_iters, int sketch_dim, uint64_t seed,
                  double tol, void* stream) {
  return run_auto(PRISM_FN_INVERSE, a, nullptr, 0, batch, m, n, (int)dt, 5, max_iters, sketch_dim, seed, tol, stream, nullptr);
}
int prism_inverse_ex(void* a, int batch, int m, int n, prism_dtype dt, int max_iters, int sketch_dim, uint64_t seed,
                     double tol, void* stream, const prism_options* opt) {
  return run_auto(PRISM_FN_INVERSE, a, nullptr, 0, batch, m, n, (int)dt, 5, max_iters, sketch_dim, seed, tol, stream, opt);
}

int prism_sqrt_newton(void* a, void* inv_out, int batch, int m, int n, prism_dtype dt, int max_iters, int fit, double tol,
                      void* stream) {
  return run_auto(PRISM_FN_SQRT_NEWTON, a, inv_out, 0, batch, m, n, (int)dt, 3, max_iters, fit ? 1 : 0, 0, tol, stream, nullptr);
}
int prism_sqrt_newton_ex(void* a, void* inv_out, int batch, int m, int n, prism_dtype dt, int max_iters, int fit, double tol,
                         void* stream, const prism_options* opt) {
  return run_auto(PRISM_FN_SQRT_NEWTON, a, inv_out, 0, batch, m, n, (int)dt, 3, max_iters, fit ? 1 : 0, 0, tol, stream, opt);
}

int prism_spd_inverse(const float* a, float* out, int batch, int n, void* stream) {
  if (!a || !out || batch <= 0 || batch > PRISM_MAX_BATCH || n <= 0 || n % 64) return PRISM_EINVAL;
  char* ws = nullptr;
  const size_t bytes = (size_t)spd_inverse_scratch_floats(n, batch, batch) * 4;
  const int rc = get_workspace(bytes + (size_t)batch * FIT_SYNC_WORDS * sizeof(unsigned), stream, nullptr, &ws);
  if (rc != PRISM_OK) return rc;
  return launch_spd_inverse(a, out, n, batch, batch, nullptr, false, (float*)ws, (unsigned*)(ws + bytes), (hipStream_t)stream);
}

int prism_run_grouped(prism_fn fn, const prism_group* groups, int ngroups, int root_p, prism_dtype dt, int degree,
                      int max_iters, int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt) {
  return run_grouped((int)fn, groups, ngroups, root_p, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, opt);
}

int prism_run_grouped_from(prism_fn fn, const prism_group* groups, const void* const* const* from, int ngroups, int root_p, prism_dtype dt,
                           int degree, int max_iters, int sketch_dim, uint64_t seed, double tol, void* stream, const prism_options* opt) {
  if (ngroups > 0 && !from) return PRISM_EINVAL;
  return run_grouped((int)fn, groups, ngroups, root_p, (int)dt, degree, max_iters, sketch_dim, seed, tol, stream, opt, false, from);
}

int prism_sketch(float* out, int n, int sketch_dim, uint64_t seed, int k, int fn, void* stream) {
  if (!out || n <= 0 || sketch_dim <= 0 || sketch_dim > PRISM_MAX_SKETCH || k < 0) return PRISM_EINVAL;
  launch_sketch(out, n, n, sketch_dim, sketch_dim, seed, k, 1, fn, (hipStream_t)stream);
  return check_hip();
}

int prism_gauss_parts(uint32_t first, uint32_t count, double* radius, double* cosv, double* sinv, void* stream) {
  if (!radius || !cosv || !sinv || count == 0 || (uint64_t)first + count > (1ull << 24)) return PRISM_EINVAL;
  launch_gauss_parts(first, count, radius, cosv, sinv, (hipStream_t)stream);
  return check_hip();
}

int prism_chain_product(const float* R, const float* V, float* out, int batch, int n, int ld, void* stream) {
  if (!R || !V || !out || batch <= 0 || batch > PRISM_MAX_BATCH || n <= 0) return PRISM_EINVAL;
  return launch_chain(R, (long long)n * n, n, V, (long long)n * ld, out, (long long)n * ld, n, ld, batch, nullptr,
                      (hipStream_t)stream);
}

int prism_chain_product_bf16(const uint16_t* Rb, const float* R, const float* V, float* out, uint16_t* planes, int batch,
                             int n, int ld, void* stream) {
  set_last_error("");
  if (!Rb || !R || !V || !out || batch <= 0 || batch > PRISM_MAX_BATCH || n <= 0) return PRISM_EINVAL;
  if (!chain_bf16_supported(n, ld, batch, n)) return PRISM_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (chain_takes_small_kernel(n, ld, batch, true))
    return launch_chain_bf16(Rb, (long long)n * n, n, R, (long long)n * n, n + 1, V, (long long)n * ld, out,
                             (long long)n * ld, n, ld, batch, nullptr, s);
  if (!planes) return PRISM_EINVAL;
  const long long pe = (long long)n * ld * 3;
  CHECK_LAUNCH(launch_split_planes(V, planes, n, ld, batch, s));
  return launch_chain_planes(Rb, (long long)n * n, n, R, (long long)n * n, n + 1, V, (long long)n * ld, planes, pe, out,
                             (long long)n * ld, planes + (long long)batch * pe, pe, n, ld, batch, nullptr, s);
}

int prism_gemm_f32(const float* A, const float* B, float* C, int batch, int M, int N, int K, int a_km, void* stream) {
  if (!A || !B || !C || batch <= 0 || batch > PRISM_MAX_BATCH || M <= 0 || N <= 0 || K <= 0) return PRISM_EINVAL;
  GemmDesc g = {};
  g.A = A; g.strideA = (long long)M * K; g.lda = (a_km & 1) ? M : K;
  g.B = B; g.strideB = (long long)K * N; g.ldb = N;
  g.M = M; g.N = N; g.K = K; g.a_km = a_km & 1; g.sym = (a_km >> 1) & 1; g.batch = batch; g.epi = EPI_STORE;
  g.C = C; g.strideC = (long long)M * N; g.ldc = N;
  const int tn = (N == 16 || N == 32 || N == 64) ? N : 128;
  if (tn == 128) return launch_gemm_f32(g, (hipStream_t)stream);
  return launch_gemm_f32(g, (tn == 64 && M % 128) ? 64 : 128, tn, (hipStream_t)stream);
}

int prism_gemm_f32_planes(const float* A, const float* B, float* C, int batch, int M, int N, int K, int a_km, void* stream) {
  if (!A || !B || !C || batch <= 0 || batch > PRISM_MAX_BATCH || M <= 0 || N <= 0 || M % 64 || N % 64 || K < 96 || K % 32) return PRISM_EINVAL;
  if ((a_km != 0 && a_km != 1) || (a_km && M != N)) return PRISM_EINVAL;
  if ((long long)M * K > MAX_ENTRIES || (long long)K * N > MAX_ENTRIES || (long long)M * N > MAX_ENTRIES) return PRISM_EUNSUPPORTED;
  const long long ca = (long long)batch * M * K, cb = (long long)batch * K * N;
  const int tiles = split_tiles(M, N, batch, a_km);
  char* ws = nullptr;
  const int rc = get_workspace((size_t)(ca + cb) * 6 + (size_t)batch * tiles * sizeof(float), stream, nullptr, &ws);
  if (rc != PRISM_OK) return rc;
  uint16_t *pa = (uint16_t*)ws, *pb = pa + 3 * ca;
  launch_split3(A, pa, ca, ca, (hipStream_t)stream);
  launch_split3(B, pb, cb, cb, (hipStream_t)stream);
  GemmDesc g = {};
  g.A3 = pa; g.psA = ca; g.strideA = (long long)M * K; g.lda = a_km ? M : K;
  g.B3 = pb; g.psB = cb; g.strideB = (long long)K * N; g.ldb = N;
  g.M = M; g.N = N; g.K = K; g.a_km = g.sym = a_km; g.batch = batch; g.n_true = M;
  g.C = C; g.strideC = (long long)M * N; g.ldc = N;
  g.epi = a_km ? EPI_RESIDUAL : EPI_AXPY;
  g.Cin = C; g.strideCin = g.strideC; g.ldcin = N; g.c_in = 1.0f;
  g.rho_part = (float*)(pb + 3 * cb);
  return launch_gemm_split(g, nullptr, (hipStream_t)stream);
}

int prism_gemm_f64a(const float* A, const double* B, double* C, int batch, int M, int N, int K, void* stream) {
  if (!A || !B || !C || batch <= 0 || batch > PRISM_MAX_BATCH || M <= 0 || N <= 0 || K <= 0) return PRISM_EINVAL;
  GemmDesc g = {};
  g.A = A; g.strideA = (long long)M * K; g.lda = K;
  g.B = B; g.strideB = (long long)K * N; g.ldb = N;
  g.M = M; g.N = N; g.K = K; g.a_km = 0; g.batch = batch; g.epi = EPI_STORE;
  g.C = C; g.strideC = (long long)M * N; g.ldc = N;
  return launch_gemm_f64a(g, 64, 64, (hipStream_t)stream);
}

int prism_gemm_bf16_nt(const uint16_t* A, const uint16_t* B, float* C, int batch, int M, int N, int K, int tile,
                       void* stream) {
  if (!A || !B || !C || batch <= 0 || batch > PRISM_MAX_BATCH || M <= 0 || N <= 0 || K <= 0) return PRISM_EINVAL;
  Bf16Desc g = {};
  g.A = A; g.strideA = (long long)M * K; g.lda = K;
  g.B = B; g.strideB = (long long)N * K; g.ldb = K;
  g.M = M; g.N = N; g.K = K; g.batch = batch; g.epi = BEPI_STORE;
  g.C32 = C; g.strideC32 = (long long)M * N; g.ldc32 = N;
  if (tile >= 20000) {          // B stored [K][N]
    tile -= 20000;
    g.km = 2; g.ldb = N;
  } else if (tile >= 10000) {   // A stored [K][M] and B stored [K][N]
    tile -= 10000;
    g.km = 3; g.lda = M; g.ldb = N;
  }
  if (tile == 2561) return launch_gemm_bf16(g, 256, 128, (hipStream_t)stream);
  return launch_gemm_bf16(g, tile, tile, (hipStream_t)stream);
}

}  // extern "C"
