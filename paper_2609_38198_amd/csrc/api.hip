// C ABI entry points: argument validation, workspace carving and the
// composition of the kernels into the operations declared in flashdiff.h.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <exception>
#include <mutex>
#include <string>
#include <vector>

#include "fd_internal.hpp"
#include "fd_solver.hpp"

namespace fd {

static thread_local std::string g_err;
void set_error(const std::string& msg) { g_err = msg; }
const char* get_error() { return g_err.c_str(); }

template <class F>
static fd_status guarded(F&& f) {
  try {
    f();
    set_error("");
    return FD_OK;
  } catch (const Error& e) {
    set_error(e.msg);
    return e.status;
  } catch (const std::exception& e) {
    set_error(std::string("internal error: ") + e.what());
    return FD_ERR_HIP;
  } catch (...) {
    set_error("internal error");
    return FD_ERR_HIP;
  }
}

constexpr int64_t MAX_POINTS = int64_t(1) << 30;

void check_points(const void* X, fd_dtype xt, int64_t N, int64_t D, int64_t ldx,
                  const char* what) {
  FD_REQUIRE(X != nullptr, FD_ERR_INVALID_ARG, std::string(what) + " is NULL");
  FD_REQUIRE(xt == FD_F32 || xt == FD_BF16, FD_ERR_INVALID_ARG, "unknown dtype");
  FD_REQUIRE(N >= 1 && N <= MAX_POINTS, FD_ERR_INVALID_ARG,
             std::string("number of points of ") + what + " out of range [1, 2^30]");
  FD_REQUIRE(D >= 1, FD_ERR_INVALID_ARG, "D must be >= 1");
  FD_REQUIRE(D <= MAX_D, FD_ERR_UNSUPPORTED, "D above 64 is not supported");
  FD_REQUIRE(ldx >= D, FD_ERR_INVALID_ARG, "ldx must be >= D");
}

void check_workspace(const void* ws, size_t ws_bytes, size_t need) {
  FD_REQUIRE(ws_bytes >= need, FD_ERR_WORKSPACE,
             "workspace too small: need " + std::to_string(need) + " bytes, got " +
                 std::to_string(ws_bytes));
  FD_REQUIRE(need == 0 || ws != nullptr, FD_ERR_WORKSPACE, "workspace is NULL");
  FD_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255) == 0, FD_ERR_WORKSPACE,
             "workspace must be 256-byte aligned");
}

// ---------------------------------------------------------------- products

ProductWs carve_product(Arena& a, int64_t Nr, int64_t Nc, int64_t D, int b) {
  ProductWs w;
  const int dp = padded_dim(D);
  w.plan = plan_product(Nr, Nc, dp, b);
  w.rows = carve_pack(a, Nr, dp, ROW_PAD);
  w.cols = carve_pack(a, Nc, dp, COL_PAD);
  w.vp = a.fspan(size_t(w.cols.npad) * w.plan.ncb * 16);
  w.vscale = a.fspan(vscale_floats(Nc));
  w.part = a.fspan(part_rows_bound(w.rows.npad, Nc) * w.plan.ncb * 16);
  if (b == 1) {
    w.colfix = a.take<unsigned long long>(size_t(w.rows.npad));
    w.colfix_lo = a.take<unsigned long long>(size_t(w.rows.npad));
  }
  w.flag = a.take<int>(1);
  w.centre = carve_centre(a, Nc, Nr);
  return w;
}

// The same regions sized for exactly the plan the call will run (the bound
// above covers every plan up to the given sizes).  sym: a single column takes the
// symmetric row sums; cap: prologue workgroups.
static ProductWs carve_product_exact(Arena& a, int64_t Nr, int64_t Nc, int64_t D, int b, bool sym,
                                     int cap) {
  ProductWs w;
  const int dp = padded_dim(D);
  w.cap = cap;
  w.plan = plan_product(Nr, Nc, dp, b);
  w.rows = carve_pack(a, Nr, dp, ROW_PAD);
  w.cols = carve_pack(a, Nc, dp, COL_PAD);
  w.vp = a.fspan(size_t(w.cols.npad) * w.plan.ncb * 16);
  w.vscale = a.fspan(vscale_floats(Nc, cap));
  const KVPlan rp = plan_rowsum(Nr, Nc, dp);
  const size_t part_prod = size_t(w.plan.nsplit) * w.rows.npad * w.plan.ncb * 16;
  size_t part_row = size_t(rp.nsplit) * w.rows.npad;
  if (sym) {
    part_row = std::max(part_row, sym_part_rows(w.rows.npad, SYM_NIB));
    w.colfix = a.take<unsigned long long>(size_t(w.rows.npad));
    w.colfix_lo = a.take<unsigned long long>(size_t(w.rows.npad));
  }
  w.part = a.fspan(b == 1 ? part_row : part_prod);
  w.flag = a.take<int>(1);
  w.centre = carve_centre(a, Nc, Nr, cap);
  return w;
}

// The fullest variant of those whose regions fit `bytes` of scratch, or else
// the smallest one: a problem near the limit gives up the symmetric row sums of
// a single column first (its words and partial sums are up to half of the
// total; the plain ones take 1.5 times as long), then prologue workgroups.
struct ExactVariant {
  bool sym = false;
  int cap = PROLOGUE_CAP;
  size_t bytes = 0;
};
static ExactVariant pick_product_exact(int64_t Nr, int64_t Nc, int64_t D, int b, bool one_set,
                                       size_t bytes) {
  ExactVariant v;
  for (int sym = b == 1 && one_set && Nr == Nc && Nr >= COLUMN_SYM_POINTS; sym >= 0; --sym)
    for (int cap : {PROLOGUE_CAP, 128, 32, 8}) {
      Arena m;
      m.measuring = true;
      carve_product_exact(m, Nr, Nc, D, b, sym != 0, cap);
      v.sym = sym != 0;
      v.cap = cap;
      v.bytes = m.used;
      if (m.used <= bytes) return v;
    }
  return v;
}

// Scratch of the allocation-free product: one array per device, held until
// the process ends.  Host code never passes the array's name to a kernel or a
// copy (on the host it is a stand-in, not a device address); it uses the
// device address that hipGetSymbolAddress returns, looked up once per device
// with that device current.
constexpr size_t SCRATCH_BYTES = size_t(256) << 20;
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

static char* scratch_on_current_device() {
  static std::mutex mu;
  static std::vector<char*> ptrs;
  int dev = -1;
  FD_HIP_CHECK(hipGetDevice(&dev));
  FD_REQUIRE(dev >= 0, FD_ERR_HIP, "no current device");
  std::lock_guard<std::mutex> lock(mu);
  if (size_t(dev) >= ptrs.size()) ptrs.resize(size_t(dev) + 1, nullptr);
  if (ptrs[size_t(dev)] == nullptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    FD_REQUIRE(e == hipSuccess && p != nullptr, FD_ERR_HIP,
               std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    FD_REQUIRE((reinterpret_cast<uintptr_t>(p) & 255) == 0, FD_ERR_HIP,
               "scratch array is not 256-byte aligned");
    ptrs[size_t(dev)] = static_cast<char*>(p);
  }
  return ptrs[size_t(dev)];
}

PointPack pack_view(const PointPack& big, int64_t n, int64_t pad) {
  PointPack p = big;
  p.n = n;
  p.npad = round_up(n, pad);
  return p;
}

DegreeWs degree_view(const DegreeWs& big, int64_t n) {
  DegreeWs w = big;
  w.rows = pack_view(big.rows, n, ROW_PAD);
  w.cols = pack_view(big.cols, n, COL_PAD);
  w.plan = plan_rowsum(n, n, big.rows.dp);
  return w;
}

ProductWs product_view(const ProductWs& big, const PointPack& rows, const PointPack& cols,
                       int width) {
  ProductWs w = big;
  w.rows = rows;
  w.cols = cols;
  w.plan = plan_product(rows.n, cols.n, rows.dp, width);
  return w;
}

// The passes of a product whose points and V are packed.
static void product_run(ProductWs& w, const float* sl, int b, float* Y, int64_t ldy, bool diag,
                        const PoisonGate& poison, hipStream_t stream) {
  if (b == 1) {
    // one right-hand side: weighted row sums K (sr v) on the vector ALUs (no
    // matrix-core contraction padded to 16 columns), then the row scale
    launch_product_column(plan_rowsum(w.rows.n, w.cols.n, w.rows.dp), w.rows, w.cols, w.vp,
                          w.vscale, diag, sl, Y, ldy, w.part, w.colfix, w.colfix_lo, poison, stream);
    return;
  }
  launch_product(w.plan, w.rows, w.cols, w.vp, w.vscale, diag, sl, Y, ldy, b, w.part, poison,
                 stream);
}

void product_apply(ProductWs& w, const float* sl, const float* sr, const float* V, int64_t ldv,
                   int b, float* Y, int64_t ldy, bool diag, hipStream_t stream) {
  launch_pack_v_split(V, w.cols.n, b, ldv, sr, b == 1 ? 0 : w.plan.ncb, w.cols.npad, w.vp,
                      w.vscale, stream,
                      b > 1 || column_sym_applies(w.rows, w.cols, diag, w.colfix));
  product_run(w, sl, b, Y, ldy, diag, PoisonGate{}, stream);
}

// One product from raw inputs: prologue, packs, product passes (whose last
// kernel writes NaN where the call is poisoned).
static void matmul_run(ProductWs& w, const void* Xr, const void* Xc, int64_t D, int64_t ldx,
                       fd_dtype xt, double beta, const float* sl, const float* sr, const float* V,
                       int b, int64_t ldv, float* Y, int64_t ldy, hipStream_t st) {
  // same base pointer and ldx: index i names the same point in both sets
  const bool diag = Xr == Xc;
  PrologueIn pro;
  // one centre for both sets: the column set's mean, the radius over both
  pro.X = Xc;
  pro.xt = xt;
  pro.n = w.cols.n;
  pro.D = D;
  pro.ldx = ldx;
  if (!diag || w.rows.n > w.cols.n) {
    pro.X2 = Xr;
    pro.n2 = w.rows.n;
  }
  const bool scaled = b > 1 || column_sym_applies(w.rows, w.cols, diag, w.colfix);
  pro.V = scaled ? V : nullptr;
  pro.nv = w.cols.n;
  pro.b = b;
  pro.ldv = ldv;
  pro.sr = sr;
  pro.cap = w.cap;
  launch_prologue(pro, w.centre, w.vscale, st);
  PackIn in;
  in.Xr = Xr;
  in.Xc = Xc;
  in.xt = xt;
  in.D = D;
  in.ldx = ldx;
  in.beta = beta;
  in.flag = w.flag;
  in.V = V;
  in.b = b;
  in.ldv = ldv;
  in.sr = sr;
  in.ncb = b == 1 ? 0 : w.plan.ncb;
  in.vp = w.vp;
  in.vscale = w.vscale;
  in.cap = w.cap;
  in.scaled = scaled;
  in.zero1 = w.colfix;
  in.zero2 = w.colfix_lo;
  in.nzero = w.colfix != nullptr ? w.rows.npad : 0;
  launch_packs(in, w.rows, w.cols, w.centre, st);
  product_run(w, sl, b, Y, ldy, diag, poison_gate(xt, w.centre, beta, w.flag), st);
}

// ---------------------------------------------------------------- degree

DegreeWs carve_degree(Arena& a, int64_t N, int64_t D, bool prefixes) {
  DegreeWs w;
  const int dp = padded_dim(D);
  w.plan = plan_rowsum(N, N, dp);
  w.rows = carve_pack(a, N, dp, ROW_PAD);
  w.cols = carve_pack(a, N, dp, COL_PAD);
  w.wp = a.fspan(size_t(w.cols.npad) * 16);  // one float4 per lane per 16-point tile
  w.q = a.take<float>(size_t(N));
  w.w = a.take<float>(size_t(N));
  w.part = a.fspan(std::max(part_rows_bound(w.rows.npad, N),
                            prefixes ? sym_part_rows_within(w.rows.npad, SYM_NIB)
                                     : sym_part_rows(w.rows.npad, SYM_NIB)));
  w.colfix = a.take<unsigned long long>(size_t(w.rows.npad));
  w.qsum = a.take<double>(2 * size_t(qsum_words(w.rows.npad)));
  w.flag = a.take<int>(1);
  w.centre = carve_centre(a, N);
  return w;
}

// Row and column packs of one point set at one bandwidth, with the column-sum
// words of the symmetric passes (and the squared kernel's, where carved) cleared.
static void degree_packs(DegreeWs& w, const void* X, fd_dtype xt, int64_t D, int64_t ldx,
                         double beta, int* flag, hipStream_t stream) {
  PackIn in;
  in.Xr = in.Xc = X;
  in.xt = xt;
  in.D = D;
  in.ldx = ldx;
  in.beta = beta;
  in.flag = flag;
  in.zero1 = w.colfix;
  in.zero2 = w.sq_colfix;
  in.nzero = w.rows.npad;
  launch_packs(in, w.rows, w.cols, w.centre, stream);
}

static void degree_prologue(DegreeWs& w, const void* X, fd_dtype xt, int64_t N, int64_t D,
                            int64_t ldx, hipStream_t stream) {
  PrologueIn pro;
  pro.X = X;
  pro.xt = xt;
  pro.n = N;
  pro.D = D;
  pro.ldx = ldx;
  launch_prologue(pro, w.centre, FSpan{}, stream);
}

// The passes of fd_degree on filled packs.
static void degree_passes(DegreeWs& w, int64_t N, double alpha, float* q, float* d, float* s,
                          double* s_off, const PoisonGate& poison, hipStream_t stream) {
  float* qq = q != nullptr ? q : w.q;
  const int64_t nq = qsum_words(w.rows.npad);
  // symmetric row sums with the epilogues fused into their reductions; the
  // first reduction leaves the column-sum words zeroed for the second pass
  const SymPass p1 = launch_rowsum_sym_pass(w.plan, w.rows, w.cols, FSpan{}, w.part, w.colfix,
                                            stream);
  launch_degree_reduce_q(p1, w.rows, w.cols, w.part, w.colfix, qq, alpha,
                         alpha == 0.0 ? FSpan{} : w.wp, w.qsum, poison, stream);
  if (alpha == 0.0) {
    launch_degree_finish(qq, qq, N, 0.0, d, s, w.qsum, nq, s_off, poison, stream);
    return;
  }
  const SymPass p2 = launch_rowsum_sym_pass(w.plan, w.rows, w.cols, w.wp, w.part, w.colfix,
                                            stream);
  launch_degree_reduce_ds(p2, w.rows, w.part, w.colfix, qq, alpha, d, s, w.qsum, s_off, poison,
                          stream);
}

void degree_run(DegreeWs& w, const void* X, fd_dtype xt, int64_t N, int64_t D, int64_t ldx,
                double beta, double alpha, float* q, float* d, float* s, double* s_off,
                bool poison, hipStream_t stream) {
  degree_prologue(w, X, xt, N, D, ldx, stream);
  int* flag = poison ? w.flag : nullptr;
  degree_packs(w, X, xt, D, ldx, beta, flag, stream);
  degree_passes(w, N, alpha, q, d, s, s_off, poison_gate(xt, w.centre, beta, flag), stream);
}

DegreeWs carve_degree_dyadic(Arena& a, int64_t N, int64_t D) {
  DegreeWs w = carve_degree(a, N, D);
  w.sq_part = a.fspan(sym_part_rows(w.rows.npad, SYM_NIB));
  w.sq_colfix = a.take<unsigned long long>(size_t(w.rows.npad));
  return w;
}

void degree_run_dyadic(DegreeWs& w, const void* X, fd_dtype xt, int64_t N, int64_t D,
                       int64_t ldx, double beta0, int nb, double alpha, float* q, float* d,
                       float* s, double* s_off, hipStream_t stream) {
  auto at = [N](float* v, int l) { return v != nullptr ? v + int64_t(l) * N : nullptr; };
  auto off_at = [s_off](int l) { return s_off != nullptr ? s_off + l : nullptr; };
  auto beta_of = [beta0](int l) { return std::ldexp(beta0, l); };
  degree_prologue(w, X, xt, N, D, ldx, stream);
  degree_packs(w, X, xt, D, ldx, beta_of(0), w.flag, stream);
  // the largest bandwidth decides (every level's outputs are poisoned)
  const PoisonGate poison = poison_gate(xt, w.centre, beta_of(nb - 1), w.flag);
  if (alpha == 0.0 || xt == FD_BF16) {
    // no weighted pass to carry the squares (alpha = 0), or bfloat16 inputs
    // (stated level by level): fd_degree's passes
    for (int l = 0; l < nb; ++l) {
      if (l > 0) degree_packs(w, X, xt, D, ldx, beta_of(l), nullptr, stream);
      degree_passes(w, N, alpha, at(q, l), at(d, l), at(s, l), off_at(l), poison, stream);
    }
    return;
  }
  // q of the current level and of the next, in the caller's arrays or in two
  // workspace vectors used in turn; likewise its partial sums
  auto q_of = [&](int l) { return q != nullptr ? q + int64_t(l) * N : (l % 2 ? w.w : w.q); };
  const int64_t nq = qsum_words(w.rows.npad);
  auto qsum_of = [&](int l) { return w.qsum + (l % 2) * nq; };
  const SymPass p1 = launch_rowsum_sym_pass(w.plan, w.rows, w.cols, FSpan{}, w.part, w.colfix,
                                            stream);
  launch_degree_reduce_q(p1, w.rows, w.cols, w.part, w.colfix, q_of(0), alpha, w.wp, qsum_of(0),
                         poison, stream);
  for (int l = 0; l < nb; ++l) {
    // (the column-sum words are zero already; clearing them again is harmless)
    if (l > 0) degree_packs(w, X, xt, D, ldx, beta_of(l), nullptr, stream);
    if (l + 1 == nb) {
      const SymPass p2 = launch_rowsum_sym_pass(w.plan, w.rows, w.cols, w.wp, w.part, w.colfix,
                                                stream);
      launch_degree_reduce_ds(p2, w.rows, w.part, w.colfix, q_of(l), alpha, at(d, l), at(s, l),
                              qsum_of(l), off_at(l), poison, stream);
      break;
    }
    // weighted pass of level l with the squared sums: t_l and q_{l+1}
    const SymPass p2 = launch_rowsum_sym_pass(w.plan, w.rows, w.cols, w.wp, w.part, w.colfix,
                                              stream, w.sq_part, w.sq_colfix);
    launch_degree_reduce_dsq(p2, w.rows, w.cols, w.part, w.colfix, q_of(l), alpha, at(d, l),
                             at(s, l), w.sq_part, w.sq_colfix, q_of(l + 1), w.wp, qsum_of(l),
                             off_at(l), qsum_of(l + 1), poison, stream);
  }
}

}  // namespace fd

using namespace fd;

extern "C" {

const char* fd_last_error(void) { return get_error(); }

const char* fd_status_string(fd_status s) {
  switch (s) {
    case FD_OK: return "FD_OK";
    case FD_ERR_INVALID_ARG: return "FD_ERR_INVALID_ARG";
    case FD_ERR_UNSUPPORTED: return "FD_ERR_UNSUPPORTED";
    case FD_ERR_WORKSPACE: return "FD_ERR_WORKSPACE";
    case FD_ERR_HIP: return "FD_ERR_HIP";
    case FD_ERR_NOT_CONVERGED: return "FD_ERR_NOT_CONVERGED";
    case FD_ERR_PERRON_WALL: return "FD_ERR_PERRON_WALL";
  }
  return "FD_UNKNOWN_STATUS";
}

void fd_lanczos_default_opts(fd_lanczos_opts* opts) {
  if (opts == nullptr) return;
  opts->tol = 1e-5;
  opts->max_restarts = 200;
  opts->max_basis_blocks = 0;
  opts->keep = -1;
  opts->max_matvecs = 0;
  opts->verbose = 0;
  opts->seed = 0x5eed;
}

size_t fd_workspace_size(fd_op op, int64_t Nr, int64_t Nc, int64_t D, int64_t b, int64_t k,
                         const fd_lanczos_opts* opts) {
  size_t out = 0;
  fd_status st = guarded([&] {
    Arena a;
    a.measuring = true;
    FD_REQUIRE(Nr >= 1 && Nr <= MAX_POINTS && D >= 1 && D <= MAX_D, FD_ERR_INVALID_ARG, "size");
    switch (op) {
      case FD_OP_KERNEL_MATMUL:
        FD_REQUIRE(Nc >= 1 && Nc <= MAX_POINTS && b >= 1 && b <= MAX_B, FD_ERR_INVALID_ARG, "size");
        carve_product(a, Nr, Nc, D, int(b));
        break;
      case FD_OP_DEGREE:
        carve_degree(a, Nr, D);
        break;
      case FD_OP_DEGREE_DYADIC:
        carve_degree_dyadic(a, Nr, D);
        break;
      case FD_OP_BLOCK_LANCZOS: {
        fd_lanczos_opts o;
        fd_lanczos_default_opts(&o);
        if (opts != nullptr) o = *opts;
        FD_REQUIRE(b >= 1 && b <= MAX_B && k >= 1 && k <= Nr, FD_ERR_INVALID_ARG, "size");
        carve_solver(a, Nr, D, int(b), int(k), o);
        break;
      }
      case FD_OP_CONTINUATION: {
        fd_lanczos_opts o;
        fd_lanczos_default_opts(&o);
        if (opts != nullptr) o = *opts;
        FD_REQUIRE(b >= 1 && b <= MAX_B && k >= 1 && k <= 64 && k <= Nr && Nc >= 1,
                   FD_ERR_INVALID_ARG, "size");
        carve_continuation_ws(a, Nr, Nc, D, int(b), int(k), o);
        break;
      }
      case FD_OP_BETA_FLOW: {
        fd_lanczos_opts o;
        fd_lanczos_default_opts(&o);
        if (opts != nullptr) o = *opts;
        FD_REQUIRE(b >= 1 && b <= MAX_B && k >= 2 && k <= Nr, FD_ERR_INVALID_ARG, "size");
        carve_flow_ws(a, Nr, D, int(b), int(k), o);
        break;
      }
      default:
        throw Error{FD_ERR_INVALID_ARG, "unknown op"};
    }
    out = a.used;
  });
  return st == FD_OK ? out : 0;
}

fd_status fd_kernel_matmul(const void* Xr, int64_t Nr, const void* Xc, int64_t Nc, int64_t D,
                           int64_t ldx, fd_dtype xt, float beta, const float* sl, const float* sr,
                           const float* V, int64_t b, int64_t ldv, float* Y, int64_t ldy,
                           void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    check_points(Xr, xt, Nr, D, ldx, "Xr");
    check_points(Xc, xt, Nc, D, ldx, "Xc");
    FD_REQUIRE(std::isfinite(beta) && beta >= 0.f, FD_ERR_INVALID_ARG, "beta must be finite and >= 0");
    FD_REQUIRE(V != nullptr && Y != nullptr, FD_ERR_INVALID_ARG, "V and Y must not be NULL");
    FD_REQUIRE(b >= 1 && b <= MAX_B, FD_ERR_INVALID_ARG, "b must be in [1, 64]");
    FD_REQUIRE(ldv >= b && ldy >= b, FD_ERR_INVALID_ARG, "ldv and ldy must be >= b");
    Arena m;
    m.measuring = true;
    carve_product(m, Nr, Nc, D, int(b));
    check_workspace(ws, ws_bytes, m.used);
    Arena a;
    a.base = static_cast<char*>(ws);
    a.cap = ws_bytes;
    ProductWs w = carve_product(a, Nr, Nc, D, int(b));
    hipStream_t st = static_cast<hipStream_t>(stream);
    matmul_run(w, Xr, Xc, D, ldx, xt, beta, sl, sr, V, int(b), ldv, Y, ldy, st);
  });
}

fd_status fd_kernel_matmul_noalloc(const void* Xr, int64_t Nr, const void* Xc, int64_t Nc,
                                   int64_t D, int64_t ldx, fd_dtype xt, float beta,
                                   const float* sl, const float* sr, const float* V, int64_t b,
                                   int64_t ldv, float* Y, int64_t ldy, void* stream) {
  return guarded([&] {
    check_points(Xr, xt, Nr, D, ldx, "Xr");
    check_points(Xc, xt, Nc, D, ldx, "Xc");
    FD_REQUIRE(std::isfinite(beta) && beta >= 0.f, FD_ERR_INVALID_ARG, "beta must be finite and >= 0");
    FD_REQUIRE(V != nullptr && Y != nullptr, FD_ERR_INVALID_ARG, "V and Y must not be NULL");
    FD_REQUIRE(b >= 1 && b <= MAX_B, FD_ERR_INVALID_ARG, "b must be in [1, 64]");
    FD_REQUIRE(ldv >= b && ldy >= b, FD_ERR_INVALID_ARG, "ldv and ldy must be >= b");
    const ExactVariant v = pick_product_exact(Nr, Nc, D, int(b), Xr == Xc, SCRATCH_BYTES);
    FD_REQUIRE(v.bytes <= SCRATCH_BYTES, FD_ERR_WORKSPACE,
               "problem too large for the built-in scratch: needs " + std::to_string(v.bytes) +
                   " bytes, the scratch holds " + std::to_string(SCRATCH_BYTES) +
                   " (use fd_kernel_matmul with a workspace)");
    Arena a;
    a.base = scratch_on_current_device();
    a.cap = SCRATCH_BYTES;
    ProductWs w = carve_product_exact(a, Nr, Nc, D, int(b), v.sym, v.cap);
    hipStream_t st = static_cast<hipStream_t>(stream);
    matmul_run(w, Xr, Xc, D, ldx, xt, beta, sl, sr, V, int(b), ldv, Y, ldy, st);
  });
}

size_t fd_kernel_matmul_noalloc_limit(void) { return SCRATCH_BYTES; }

fd_status fd_degree(const void* X, fd_dtype xt, int64_t N, int64_t D, int64_t ldx, float beta,
                    float alpha, float* q, float* d, float* s, double* s_off, void* ws,
                    size_t ws_bytes, void* stream) {
  return guarded([&] {
    check_points(X, xt, N, D, ldx, "X");
    FD_REQUIRE(std::isfinite(beta) && beta > 0.f, FD_ERR_INVALID_ARG, "beta must be finite and > 0");
    FD_REQUIRE(alpha >= 0.f && alpha <= 1.f, FD_ERR_INVALID_ARG, "alpha must be in [0, 1]");
    Arena m;
    m.measuring = true;
    carve_degree(m, N, D);
    check_workspace(ws, ws_bytes, m.used);
    Arena a;
    a.base = static_cast<char*>(ws);
    a.cap = ws_bytes;
    DegreeWs w = carve_degree(a, N, D);
    hipStream_t st = static_cast<hipStream_t>(stream);
    degree_run(w, X, xt, N, D, ldx, beta, alpha, q, d, s, s_off, true, st);
  });
}

fd_status fd_degree_dyadic(const void* X, fd_dtype xt, int64_t N, int64_t D, int64_t ldx,
                           float beta0, int32_t nbeta, float alpha, float* q, float* d, float* s,
                           double* s_off, void* ws, size_t ws_bytes, void* stream) {
  return guarded([&] {
    check_points(X, xt, N, D, ldx, "X");
    FD_REQUIRE(nbeta >= 1 && nbeta <= 32, FD_ERR_INVALID_ARG, "nbeta must be in [1, 32]");
    FD_REQUIRE(std::isfinite(beta0) && beta0 > 0.f &&
                   std::isfinite(std::ldexp(double(beta0), nbeta - 1)) &&
                   std::ldexp(double(beta0), nbeta - 1) <= double(FLT_MAX),
               FD_ERR_INVALID_ARG, "beta0 must be > 0 with beta0 2^(nbeta-1) finite");
    FD_REQUIRE(alpha >= 0.f && alpha <= 1.f, FD_ERR_INVALID_ARG, "alpha must be in [0, 1]");
    Arena m;
    m.measuring = true;
    carve_degree_dyadic(m, N, D);
    check_workspace(ws, ws_bytes, m.used);
    Arena a;
    a.base = static_cast<char*>(ws);
    a.cap = ws_bytes;
    DegreeWs w = carve_degree_dyadic(a, N, D);
    hipStream_t st = static_cast<hipStream_t>(stream);
    degree_run_dyadic(w, X, xt, N, D, ldx, beta0, int(nbeta), alpha, q, d, s, s_off, st);
  });
}

}  // extern "C"
