// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>

#include "fd_plans.hpp"
#include "flashdiff.h"

namespace fd {

// ---------------------------------------------------------------- errors
void set_error(const std::string& msg);
const char* get_error();

struct Error {
  fd_status status;
  std::string msg;
};

#define FD_HIP_CHECK(expr)                                                               \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      throw ::fd::Error{FD_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)}; \
  } while (0)

#define FD_LAUNCH_CHECK() FD_HIP_CHECK(hipGetLastError())

#define FD_REQUIRE(cond, status, msg)                 \
  do {                                                \
    if (!(cond)) throw ::fd::Error{(status), (msg)}; \
  } while (0)

// ---------------------------------------------------------------- workspace
// A carved region of float32 elements.
struct FSpan {
  float* p = nullptr;
  size_t n = 0;
};

inline void check_span(const FSpan& s, size_t need, const char* what) {
  if (s.p == nullptr || s.n < need)
    throw Error{FD_ERR_WORKSPACE, std::string("internal: region '") + what +
                                      "' smaller than the extent its kernel touches"};
}

// Bump allocator over the caller's workspace (never allocates device memory).
struct Arena {
  char* base = nullptr;
  size_t cap = 0;
  size_t used = 0;
  bool measuring = false;  // when true only counts bytes
  template <class T>
  T* take(size_t count) {
    size_t bytes = (count * sizeof(T) + 255) & ~size_t(255);
    size_t off = used;
    used += bytes;
    if (measuring) return nullptr;
    if (used > cap) throw Error{FD_ERR_WORKSPACE, "workspace too small"};
    return reinterpret_cast<T*>(base + off);
  }
  FSpan fspan(size_t count) { return FSpan{take<float>(count), count}; }
};

// ---------------------------------------------------------------- geometry
// Padded contraction width used for a feature dimension D (multiple of 4).
int padded_dim(int64_t D);
// Supported feature dimensions and block widths.
constexpr int MAX_D = 64;
constexpr int MAX_B = 64;

// Packed operands of one point set, produced by launch_packs.
// float32 X: xp holds the split float16 exponent chunks ([tiles][chunks][64]
//   uint4; chunk layout by recipe rid, row or column side).
// bfloat16 X: xp holds [tiles][dc][64] uint4 of raw bfloat16 features,
//   ap [tiles][64][4] the column offsets -||x_j||^2/2 in accumulator order,
//   ar [npad] the row offsets.
struct PointPack {
  FSpan xp, ap, ar;
  int64_t n = 0;      // real points
  int64_t npad = 0;   // padded points
  int dp = 0;         // padded feature width the region was sized for
  bool bf16 = false;  // filled from bfloat16 X
  int dc = 0;         // bfloat16: 32-feature chunks
  int rid = -1;       // float32: split-exponent recipe
  bool row_side = false;
  double beta = 0.0;  // bandwidth the pack was made for
  // float32 packs of a D whose short layout drops the third offset piece
  // (13 < D <= 30, 32 < D <= 62): the layout with all three pieces too (xp2,
  // recipe rid2), and the device word the kernels choose between them by
  // (max ||x - mu||^2 as float64 bits); variant 1 / 2 = this pack is the
  // short / the full-offset one, 0 = no choice.
  FSpan xp2;
  int rid2 = -1;
  const unsigned long long* r2max = nullptr;
  int variant = 0;
  // single-column products (HxGate): the device word and the case to serve
  const float* vbad = nullptr;
  int serves_bad = 0;
};

// Centring of a float32 point set (the kernel is translation invariant, and
// the Gram-form exponent is most accurate around the mean): partial column sums
// (float64, one row of D per prologue workgroup; every consumer adds them in
// the same order) and the largest squared distance of a point from the mean.
// flags: one word per prologue workgroup, non-zero where it met a NaN or an
// infinity.
constexpr int PROLOGUE_CAP = 1024;  // prologue workgroups per set at most
struct CentreWs {
  double* part = nullptr;               // D finished column sums, then nblk x D partial ones
  const double* sums = nullptr;         // nsums x D sums that the consumers add (set by the prologue)
  unsigned long long* r2max = nullptr;  // float64 bits of max ||x - mean||^2
  int* flags = nullptr;                 // nblk words, then nblk2 of a second point set
  int64_t n = 0;                        // points the partial sums cover (set by the prologue)
  int nblk = 0, nblk2 = 0;              // workgroups carved for
  int used = 0, used2 = 0;              // workgroups the last prologue ran
  int nsums = 0;
};
CentreWs carve_centre(Arena& a, int64_t n, int64_t n2 = 0, int cap = PROLOGUE_CAP);

// What one call reads before its kernel passes: the points X (column sums and
// finiteness), a second point set X2 (finiteness), and a block V (column
// maxima of sr V for the split pack).
struct PrologueIn {
  const void* X = nullptr;
  fd_dtype xt = FD_F32;
  int64_t n = 0, D = 0, ldx = 0;
  const void* X2 = nullptr;
  int64_t n2 = 0;
  const float* V = nullptr;
  int64_t nv = 0, b = 0, ldv = 0;
  const float* sr = nullptr;
  int cap = PROLOGUE_CAP;  // what the regions were carved for
};
// Everything in one launch (two for large sets): centre.part, centre.flags,
// vscale's maxima; clears centre.r2max (the packs raise it).
void launch_prologue(const PrologueIn& in, CentreWs& c, FSpan vscale, hipStream_t stream);
// r2max over X[0:n] from the prologue's sums, without packing (a no-op for bfloat16).
void launch_radius(const void* X, fd_dtype xt, int64_t n, int64_t D, int64_t ldx,
                   const CentreWs& c, hipStream_t stream);

// Exponent budget of the short split layouts: above beta log2(e) max ||x - mu||^2
// = 64 the kernels take the layout that keeps all three offset pieces (the
// dropped third piece is a coherent row / column scale error of up to
// 2^-22 ln 2 times that, 3.7e-6 relative at 64, against measured K V errors of
// 2.8e-6 at 50 and 5.4e-6 at 100 on the molecule-like set).
constexpr double EXP_BUDGET = 64.0;

// Exponent range of the float32 path: the row and column offsets
// -beta log2(e) ||x - mu||^2 (+15 on the row side) enter the contraction as
// float16 pieces, which hold magnitudes up to 65504.  Above
// beta log2(e) max ||x - mu||^2 = HX_EXP_RANGE the exponent cannot be formed:
// the asynchronous entry points fill their outputs with NaN, the synchronous
// ones refuse (FD_ERR_UNSUPPORTED) and the flow stops before such a probe.
// (bfloat16 X forms its exponent in float32 and has no such limit.)
constexpr double HX_EXP_RANGE = 65504.0 - 16.0;
// The coordinates enter as float16 pieces of s (x - mu) (column side) and
// 2 beta log2(e) (x - mu) / s (row side): both must stay within 65504 too.
// The balanced s keeps them below 512 inside the offset range; only its clamp
// at the float32 extremes of beta (below about 1e-39) could break that.
constexpr double HX_PIECE_MAX = 65504.0;
// s of the float32 packs for bandwidth beta (a power of two).
double hx_coord_scale(double beta);
// Whether bandwidth beta is inside the exponent range (offsets and
// coordinate pieces) for points of squared centred radius r2max (always for
// bfloat16 X).
bool exponent_in_range(fd_dtype xt, double beta, double r2max);
// r2max of a centring (host copy; synchronises the stream; 0 for bfloat16).
double exponent_radius(fd_dtype xt, const CentreWs& c, hipStream_t stream);
// Synchronous check: FD_ERR_UNSUPPORTED when beta is outside the range.
void require_exponent_range(fd_dtype xt, const CentreWs& c, double beta, hipStream_t stream);
// Asynchronous check: where it holds, the kernel that writes an output of the
// call writes NaN instead (a point is not finite, or beta is outside the
// exponent range).  flag == NULL: no check.
struct PoisonGate {
  const int* flag = nullptr;
  const unsigned long long* r2max = nullptr;  // NULL for bfloat16 X
  double bl = 0.0;                            // beta log2(e)
  double f2 = 0.0;                            // square of the larger coordinate scale
};
PoisonGate poison_gate(fd_dtype xt, const CentreWs& c, double beta, const int* flag);

// Floats per point of a pack region (large enough for either pack kind).
int pack_floats_per_point(int64_t D);

// Workspace carving helpers (size when arena.measuring).
PointPack carve_pack(Arena& a, int64_t n, int dp, int64_t pad);

// Launchers (enqueue on stream; throw Error on failure).
// The packs of one call in one launch: the row pack of Xr and the column pack
// of Xc (float32: centred on the prologue's mean, r2max raised to both sets'
// radius), the block V (split pack, or with ncb = 0 the weight pack of its one
// column), and 64-bit words to clear.  flag: receives whether the prologue met
// a non-finite value.
struct PackIn {
  const void *Xr = nullptr, *Xc = nullptr;
  fd_dtype xt = FD_F32;
  int64_t D = 0, ldx = 0;
  double beta = 0.0;
  int* flag = nullptr;
  const float* V = nullptr;
  int64_t b = 0, ldv = 0;
  const float* sr = nullptr;
  int ncb = 0;
  FSpan vp, vscale;
  int cap = PROLOGUE_CAP;  // the prologue's
  bool scaled = true;      // the prologue left V's maxima (else the weight pack is of V itself)
  unsigned long long *zero1 = nullptr, *zero2 = nullptr;
  int64_t nzero = 0;
};
void launch_packs(const PackIn& in, PointPack& rows, PointPack& cols, const CentreWs& centre,
                  hipStream_t stream);
void launch_pack_w(const float* w, int64_t n, int64_t npad, FSpan wp, hipStream_t stream);
// Split float16 pack of sr * V with per-column power-of-two scales, in two
// launches (column maxima, pack).  vscale (vscale_floats(n)): 64 inverse scales,
// 64 column maxima where the prologue finishes them, then its partial maxima.
size_t vscale_floats(int64_t n, int cap = PROLOGUE_CAP);
void launch_pack_v_split(const float* V, int64_t n, int64_t b, int64_t ldv, const float* sr,
                         int ncb, int64_t npad, FSpan vp, FSpan vscale, hipStream_t stream,
                         bool scaled = true);
// Y = diag(sl) K diag(sr) V from packed operands (V packed with sr applied).
void launch_product(const KVPlan& p, const PointPack& rows, const PointPack& cols, FSpan vp,
                    FSpan vscale, bool diag, const float* sl, float* Y, int64_t ldy, int b,
                    FSpan part, const PoisonGate& poison, hipStream_t stream);
// Y[:, 0] = diag(sl) K diag(sr) v for one column from its weight pack: on one
// point set (colfix, colfix_lo set: npad cleared words each, left cleared) the
// symmetric row sums, or the plain ones where the column holds a NaN or an
// infinity or spans more than column_range; else the plain ones.  The weight
// pack is a scaled one where column_sym_applies.
void launch_product_column(const KVPlan& p, const PointPack& rows, const PointPack& cols, FSpan wp,
                           FSpan vscale, bool diag, const float* sl, float* Y, int64_t ldy,
                           FSpan part, unsigned long long* colfix, unsigned long long* colfix_lo,
                           const PoisonGate& poison, hipStream_t stream);
// out = K w.
void launch_rowsum(const KVPlan& p, const PointPack& rows, const PointPack& cols, FSpan wp,
                   bool diag, float* out, FSpan part, hipStream_t stream);
// The symmetric path piece by piece (the two normalisation passes fuse their
// epilogues into its reduction): whether it applies, one pass of the kernel
// (row partials in part, fixed-point column sums added into colfix, which the
// pack or the last reduction cleared), and the fused reductions.  Each reduction leaves
// colfix zeroed.  launch_degree_reduce_q: q, and w = q^-alpha into the weight
// pack (the column pack's extent) when wp.p is set; launch_degree_reduce_ds: d = w t and s = w d^-1/2
// (either may be NULL).  Each workgroup of a reduction that makes q leaves the
// sum of its q in qsum; the next reduction's first workgroup adds those to
// s_off = sum(q) - n.
struct SymPass {
  int nsplit = 0;
  double inv_fix = 0.0;
};
// Second output of a weighted symmetric pass: the unit-weight row sums (per
// split, part) and fixed-point column sums (colfix) of the squared kernel.
// Fixed-point column sums: one word per point with `frac` fractional bits, or
// (lo set) two, the workgroups' words split at WIDE_SPLIT bits (fd_plans.hpp).
struct ColumnWords {
  unsigned long long* hi = nullptr;
  unsigned long long* lo = nullptr;
  int frac = 0;
};
struct SymSquares {
  float* part = nullptr;
  unsigned long long* colfix = nullptr;
};
// Whether a single-column product takes them.
bool column_sym_applies(const PointPack& rows, const PointPack& cols, bool diag,
                        const unsigned long long* colfix);
bool rowsum_sym_applies(const PointPack& rows, const PointPack& cols, bool diag,
                        const unsigned long long* colfix);
// sq_part / sq_colfix (weighted passes only): also the squared-kernel sums, whose
// reduction uses the returned inv_fix as well.  colfix_lo (weighted passes
// only): two words per column sum.
SymPass launch_rowsum_sym_pass(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                               FSpan wp, FSpan part, unsigned long long* colfix,
                               hipStream_t stream, FSpan sq_part = FSpan{},
                               unsigned long long* sq_colfix = nullptr,
                               unsigned long long* colfix_lo = nullptr);
void launch_degree_reduce_q(const SymPass& sp, const PointPack& rows, const PointPack& cols,
                            FSpan part, unsigned long long* colfix, float* q, double alpha,
                            FSpan wp, double* qsum, const PoisonGate& poison, hipStream_t stream);
void launch_degree_reduce_ds(const SymPass& sp, const PointPack& rows, FSpan part,
                             unsigned long long* colfix, const float* q, double alpha, float* d,
                             float* s, const double* qsum, double* s_off,
                             const PoisonGate& poison, hipStream_t stream);
// launch_degree_reduce_ds plus the squared-kernel sums of the same pass: the
// next dyadic level's q_next = K(2 beta) 1 and its w = q_next^-alpha into the
// weight pack wp (the column pack's extent); leaves both colfix arrays zeroed.
void launch_degree_reduce_dsq(const SymPass& sp, const PointPack& rows, const PointPack& cols,
                              FSpan part, unsigned long long* colfix, const float* q,
                              double alpha, float* d, float* s, FSpan sq_part,
                              unsigned long long* sq_colfix, float* q_next, FSpan wp,
                              const double* qsum, double* s_off, double* qsum_next,
                              const PoisonGate& poison, hipStream_t stream);
// Words of a partial-sum buffer of q (one per reduction workgroup).
int64_t qsum_words(int64_t npad);
// d, s from q and t; with qsum (nqsum words) also s_off.
void launch_degree_finish(const float* q, const float* t, int64_t n, double alpha, float* d,
                          float* s, const double* qsum, int64_t nqsum, double* s_off,
                          const PoisonGate& poison, hipStream_t stream);
void launch_pow_neg(const float* q, int64_t n, double alpha, float* w, hipStream_t stream);

}  // namespace fd
