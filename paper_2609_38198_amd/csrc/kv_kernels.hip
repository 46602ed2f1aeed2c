// Shared pieces of the fused Gaussian-kernel products: V and weight packs,
// the bfloat16-input kernels, partial-sum reductions, the degree epilogues and
// the host-side planning and dispatch.  The float32-input kernels (split
// float16 exponent contraction) are in hx_kernels.hip.
//
// Operation (FlashDiffusion Sec. 2.1 eq. matmat, Sec. 2.2 eq. tiled_rbf):
//   Y_I = diag(sl_I) * sum_J exp(-beta * ||x_i - x_j||^2) * (sr_J * V_J),
// and the row sums q = K 1, K w of the normalisation (Sec. 2.1).  The N x N
// kernel matrix is never stored.
#include <hip/hip_runtime.h>

#include <cstring>

#include <algorithm>
#include <cmath>

#include "fd_profile.hpp"
#include "kv_common.hpp"
#include "sym_rowsum.hpp"

namespace fd {

int padded_dim(int64_t D) {
  static const int dims[] = {4, 8, 12, 16, 24, 32, 48, 64};
  for (int d : dims)
    if (D <= d) return d;
  return 0;
}

// Floats per point of a pack region: large enough for the float32 (split
// float16 chunks of 16 floats) and the bfloat16 pack of any D with this
// padded width; chunk counts grow with D, so the largest D decides.
int pack_floats_per_point(int64_t D) {
  const int dp = padded_dim(D);
  const int dc16 = int(ceil_div(dp, 32)) * 16;
  const int rid = hx_recipe_for(dp);
  const int hx = 16 * std::max(hx_col_chunks(rid), hx_row_chunks(rid));
  return std::max({dp, dc16, hx});
}

PointPack carve_pack(Arena& a, int64_t n, int dp, int64_t pad) {
  PointPack p;
  p.n = n;
  p.npad = round_up(n, pad);
  p.dp = dp;
  p.xp = a.fspan(size_t(p.npad) * pack_floats_per_point(dp));
  p.ap = a.fspan(size_t(p.npad) * 16);  // [tiles][64][4]: 16 floats per point
  p.ar = a.fspan(size_t(p.npad));
  // the full-offset layout of a short recipe: every D of this padded width
  // whose recipe drops the third offset piece takes the same wider recipe
  const int wide = hx_full_offset_recipe(hx_recipe_for(dp == 32 ? 30 : dp == 64 ? 62 : dp));
  if (wide >= 0)
    p.xp2 = a.fspan(size_t(p.npad) * 16 * std::max(hx_col_chunks(wide), hx_row_chunks(wide)));
  return p;
}

// ------------------------------------------------------------------ prologue
//
// One launch reads everything a call's packs depend on: the column sums of X
// (float64), whether X (and a second point set X2) is finite, and the column
// maxima of sr V.  These are reductions over inputs of at most a few hundred MB
// in front of an N^2 pass, so what counts is the number of launches and the
// latency of each, not their bandwidth: workgroups own consecutive rows, the
// lanes of a wave lie along the columns (coalesced; the earlier sums, one
// column after the other with lanes along the rows, took 61 us at 5,003 x 30
// and 101 us at 65,536 x 32), four rows in flight per lane, and every
// workgroup leaves its partial result for the consumer to add, so that nothing
// has to be cleared beforehand.
//
// For a large set the bandwidth counts after all: up to 1024 workgroups, and a
// second launch (prologue_finish_kernel) that adds their results once, where
// every pack workgroup would add them again.  300 rows against n columns, one
// launch of 128 workgroups / two (us): for the maxima of V, D = 12, b = 64
// n = 65,536 100 / 74, 200,000 243 / 170, b = 16 n = 50,000 49 / 49, 65,536 58 / 56,
// b = 1 n = 36,000 42 / 45: from 3 * 2^18 values on.  For the column sums,
// b = 8, D = 30 n = 200,000 137 / 107, D = 64 n = 262,144 244 / 189, D = 12
// n = 524,288 236 / 213, but D = 12 n = 65,536 74 / 85, D = 4 n = 200,000 102 / 127:
// adding 128 partial sums first spreads the pack's waves, which otherwise all
// raise the radius word at once: from 2^22 values on.

constexpr int PRO_BLOCKS = 128;     // workgroups per point set in one launch
constexpr int PRO_MIN_ROWS = 128;   // rows a workgroup should at least have
constexpr int64_t PRO_LARGE_N = 32768, PRO_LARGE_VALUES = int64_t(3) << 18;
constexpr int64_t PRO_LARGE_SUMS = int64_t(1) << 22;
constexpr int PRO_LARGE_ROWS = 256;

// Workgroups over n rows of `width` values (sums: of column sums), at most `cap`;
// more than PRO_BLOCKS: two launches.
static int prologue_blocks(int64_t n, int64_t width, int cap, bool sums = false) {
  if (n > PRO_LARGE_N && n * width >= (sums ? PRO_LARGE_SUMS : PRO_LARGE_VALUES))
    return int(std::min<int64_t>(cap, ceil_div(n, PRO_LARGE_ROWS)));
  return int(std::min<int64_t>(std::min(cap, PRO_BLOCKS),
                               std::max<int64_t>(1, ceil_div(n, PRO_MIN_ROWS))));
}

size_t vscale_floats(int64_t n, int cap) { return 128 + 64 * size_t(prologue_blocks(n, MAX_B, cap)); }

__device__ __forceinline__ bool x_load(const float* X, int64_t e, float& v) {
  v = X[e];
  return isfinite(v);
}
__device__ __forceinline__ bool x_load(const uint16_t* X, int64_t e, float& v) {
  const uint32_t u = X[e];
  v = __uint_as_float(u << 16);
  return (u & 0x7F80u) != 0x7F80u;
}

struct PrologueArgs {
  const void* X;
  const void* X2;
  int64_t n, n2, ldx;
  int D, tcx, nblk, nblk2;
  double* part;
  unsigned long long* r2max;
  int* flags;
  const float* V;
  const float* sr;
  int64_t nv, ldv;
  int b, tcv, nblkv;
  float* vpart;
};

// Rows [blk rpb, (blk + 1) rpb) of X: whether they are finite and, with part,
// their column sums (thread (row lane, column); four rows in flight).
template <typename T>
__device__ __forceinline__ void prologue_points(const T* __restrict__ X, int64_t n, int D,
                                                int64_t ldx, int tc, int nblk, int blk,
                                                double* __restrict__ part, int* __restrict__ flag,
                                                double* red) {
  const int f = int(threadIdx.x) % tc, rl = int(threadIdx.x) / tc, nrl = 256 / tc;
  const int64_t rpb = (n + nblk - 1) / nblk;
  const int64_t r0 = int64_t(blk) * rpb, r1 = min(n, r0 + rpb);
  double acc = 0.0;
  bool ok = true;
  if (f < D) {
    for (int64_t i = r0 + rl; i < r1; i += 4 * nrl) {
      float v[4];
      bool fin[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) fin[u] = x_load(X, min(i + u * nrl, r1 - 1) * ldx + f, v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        ok = ok && fin[u];
        if (i + u * nrl < r1) acc += double(v[u]);
      }
    }
  }
  const int bad = __syncthreads_or(ok ? 0 : 1);
  if (threadIdx.x == 0) *flag = bad;
  if (part == nullptr) return;
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w >= tc; w >>= 1) {
    if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (int(threadIdx.x) < D) part[int64_t(blk) * D + threadIdx.x] = red[threadIdx.x];
}

// Largest |sr_j V[j][c]| per column c over the workgroup's rows.
__device__ __forceinline__ void prologue_vmax(const PrologueArgs& a, int blk, float* red) {
  const int c = int(threadIdx.x) % a.tcv, rl = int(threadIdx.x) / a.tcv, nrl = 256 / a.tcv;
  const int64_t rpb = (a.nv + a.nblkv - 1) / a.nblkv;
  const int64_t r0 = int64_t(blk) * rpb, r1 = min(a.nv, r0 + rpb);
  float m = 0.f, mn = __builtin_inff();
  bool ok = true;
  if (c < a.b) {
    for (int64_t i = r0 + rl; i < r1; i += 4 * nrl) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t r = min(i + u * nrl, r1 - 1);
        v[u] = a.V[r * a.ldv + c];
        if (a.sr != nullptr) v[u] *= a.sr[r];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        m = fmaxf(m, fabsf(v[u]));
        mn = fminf(mn, fabsf(v[u]));
        ok = ok && isfinite(v[u]);
      }
    }
  }
  if (a.b == 1) {
    // one column: also whether it is finite and its smallest value (pack_v_block)
    const int bad = __syncthreads_or(ok ? 0 : 1);
    red[threadIdx.x] = mn;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
      if (int(threadIdx.x) < w) red[threadIdx.x] = fminf(red[threadIdx.x], red[threadIdx.x + w]);
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      a.vpart[blk * 64 + 1] = bad ? 1.f : 0.f;
      a.vpart[blk * 64 + 2] = red[0];
    }
    __syncthreads();
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w >= a.tcv; w >>= 1) {
    if (int(threadIdx.x) < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (int(threadIdx.x) < a.b) a.vpart[blk * 64 + threadIdx.x] = red[threadIdx.x];
}

// The partial results of a large set's prologue added (float64 sums) or compared
// (maxima; with b = 1 the column's flag and its smallest value too) over its
// workgroups, eight columns per workgroup: [0, ceil(D / 8)) of X, then of V.
__global__ __launch_bounds__(256) void prologue_finish_kernel(
    const double* __restrict__ part, int nblk, int D, int nxb, double* __restrict__ sums,
    const float* __restrict__ vpart, int nblkv, int b, float* __restrict__ vmax) {
  __shared__ double red[256];
  const bool points = int(blockIdx.x) < nxb;
  const int c = 8 * (int(blockIdx.x) - (points ? 0 : nxb)) + int(threadIdx.x) % 8;
  const int rl = int(threadIdx.x) / 8;
  const bool least = !points && b == 1 && c == 2;
  double r = least ? double(__builtin_inff()) : 0.0;
  if (points) {
    if (c < D) {
#pragma unroll 8
      for (int k = rl; k < nblk; k += 32) r += part[int64_t(k) * D + c];
    }
  } else if (c < (b == 1 ? 3 : b)) {
#pragma unroll 8
    for (int k = rl; k < nblkv; k += 32) {
      const double v = double(vpart[k * 64 + c]);
      r = least ? fmin(r, v) : fmax(r, v);
    }
  }
  red[threadIdx.x] = r;
  __syncthreads();
  for (int w = 128; w >= 8; w >>= 1) {
    if (int(threadIdx.x) < w) {
      const double o = red[threadIdx.x + w];
      red[threadIdx.x] = points ? red[threadIdx.x] + o
                         : least ? fmin(red[threadIdx.x], o)
                                 : fmax(red[threadIdx.x], o);
    }
    __syncthreads();
  }
  if (threadIdx.x >= 8) return;
  if (points) {
    if (c < D) sums[c] = red[threadIdx.x];
  } else if (c < (b == 1 ? 3 : b)) {
    vmax[c] = float(red[threadIdx.x]);
  }
}

// Workgroups [0, nblk): X; [nblk, nblk + nblk2): X2; the rest: V.
template <typename T>
__global__ __launch_bounds__(256) void prologue_kernel(PrologueArgs a) {
  __shared__ double red[256];
  int blk = int(blockIdx.x);
  if (blk == 0 && threadIdx.x == 0 && a.r2max != nullptr) *a.r2max = 0ull;
  if (blk < a.nblk) {
    prologue_points<T>(static_cast<const T*>(a.X), a.n, a.D, a.ldx, a.tcx, a.nblk, blk, a.part,
                       a.flags + blk, red);
    return;
  }
  blk -= a.nblk;
  if (blk < a.nblk2) {
    prologue_points<T>(static_cast<const T*>(a.X2), a.n2, a.D, a.ldx, a.tcx, a.nblk2, blk, nullptr,
                       a.flags + a.nblk + blk, red);
    return;
  }
  prologue_vmax(a, blk - a.nblk2, reinterpret_cast<float*>(red));
}

CentreWs carve_centre(Arena& a, int64_t n, int64_t n2, int cap) {
  CentreWs c;
  c.nblk = prologue_blocks(n, MAX_D, cap);
  c.nblk2 = n2 > 0 ? prologue_blocks(n2, MAX_D, cap) : 0;
  c.part = a.take<double>((size_t(c.nblk) + 1) * MAX_D);
  c.r2max = a.take<unsigned long long>(1);
  c.flags = a.take<int>(size_t(c.nblk) + size_t(c.nblk2));
  return c;
}

void launch_prologue(const PrologueIn& in, CentreWs& c, FSpan vscale, hipStream_t stream) {
  PrologueArgs a{};
  a.X = in.X;
  a.X2 = in.X2;
  a.n = in.n;
  a.n2 = in.n2;
  a.ldx = in.ldx;
  a.D = int(in.D);
  a.nblk = in.X != nullptr ? prologue_blocks(in.n, in.D, in.cap, in.xt == FD_F32) : 0;
  a.nblk2 = in.X2 != nullptr ? prologue_blocks(in.n2, in.D, in.cap) : 0;
  FD_REQUIRE(a.nblk <= c.nblk && a.nblk2 <= c.nblk2 && in.D <= MAX_D && in.b <= MAX_B,
             FD_ERR_INVALID_ARG, "internal: prologue workspace");
  a.tcx = a.nblk > 0 ? column_lanes(in.D) : 1;
  a.part = in.xt == FD_F32 && a.nblk > 0 ? c.part + MAX_D : nullptr;
  a.r2max = a.nblk > 0 ? c.r2max : nullptr;
  a.flags = c.flags;
  if (in.V != nullptr) {
    check_span(vscale, vscale_floats(in.nv, in.cap), "column scales");
    a.V = in.V;
    a.sr = in.sr;
    a.nv = in.nv;
    a.ldv = in.ldv;
    a.b = int(in.b);
    a.tcv = column_lanes(in.b);
    a.nblkv = prologue_blocks(in.nv, in.b, in.cap);
    a.vpart = vscale.p + 128;
  }
  c.n = in.n;
  c.used = a.nblk;
  c.used2 = a.nblk2;
  const dim3 grid{unsigned(a.nblk + a.nblk2 + a.nblkv)};
  if (in.xt == FD_BF16)
    hipLaunchKernelGGL(prologue_kernel<uint16_t>, grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(prologue_kernel<float>, grid, dim3(256), 0, stream, a);
  FD_LAUNCH_CHECK();
  c.sums = a.part;
  c.nsums = a.nblk;
  const int nxb = a.part != nullptr && a.nblk > PRO_BLOCKS ? int(ceil_div(in.D, 8)) : 0;
  const int nvb = a.nblkv > PRO_BLOCKS ? int(ceil_div(in.b == 1 ? 3 : in.b, 8)) : 0;
  if (nxb + nvb == 0) return;
  hipLaunchKernelGGL(prologue_finish_kernel, dim3(unsigned(nxb + nvb)), dim3(256), 0, stream,
                     a.part, a.nblk, a.D, nxb, c.part, a.vpart, a.nblkv, a.b, vscale.p + 64);
  FD_LAUNCH_CHECK();
  if (nxb > 0) {
    c.sums = c.part;
    c.nsums = 1;
  }
}

// r2max = max_i ||x_i - mu||^2 over X[0:n] (raise_r2max).
__global__ __launch_bounds__(256) void radius_max_kernel(const float* __restrict__ X, int64_t n,
                                                         int D, int64_t ldx,
                                                         const double* __restrict__ part, int nblk,
                                                         unsigned long long* r2max) {
  __shared__ double mu[MAX_D], red[128];
  centre_means(part, nblk, D, n, mu, red);
  double best = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x) {
    double r = 0.0;
    for (int f = 0; f < D; ++f) {
      const double v = double(X[i * ldx + f]) - mu[f];
      r += v * v;
    }
    best = r > best ? r : best;  // a NaN row is skipped; the flag words report it
  }
  raise_r2max(best, r2max);
}

void launch_radius(const void* X, fd_dtype xt, int64_t n, int64_t D, int64_t ldx,
                   const CentreWs& c, hipStream_t stream) {
  if (xt != FD_F32) return;
  FD_REQUIRE(c.n == n && c.nsums > 0, FD_ERR_INVALID_ARG, "internal: radius before the prologue");
  const unsigned grid = unsigned(std::min<int64_t>(1024, std::max<int64_t>(1, ceil_div(n, 256))));
  hipLaunchKernelGGL(radius_max_kernel, dim3(grid), dim3(256), 0, stream,
                     static_cast<const float*>(X), n, int(D), ldx, c.sums, c.nsums, c.r2max);
  FD_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ exponent range

static double coord_scale_sq(double beta) {
  const double s = hx_coord_scale(beta);
  const double f = std::max(s, 2.0 * beta * LOG2E / s);
  return f * f;
}

bool exponent_in_range(fd_dtype xt, double beta, double r2max) {
  return xt != FD_F32 || (beta * LOG2E * r2max <= HX_EXP_RANGE &&
                          coord_scale_sq(beta) * r2max <= HX_PIECE_MAX * HX_PIECE_MAX);
}

double exponent_radius(fd_dtype xt, const CentreWs& c, hipStream_t stream) {
  if (xt != FD_F32) return 0.0;
  unsigned long long bits = 0;
  FD_HIP_CHECK(hipMemcpyAsync(&bits, c.r2max, sizeof(bits), hipMemcpyDeviceToHost, stream));
  FD_HIP_CHECK(hipStreamSynchronize(stream));
  double r2 = 0.0;
  std::memcpy(&r2, &bits, sizeof(r2));
  return r2;
}

void require_exponent_range(fd_dtype xt, const CentreWs& c, double beta, hipStream_t stream) {
  if (xt != FD_F32) return;
  const double r2 = exponent_radius(xt, c, stream);
  if (!exponent_in_range(xt, beta, r2))
    throw Error{FD_ERR_UNSUPPORTED,
                "beta log2(e) max ||x - mean||^2 = " + std::to_string(beta * LOG2E * r2) +
                    " with max ||x - mean|| = " + std::to_string(std::sqrt(r2)) +
                    " is beyond the float32 path's exponent range (offsets up to " +
                    std::to_string(HX_EXP_RANGE) + ", coordinate pieces up to 65504)"};
}

PoisonGate poison_gate(fd_dtype xt, const CentreWs& c, double beta, const int* flag) {
  PoisonGate g;
  g.flag = flag;
  if (xt == FD_F32) {
    g.r2max = c.r2max;
    g.bl = beta * LOG2E;
    g.f2 = coord_scale_sq(beta);
  }
  return g;
}

// ------------------------------------------------------------------ packing

__global__ void pack_w_kernel(const float* __restrict__ w, int64_t n, int64_t ntiles,
                              floatx4* __restrict__ wp) {
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= ntiles * 64) return;
  const int lane = int(idx & 63);
  const int64_t jb = idx >> 6;
  const int g = lane >> 4;
  floatx4 out;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t j = jb * TILE + 4 * g + r;
    out[r] = (j < n) ? w[j] : 0.f;
  }
  wp[idx] = out;
}

// 2^t clamped to [0, 1]: the exponent of a true kernel value is <= 0 and
// rounding can only push it a few ulps above.  The median-of-three with 0 and 1
// folds into the output clamp bit of v_exp_f32 (one instruction).  Written with
// builtins, not inline asm, so the compiler sees the read of the MFMA result
// and inserts the wait states that hazard requires.
__device__ __forceinline__ float exp2_unit(float t) {
  return __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t), 0.f, 1.f);
}

// ------------------------------------------------------------------ split V pack
//
// The K*V contraction runs in float16 with a two-term split of both factors:
//   K' = 2^15 K = Kh + Kl,  V' = 2^e_c sr V = Vh + Vl  (Kh, Kl, Vh, Vl float16),
//   K' V' ~= Kh Vh + Kh Vl + Kl Vh       (the dropped Kl Vl is 2^-22 relative),
// with float32 accumulation; the result is scaled back by 2^(-15 - e_c).  e_c
// puts the largest |V'| of column c just below 2^14; the representation error
// of each split is below 2^-21 relative.  Two consecutive 16-point column tiles
// form the 32-wide contraction; the pack stores, per lane (g, p), the 8 rows
// {4g + r, 16 + 4g + r} of column 16 cb + p as hi and lo halves.

__global__ __launch_bounds__(PACK_THREADS) void pack_v_kernel(PackV a) {
  __shared__ int ex[64];
  pack_v_block(a, a.blk0 + blockIdx.x, ex);
}

// ------------------------------------------------------------------ bfloat16 inputs
//
// For X in bfloat16 the exponent contraction runs on v_mfma_f32_16x16x32_bf16:
// products of bfloat16 values are exact in float32, so the tile
//   C[j][i] = -(r_i + r_j) / 2 + x_j . x_i = -||x_i - x_j||^2 / 2
// is computed on raw (unscaled) bfloat16 operands with float32 accumulation,
// and t = 2 beta log2(e) C is applied afterwards on the vector ALUs.  In the
// K*V contraction K' = 2^15 K is rounded once to the nearest float16 (relative
// error <= 2^-12, well inside the bfloat16-input tolerance) and multiplied by
// the split V (hi + lo): the product is then a fixed matrix applied linearly
// to 2^-22, so an eigensolver built on it can converge to its tolerance.
//
// Pack layout (per 16-point tile and 32-feature chunk c): lane (g, p) holds
// the 8 bfloat16 x[16 tile + p][32 c + 8 g + e], e = 0..7, as one uint4; that
// is the A operand of the column tile and the B operand of the row tile.

// One wave per 16-point tile: lane (g, p) holds eight features of point p per
// chunk, sums their squares in float64 (exact products) and adds the four lanes
// of a point.  Workgroups [0, nbr): the row pack, then the column pack, then V.
struct PackBf16Side {
  const uint16_t* X;
  int64_t n, ntiles;
  uintx4* xp;
  float* ar;      // row side: offsets per point
  floatx4* ap;    // column side: offsets in accumulator order
};
struct PackBf16Args {
  PackBf16Side row, col;
  int64_t ldx, nbr, nbc, blk0;
  int D, dc, vec;
  float pad;  // offset of the padding points
  const int* flags;
  int nflags;
  int* flag;
  PackV v;
  unsigned long long *zero1, *zero2;
  int64_t nzero;
};
__global__ __launch_bounds__(PACK_THREADS) void pack_bf16_kernel(PackBf16Args a) {
  __shared__ int ex[64];
  int64_t blk = a.blk0 + blockIdx.x;
  if (blk == 0 && a.flag != nullptr) pack_flag(a.flags, a.nflags, a.flag);
  if (blk >= a.nbr + a.nbc) {
    pack_v_block(a.v, blk - a.nbr - a.nbc, ex);
    return;
  }
  const bool row_side = blk < a.nbr;
  if (row_side) {
    const int64_t z = blk * PACK_THREADS + threadIdx.x;
    // a workgroup clears 1/nbr of the words
    for (int64_t e = z; e < a.nzero; e += a.nbr * PACK_THREADS) {
      if (a.zero1 != nullptr) a.zero1[e] = 0ull;
      if (a.zero2 != nullptr) a.zero2[e] = 0ull;
    }
  }
  const PackBf16Side s = row_side ? a.row : a.col;
  if (!row_side) blk -= a.nbr;
  const int lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  const int64_t tile = blk * (PACK_THREADS / 64) + (threadIdx.x >> 6);
  if (tile >= s.ntiles) return;
  const int64_t i = tile * TILE + p;
  const bool real = i < s.n;
  const uint16_t* xi = s.X + min(i, s.n - 1) * a.ldx;
  double r = 0.0;
  for (int c = 0; c < a.dc; ++c) {
    const int k0 = 32 * c + 8 * g;
    uintx4 out = uintx4{0u, 0u, 0u, 0u};
    if (a.vec && k0 + 8 <= a.D) {
      out = *reinterpret_cast<const uintx4*>(xi + k0);
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = k0 + 2 * w + h;
          const uint32_t v = uint32_t(xi[min(k, a.D - 1)]);
          out[w] |= (k < a.D ? v : 0u) << (16 * h);
        }
    }
    if (!real) out = uintx4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const double lo = double(__uint_as_float(out[w] << 16));
      const double hi = double(__uint_as_float(out[w] & 0xFFFF0000u));
      r += lo * lo;
      r += hi * hi;
    }
    s.xp[(tile * a.dc + c) * 64 + lane] = out;
  }
  r += __shfl_xor(r, 16);
  r += __shfl_xor(r, 32);
  const float off = real ? float(-0.5 * r) : a.pad;
  if (s.ar != nullptr && g == 0) s.ar[i] = off;
  if (s.ap != nullptr) {
    floatx4 q;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = __shfl(off, 4 * g + e);
    s.ap[tile * 64 + lane] = q;
  }
}


template <int DC, bool DIAG>
__device__ __forceinline__ floatx4 half_sqdist(const uintx4* xa, const floatx4& aj,
                                               const uintx4* xb, float ai, int g, int p) {
  floatx4 t;
#pragma unroll
  for (int r = 0; r < 4; ++r) t[r] = ai + aj[r];
#pragma unroll
  for (int c = 0; c < DC; ++c)
    t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[c]),
                                                __builtin_bit_cast(bf16x8, xb[c]), t, 0, 0, 0);
  if (DIAG) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * g + r == p) t[r] = 0.f;
  }
  return t;
}

template <int DC, int NCB>
struct ColPairB {
  uintx4 xa[2][DC];
  floatx4 aj[2];
  VSplit v[NCB];
};

template <int DC, int NCB>
__device__ __forceinline__ void load_pair_b(ColPairB<DC, NCB>& cp, const uintx4* __restrict__ xa,
                                            const floatx4* __restrict__ aj,
                                            const VSplit* __restrict__ vp, int64_t jp, int lane) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int64_t jb = 2 * jp + t;
#pragma unroll
    for (int c = 0; c < DC; ++c) cp.xa[t][c] = xa[(jb * DC + c) * 64 + lane];
    cp.aj[t] = aj[jb * 64 + lane];
  }
  // unconditional: a branch here would leave the compiler unsure whether the
  // V loads were issued, and its merged load counts would then make every
  // exponent contraction wait for the V loads as well
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) cp.v[cb] = vp[(jp * NCB + cb) * 64 + lane];
}

// Exponents of one pair of column tiles against row tile ib, in accumulator
// layout with the column offsets as the initial accumulator:
//   u_ij = -||x_j||^2 / 2 + x_j . x_i,  K'_ij = 2^(scale2 u_ij + c_i) = 2^15 K_ij,
// with c_i = 15 - scale2 ||x_i||^2 / 2 per row (one FMA per entry).  K' is
// rounded to float16 (nearest, two per instruction) and multiplied into the
// split V on the float16 matrix cores; lane (g, p) holds K'[p][J0 + 4g + r]
// and K'[p][J1 + 4g + r], its A-operand values k = 8g + 4u + r.
template <int DC, bool DIAG>
__device__ __forceinline__ halfx8 bf16_kpair(const uintx4 (&xa)[2][DC], const floatx4 (&aj)[2],
                                             const uintx4 (&xb)[DC], float ci, float scale2,
                                             int64_t jp, int64_t ib, int g, int p) {
  floatx4 t[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    t[u] = aj[u];
#pragma unroll
    for (int cc = 0; cc < DC; ++cc)
      t[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[u][cc]),
                                                     __builtin_bit_cast(bf16x8, xb[cc]), t[u], 0,
                                                     0, 0);
  }
  float e[8];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      e[4 * u + r] = fmaf(t[u][r], scale2, ci);
      // the diagonal of one point set: K'_ii = 2^15 exactly
      if (DIAG && 2 * jp + u == ib && 4 * g + r == p) e[4 * u + r] = 15.f;
    }
  halfx8 k;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const floatx2 kk = floatx2{__builtin_amdgcn_exp2f(e[2 * q]), __builtin_amdgcn_exp2f(e[2 * q + 1])};
    const halfx2 hk = __builtin_convertvector(kk, halfx2);
    k[2 * q] = hk[0];
    k[2 * q + 1] = hk[1];
  }
  return k;
}

template <int NCB>
__device__ __forceinline__ void bf16_kv(const halfx8& k, const VSplit (&v)[NCB],
                                        floatx4 (&acc)[NCB]) {
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k, v[cb].hi, acc[cb], 0, 0, 0);
    acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k, v[cb].lo, acc[cb], 0, 0, 0);
  }
}

template <int DC, int NCB, int NIB, bool DIAG>
__device__ __forceinline__ void bf16_pair(const ColPairB<DC, NCB>& c, const uintx4 (&xbr)[NIB][DC],
                                          const float (&ci)[NIB], float scale2,
                                          floatx4 (&acc)[NIB][NCB], int64_t jp, int64_t ib0,
                                          int g, int p) {
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    const halfx8 k = bf16_kpair<DC, DIAG>(c.xa, c.aj, xbr[ib], ci[ib], scale2, jp, ib0 + ib, g, p);
    bf16_kv<NCB>(k, c.v, acc[ib]);
  }
}

// Waves per SIMD asked of the compiler (at 2 a wave has at most 256
// registers and accumulates in ordinary VGPRs; the widest blocks take 1).
template <int DC, int NCB, int NIB>
constexpr int bf16_waves() {
  constexpr int buffers = NCB >= 3 ? 1 : 2;
  return (NIB * NCB * 4 + NIB * DC * 4 + buffers * (DC * 8 + 8 + NCB * 8) > 200) ? 1 : 2;
}

// One workgroup = 4 waves; wave w owns row tiles [ib0, ib0 + NIB).  Column
// tiles stream in pairs through two operand buffers used in turn (each
// refilled right after its pair is consumed); chunk totals of the two-level
// column sum live in LDS.
template <int DC, int NCB, int NIB>
__global__ __launch_bounds__(WG_THREADS)
__attribute__((amdgpu_waves_per_eu(bf16_waves<DC, NCB, NIB>()))) void product_bf16_kernel(
    const uintx4* __restrict__ xa, const floatx4* __restrict__ aj, const VSplit* __restrict__ vp,
    const uintx4* __restrict__ xb, const float* __restrict__ ar, int64_t nrt, int64_t njp,
    int64_t jp_per_split, int diag, float scale2, const float* __restrict__ colscale,
    const float* __restrict__ sl, float* __restrict__ Y, int64_t ldy, int64_t Nr, int b,
    float* __restrict__ part, int64_t nrpad, PoisonGate poison) {
  __shared__ floatx4 tot[4][NIB][NCB][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t split = wr / nrt;
  const int64_t rt = wr % nrt;
  const int64_t ib0 = (rt * 4 + wave) * NIB;
  const int64_t jp_begin = split * jp_per_split;
  const int64_t jp_end = min(njp, jp_begin + jp_per_split);
  const int g = lane >> 4, p = lane & 15;

  uintx4 xbr[NIB][DC];
  float ci[NIB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
#pragma unroll
    for (int cc = 0; cc < DC; ++cc) xbr[ib][cc] = xb[((ib0 + ib) * DC + cc) * 64 + lane];
    ci[ib] = fmaf(scale2, ar[(ib0 + ib) * TILE + p], 15.f);
  }
  floatx4 acc[NIB][NCB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      acc[ib][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
      tot[wave][ib][cb][lane] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

  if constexpr (NCB >= 3) {
    // Wide blocks: one buffer each for the exponent operands and for V.  A
    // step first forms K' of all the wave's row tiles (then refills the
    // exponent operands), then multiplies them into V (then refills V); each
    // load has the other phase's work to land, and the registers saved by
    // single buffering keep two waves per SIMD.
    ColPairB<DC, NCB> c;
    load_pair_b(c, xa, aj, vp, jp_begin, lane);
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib) {
#pragma unroll
      for (int cc = 0; cc < DC; ++cc) asm volatile("" ::"v"(xbr[ib][cc]));
      asm volatile("" ::"v"(ci[ib]));
    }
    int chunk = 0;
    for (int64_t jp = jp_begin; jp < jp_end; ++jp) {
      const int64_t jn = min(jp + 1, jp_end - 1);
      halfx8 k[NIB];
      if (diag && 2 * jp + 1 >= ib0 && 2 * jp < ib0 + NIB) {
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib)
          k[ib] = bf16_kpair<DC, true>(c.xa, c.aj, xbr[ib], ci[ib], scale2, jp, ib0 + ib, g, p);
      } else {
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib)
          k[ib] = bf16_kpair<DC, false>(c.xa, c.aj, xbr[ib], ci[ib], scale2, jp, ib0 + ib, g, p);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int64_t jb = 2 * jn + t;
#pragma unroll
        for (int cc = 0; cc < DC; ++cc) c.xa[t][cc] = xa[(jb * DC + cc) * 64 + lane];
        c.aj[t] = aj[jb * 64 + lane];
      }
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) bf16_kv<NCB>(k[ib], c.v, acc[ib]);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) c.v[cb] = vp[(jn * NCB + cb) * 64 + lane];
      if (++chunk == CHUNK_TILES / 2) {
        chunk = 0;
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            tot[wave][ib][cb][lane] += acc[ib][cb];
            acc[ib][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  } else {
  auto step = [&](const ColPairB<DC, NCB>& c, int64_t jp) {
    if (diag && 2 * jp + 1 >= ib0 && 2 * jp < ib0 + NIB)
      bf16_pair<DC, NCB, NIB, true>(c, xbr, ci, scale2, acc, jp, ib0, g, p);
    else
      bf16_pair<DC, NCB, NIB, false>(c, xbr, ci, scale2, acc, jp, ib0, g, p);
  };
  ColPairB<DC, NCB> b0, b1;
  load_pair_b(b0, xa, aj, vp, jp_begin, lane);
  __builtin_amdgcn_sched_barrier(0);  // b0's loads ahead of b1's, as in the loop
  load_pair_b(b1, xa, aj, vp, min(jp_begin + 1, jp_end - 1), lane);
  // consume the row operands before the loop (an empty statement reading
  // them): their loads then complete here, and the loop's waits only ever
  // cover the column buffer a step consumes
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
#pragma unroll
    for (int cc = 0; cc < DC; ++cc) asm volatile("" ::"v"(xbr[ib][cc]));
    asm volatile("" ::"v"(ci[ib]));
  }
  int chunk = 0;
  for (int64_t jp = jp_begin; jp < jp_end; jp += 2) {
    step(b0, jp);
    // the refills are unconditional (clamped index): every path reaches the
    // loop top with the same loads in flight
    load_pair_b(b0, xa, aj, vp, min(jp + 2, jp_end - 1), lane);
    if (jp + 1 < jp_end) step(b1, jp + 1);
    load_pair_b(b1, xa, aj, vp, min(jp + 3, jp_end - 1), lane);
    chunk += 2;
    if (chunk >= CHUNK_TILES / 2) {
      chunk = 0;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          tot[wave][ib][cb][lane] += acc[ib][cb];
          acc[ib][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  }

  // read once: between stores to Y the compiler would read the words again for
  // every element (32% of a product of 2^20 rows and 512 columns)
  const bool bad = part == nullptr && poisoned(poison);
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const floatx4 v = tot[wave][ib][cb][lane] + acc[ib][cb];
      const int c = cb * 16 + p;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = (ib0 + ib) * TILE + 4 * g + e;
        if (part != nullptr) {
          part[(split * nrpad + i) * (NCB * 16) + c] = v[e];
        } else if (i < Nr && c < b) {
          const float y = v[e] * colscale[c];
          Y[i * ldy + c] = bad ? __builtin_nanf("") : (sl != nullptr) ? y * sl[i] : y;
        }
      }
    }
}


// Row sums for bfloat16 inputs: the same half squared distances, K = 2^t
// clamped to [0, 1], summed times the weights on the vector ALUs.  Two waves
// per SIMD (every variant fits 256 registers): the matrix instructions then
// accumulate in VGPRs, with no copies out of accumulation registers (bitwise
// equal results, 13-17% faster bfloat16 degree passes at D = 30 and 64).
template <int DC, int NIB>
__global__ __launch_bounds__(WG_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void
rowsum_bf16_kernel(
    const uintx4* __restrict__ xa, const floatx4* __restrict__ aj, const floatx4* __restrict__ wp,
    const uintx4* __restrict__ xb, const float* __restrict__ ar, int64_t nrt, int64_t njb,
    int64_t jb_per_split, int diag, float scale2, float* __restrict__ out, int64_t Nr,
    float* __restrict__ part, int64_t nrpad, HxGate gate) {
  if (hx_gate_closed(gate)) return;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wr = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t split = wr / nrt;
  const int64_t rt = wr % nrt;
  const int64_t ib0 = (rt * 4 + wave) * NIB;
  const int64_t jb_begin = split * jb_per_split;
  const int64_t jb_end = min(njb, jb_begin + jb_per_split);
  const int g = lane >> 4, p = lane & 15;

  uintx4 xbr[NIB][DC];
  float ai[NIB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
#pragma unroll
    for (int c = 0; c < DC; ++c) xbr[ib][c] = xb[((ib0 + ib) * DC + c) * 64 + lane];
    ai[ib] = ar[(ib0 + ib) * TILE + p];
  }
  float acc[NIB], tot[NIB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) acc[ib] = tot[ib] = 0.f;
  int chunk = 0;
  for (int64_t jb = jb_begin; jb < jb_end; ++jb) {
    uintx4 xar[DC];
#pragma unroll
    for (int c = 0; c < DC; ++c) xar[c] = xa[(jb * DC + c) * 64 + lane];
    const floatx4 ajr = aj[jb * 64 + lane];
    const floatx4 w4 = wp[jb * 64 + lane];
    const bool dtile = diag && jb >= ib0 && jb < ib0 + NIB;
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib) {
      floatx4 t;
      if (dtile && jb == ib0 + ib)
        t = half_sqdist<DC, true>(xar, ajr, xbr[ib], ai[ib], g, p);
      else
        t = half_sqdist<DC, false>(xar, ajr, xbr[ib], ai[ib], g, p);
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float k = exp2_unit(t[r] * scale2);
        sum = fmaf(k, w4[r], sum);
      }
      acc[ib] += sum;
    }
    if (++chunk == CHUNK_TILES) {
      chunk = 0;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        tot[ib] += acc[ib];
        acc[ib] = 0.f;
      }
    }
  }
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    float v = tot[ib] + acc[ib];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (g == 0) {
      const int64_t i = (ib0 + ib) * TILE + p;
      if (part != nullptr)
        part[split * nrpad + i] = v;
      else if (i < Nr)
        out[i] = v;
    }
  }
}

// Tile policy of the symmetric row sums (sym_rowsum.hpp).  fd_degree plus a
// 64-column product at N = 131,072, D = 64 takes 10.7 ms with it and 14.1 ms
// with the plain sums (each entry evaluated twice).  The accumulator
// starts at the offsets -r_i / 2 - r_j / 2, as in the plain sums (half_sqdist), and
// K = 2^(scale2 u), clamped to [0, 1]: large offsets of near points cancel
// before anything is scaled, so that points that coincide give K = 1 where the
// sums are exact (scaled on its own, a row offset loses 2^-25 of 2 beta r^2).
template <int DC>
struct Bf16Tile {
  static constexpr float ONE = 1.f;
  static constexpr int NM = DC, EXTRA = 3;
  struct Args {
    const uintx4* xa;
    const floatx4* aj;
    const uintx4* xb;
    const float* ar;
    float scale2;
  };
  struct Row {
    uintx4 b[DC];
    float off;
  };
  struct Col {
    uintx4 a[DC];
    floatx4 off;
  };
  template <int NIB, bool SQ>
  static constexpr int waves() {
    return 2;
  }
  static __device__ __forceinline__ void load_row(Row& r, const Args& a, int64_t tile, int lane) {
#pragma unroll
    for (int c = 0; c < DC; ++c) r.b[c] = a.xb[(tile * DC + c) * 64 + lane];
    r.off = a.ar[tile * TILE + (lane & 15)];
  }
  static __device__ __forceinline__ void load_col(Col& c, const Args& a, int64_t tile, int lane) {
#pragma unroll
    for (int k = 0; k < DC; ++k) c.a[k] = a.xa[(tile * DC + k) * 64 + lane];
    c.off = a.aj[tile * 64 + lane];
  }
  static __device__ __forceinline__ void consume(const Row& r) {
#pragma unroll
    for (int c = 0; c < DC; ++c) asm volatile("" ::"v"(r.b[c]));
    asm volatile("" ::"v"(r.off));
  }
  static __device__ __forceinline__ floatx4 tile(const Col& c, const Row& r) {
    floatx4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = r.off + c.off[e];
#pragma unroll
    for (int k = 0; k < DC; ++k)
      t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, c.a[k]),
                                                  __builtin_bit_cast(bf16x8, r.b[k]), t, 0, 0, 0);
    return t;
  }
  static __device__ __forceinline__ float value(float t, const Row&, const Args& a) {
    return exp2_unit(t * a.scale2);
  }
};

// One column on one point set: Y_i = sl_i 2^e (row partials + fixed-point column
// sums in two words), which are left cleared; where the column could not be
// taken so (bad != 0) from the plain row sums' partials instead.
__global__ __launch_bounds__(256) void column_finish_kernel(
    const float* __restrict__ part, int nsplit_plain, int nsplit_sym, int64_t nrpad,
    unsigned long long* __restrict__ colfix, unsigned long long* __restrict__ colfix_lo,
    const float* __restrict__ colscale, const float* __restrict__ sl, int64_t n, int64_t npad,
    float* __restrict__ Y, int64_t ldy, PoisonGate poison) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const bool sym = colfix != nullptr && colscale[1] == 0.f;
  if (i < n) {
    const int ns = sym ? nsplit_sym : nsplit_plain;
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < ns; ++k) s += double(part[k * nrpad + i]);
    if (sym)
      s += (double(static_cast<long long>(colfix[i])) * (1ull << WIDE_SPLIT) +
            double(colfix_lo[i])) *
           (1.0 / double(1ull << WIDE_FRAC));
    float y = float(ldexp(s, int(colscale[0])));
    if (sl != nullptr) y = sl[i] * y;
    Y[i * ldy] = poisoned(poison) ? __builtin_nanf("") : y;
  }
  if (colfix != nullptr && i < npad) colfix[i] = colfix_lo[i] = 0ull;
}

// Y = diag(sl) (sum over splits of part) diag(colscale), NaN where the call is
// poisoned.  A thread sums four consecutive columns of a row over every
// TEAMS-th split (float64, one 16-byte load per split); the teams are added in
// LDS in a fixed order.  Small outputs take more teams: a chain of up to 64
// dependent loads per thread is what their time was (6-12 us below 2^13 rows).
template <int TEAMS>
__global__ __launch_bounds__(256) void reduce_product_kernel(
    const float* __restrict__ part, int nsplit, int64_t nrpad, int width,
    const float* __restrict__ colscale, const float* __restrict__ sl, float* __restrict__ Y,
    int64_t ldy, int64_t Nr, int b, int vec, PoisonGate poison) {
  constexpr int OUT = 256 / TEAMS;
  __shared__ double red[TEAMS > 1 ? TEAMS : 1][TEAMS > 1 ? OUT : 1][4];
  const int o = int(threadIdx.x) % OUT, team = int(threadIdx.x) / OUT;
  const int quads = (b + 3) / 4;
  const int64_t idx = int64_t(blockIdx.x) * OUT + o;
  const bool live = idx < Nr * quads;
  const int64_t i = live ? idx / quads : 0;
  const int c = live ? 4 * int(idx % quads) : 0;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  const float* src = part + i * width + c;
#pragma unroll 4
  for (int k = team; k < nsplit; k += TEAMS) {
    const floatx4 v = *reinterpret_cast<const floatx4*>(src + int64_t(k) * nrpad * width);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += double(v[e]);
  }
  if constexpr (TEAMS > 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) red[team][o][e] = s[e];
    __syncthreads();
    if (team != 0) return;
#pragma unroll
    for (int k = 1; k < TEAMS; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += red[k][o][e];
  }
  if (!live) return;
  const bool bad = poisoned(poison);
  floatx4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    double v = s[e] * double(colscale[min(c + e, b - 1)]);
    if (sl != nullptr) v *= double(sl[i]);
    out[e] = bad ? __builtin_nanf("") : float(v);
  }
  if (vec && c + 4 <= b) {
    *reinterpret_cast<floatx4*>(Y + i * ldy + c) = out;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (c + e < b) Y[i * ldy + c + e] = out[e];
}

__global__ void reduce_rowsum_kernel(const float* __restrict__ part, int nsplit, int64_t nrpad,
                                     float* __restrict__ out, int64_t Nr) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= Nr) return;
  double s = 0.0;
  for (int k = 0; k < nsplit; ++k) s += double(part[k * nrpad + i]);
  out[i] = float(s);
}

// Sum of v over the workgroup of 256 threads (fixed order); on thread 0.
__device__ __forceinline__ double block_sum_256(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double s = red[0];
  __syncthreads();
  return s;
}

// s_off = sum(q) - n from the partial sums of q (one workgroup of 256, fixed
// order).
__device__ __forceinline__ void finish_s_off(const double* __restrict__ qsum, int64_t nq,
                                             int64_t n, double* __restrict__ s_off, bool bad,
                                             double* red) {
  double v = 0.0;
#pragma unroll 4
  for (int64_t k = threadIdx.x; k < nq; k += 256) v += qsum[k];
  v = block_sum_256(v, red);
  if (threadIdx.x == 0) *s_off = bad ? __builtin_nan("") : v - double(n);
}

// w = q^-alpha
__global__ void pow_neg_kernel(const float* __restrict__ q, int64_t n, double alpha,
                               float* __restrict__ w) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) w[i] = float(pow(double(q[i]), -alpha));
}

// d = w * t, s = w * d^-1/2 (w = q^-alpha recomputed in double from q)
__global__ __launch_bounds__(256) void degree_finish_kernel(
    const float* __restrict__ q, const float* __restrict__ t, int64_t n, double alpha,
    float* __restrict__ d, float* __restrict__ s, const double* __restrict__ qsum, int64_t nq,
    double* __restrict__ s_off, PoisonGate poison) {
  __shared__ double red[256];
  const bool bad = poisoned(poison);
  if (blockIdx.x == 0 && s_off != nullptr) finish_s_off(qsum, nq, n, s_off, bad, red);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double w = pow(double(q[i]), -alpha);
  const double dd = w * double(t[i]);
  if (d != nullptr) d[i] = bad ? __builtin_nanf("") : float(dd);
  if (s != nullptr) s[i] = bad ? __builtin_nanf("") : float(w / sqrt(dd));
}

// The two normalisation passes on the symmetric path with their epilogues in
// the reductions.  One thread per padded point; each clears its fixed-point
// column sum for the next pass.

// Row sum of point i: the split partials, then the fixed-point column sum.
__device__ __forceinline__ double sym_row_total(const float* __restrict__ part, int nsplit,
                                                int64_t nrpad, unsigned long long col,
                                                double inv_fix, int64_t i) {
  double sum = 0.0;
#pragma unroll 8
  for (int k = 0; k < nsplit; ++k) sum += double(part[k * nrpad + i]);
  return sum + double(static_cast<long long>(col)) * inv_fix;
}

// w_j into the weight pack (pack_w_kernel's layout: w_j in lanes 16 g + p,
// p = 0..15, component r of tile j / 16, j % 16 = 4 g + r).
__device__ __forceinline__ void put_weight(float* __restrict__ wpk, int64_t i, float w) {
  const int64_t jb = i / TILE;
  const int jj = int(i % TILE), g = jj / 4, r = jj % 4;
  float* base = wpk + (jb * 64 + 16 * g) * 4 + r;
#pragma unroll
  for (int p = 0; p < 16; ++p) base[4 * p] = w;
}

// Pass 1: q_i, and if wpk is set w_i = q_i^-alpha written to the weight pack
// (0 for padding points) for the wnpad points of the column pack.  qsum: the
// workgroup's sum of q.
__global__ __launch_bounds__(256) void degree_reduce_q_kernel(
    const float* __restrict__ part, int nsplit, int64_t nrpad,
    unsigned long long* __restrict__ colfix, double inv_fix, float* __restrict__ q, int64_t n,
    int64_t npad, double alpha, float* __restrict__ wpk, int64_t wnpad, double* __restrict__ qsum,
    PoisonGate poison) {
  __shared__ double red[256];
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  float qi = 0.f, w = 0.f;
  if (i < n) {
    qi = float(sym_row_total(part, nsplit, nrpad, colfix[i], inv_fix, i));
    w = float(pow(double(qi), -alpha));
    q[i] = poisoned(poison) ? __builtin_nanf("") : qi;
  }
  if (i < npad) colfix[i] = 0ull;
  if (wpk != nullptr && i < wnpad) put_weight(wpk, i, w);
  const double s = block_sum_256(double(qi), red);
  if (threadIdx.x == 0) qsum[blockIdx.x] = s;
}

// Pass 2: t_i (the weighted row sums), then d_i = w_i t_i and
// s_i = w_i d_i^-1/2 with w_i = q_i^-alpha in double.  The first workgroup also
// finishes s_off.
__global__ __launch_bounds__(256) void degree_reduce_ds_kernel(
    const float* __restrict__ part, int nsplit, int64_t nrpad,
    unsigned long long* __restrict__ colfix, double inv_fix, const float* __restrict__ q,
    int64_t n, int64_t npad, double alpha, float* __restrict__ d, float* __restrict__ s,
    const double* __restrict__ qsum, int64_t nq, double* __restrict__ s_off, PoisonGate poison) {
  __shared__ double red[256];
  const bool bad = poisoned(poison);
  if (blockIdx.x == 0 && s_off != nullptr) finish_s_off(qsum, nq, n, s_off, bad, red);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= npad) return;
  if (i < n) {
    const float ti = float(sym_row_total(part, nsplit, nrpad, colfix[i], inv_fix, i));
    const double w = pow(double(q[i]), -alpha);
    const double dd = w * double(ti);
    if (d != nullptr) d[i] = bad ? __builtin_nanf("") : float(dd);
    if (s != nullptr) s[i] = bad ? __builtin_nanf("") : float(w / sqrt(dd));
  }
  colfix[i] = 0ull;
}

// Pass 2 of a dyadic level: degree_reduce_ds_kernel's outputs, and from the
// squared-kernel sums of the same pass the next level's q (K(2 beta) 1, the
// reduction in the same order as degree_reduce_q_kernel's) with its
// w = q^-alpha written to the weight pack as degree_reduce_q_kernel writes it.
__global__ __launch_bounds__(256) void degree_reduce_dsq_kernel(
    const float* __restrict__ part, int nsplit, int64_t nrpad,
    unsigned long long* __restrict__ colfix, double inv_fix, const float* __restrict__ q,
    int64_t n, int64_t npad, double alpha, float* __restrict__ d, float* __restrict__ s,
    const float* __restrict__ part2, unsigned long long* __restrict__ colfix2,
    float* __restrict__ q_next, float* __restrict__ wpk, int64_t wnpad,
    const double* __restrict__ qsum, int64_t nq, double* __restrict__ s_off,
    double* __restrict__ qsum_next, PoisonGate poison) {
  __shared__ double red[256];
  const bool bad = poisoned(poison);
  if (blockIdx.x == 0 && s_off != nullptr) finish_s_off(qsum, nq, n, s_off, bad, red);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  float qn = 0.f, wn = 0.f;
  if (i < n) {
    const float ti = float(sym_row_total(part, nsplit, nrpad, colfix[i], inv_fix, i));
    const double w = pow(double(q[i]), -alpha);
    const double dd = w * double(ti);
    if (d != nullptr) d[i] = bad ? __builtin_nanf("") : float(dd);
    if (s != nullptr) s[i] = bad ? __builtin_nanf("") : float(w / sqrt(dd));
    qn = float(sym_row_total(part2, nsplit, nrpad, colfix2[i], inv_fix, i));
    q_next[i] = bad ? __builtin_nanf("") : qn;
    wn = float(pow(double(qn), -alpha));
  }
  if (i < npad) {
    colfix[i] = 0ull;
    colfix2[i] = 0ull;
  }
  if (i < wnpad) put_weight(wpk, i, wn);
  const double sq = block_sum_256(double(qn), red);
  if (threadIdx.x == 0) qsum_next[blockIdx.x] = sq;
}

int64_t qsum_words(int64_t npad) { return ceil_div(npad, 256); }

// ------------------------------------------------------------------ host side

static inline size_t lane4_extent(int64_t tiles, int groups) {
  return size_t(tiles) * groups * 64 * 4;
}

static PackBf16Side bf16_side(const void* X, PointPack& out, int dc, bool row_side) {
  FD_REQUIRE(out.npad % TILE == 0 && out.npad >= out.n && dc <= 2, FD_ERR_INVALID_ARG,
             "internal: bad bf16 pack geometry");
  const int64_t ntiles = out.npad / TILE;
  check_span(out.xp, size_t(ntiles) * dc * 64 * 4, "bf16 point pack");
  if (row_side) check_span(out.ar, size_t(out.npad), "row offsets");
  else check_span(out.ap, lane4_extent(ntiles, 1), "column offsets");
  out.bf16 = true;
  out.dc = dc;
  out.rid = -1;
  out.rid2 = -1;
  out.variant = 0;
  out.row_side = row_side;
  return PackBf16Side{static_cast<const uint16_t*>(X), out.n, ntiles,
                      reinterpret_cast<uintx4*>(out.xp.p), row_side ? out.ar.p : nullptr,
                      row_side ? nullptr : reinterpret_cast<floatx4*>(out.ap.p)};
}

static void launch_packs_bf16(const PackIn& in, const PackV& v, PointPack& rows, PointPack& cols,
                              const CentreWs& centre, hipStream_t stream) {
  PackBf16Args a{};
  const int dc = int(ceil_div(in.D, 32));
  a.row = bf16_side(in.Xr, rows, dc, true);
  a.col = bf16_side(in.Xc, cols, dc, false);
  a.ldx = in.ldx;
  a.D = int(in.D);
  a.dc = dc;
  // eight features at a time where every row starts on 16 bytes
  a.vec = in.ldx % 8 == 0 && reinterpret_cast<uintptr_t>(in.Xr) % 16 == 0 &&
          reinterpret_cast<uintptr_t>(in.Xc) % 16 == 0;
  // padding points: an infinite offset makes their kernel values 0 at any
  // bandwidth (a finite one, -1e30, was too near below beta = 5e-29); at
  // beta = 0, where only products go, it is finite (0 times it is 0) and their
  // rows of V are 0
  a.pad = in.beta > 0.0 ? -__builtin_inff() : -1e30f;
  constexpr int TPB = PACK_THREADS / 64;
  a.nbr = ceil_div(a.row.ntiles, TPB);
  a.nbc = ceil_div(a.col.ntiles, TPB);
  a.flags = centre.flags;
  a.nflags = centre.used + centre.used2;
  a.flag = in.flag;
  a.v = v;
  a.zero1 = in.zero1;
  a.zero2 = in.zero2;
  a.nzero = in.nzero;
  launch_pack_blocks(pack_bf16_kernel,
                     a.nbr + a.nbc + ceil_div(pack_v_items(v), PACK_THREADS), a, stream);
}

// The V part of a pack: the split pack of V[0:n, 0:b] (ncb > 0) or the weight
// pack of its one column (ncb = 0) for a column side of npad points.
static PackV pack_v_args(const float* V, int64_t n, int64_t b, int64_t ldv, const float* sr,
                         int ncb, int64_t npad, FSpan vp, FSpan vscale, int cap, bool scaled) {
  PackV v;
  if (V == nullptr) return v;
  check_span(vscale, vscale_floats(n, cap), "column scales");
  v.colscale = vscale.p;
  // the finished maxima, or the prologue's partial ones
  const int nblk = prologue_blocks(n, b, cap);
  const bool finished = nblk > PRO_BLOCKS;
  v.nvmax = finished ? 1 : nblk;
  v.vpart = vscale.p + (finished ? 64 : 128);
  v.V = V;
  v.sr = sr;
  v.n = n;
  v.ldv = ldv;
  v.b = int(b);
  v.ncb = ncb;
  if (!scaled) v.nvmax = 0;
  FD_REQUIRE(scaled || ncb == 0, FD_ERR_INVALID_ARG, "internal: split V pack without maxima");
  if (ncb == 0) {
    FD_REQUIRE(npad % TILE == 0 && npad >= n && b == 1, FD_ERR_INVALID_ARG,
               "internal: bad w pack geometry");
    v.ntiles = npad / TILE;
    check_span(vp, lane4_extent(v.ntiles, 1), "weight pack");
    v.wp = reinterpret_cast<floatx4*>(vp.p);
    v.range = column_range(round_up(n, ROW_PAD));
    return v;
  }
  FD_REQUIRE(npad % (2 * TILE) == 0 && npad >= n && b <= ncb * 16 && b <= 64, FD_ERR_INVALID_ARG, "internal: bad split V pack geometry");
  v.npairs = npad / (2 * TILE);
  // one VSplit (32 bytes = 8 floats) per lane per pair per column block
  check_span(vp, size_t(v.npairs) * ncb * 64 * 8, "split V pack");
  v.vp = reinterpret_cast<VSplit*>(vp.p);
  return v;
}

void launch_packs(const PackIn& in, PointPack& rows, PointPack& cols, const CentreWs& centre,
                  hipStream_t stream) {
  rows.beta = cols.beta = in.beta;
  const PackV v = pack_v_args(in.V, cols.n, in.b, in.ldv, in.sr, in.ncb, cols.npad, in.vp,
                              in.vscale, in.cap, in.scaled);
  if (in.xt == FD_BF16) {
    launch_packs_bf16(in, v, rows, cols, centre, stream);
    return;
  }
  rows.bf16 = cols.bf16 = false;
  rows.dc = cols.dc = 0;
  FD_REQUIRE(rows.dp == cols.dp && rows.dp % 4 == 0 && in.D <= rows.dp, FD_ERR_INVALID_ARG,
             "internal: bad point pack geometry");
  launch_packs_hx(in, v, rows, cols, centre, stream);
}

void launch_pack_w(const float* w, int64_t n, int64_t npad, FSpan wp, hipStream_t stream) {
  FD_REQUIRE(npad % TILE == 0 && npad >= n, FD_ERR_INVALID_ARG, "internal: bad w pack geometry");
  const int64_t ntiles = npad / TILE;
  check_span(wp, lane4_extent(ntiles, 1), "weight pack");
  hipLaunchKernelGGL(pack_w_kernel, dim3(blocks_for(ntiles * 64, 256)), dim3(256), 0, stream, w,
                     n, ntiles, reinterpret_cast<floatx4*>(wp.p));
  FD_LAUNCH_CHECK();
}

// Geometry shared by the product and row-sum launches.
static void check_tiles(const KVPlan& p, const PointPack& rows, const PointPack& cols) {
  const int64_t row_tiles = p.nrt * 4 * p.nib;  // 16-row tiles the grid reads
  FD_REQUIRE(rows.dp == p.dp && cols.dp == p.dp, FD_ERR_INVALID_ARG, "internal: pack width");
  FD_REQUIRE(row_tiles * TILE == rows.npad, FD_ERR_INVALID_ARG,
             "internal: row pack not padded to the workgroup tile");
  FD_REQUIRE(p.njb * TILE <= cols.npad && cols.n <= p.njb * TILE, FD_ERR_INVALID_ARG,
             "internal: column pack does not match the plan");
  FD_REQUIRE(p.nsplit >= 1 && (p.nsplit - 1) * p.jb_per_split < p.njb &&
                 p.nsplit * p.jb_per_split >= p.njb,
             FD_ERR_INVALID_ARG, "internal: bad column split");
  if (rows.bf16) {
    check_span(rows.xp, size_t(row_tiles) * rows.dc * 64 * 4, "bf16 row pack");
    check_span(cols.xp, size_t(round_up(p.njb, 2)) * cols.dc * 64 * 4, "bf16 column pack");
    check_span(rows.ar, size_t(rows.npad), "row offsets");
    check_span(cols.ap, lane4_extent(round_up(p.njb, 2), 1), "column offsets");
  }
}

void launch_pack_v_split(const float* V, int64_t n, int64_t b, int64_t ldv, const float* sr,
                         int ncb, int64_t npad, FSpan vp, FSpan vscale, hipStream_t stream,
                         bool scaled) {
  if (scaled) {
    PrologueIn in;
    in.V = V;
    in.nv = n;
    in.b = b;
    in.ldv = ldv;
    in.sr = sr;
    CentreWs none;
    launch_prologue(in, none, vscale, stream);
  }
  const PackV v = pack_v_args(V, n, b, ldv, sr, ncb, npad, vp, vscale, PROLOGUE_CAP, scaled);
  launch_pack_blocks(pack_v_kernel, ceil_div(pack_v_items(v), PACK_THREADS), v, stream);
}

template <int DC, int NCB, int NIB>
static void product_bf16_nib(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                             const float* vp, const float* colscale, bool diag, const float* sl,
                             float* Y, int64_t ldy, int b, float* part,
                             const PoisonGate& poison, hipStream_t stream) {
  const unsigned grid = unsigned(p.nrt * p.nsplit);
  const float scale2 = float(2.0 * rows.beta * LOG2E);
  ProfScope prof(FD_KERNEL_PRODUCT, stream);
  hipLaunchKernelGGL((product_bf16_kernel<DC, NCB, NIB>), dim3(grid), dim3(WG_THREADS), 0, stream,
                     reinterpret_cast<const uintx4*>(cols.xp.p),
                     reinterpret_cast<const floatx4*>(cols.ap.p),
                     reinterpret_cast<const VSplit*>(vp),
                     reinterpret_cast<const uintx4*>(rows.xp.p), rows.ar.p, p.nrt,
                     ceil_div(p.njb, 2), p.jb_per_split / 2, int(diag), scale2, colscale, sl, Y,
                     ldy, rows.n, b, part, rows.npad, poison);
  FD_LAUNCH_CHECK();
}

template <int DC, int NCB>
static void product_bf16_launch(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                                const float* vp, const float* cs, bool diag, const float* sl,
                                float* Y, int64_t ldy, int b, float* part,
                             const PoisonGate& poison, hipStream_t stream) {
  // eight row tiles per wave only for the shapes plan_product gives them to
  if constexpr (DC == 1 && NCB == 1) {
    if (p.nib == 8)
      return product_bf16_nib<DC, NCB, 8>(p, rows, cols, vp, cs, diag, sl, Y, ldy, b, part,
                                          poison, stream);
  }
  FD_REQUIRE(p.nib == 4, FD_ERR_INVALID_ARG, "internal: bf16 rows per wave");
  product_bf16_nib<DC, NCB, 4>(p, rows, cols, vp, cs, diag, sl, Y, ldy, b, part, poison, stream);
}

template <int DC>
static void product_bf16_ncb(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                             const float* vp, const float* cs, bool diag, const float* sl,
                             float* Y, int64_t ldy, int b, float* part,
                             const PoisonGate& poison, hipStream_t stream) {
  switch (p.ncb) {
    case 1: return product_bf16_launch<DC, 1>(p, rows, cols, vp, cs, diag, sl, Y, ldy, b, part, poison, stream);
    case 2: return product_bf16_launch<DC, 2>(p, rows, cols, vp, cs, diag, sl, Y, ldy, b, part, poison, stream);
    case 3: return product_bf16_launch<DC, 3>(p, rows, cols, vp, cs, diag, sl, Y, ldy, b, part, poison, stream);
    case 4: return product_bf16_launch<DC, 4>(p, rows, cols, vp, cs, diag, sl, Y, ldy, b, part, poison, stream);
  }
  throw Error{FD_ERR_UNSUPPORTED, "block width above 64"};
}

void launch_product(const KVPlan& p, const PointPack& rows, const PointPack& cols, FSpan vp,
                    FSpan vscale, bool diag, const float* sl, float* Y, int64_t ldy, int b,
                    FSpan part, const PoisonGate& poison, hipStream_t stream) {
  check_tiles(p, rows, cols);
  FD_REQUIRE(b >= 1 && b <= p.ncb * 16 && (p.nib == 4 || p.nib == 8),
             FD_ERR_INVALID_ARG, "internal: block width does not match the plan");
  FD_REQUIRE(p.jb_per_split % 2 == 0 && round_up(p.njb, 2) * TILE <= cols.npad,
             FD_ERR_INVALID_ARG, "internal: column pairs do not fit the pack");
  check_span(vscale, 64, "column scales");
  const float* cs = vscale.p;
  float* pp = nullptr;
  if (p.nsplit > 1) {
    check_span(part, size_t(p.nsplit) * rows.npad * p.ncb * 16, "partial products");
    pp = part.p;
  }
  if (rows.bf16 || cols.bf16) {
    FD_REQUIRE(rows.bf16 && cols.bf16 && rows.dc == cols.dc, FD_ERR_INVALID_ARG,
               "internal: mixed pack kinds");
    check_span(vp, size_t(ceil_div(p.njb, 2)) * p.ncb * 64 * 8, "split V pack");
    if (rows.dc == 1)
      product_bf16_ncb<1>(p, rows, cols, vp.p, cs, diag, sl, Y, ldy, b, pp, poison, stream);
    else
      product_bf16_ncb<2>(p, rows, cols, vp.p, cs, diag, sl, Y, ldy, b, pp, poison, stream);
  } else {
    check_span(vp, size_t(ceil_div(p.njb, 2)) * p.ncb * 64 * 8, "split V pack");
    launch_product_hx(p, rows, cols, vp.p, cs, diag, sl, Y, ldy, b, pp, poison, stream);
  }
  if (p.nsplit > 1) {
    // eight or four teams of threads share an output's splits where one thread
    // per output would leave most of the chip idle (N = 2,048, b = 8, 16 splits:
    // 6.0 -> 4.0 us); from 2^18 threads' worth of outputs one is as fast
    const int64_t total = rows.n * ceil_div(b, 4);
    const int teams = total < (int64_t(1) << 16) && p.nsplit >= 16  ? 8
                      : total < (int64_t(1) << 18) && p.nsplit >= 8 ? 4
                                                                     : 1;
    const int vec = ldy % 4 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(blocks_for(total * teams, 256)), dim3(256), 0, stream, pp,
                         p.nsplit, rows.npad, p.ncb * 16, cs, sl, Y, ldy, rows.n, b, vec, poison);
    };
    if (teams == 8) go(reduce_product_kernel<8>);
    else if (teams == 4) go(reduce_product_kernel<4>);
    else go(reduce_product_kernel<1>);
    FD_LAUNCH_CHECK();
  }
}

template <int DC>
static void rowsum_bf16_launch(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                               const float* wp, bool diag, float* out, float* part,
                               hipStream_t stream) {
  const unsigned grid = unsigned(p.nrt * p.nsplit);
  const float scale2 = float(2.0 * rows.beta * LOG2E);
  ProfScope prof(FD_KERNEL_ROWSUM, stream);
  hipLaunchKernelGGL((rowsum_bf16_kernel<DC, 8>), dim3(grid), dim3(WG_THREADS), 0, stream,
                     reinterpret_cast<const uintx4*>(cols.xp.p),
                     reinterpret_cast<const floatx4*>(cols.ap.p),
                     reinterpret_cast<const floatx4*>(wp),
                     reinterpret_cast<const uintx4*>(rows.xp.p), rows.ar.p, p.nrt, p.njb,
                     p.jb_per_split, int(diag), scale2, out, rows.n, part, rows.npad, gate_of(rows));
  FD_LAUNCH_CHECK();
}

bool column_sym_applies(const PointPack& rows, const PointPack& cols, bool diag,
                        const unsigned long long* colfix) {
  return rowsum_sym_applies(rows, cols, diag, colfix) && rows.n >= COLUMN_SYM_POINTS;
}

bool rowsum_sym_applies(const PointPack& rows, const PointPack& cols, bool diag,
                        const unsigned long long* colfix) {
  return colfix != nullptr && diag && rows.bf16 == cols.bf16 && rows.n == cols.n;
}

template <int DC, bool UNIT, bool TWO = false>
static void rowsum_sym_bf16(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                            const float* wp, float* part, const ColumnWords& col,
                            hipStream_t stream) {
  using T = Bf16Tile<DC>;
  const typename T::Args ta{reinterpret_cast<const uintx4*>(cols.xp.p),
                            reinterpret_cast<const floatx4*>(cols.ap.p),
                            reinterpret_cast<const uintx4*>(rows.xp.p), rows.ar.p,
                            float(2.0 * rows.beta * LOG2E)};
  ProfScope prof(FD_KERNEL_ROWSUM, stream);
  hipLaunchKernelGGL((rowsum_sym_kernel<T, 8, UNIT, false, TWO>), dim3(unsigned(p.nrt * p.nsplit)),
                     dim3(WG_THREADS), 0, stream, ta, reinterpret_cast<const floatx4*>(wp), p.nrt,
                     p.njb, p.jb_per_split, int64_t(p.nsplit), part, rows.npad, col.hi, col.lo,
                     std::ldexp(1.0, col.frac), nullptr, nullptr, 0.0, gate_of(rows));
  FD_LAUNCH_CHECK();
}

SymPass launch_rowsum_sym_pass(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                               FSpan wp, FSpan part, unsigned long long* colfix, hipStream_t stream,
                               FSpan sq_part, unsigned long long* sq_colfix,
                               unsigned long long* colfix_lo) {
  check_tiles(p, rows, cols);
  FD_REQUIRE(rowsum_sym_applies(rows, cols, true, colfix), FD_ERR_INVALID_ARG,
             "internal: symmetric row sums need one point set");
  const KVPlan sp = plan_rowsum_sym(rows.n, rows.npad, p.dp, SYM_NIB);
  if (wp.p != nullptr) check_span(wp, lane4_extent(sp.njb, 1), "weight pack");
  check_span(part, size_t(sp.nsplit) * rows.npad, "partial row sums");
  // fixed point with F fractional bits: the total of weights in [-1, 1] over
  // npad columns stays below 2^62 / 4 (and so does that of K^2 <= 1); two words
  // have no total to leave room for
  FD_REQUIRE(colfix_lo == nullptr || (wp.p != nullptr && sq_part.p == nullptr),
             FD_ERR_INVALID_ARG, "internal: column words");
  const int F = colfix_lo != nullptr ? WIDE_FRAC
                                     : 62 - int(std::ceil(std::log2(double(rows.npad)))) - 2;
  const ColumnWords col{colfix, colfix_lo, F};
  SymSquares sq;
  if (sq_part.p != nullptr) {
    FD_REQUIRE(wp.p != nullptr && sq_colfix != nullptr, FD_ERR_INVALID_ARG,
               "internal: squared sums ride on a weighted pass");
    check_span(sq_part, size_t(sp.nsplit) * rows.npad, "partial squared row sums");
    sq = SymSquares{sq_part.p, sq_colfix};
  }
  if (rows.bf16) {
    FD_REQUIRE(rows.dc == cols.dc && sq.part == nullptr && sp.nrt * 4 * sp.nib * TILE == rows.npad, FD_ERR_INVALID_ARG,
               "internal: symmetric row-sum plan");
    const bool unit = wp.p == nullptr, two = colfix_lo != nullptr;
    if (rows.dc == 1)
      unit  ? rowsum_sym_bf16<1, true>(sp, rows, cols, wp.p, part.p, col, stream)
      : two ? rowsum_sym_bf16<1, false, true>(sp, rows, cols, wp.p, part.p, col, stream)
            : rowsum_sym_bf16<1, false>(sp, rows, cols, wp.p, part.p, col, stream);
    else
      unit  ? rowsum_sym_bf16<2, true>(sp, rows, cols, wp.p, part.p, col, stream)
      : two ? rowsum_sym_bf16<2, false, true>(sp, rows, cols, wp.p, part.p, col, stream)
            : rowsum_sym_bf16<2, false>(sp, rows, cols, wp.p, part.p, col, stream);
  } else {
    launch_rowsum_sym_hx(sp, rows, cols, wp.p, part.p, col, sq, stream);
  }
  return SymPass{int(sp.nsplit), std::ldexp(1.0, -F)};
}

void launch_degree_reduce_q(const SymPass& sp, const PointPack& rows, const PointPack& cols,
                            FSpan part, unsigned long long* colfix, float* q, double alpha,
                            FSpan wp, double* qsum, const PoisonGate& poison, hipStream_t stream) {
  FD_REQUIRE(cols.npad % TILE == 0 && cols.npad <= rows.npad && cols.n == rows.n,
             FD_ERR_INVALID_ARG, "internal: bad weight pack geometry");
  if (wp.p != nullptr) check_span(wp, lane4_extent(cols.npad / TILE, 1), "weight pack");
  hipLaunchKernelGGL(degree_reduce_q_kernel, dim3(blocks_for(rows.npad, 256)), dim3(256), 0,
                     stream, part.p, sp.nsplit, rows.npad, colfix, sp.inv_fix, q, rows.n,
                     rows.npad, alpha, wp.p, cols.npad, qsum, poison);
  FD_LAUNCH_CHECK();
}

void launch_degree_reduce_ds(const SymPass& sp, const PointPack& rows, FSpan part,
                             unsigned long long* colfix, const float* q, double alpha, float* d,
                             float* s, const double* qsum, double* s_off,
                             const PoisonGate& poison, hipStream_t stream) {
  hipLaunchKernelGGL(degree_reduce_ds_kernel, dim3(blocks_for(rows.npad, 256)), dim3(256), 0,
                     stream, part.p, sp.nsplit, rows.npad, colfix, sp.inv_fix, q, rows.n,
                     rows.npad, alpha, d, s, qsum, qsum_words(rows.npad), s_off, poison);
  FD_LAUNCH_CHECK();
}

void launch_degree_reduce_dsq(const SymPass& sp, const PointPack& rows, const PointPack& cols,
                              FSpan part, unsigned long long* colfix, const float* q,
                              double alpha, float* d, float* s, FSpan sq_part,
                              unsigned long long* sq_colfix, float* q_next, FSpan wp,
                              const double* qsum, double* s_off, double* qsum_next,
                              const PoisonGate& poison, hipStream_t stream) {
  FD_REQUIRE(cols.npad % TILE == 0 && cols.npad <= rows.npad && cols.n == rows.n,
             FD_ERR_INVALID_ARG, "internal: bad weight pack geometry");
  check_span(wp, lane4_extent(cols.npad / TILE, 1), "weight pack");
  check_span(sq_part, size_t(sp.nsplit) * rows.npad, "partial squared row sums");
  FD_REQUIRE(q_next != nullptr && sq_colfix != nullptr, FD_ERR_INVALID_ARG,
             "internal: dyadic reduction outputs");
  hipLaunchKernelGGL(degree_reduce_dsq_kernel, dim3(blocks_for(rows.npad, 256)), dim3(256), 0,
                     stream, part.p, sp.nsplit, rows.npad, colfix, sp.inv_fix, q, rows.n,
                     rows.npad, alpha, d, s, sq_part.p, sq_colfix, q_next, wp.p, cols.npad, qsum,
                     qsum_words(rows.npad), s_off, qsum_next, poison);
  FD_LAUNCH_CHECK();
}

// The plain row-sum kernel: partials into pp, or (pp NULL, one split) out.
static void launch_rowsum_pass(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                               FSpan wp, bool diag, float* out, float* pp, hipStream_t stream) {
  FD_REQUIRE(p.nib == 8, FD_ERR_INVALID_ARG, "internal: row-sum plan");
  check_span(wp, lane4_extent(p.njb, 1), "weight pack");
  if (rows.bf16 || cols.bf16) {
    FD_REQUIRE(rows.bf16 && cols.bf16 && rows.dc == cols.dc, FD_ERR_INVALID_ARG,
               "internal: mixed pack kinds");
    if (rows.dc == 1) rowsum_bf16_launch<1>(p, rows, cols, wp.p, diag, out, pp, stream);
    else rowsum_bf16_launch<2>(p, rows, cols, wp.p, diag, out, pp, stream);
  } else {
    launch_rowsum_hx(p, rows, cols, wp.p, diag, out, pp, stream);
  }
}

void launch_rowsum(const KVPlan& p, const PointPack& rows, const PointPack& cols, FSpan wp,
                   bool diag, float* out, FSpan part, hipStream_t stream) {
  check_tiles(p, rows, cols);
  float* pp = nullptr;
  if (p.nsplit > 1) {
    check_span(part, size_t(p.nsplit) * rows.npad, "partial row sums");
    pp = part.p;
  }
  launch_rowsum_pass(p, rows, cols, wp, diag, out, pp, stream);
  if (p.nsplit > 1) {
    hipLaunchKernelGGL(reduce_rowsum_kernel, dim3(blocks_for(rows.n, 256)), dim3(256), 0, stream,
                       pp, p.nsplit, rows.npad, out, rows.n);
    FD_LAUNCH_CHECK();
  }
}

void launch_product_column(const KVPlan& p, const PointPack& rows, const PointPack& cols, FSpan wp,
                           FSpan vscale, bool diag, const float* sl, float* Y, int64_t ldy,
                           FSpan part, unsigned long long* colfix, unsigned long long* colfix_lo,
                           const PoisonGate& poison, hipStream_t stream) {
  check_tiles(p, rows, cols);
  check_span(part, size_t(p.nsplit) * rows.npad, "partial row sums");
  check_span(vscale, 64, "column scales");
  SymPass sp;
  if (column_sym_applies(rows, cols, diag, colfix)) {
    ProfScope prof(FD_KERNEL_ROWSUM, stream);  // one of the two variants runs
    // K is symmetric: each tile off the diagonal blocks once (the whole call on
    // the 6-torus set-up, N = 65,536, D = 32: 885 -> 590 us).  Column sums are
    // fixed point against the column's largest weight, so a NaN, an infinity or
    // a wide range (zeros among others, column_range) takes the plain sums: both
    // are launched, and the column's flag closes one of them.  (No colfix: a
    // caller without room for the words takes the plain sums.)
    PointPack r = rows, c = cols;
    r.vbad = c.vbad = vscale.p + 1;
    FD_REQUIRE(colfix_lo != nullptr, FD_ERR_INVALID_ARG, "internal: column words");
    sp = launch_rowsum_sym_pass(p, r, c, wp, part, colfix, stream, FSpan{}, nullptr, colfix_lo);
    r.serves_bad = c.serves_bad = 1;
    launch_rowsum_pass(p, r, c, wp, diag, nullptr, part.p, stream);
  } else {
    colfix = nullptr;
    launch_rowsum_pass(p, rows, cols, wp, diag, nullptr, part.p, stream);
  }
  hipLaunchKernelGGL(column_finish_kernel, dim3(blocks_for(rows.npad, 256)), dim3(256), 0, stream,
                     part.p, p.nsplit, sp.nsplit, rows.npad, colfix, colfix_lo, vscale.p, sl,
                     rows.n, rows.npad, Y, ldy, poison);
  FD_LAUNCH_CHECK();
}

void launch_pow_neg(const float* q, int64_t n, double alpha, float* w, hipStream_t stream) {
  hipLaunchKernelGGL(pow_neg_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, stream, q, n, alpha,
                     w);
  FD_LAUNCH_CHECK();
}

void launch_degree_finish(const float* q, const float* t, int64_t n, double alpha, float* d,
                          float* s, const double* qsum, int64_t nqsum, double* s_off,
                          const PoisonGate& poison, hipStream_t stream) {
  hipLaunchKernelGGL(degree_finish_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, stream, q, t,
                     n, alpha, d, s, qsum, nqsum, s_off, poison);
  FD_LAUNCH_CHECK();
}

}  // namespace fd
