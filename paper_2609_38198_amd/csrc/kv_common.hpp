// Device-side types and helpers shared by the fused-product translation units.
#pragma once

#include <hip/hip_runtime.h>

#include "fd_internal.hpp"

namespace fd {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __fp16 pkhalf2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

constexpr double LOG2E = 1.4426950408889634073599;

// Which of the two layouts of a float32 pack a launch serves (PointPack):
// every launch of such a pair reads the same device word, and the one whose
// layout does not match the exponent budget exits before any work.
// vbad (single-column products): whether the column holds a value that the
// symmetric row sums cannot take; the launch serves one of the two cases.
struct HxGate {
  const unsigned long long* r2max = nullptr;
  double bl = 0.0;  // beta log2(e) of the pack
  int variant = 0;  // 0: no choice, 1: short layout, 2: full-offset layout
  const float* vbad = nullptr;
  int serves_bad = 0;
};
__device__ __forceinline__ bool hx_gate_closed(const HxGate& g) {
  if (g.vbad != nullptr && (*g.vbad != 0.f) != (g.serves_bad != 0)) return true;
  if (g.variant == 0) return false;
  const double r2 = __longlong_as_double(static_cast<long long>(*g.r2max));
  const bool wide = g.bl * r2 > EXP_BUDGET;
  return wide != (g.variant == 2);
}
inline HxGate gate_of(const PointPack& rows) {
  HxGate g;
  g.r2max = rows.r2max;
  g.bl = rows.beta * LOG2E;
  g.variant = rows.variant;
  g.vbad = rows.vbad;
  g.serves_bad = rows.serves_bad;
  return g;
}

// Workgroups of one dispatch are spread over the eight XCDs round-robin by
// id.  Re-number them so that each XCD owns a contiguous block of logical
// work items (same column split, hence a shared working set in its L2).
__device__ __forceinline__ int xcd_remap(int w, int total) {
  if ((total & 7) != 0) return w;
  const int per = total >> 3;
  return (w & 7) * per + (w >> 3);
}

// Split float16 pack of V for one pair of 16-point column tiles: lane (g, p)
// holds rows {4g + r} of the first tile and {16 + 4g + r} of the second
// (r = 0..3) of column 16 cb + p, as hi and lo halves.
struct VSplit {
  halfx8 hi;
  halfx8 lo;
};

// Round two floats toward zero to float16 (hi) and the remainders likewise
// (lo); returns both packed pairs as 32-bit words.
__device__ __forceinline__ void split2(float a, float b, unsigned& hi, unsigned& lo) {
  const pkhalf2 h = __builtin_amdgcn_cvt_pkrtz(a, b);
  const pkhalf2 l = __builtin_amdgcn_cvt_pkrtz(a - float(h[0]), b - float(h[1]));
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, l);
}

// The same split with each remainder formed by one mixed-precision FMA,
// k - h = fma(h, m1, k) reading h straight from the packed float16 word (exact
// in float32) and rounded to nearest float16.
// m1 must be -1; it is a run-time value (a kernel argument) so that the
// compiler keeps the FMA form instead of turning it into a subtraction.
__device__ __forceinline__ void split2m(float a, float b, float m1, unsigned& hi, unsigned& lo) {
  const pkhalf2 h = __builtin_amdgcn_cvt_pkrtz(a, b);
  // each remainder rounded straight into its half of the packed word
  // (v_fma_mixlo_f16 / v_fma_mixhi_f16: two instructions instead of two
  // float32 FMAs and a conversion)
  pkhalf2 l;
  l[0] = (_Float16)__builtin_fmaf(float(h[0]), m1, a);
  l[1] = (_Float16)__builtin_fmaf(float(h[1]), m1, b);
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, l);
}

// Whether a call's outputs are NaN (PoisonGate).
__device__ __forceinline__ bool poisoned(const PoisonGate& g) {
  if (g.flag == nullptr) return false;
  if (*g.flag != 0) return true;
  if (g.r2max == nullptr) return false;
  const double r2 = __longlong_as_double(static_cast<long long>(*g.r2max));
  return !(g.bl * r2 <= HX_EXP_RANGE && g.f2 * r2 <= HX_PIECE_MAX * HX_PIECE_MAX);
}

// ---------------------------------------------------------------- V and weight packs

constexpr int PACK_THREADS = 128;  // workgroup of the pack kernels

// Launches `blocks` workgroups of a pack kernel.  A launch holds fewer than 2^32
// threads, and a side of a set takes up to four threads a point, its V eight:
// beyond 2^31 threads the packs go in slices (args.blk0 is a slice's first block).
template <class K, class A>
void launch_pack_blocks(K kernel, int64_t blocks, A args, hipStream_t stream) {
  constexpr int64_t SLICE = (int64_t(1) << 31) / PACK_THREADS;
  for (args.blk0 = 0; args.blk0 < blocks; args.blk0 += SLICE) {
    hipLaunchKernelGGL(kernel, dim3(unsigned(std::min(SLICE, blocks - args.blk0))),
                       dim3(PACK_THREADS), 0, stream, args);
    FD_LAUNCH_CHECK();
  }
}

// The V part of a pack launch: V (n x b, ldv) times sr, as the split pack of
// ncb 16-column blocks over npairs pairs of 16-point tiles, or (ncb = 0) as the
// weight pack of its one column over ntiles tiles; with nvmax that column is
// scaled by 2^-e to below 1 (colscale[0] = e or 0, colscale[1] = 1 where it holds a
// NaN or an infinity or spans more than `range`, else 0).
struct PackV {
  const float* V = nullptr;
  const float* sr = nullptr;
  int64_t n = 0, ldv = 0, npairs = 0, ntiles = 0;
  int64_t blk0 = 0;
  int b = 0, ncb = 0, nvmax = 0;
  float range = 0.f;             // column_range
  const float* vpart = nullptr;  // nvmax x 64 partial column maxima
  float* colscale = nullptr;
  VSplit* vp = nullptr;
  floatx4* wp = nullptr;
};
inline int64_t pack_v_items(const PackV& a) {
  return a.V == nullptr ? 0 : a.ncb > 0 ? a.npairs * a.ncb * 64 : a.ntiles * 64;
}

__device__ __forceinline__ int vscale_exponent(float mx) {
  if (!(mx > 0.f)) return 0;
  int e;
  (void)frexpf(mx, &e);  // max < 2^e
  return 14 - e;         // scaled max < 2^14
}

// Workgroup `blk` of the V part (PACK_THREADS threads); ex: 64 LDS words.
__device__ __forceinline__ void pack_v_block(const PackV& a, int64_t blk, int* ex) {
  const int64_t idx = blk * PACK_THREADS + threadIdx.x;
  const int lane = int(threadIdx.x & 63);
  const int g = lane >> 4, p = lane & 15;
  if (a.ncb == 0) {
    int ex1 = 0;
    float bad = 0.f;
    if (a.nvmax > 0) {
      float m = 0.f, mn = __builtin_inff();
      for (int k = lane; k < a.nvmax; k += 64) {
        m = fmaxf(m, a.vpart[k * 64]);
        bad = fmaxf(bad, a.vpart[k * 64 + 1]);
        mn = fminf(mn, a.vpart[k * 64 + 2]);
      }
      for (int o = 32; o > 0; o >>= 1) {
        m = fmaxf(m, __shfl_xor(m, o));
        bad = fmaxf(bad, __shfl_xor(bad, o));
        mn = fminf(mn, __shfl_xor(mn, o));
      }
      if (mn * a.range < m) bad = 1.f;
      ex1 = bad != 0.f ? 0 : 14 - vscale_exponent(m);
    }
    if (idx == 0) {
      a.colscale[0] = float(ex1);
      a.colscale[1] = bad;
    }
    if (idx >= a.ntiles * 64) return;
    floatx4 out;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t j = (idx >> 6) * TILE + 4 * g + r;
      out[r] = 0.f;
      if (j < a.n) out[r] = a.sr != nullptr ? a.sr[j] * a.V[j * a.ldv] : a.V[j * a.ldv];
      out[r] = ldexpf(out[r], -ex1);
    }
    a.wp[idx] = out;
    return;
  }
  // column exponents from the prologue's partial maxima: two threads a column
  // (a maximum does not depend on the order)
  {
    const int c = int(threadIdx.x) >> 1, h = int(threadIdx.x) & 1;
    float m = 0.f;
    if (c < a.b) {
#pragma unroll 8
      for (int k = h; k < a.nvmax; k += 2) m = fmaxf(m, a.vpart[k * 64 + c]);
    }
    m = fmaxf(m, __shfl_xor(m, 1));
    if (h == 0) ex[c] = vscale_exponent(m);
  }
  __syncthreads();
  if (blk == 0 && int(threadIdx.x) < a.b) a.colscale[threadIdx.x] = ldexpf(1.f, -ex[threadIdx.x] - 15);
  if (idx >= a.npairs * a.ncb * 64) return;
  const int cb = int((idx >> 6) % a.ncb);
  const int64_t jp = idx / (64 * a.ncb);
  const int c = cb * 16 + p;
  const float scale = ldexpf(1.f, c < a.b ? ex[c] : 0);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t j = jp * 32 + (e < 4 ? 4 * g + e : 16 + 4 * g + (e - 4));
    float x = 0.f;
    if (j < a.n && c < a.b) {
      x = a.V[j * a.ldv + c];
      if (a.sr != nullptr) x *= a.sr[j];
    }
    v[e] = x * scale;
  }
  uintx4 hw, lw;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    unsigned h, l;
    split2(v[e], v[e + 1], h, l);
    hw[e / 2] = h;
    lw[e / 2] = l;
  }
  VSplit out;
  out.hi = __builtin_bit_cast(halfx8, hw);
  out.lo = __builtin_bit_cast(halfx8, lw);
  a.vp[idx] = out;
}

// The flag word of a call from the prologue's words (one workgroup).
__device__ __forceinline__ void pack_flag(const int* __restrict__ flags, int nflags,
                                          int* __restrict__ flag) {
  int bad = 0;
  for (int k = threadIdx.x; k < nflags; k += PACK_THREADS) bad |= flags[k];
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) *flag = bad;
}

// Columns side by side in a row-major sweep: the power of two >= b.
inline int column_lanes(int64_t b) {
  int tc = 1;
  while (tc < b) tc *= 2;
  return tc;
}

// Means of the D columns from the prologue's partial sums, in LDS (mu: MAX_D
// doubles, red: 128 doubles); every workgroup of every kernel adds
// them in the same order (two teams; workgroups of at least 128 threads).
__device__ __forceinline__ void centre_means(const double* __restrict__ part, int nblk, int D,
                                             int64_t n, double* mu, double* red) {
  const int f = int(threadIdx.x) % 64, team = int(threadIdx.x) / 64;
  double acc = 0.0;
  if (f < D && team < 2) {
#pragma unroll 8
    for (int k = team; k < nblk; k += 2) acc += part[int64_t(k) * D + f];
  }
  if (team < 2) red[threadIdx.x] = acc;
  __syncthreads();
  if (int(threadIdx.x) < D) mu[threadIdx.x] = (red[threadIdx.x] + red[64 + threadIdx.x]) / double(n);
  __syncthreads();
}

// Raises *r2max (float64 bits; non-negative values order like them) to the
// wave's maximum.  The word only grows during a launch, so a wave that reads a
// value at least as large has nothing to add; most do after the first few.
__device__ __forceinline__ void raise_r2max(double r, unsigned long long* r2max) {
  for (int o = 32; o > 0; o >>= 1) r = fmax(r, __shfl_xor(r, o));
  if ((threadIdx.x & 63) != 0) return;
  const unsigned long long bits = static_cast<unsigned long long>(__double_as_longlong(r));
  if (r > 0.0 && bits > __hip_atomic_load(r2max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(r2max, bits);
}

inline unsigned blocks_for(int64_t n, int t) { return unsigned(ceil_div(n, t)); }

// ---------------------------------------------------------------- float32 path
// (split float16 exponent contraction; hx_kernels.hip)

// Recipe index and chunk counts of the split-exponent pack for a feature
// dimension D (1 <= D <= 64).
int hx_recipe_for(int64_t D);
int hx_col_chunks(int rid);
int hx_row_chunks(int rid);

void launch_packs_hx(const PackIn& in, const PackV& v, PointPack& rows, PointPack& cols,
                     const CentreWs& centre, hipStream_t stream);
// Recipe that keeps all three offset pieces for a short recipe that drops the
// third (-1: the recipe keeps them).
int hx_full_offset_recipe(int rid);
void launch_product_hx(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                       const float* vp, const float* colscale, bool diag, const float* sl,
                       float* Y, int64_t ldy, int b, float* part, const PoisonGate& poison,
                       hipStream_t stream);
void launch_rowsum_hx(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                      const float* wp, bool diag, float* out, float* part, hipStream_t stream);
// Symmetric row sums of one point set (rows.n == cols.n): per-split row partials
// into part ([nsplit][rows.npad]) and column sums added into col (fixed point;
// weights in [-1, 1]).  With sq.part set
// (weighted passes only), the unit-weight sums of the squared kernel K^2 (the
// kernel at twice the bandwidth) go the same way into sq.part and sq.colfix.
void launch_rowsum_sym_hx(const KVPlan& p, const PointPack& rows, const PointPack& cols,
                          const float* wp, float* part, const ColumnWords& col,
                          const SymSquares& sq, hipStream_t stream);

// Scheduling pattern for a region holding M matrix instructions and E
// exponentials: each matrix instruction followed by its share of the
// exponentials and V other vector instructions.
template <int M, int E, int V, int m = 0>
__device__ __forceinline__ void sched_interleave() {
  if constexpr (m < M) {
    constexpr int ne = (m + 1) * E / M - m * E / M;
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // matrix
    if constexpr (ne > 0) __builtin_amdgcn_sched_group_barrier(0x400, ne, 0);  // transcendental
    __builtin_amdgcn_sched_group_barrier(0x002, V, 0);  // vector
    sched_interleave<M, E, V, m + 1>();
  }
}

}  // namespace fd
