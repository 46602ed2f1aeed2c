// Symmetric row sums of one point set: sum_j K_ij w_j with every kernel tile
// off the diagonal blocks evaluated once.  Shared by the float32 and the
// bfloat16 path.
#pragma once

#include <type_traits>

#include "kv_common.hpp"

namespace fd {

namespace {

// When rows and columns are the same N points, K is symmetric and each
// off-diagonal tile K_IJ can serve both sums: q_I += K_IJ w_J along its rows and
// q_J += K_IJ^T w_I along its columns, so every kernel entry off the diagonal
// blocks is evaluated (and exponentiated) once instead of twice.
//
// Points are grouped in blocks of 512 (one workgroup's 4 waves x 8 row tiles);
// with B blocks and h = (B - 1) / 2, the workgroup of block P takes its own
// block (row sums only, exact diagonal) and then the blocks P + 1 .. P + h
// (mod B), plus P + B/2 when B is even and P < B/2: every unordered pair of
// distinct blocks is then taken exactly once.  That column range is split over
// nsplit workgroups.  Row sums go to per-split partials as in the plain kernel.
// Column sums are reduced over the wave's 128 rows (in-lane over its row
// tiles, then across the 16 lanes of a DPP row), converted to 64-bit fixed
// point and added into a per-workgroup LDS array with integer LDS atomics; every
// SYM_CHUNK column tiles the workgroup adds that array into the global
// per-point accumulator with integer atomics.  Integer addition is exact and
// order-free, so the result is bitwise reproducible.  (Global atomics inside
// the tile loop would make each operand-load wait also wait for an atomic's
// round trip, since vector memory operations retire in order.)  The
// fixed-point scale assumes weights in [-1, 1] (the normalisation weights
// q^-alpha with q >= 1 are; a single right-hand side is scaled by a power of
// two) and leaves a factor 4 of headroom below 2^63 for
// the total, or (TWO) for the workgroup's own sums only, whose words
// then go to two global words (WIDE_FRAC in fd_plans.hpp).

// Column tiles whose fixed-point column sums a workgroup gathers in LDS
// (SYM_CHUNK x 16 x 8 bytes) before adding them into global memory; even.
constexpr int SYM_CHUNK = 256;

// Sum of v over the 16 lanes of the lane's DPP row (every lane gets the sum).
__device__ __forceinline__ float dpp_row_sum(float v) {
  // xor 1 and xor 2 inside quads, then mirrored quads and mirrored half-rows
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1,
                                                             0xF, 0xF, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E,
                                                             0xF, 0xF, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141,
                                                             0xF, 0xF, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140,
                                                             0xF, 0xF, false));
  return v;
}

// The kernel is written over a tile policy T (the float32 path's split-float16
// exponent contraction in hx_kernels.hip, the bfloat16 one in kv_kernels.hip):
//   T::Row, T::Col        operands of a row tile / a column tile per lane,
//   T::Args, load_row, load_col, consume (an empty statement reading a Row),
//   tile(col, row)        the contraction of a tile,
//   value(x, row, args)   ONE K from an element of it (ONE a power of two),
//   waves<NIB, SQ>()      waves per SIMD asked of the compiler.

// One pipeline step of the symmetric row sums.  t holds the exponent tiles of
// an off-diagonal column tile J against the wave's NIB row tiles; each is
// exponentiated and then overwritten with the exponent tile of the next column
// tile (operands xn), so the matrix-core chain of row tile ib runs alongside
// the vector work of row tiles ib + 1, ...  SUMS: add J's row sums into acc and
// its column sums into the fixed-point accumulator (false for padding tiles).
template <class T, int NIB, bool UNIT, bool SUMS, bool SQ>
__device__ __forceinline__ void sym_step(floatx4 (&t)[NIB], const typename T::Col& xn,
                                         const typename T::Row (&br)[NIB], const floatx4& w,
                                         const float (&wi)[NIB], float (&acc)[NIB],
                                         float (&acc2)[NIB], int64_t jl, double fix_scale,
                                         double fix_scale2, unsigned long long* lds_col,
                                         unsigned long long* lds_col2, int g, int p,
                                         const typename T::Args& ta) {
  float cs[4] = {0.f, 0.f, 0.f, 0.f};
  float cs2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    float k[4];
    if (SUMS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) k[r] = T::value(t[ib][r], br[ib], ta);
    }
    t[ib] = T::tile(xn, br[ib]);
    if (SUMS) {
      if (UNIT) {
        acc[ib] += (k[0] + k[1]) + (k[2] + k[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r) cs[r] += k[r];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[ib] = fmaf(k[r], w[r], acc[ib]);
          cs[r] = fmaf(k[r], wi[ib], cs[r]);
        }
        if constexpr (SQ) {
          // the squared kernel (K at twice the bandwidth) with unit weights,
          // along the rows and along the columns of the tile
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            acc2[ib] = fmaf(k[r], k[r], acc2[ib]);
            cs2[r] = fmaf(k[r], k[r], cs2[r]);
          }
        }
      }
    }
  }
  if (!SUMS) return;
  // the row sums are due here (an empty statement reading them), not sunk
  // past the column-sum atomic below, so that they interleave too
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    asm volatile("" ::"v"(acc[ib]));
    if constexpr (SQ) asm volatile("" ::"v"(acc2[ib]));
  }
  // Interleave the contraction with the exponentials and sums (left to
  // itself the scheduler issues the exponentials first, then the matrix
  // instructions with little vector work between them).
  sched_interleave<T::NM * NIB, 4 * NIB, (SQ ? 5 : 3) + T::EXTRA>();
  // lane (g, p) holds, for column 4g + r of the tile, the sum over rows p of
  // the wave's tiles; the 16 lanes of DPP row g hold the wave's other rows
#pragma unroll
  for (int r = 0; r < 4; ++r) cs[r] = dpp_row_sum(cs[r]);
  // lane p < 4 adds column 4g + p (selects, no branches)
  const float v01 = (p & 1) ? cs[1] : cs[0];
  const float v23 = (p & 1) ? cs[3] : cs[2];
  const float v = (p & 2) ? v23 : v01;
  const long long fx = __double2ll_rn(double(v) * fix_scale);
  if (p < 4) atomicAdd(lds_col + jl * TILE + 4 * g + p, static_cast<unsigned long long>(fx));
  if constexpr (SQ) {
#pragma unroll
    for (int r = 0; r < 4; ++r) cs2[r] = dpp_row_sum(cs2[r]);
    const float u01 = (p & 1) ? cs2[1] : cs2[0];
    const float u23 = (p & 1) ? cs2[3] : cs2[2];
    const float u = (p & 2) ? u23 : u01;
    const long long fx2 = __double2ll_rn(double(u) * fix_scale2);
    if (p < 4) atomicAdd(lds_col2 + jl * TILE + 4 * g + p, static_cast<unsigned long long>(fx2));
  }
}

// One column tile of the workgroup's own block against the wave's row tiles:
// row sums only, K_ii = 1 exactly.
template <class T, int NIB, bool UNIT, bool DIAG, bool SQ>
__device__ __forceinline__ void sym_own_tile(const typename T::Col& c, const floatx4& w,
                                             const typename T::Row (&br)[NIB], float (&acc)[NIB],
                                             float (&acc2)[NIB], int64_t jb, int64_t ib0, int g,
                                             int p, const typename T::Args& ta) {
  floatx4 t[NIB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) t[ib] = T::tile(c, br[ib]);
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    float k[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      k[r] = T::value(t[ib][r], br[ib], ta);
      if (DIAG && jb == ib0 + ib && 4 * g + r == p) k[r] = T::ONE;
    }
    if (UNIT) {
      acc[ib] += (k[0] + k[1]) + (k[2] + k[3]);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[ib] = fmaf(k[r], w[r], acc[ib]);
    }
    if constexpr (SQ) {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc2[ib] = fmaf(k[r], k[r], acc2[ib]);
    }
  }
}

// SQ (weighted passes only): also the row and column sums of the squared
// kernel, K^2 1 = K(2 beta) 1 (eq. kernel), into part2 / colfix2 with the scale
// fix_scale2 per unit of (ONE K)^2.
// TWO (weighted passes only): column sums in two words, into colfix and
// colfix_lo (an instantiation of its own: chosen at run time, the normalisation's
// weighted pass came out 1% slower at N = 200,003, D = 30).
template <class T, int NIB, bool UNIT, bool SQ = false, bool TWO = false>
__global__ __launch_bounds__(WG_THREADS)
__attribute__((amdgpu_waves_per_eu(T::template waves<NIB, SQ>()))) void rowsum_sym_kernel(
    typename T::Args ta, const floatx4* __restrict__ wp, int64_t nblk, int64_t njb,
    int64_t jb_per_split, int64_t nsplit, float* __restrict__ part, int64_t nrpad,
    unsigned long long* __restrict__ colfix, unsigned long long* __restrict__ colfix_lo,
    double fix_scale, float* __restrict__ part2,
    unsigned long long* __restrict__ colfix2, double fix_scale2, HxGate gate) {
  static_assert(!((SQ || TWO) && UNIT), "squared sums and two words are weighted passes'");
  if (hx_gate_closed(gate)) return;
  constexpr int BT = 4 * NIB;  // tiles per block
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = xcd_remap(blockIdx.x, gridDim.x);
  // whole-block splits: number the workgroups by the block c their window
  // starts at (c = P + split * blocks per split), so that consecutive ids (run
  // together on one XCD) read the same column tiles
  const int64_t jbk = jb_per_split / BT;
  int64_t split, P;
  if (jb_per_split % BT == 0) {
    const int64_t c = wr / nsplit;
    split = wr % nsplit;
    P = ((c - split * jbk) % nblk + nblk) % nblk;
  } else {
    split = wr / nblk;
    P = wr % nblk;
  }
  const int64_t ib0 = P * BT + wave * NIB;
  const int64_t h = (nblk - 1) / 2;
  const int64_t span = BT * (1 + h + ((nblk % 2 == 0 && 2 * P < nblk) ? 1 : 0));
  const int64_t jj_begin = split * jb_per_split;
  const int64_t jj_end = min(span, jj_begin + jb_per_split);
  const int64_t ntile = nblk * BT;
  const int g = lane >> 4, p = lane & 15;
  // fixed-point column sums of the current chunk of SYM_CHUNK tiles
  __shared__ unsigned long long lds_col[SYM_CHUNK * TILE];
  __shared__ unsigned long long lds_col2[SQ ? SYM_CHUNK * TILE : 1];
  for (int e = threadIdx.x; e < SYM_CHUNK * TILE; e += WG_THREADS) {
    lds_col[e] = 0ull;
    if constexpr (SQ) lds_col2[e] = 0ull;
  }
  __syncthreads();

  typename T::Row br[NIB];
  float wi[NIB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    T::load_row(br[ib], ta, ib0 + ib, lane);
    // weight of own row 16 (ib0 + ib) + p: pack element (tile, lane 16 (p / 4), p % 4);
    // own tiles past the column pack are padding rows (their kernel values are 0)
    wi[ib] = 0.f;
    if (!UNIT && ib0 + ib < njb)
      wi[ib] = reinterpret_cast<const float*>(wp)[((ib0 + ib) * 64 + 16 * (p >> 2)) * 4 + (p & 3)];
  }
  float acc[NIB], tot[NIB], acc2[NIB], tot2[NIB];
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) acc[ib] = tot[ib] = acc2[ib] = tot2[ib] = 0.f;

  // column tile of range position jj (0 <= jj < span <= ntile + BT, cyclic over
  // the blocks); -1 for the padding tiles past the real columns
  const int base = int(P * BT), nt32 = int(ntile), njb32 = int(njb);
  auto tile_of = [&](int64_t jj) -> int {
    int J = base + int(jj);
    if (J >= nt32) J -= nt32;
    return J < njb32 ? J : -1;
  };
  // tile loaded for range position jj of [lo, jj_end): clamped into the range,
  // padding tiles read tile 0, so that loads are unconditional and every path
  // keeps the same loads in flight
  auto load_tile = [&](int64_t jj, int64_t lo) -> int64_t {
    const int J = tile_of(max(min(jj, jj_end - 1), lo));
    return J < 0 ? 0 : J;
  };
  int chunk = 0;
  auto row_chunk = [&](int tiles) {
    chunk += tiles;
    if (chunk >= CHUNK_TILES) {
      chunk = 0;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        tot[ib] += acc[ib];
        acc[ib] = 0.f;
        if constexpr (SQ) {
          tot2[ib] += acc2[ib];
          acc2[ib] = 0.f;
        }
      }
    }
  };

  // The workgroup's own block (range positions below BT, in split 0 only):
  // plain row sums, exact diagonal.  Column tiles stream through two buffers
  // used in turn.
  const int64_t own_end = min(jj_end, int64_t(BT));
  if (jj_begin < own_end) {
    typename T::Col c0, c1;
    floatx4 w0, w1;
    w0 = w1 = floatx4{1.f, 1.f, 1.f, 1.f};
    auto step = [&](const typename T::Col& c, const floatx4& w, int64_t jj) {
      const int J = tile_of(jj);
      if (J < 0) return;
      if (J >= ib0 && J < ib0 + NIB)
        sym_own_tile<T, NIB, UNIT, true, SQ>(c, w, br, acc, acc2, J, ib0, g, p, ta);
      else
        sym_own_tile<T, NIB, UNIT, false, SQ>(c, w, br, acc, acc2, J, ib0, g, p, ta);
    };
    auto load = [&](typename T::Col& c, floatx4& w, int64_t jj) {
      const int64_t J = load_tile(min(jj, own_end - 1), jj_begin);
      T::load_col(c, ta, J, lane);
      if (!UNIT) w = wp[J * 64 + lane];
    };
    load(c0, w0, jj_begin);
    __builtin_amdgcn_sched_barrier(0);  // c0's loads ahead of c1's, as in the loop
    load(c1, w1, jj_begin + 1);
    for (int64_t jj = jj_begin; jj < own_end; jj += 2) {
      step(c0, w0, jj);
      load(c0, w0, jj + 2);
      if (jj + 1 < own_end) step(c1, w1, jj + 1);
      load(c1, w1, jj + 3);
      row_chunk(2);
    }
  }

  // The other blocks: each tile serves both sums.  Two-stage pipeline over
  // the tiles u = 0, 1, ... of [s0, jj_end): step u exponentiates and sums
  // tile u, whose exponents the previous step made, while the matrix cores
  // make those of tile u + 1 (sym_step).  Tile v's column operands sit in
  // slot v % 2 and are loaded two steps ahead of their contraction, its
  // weights one step ahead of its sums.
  const int64_t s0 = max(jj_begin, int64_t(BT));
  const int64_t n2 = jj_end - s0;
  if (n2 > 0) {
    typename T::Col xa[2];
    floatx4 w[2];
    floatx4 t[NIB];
    w[0] = w[1] = floatx4{1.f, 1.f, 1.f, 1.f};
    auto load_xa = [&](typename T::Col& dst, int64_t u) {
      T::load_col(dst, ta, load_tile(s0 + u, s0), lane);
    };
    auto load_w = [&](floatx4& dst, int64_t u) {
      if (!UNIT) dst = wp[load_tile(s0 + u, s0) * 64 + lane];
    };
    load_xa(xa[0], 0);
    load_w(w[0], 0);
    __builtin_amdgcn_sched_barrier(0);
    load_xa(xa[1], 1);
    // consume the row operands here (an empty statement reading them): their
    // loads complete before the loop, whose waits then only ever cover the
    // column operands a step consumes (left to itself the compiler sinks these
    // loads past the loop entry and every iteration waits for all loads)
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib) T::consume(br[ib]);
    // likewise the scalar kernel argument used in the loop: with its load done
    // here, the loop's LDS atomics (which share the counter) are never waited on
    asm volatile("" ::"s"(fix_scale));
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib) t[ib] = T::tile(xa[0], br[ib]);
    // step u (slot S = u % 2): operands of tile u + 2 into slot S, weights of
    // tile u + 1 into slot S ^ 1, sums of tile u with weights from slot S,
    // contraction of tile u + 1 from slot S ^ 1
    auto pipe_step = [&](auto S_, int64_t u) {
      constexpr int S = decltype(S_)::value;
      load_xa(xa[S], u + 2);
      load_w(w[S ^ 1], u + 1);
      const int J = tile_of(s0 + u);
      const int64_t jl = (s0 + u - jj_begin) % SYM_CHUNK;
      if (J >= 0)
        sym_step<T, NIB, UNIT, true, SQ>(t, xa[S ^ 1], br, w[S], wi, acc, acc2, jl, fix_scale,
                                         fix_scale2, lds_col, lds_col2, g, p, ta);
      else
        sym_step<T, NIB, UNIT, false, SQ>(t, xa[S ^ 1], br, w[S], wi, acc, acc2, jl, fix_scale,
                                          fix_scale2, lds_col, lds_col2, g, p, ta);
      row_chunk(1);
      // end of a chunk of column tiles (the trip count is uniform over the
      // workgroup): add the chunk's column sums into the global accumulator
      const int64_t done = s0 + u + 1 - jj_begin;
      if (done % SYM_CHUNK == 0 || s0 + u + 1 >= jj_end) {
        const int64_t c0 = jj_begin + (done - 1) / SYM_CHUNK * SYM_CHUNK;
        __syncthreads();
        for (int e = threadIdx.x; e < SYM_CHUNK * TILE; e += WG_THREADS) {
          const unsigned long long v = lds_col[e];
          const int Jc = c0 + e / TILE < jj_end ? tile_of(c0 + e / TILE) : -1;
          if (v != 0ull && Jc >= 0) {
            const int64_t j = int64_t(Jc) * TILE + e % TILE;
            if constexpr (!TWO) {
              atomicAdd(colfix + j, v);
            } else {
              // arithmetic shift: hi 2^WIDE_SPLIT + lo is the signed word
              atomicAdd(colfix + j, static_cast<unsigned long long>(static_cast<long long>(v) >>
                                                                    WIDE_SPLIT));
              atomicAdd(colfix_lo + j, v & ((1ull << WIDE_SPLIT) - 1));
            }
          }
          lds_col[e] = 0ull;
          if constexpr (SQ) {
            const unsigned long long v2 = lds_col2[e];
            if (v2 != 0ull && Jc >= 0) atomicAdd(colfix2 + int64_t(Jc) * TILE + e % TILE, v2);
            lds_col2[e] = 0ull;
          }
        }
        __syncthreads();
      }
    };
    for (int64_t u = 0; u < n2; u += 2) {
      pipe_step(std::integral_constant<int, 0>{}, u);
      if (u + 1 < n2) pipe_step(std::integral_constant<int, 1>{}, u + 1);
    }
  }
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    float v = (tot[ib] + acc[ib]) * (1.f / T::ONE);
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (g == 0) part[split * nrpad + (ib0 + ib) * TILE + p] = v;
    if constexpr (SQ) {
      float v2 = (tot2[ib] + acc2[ib]) * (1.f / (T::ONE * T::ONE));
      v2 += __shfl_xor(v2, 16);
      v2 += __shfl_xor(v2, 32);
      if (g == 0) part2[split * nrpad + (ib0 + ib) * TILE + p] = v2;
    }
  }
}

}  // namespace

}  // namespace fd
