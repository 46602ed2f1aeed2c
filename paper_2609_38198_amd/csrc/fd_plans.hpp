// Work split of the products and the row sums, and the extents of their partial
// sums: host code free of HIP, which a CPU test sweeps over its whole range.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace fd {

// ---------------------------------------------------------------- geometry
constexpr int TILE = 16;          // points per MFMA tile
constexpr int WG_THREADS = 256;   // four wave64 per workgroup
constexpr int ROW_PAD = 512;      // row packs: whole workgroups of 4 waves x 8 row tiles
constexpr int COL_PAD = 32;       // column packs: whole pairs of 16-point tiles
// Longest column range one workgroup of a product or row-sum plan streams
// (tiles of 16 points); longer ranges are split.  The workgroups that run
// together on an XCD start a split together and drift apart; over 4,096
// tiles (a few tens of MB of column operands) their working set stays
// cache-resident, over 32,768 it did not always (the bfloat16 product at
// N = 2^21, b = 64 then ran 1.5 to 2.2 s against 1.43 s).
constexpr int64_t SPLIT_SPAN_TILES = 4096;

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline int64_t ceil_div(int64_t x, int64_t m) { return (x + m - 1) / m; }

// Column tiles per partial accumulator: the sums over a longer range go to a
// running total (float32).
constexpr int CHUNK_TILES = 64;

// Plan of one fused product / degree launch.
struct KVPlan {
  int dp = 0, ncb = 0, nib = 0;
  int64_t njb = 0;        // column tiles of 16
  int64_t nrt = 0;        // row tiles of 64*nib
  int nsplit = 1;         // column splits
  int64_t jb_per_split = 0;
  int chunk = CHUNK_TILES;  // column tiles per partial accumulator (float32 products)
};

// Row tiles per wave of the symmetric row sums, and the fewest column splits
// of their large-problem plans.
constexpr int SYM_NIB = 8;
constexpr int64_t SYM_MIN_SPLITS = 16;

// Workgroups of one resident round: products and most symmetric row sums hold
// two waves per SIMD, so 256 CUs take two four-wave workgroups each.  The row
// sums of float32 points with D > 32 (and D = 31, 32 with squared sums) hold one,
// so that 512 of their workgroups are two rounds: still better than 2048
// (fd_degree, 2048 / 512 / 256 workgroups, us: D = 40, N = 5,000 74 / 74 / 62,
// 9,000 126 / 103 / 93, 16,000 269 / 192 / 176, 24,000 389 / 332 / 319; D = 64,
// N = 16,000 295 / 205 / 188).
constexpr int64_t ONE_ROUND = 512;

// `round`: split the columns for one resident round of workgroups (never more
// than ONE_ROUND) instead of for >= 2048
inline KVPlan plan_tiles(int64_t Nr, int64_t Nc, int dp, int b, int nib, bool round) {
  KVPlan p;
  p.dp = dp;
  p.ncb = int(ceil_div(b, 16));
  p.nib = nib;
  p.njb = ceil_div(Nc, TILE);
  const int64_t rows_per_wg = 4 * p.nib * TILE;
  p.nrt = ceil_div(round_up(Nr, ROW_PAD), rows_per_wg);
  // aim for >= 2048 workgroups (eight per CU), keep >= 8 column tiles per split
  int64_t ns = std::max<int64_t>(1, round ? ONE_ROUND / p.nrt : ceil_div(2048, p.nrt));
  ns = std::min<int64_t>(ns, std::max<int64_t>(1, p.njb / 8));
  // at most SPLIT_SPAN_TILES column tiles per workgroup: the workgroups that
  // run together on an XCD start a split together and drift apart as they go;
  // over a shorter span they stay close enough to share column tiles in L2
  ns = std::max<int64_t>(ns, ceil_div(p.njb, SPLIT_SPAN_TILES));
  ns = std::min<int64_t>(ns, 64);
  // splits hold an even number of column tiles (the split product takes them in pairs)
  p.jb_per_split = round_up(ceil_div(p.njb, ns), 2);
  p.nsplit = int(ceil_div(p.njb, p.jb_per_split));
  // the long ranges of one round would also be longer chains of float32 sums than
  // those of 2048 workgroups, whose ranges were added in float64: shorter chunks
  // keep the error (against float64, 2048 workgroups / one round with 64, 16, 8
  // tiles, 1e-7: N = 16,000, D = 12, b = 32 8.12 / 8.56, 7.93, 7.83; N = 8,000,
  // D = 30, b = 32 9.33 / 9.56, 9.40, 9.32) for 2% of the time (with 64 tiles / as
  // here, us: N = 16,384, D = 12, b = 32 99 / 101, b = 64 141 / 144; N = 8,192,
  // D = 30, b = 32 54.2 / 55.2)
  if (round) p.chunk = p.jb_per_split <= 32 ? 8 : 16;
  return p;
}

// Row tiles per wave and splits of the fused product.
//
// Eight row tiles for one 16-column block at D <= 12 above 2^28 pairs (6-torus,
// b = 16, microseconds for eight / four: N = 65,536 862 / 898, N = 32,768
// 256 / 270, N = 18,000 104 / 106: two instructions per exponent tile leave room
// for more independent chains).  Four below, where twice the workgroups count
// for more (N = 8,192 43 / 38, N = 4,096 27 / 26, N = 1,000 25 / 21; equal at
// 16,384), and on every other shape (the fastest or tied in D in {4, 12, 30, 64},
// b in {8 .. 64}; two and eight are 11-17% slower at D = 30, b = 32).
//
// One round of workgroups up to 3 * 2^27 pairs (about N = 20,000): each
// workgroup's start and its partial product, written and read again, cost more
// there than the uneven end of a few long workgroups (2048 workgroups / one
// round: D = 30, b = 32, N = 8,192 67 / 57, 20,000 173 / 165; 6-torus, b = 32,
// N = 16,384 115 / 102, b = 16, N = 16,384 95 / 87).  Beyond, the uneven end
// does (D = 30, b = 32, N = 28,000 289 / 296; b = 16, N = 24,000 182 / 186).  Both
// lines are by pairs alone and were measured at b = 16 and 32; partial products
// grow with b (b = 64, 30,011 x 16,384: 18 splits, 139 MB written and read again).
constexpr int64_t WIDE_ROWS_PAIRS = int64_t(1) << 28;
constexpr int64_t ONE_ROUND_PAIRS = int64_t(3) << 27;

inline KVPlan plan_product(int64_t Nr, int64_t Nc, int dp, int b) {
  const double pairs = double(Nr) * double(Nc);
  const int nib = (b <= 16 && dp <= 12 && pairs > double(WIDE_ROWS_PAIRS)) ? 8 : 4;
  return plan_tiles(Nr, Nc, dp, b, nib, pairs <= double(ONE_ROUND_PAIRS));
}

// Row sums: eight row tiles per wave (more independent exponent chains per
// column tile than four; measured faster on every shape).
inline KVPlan plan_rowsum(int64_t Nr, int64_t Nc, int dp) {
  return plan_tiles(Nr, Nc, dp, 1, 8, false);
}

// Symmetric row sums (one point set): workgroups of 4 waves x nib row tiles
// own blocks of 64 nib points; a block's column range (its own block and about
// half of the others) is split.  nrt holds the number of blocks.  From 64
// blocks up, for >= 2048 workgroups and by whole blocks (at least
// SYM_MIN_SPLITS of them): the workgroups whose windows start at the same
// block then read the same column tiles, and the kernel runs them side by side
// on one XCD so that they share its L2.  Up to 48 blocks, for one resident
// round: a workgroup's column sums end in atomic adds, and fewer, longer
// workgroups make fewer of them (fd_degree, 2048 workgroups / one round in
// microseconds: D = 30, N = 9,000 79 / 66, N = 16,000 140 / 115; D = 12,
// N = 20,000 168 / 151; bfloat16 points, D = 30, N = 9,000 59 / 54), down to four
// column tiles a workgroup (eight / four: N = 2,048 37 / 33, N = 512 34 / 29).
// In between the uneven end of one round begins to cost more than it saves
// (bfloat16 points, D = 30, N = 28,000: 215 / 221).
inline KVPlan plan_rowsum_sym(int64_t N, int64_t npad, int dp, int nib) {
  KVPlan p;
  p.dp = dp;
  p.ncb = 1;
  p.nib = nib;
  p.njb = ceil_div(N, TILE);
  const int64_t BT = 4 * nib;
  p.nrt = npad / (BT * TILE);
  const int64_t span_blocks = 1 + (p.nrt - 1) / 2 + (p.nrt % 2 == 0 ? 1 : 0);  // longest range
  if (p.nrt >= 64) {
    const int64_t ns = std::max<int64_t>(SYM_MIN_SPLITS, ceil_div(2048, p.nrt));
    const int64_t jbk = std::max<int64_t>(1, span_blocks / ns);
    p.jb_per_split = jbk * BT;
    p.nsplit = int(ceil_div(span_blocks, jbk));
    return p;
  }
  const int64_t span = BT * span_blocks;
  int64_t ns =
      std::max<int64_t>(1, p.nrt <= 48 ? ONE_ROUND / p.nrt : ceil_div(2048, p.nrt));
  ns = std::min<int64_t>(ns, std::max<int64_t>(1, span / 4));
  ns = std::min<int64_t>(ns, 64);
  p.jb_per_split = round_up(ceil_div(span, ns), 2);
  p.nsplit = int(ceil_div(span, p.jb_per_split));
  return p;
}

// Row slots of the partial sums of a symmetric row-sum plan with npad rows.
inline size_t sym_part_rows(int64_t npad, int nib) {
  return size_t(plan_rowsum_sym(npad, npad, 4, nib).nsplit) * size_t(npad);
}

// The same for every plan with at most npad rows (a continuation plans each of
// its prefixes in regions carved for the longest one).  Splits by whole blocks
// make the need no monotone function of the rows: 89 blocks of 512 points take
// 45 splits of one block, 128 blocks 18 of four.  Beyond SWEEP blocks a split
// holds at least 64 of them, so that there are at most 17.
inline size_t sym_part_rows_within(int64_t npad, int nib) {
  constexpr int64_t SWEEP = 2048;
  const int64_t block = 4 * int64_t(nib) * TILE, nblk = npad / block;
  size_t need = nblk > SWEEP ? size_t(SYM_MIN_SPLITS + 1) * size_t(npad) : 0;
  for (int64_t k = 1; k <= std::min(nblk, SWEEP); ++k)
    need = std::max(need, sym_part_rows(k * block, nib));
  return need;
}

// Points from which a single-column product on one point set takes the symmetric
// row sums.  Below, a call is its launches: the plain sums need neither the
// column's maxima nor the second variant of the pass (symmetric / plain, us:
// D = 4 N = 2,048 22 / 19, 5,000 27 / 24; D = 64 N = 6,000 57 / 52, 8,000 66 / 74,
// 16,000 121 / 179; bfloat16, D = 12 N = 6,000 29 / 25, 8,000 33 / 34, 16,000
// 60 / 70; all 700 eigenpairs of 700 points with b = 1 28.8 / 24.6 ms).  At
// D = 4 in float32 the plain sums stay 3-9% ahead to N = 24,000.
constexpr int64_t COLUMN_SYM_POINTS = 6144;

// Column sums of a single-column product over the symmetric row sums.  A wave's
// contribution (weights below 1, 128 rows) is rounded to WIDE_FRAC fractional
// bits; a workgroup adds at most four of them to a column (below 2^9, so that
// its 64-bit word holds them), splits the word and adds its signed upper part
// and its lower WIDE_SPLIT bits to two global words: no sum over the up to 2^21
// blocks takes bits from the fraction (one 64-bit word would have 40 at 2^20
// points, where results of small weights lost up to 2% of themselves).
constexpr int WIDE_FRAC = 53;
constexpr int WIDE_SPLIT = 32;

// Widest column (largest over smallest |weight|) that takes them.  A result
// holds its own point's weight (K_ii = 1), at least half of 1 / range, and up to
// npad / 256 roundings of 2^-(WIDE_FRAC + 1) each: at this range they come to
// 2^-18 of that weight if all have one sign and their full size (the float32 sums of a
// row's 256-term chains may lose 2^-16).  Wider columns, sparse ones among them,
// take the plain float32 sums.
inline float column_range(int64_t npad) { return std::ldexp(1.f, 43) / float(npad); }

// Every plan has nsplit <= max(ceil(2048 / row blocks), ceil(column tiles /
// SPLIT_SPAN_TILES)), so the partial buffers of any problem with at most npad
// rows and nc columns fit in this many row slots.
inline size_t part_rows_bound(int64_t npad, int64_t nc) {
  return size_t(2048) * ROW_PAD + size_t(npad) * size_t(1 + ceil_div(ceil_div(nc, TILE), SPLIT_SPAN_TILES));
}

}  // namespace fd
