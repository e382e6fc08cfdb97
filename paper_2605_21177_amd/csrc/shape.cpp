// Host-side shape logic of the weight-gradient calls: which rows the MFMA kernel tiles, whether
// a call can take the MFMA path, and into how many token slabs it is split.  Pure functions of
// their arguments (no HIP), so that they can be built and fuzzed on a machine without a GPU.

#include <cstdint>

#include "internal.h"

namespace chunkft {

namespace {
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// rounds of work for w tiles per compute unit: a partly filled round costs 0.6 + 0.4 x its fill
inline double round_cost(double w) {
  const double fl = (double)(int64_t)w, fr = w - fl;
  return fl + (fr > 1e-9 ? 0.6 + 0.4 * fr : 0.0);
}
}  // namespace

// Body = complete rows from the first multiple of 8 on.  Everything before it
// lies in the one 8-row group [rb0 - 8, rb0) (at most the partial first row and
// 7 complete rows); after it there is at most the partial last row.
RowSplit split_rows(const WgradProblem& p) {
  RowSplit rs{};
  const int64_t r0 = p.begin / p.in, c0 = p.begin % p.in;
  const int64_t r1 = (p.end - 1) / p.in, c1 = (p.end - 1) % p.in + 1;
  const int64_t full0 = r0 + (c0 != 0 ? 1 : 0);           // first complete row
  const int64_t full1 = r1 + 1 - (c1 != p.in ? 1 : 0);    // one past the last complete row
  const int64_t rb0 = (full0 + 7) / 8 * 8;
  const bool body = full1 > rb0;
  rs.rb0 = rb0;
  rs.rb1 = body ? full1 : rb0;
  rs.lead_base = r0 < rb0 ? rb0 - 8 : -1;
  const int64_t first_after = body ? full1 : rb0;          // rows from here on are not in the lead group
  rs.trail_row = r1 >= first_after ? r1 : -1;
  return rs;
}

// The edge rows ride in the large-tile kernel if it has the tile rows that carry them (more than 128 body
// rows = two tile rows of the 128 x 256 tile); a chunk with edge rows and a shorter body goes to the small
// tiles, which have no edge rows.
bool edge_rows_folded(const RowSplit& rs) { return rs.rb1 - rs.rb0 > 128; }

namespace {
// 64 x 64 tiles over the rows of [begin, end), the first one rounded down to a multiple of 8
int64_t small_tiles(int64_t in, int64_t begin, int64_t end) {
  const int64_t rows = (end - 1) / in - begin / in / 8 * 8 + 1;
  return ceil_div(rows, 64) * ceil_div(in, 64);
}
}  // namespace

// Which chunks go to the 64 x 64 tiles.  A 256 x 256 or 128 x 256 tile per compute unit needs millions of
// elements; below that most of the device has no work (1 Mi elements of 1024 x 1024 at 256 tokens are 32
// tiles: the fused call needed 30 us, 9 us of it latency in small tiles).  Small tiles read their operands
// 1.5 - 4 times as often, so they lose where the token loop decides.  Fused call in us, small tiles against the
// better of the large ones, each at its best split (chunks of 4096-wide rows):
//   256 tokens: 1 Mi elements 9 against 27, 4 Mi 27 - 37, 8 Mi (2112 tiles) 46 - 49;  1024 tokens: 1 Mi 15 - 25, 2 Mi 23 - 32,
//   4 Mi 41 - 47, 8 Mi 67 - 63;   2048 tokens: 1 Mi 22 - 28, 2 Mi (528 tiles) 33 - 35, 4 Mi 59 - 51;   4096 tokens: 0.5 Mi (144
//   tiles) 22 - 24, 1 Mi (272) 34 - 31, 2 Mi 51 - 42;   8192 tokens: 0.25 Mi 27 - 28, 0.5 Mi 36 - 36, 1 Mi 55 - 41;
//   184-wide rows, 3620 tokens, 1.2 Mi (324 tiles) 44 - 38.  The gradient by itself crosses at the same products of tiles
//   and tokens.
// Bodies of at most 128 rows: with edge rows the large kernel cannot take them at all.  Without, it can, and the line is the
// same (72 - 128 rows; 512 tiles 2048 tokens 27 - 37, 4096 tokens 43 - 38, 2048 tiles 1024 tokens 52 - 45, 8192 tokens 389 -
// 280), but a body of at most 64 rows fills half a large tile and all of a small one: twice the line (64 rows; 256 tiles
// 8192 tokens 54 - 67, 1024 tiles 1024 tokens 43 - 43, 2048 tokens 65 - 61, 4096 tokens 136 - 106).
bool takes_small_tiles(int64_t in, int64_t T, int64_t begin, int64_t end, int compute_units) {
  const int64_t cus = compute_units > 0 ? compute_units : kDefaultComputeUnits;
  WgradProblem p{};
  p.begin = begin;
  p.end = end;
  p.in = in;
  const RowSplit rs = split_rows(p);
  const int64_t body = rs.rb1 - rs.rb0;
  if (body <= 0 || ((rs.lead_base >= 0 || rs.trail_row >= 0) && !edge_rows_folded(rs))) return true;
  const int64_t tiles = small_tiles(in, begin, end);
  return tiles <= cus * 43 / 10 && tiles * T <= cus * (body <= 64 ? 8600 : 4300);
}

// Four small tiles share a compute unit; the gradient has nothing but its loop to run under a fifth one's.  Small tiles against the
// large ones, gradient in us (the fused call, whose update does run under it, gains to the end of the line): 1050 tiles of 280 x
// 13408 200 tokens 11.4 - 11.6, 436 tokens 15.6 - 13.9, 1000 tokens 26 - 19 (fused 40 - 43); 1088 of 1032 x 4096 436 tokens
// 14.6 - 14.2, 1000 tokens 25 - 19; 1024 of 1024 x 4096 700 tokens 14.2 - 15.8, 1000 tokens 17.8 - 18.9.  Rows that are not whole
// 128-byte lines get there a little earlier: 968 of 1400 x 2800 436 tokens 13.3 - 14.1, 1000 tokens 22 - 19; 768 of 1024 x 3016
// 1400 tokens 20 - 22.
bool plain_leaves_small_tiles(const WgradProblem& p, int compute_units) {
  const int64_t cus = compute_units > 0 ? compute_units : kDefaultComputeUnits;
  const RowSplit rs = split_rows(p);
  if (rs.rb1 <= rs.rb0 || !(edge_rows_folded(rs) || (rs.lead_base < 0 && rs.trail_row < 0))) return false;   // only they can take it
  const int64_t tiles = small_tiles(p.in, p.begin, p.end), slab_tokens = p.S > 1 ? p.kslab : p.T;
  const bool whole_lines = p.ldx % 64 == 0 && (reinterpret_cast<uintptr_t>(p.X) & 127u) == 0;
  return (tiles > 4 * cus && slab_tokens > 256) || (!whole_lines && tiles > cus * 15 / 4 && slab_tokens > 440);
}

bool group_takes_segment(const WgradProblem& p, bool vector) {
  if (vector) return true;
  const RowSplit rs = split_rows(p);
  // a body for the MFMA kernel, its edge rows (if any) carried by it, one token slab
  return p.S == 1 && rs.rb1 > rs.rb0 && (edge_rows_folded(rs) || (rs.lead_base < 0 && rs.trail_row < 0));
}

bool mfma_path_ok(const WgradProblem& p) {
  const auto a16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
  if (!(p.in % 8 == 0 && p.out % 8 == 0 && p.ldx % 8 == 0 && p.lddy % 8 == 0 && a16(p.X) && a16(p.dY)))
    return false;
  if (p.in >= (1 << 21)) return false;      // the epilogue's 32-bit tile offsets
  // the 32-bit byte offsets of the global->LDS loads: a row / column index plus up to 63 tokens
  if (p.out + 64 * p.lddy >= (int64_t(1) << 31) || p.in + 64 * p.ldx >= (int64_t(1) << 31)) return false;
  return true;
}

// Which tile the plain gradient takes.  The 256 x 256 tile (one workgroup per compute unit) runs its
// rounds faster the more tokens a slab has -- measured ratio of a full round against the 128 x 256
// tile's (two workgroups per unit): 1.05 at 768 tokens, 0.99 at 1024, 0.95 at 1536, 0.91 at 2048,
// 0.88 at 3072, 0.85 at 8192, fitted by 0.83 + 160 / T -- but pays for a partly filled last round in
// whole tiles where the small tile pays in half ones.  With w = tiles / compute units, a partly
// filled round costs about 0.6 + 0.4 x (its fill) of a full one (the units that work alone run
// faster): cost(w) = floor(w) + (0.6 + 0.4 frac(w) if frac(w) > 0), and the small tile's cost in the
// same unit is cost(2 w) / 2.  On 75 measured cases (12 shapes, 768 - 8192 tokens) the rule below is
// within 0.3 % of the better tile on average and never more than 4 % off; "small tile up to 2048
// tokens" was 2.5 % off on average and up to 15 %.
bool plain_takes_large_tile(int64_t large_tiles, int64_t slab_tokens, int compute_units) {
  const double cus = compute_units > 0 ? compute_units : kDefaultComputeUnits;
  if (large_tiles <= (int64_t)(cus / 2)) return false;          // too few tiles to fill the device: twice as many small ones
  const double w = (double)large_tiles / cus;
  const double round_ratio = 0.83 + 160.0 / (double)(slab_tokens > 0 ? slab_tokens : 1);
  return round_ratio * round_cost(w) / (round_cost(2.0 * w) / 2.0) < 0.99;
}

// Which tile the fused call takes.  Its AdamW epilogue is HBM-bound and overlaps the partner's loop
// only on the small tile, so the large tile pays only when the loops dominate: the ratio of the large tile's time
// to the small one's on fully filled rounds was fitted by 0.55 + 2600 / T, and partly filled rounds are priced as for the plain
// gradient, before either tile's update took its present form (the small one's requests its state ahead up to 1024 tokens, the
// large one's always, and no unit of it starts late).  With the present kernels the rule is within 3 % of the faster tile in 49 of 54
// measured cases (nine shapes of 1 - 16 rounds, 2048 - 8192 tokens).  In the other five, of many rounds at 4096 - 6144 tokens, it takes the small tile
// where the large one is ahead: 256 Mi of 4096-wide rows 4096 tokens 2642 / 2563 us, 5120 tokens 3100 / 2909, 200 Mi of 8192-wide 5120 tokens 2340 / 2265 and 6144 tokens
// 2796 / 2605, 100 Mi of 14336-wide 6144 tokens 1534 / 1380.  (32 Mi of 4096-wide rows, small / large: 3072 tokens 261 / 312, 5120 365 / 398, 6144
// 419 / 426, 8192 542 / 510.)
bool fused_takes_large_tile(const WgradProblem& p, int compute_units) {
  const double cus = compute_units > 0 ? compute_units : kDefaultComputeUnits;
  const RowSplit rs = split_rows(p);
  const int64_t rows = rs.rb1 > rs.rb0 ? rs.rb1 - rs.rb0 : 0;
  const int64_t tiles = ceil_div(rows, kMainTileM) * ceil_div(p.in, kMainTileN) * (p.S > 0 ? p.S : 1);
  if (tiles <= (int64_t)(cus / 2)) return false;
  const int64_t slab_tokens = p.S > 1 ? p.kslab : p.T;
  const double w = (double)tiles / cus;
  const double round_ratio = 0.55 + 2600.0 / (double)(slab_tokens > 0 ? slab_tokens : 1);
  return round_ratio * round_cost(w) / (round_cost(2.0 * w) / 2.0) < 0.99;
}

// Whether the update on 128-row tiles requests its state ahead (tile_epilogue in kernels.hip): where the update's streams
// decide and not the loops.  The lines are where measurements cross, per width and not per size: up to 1024 tokens, 768 on rows of more
// than 8192 elements.  Fused call in us, without / with, each at its start delay:
//   4096-wide rows, 32 Mi elements 256 tokens 163.4 / 159.4, 512 176.8 / 167.3, 1024 182.5 / 179.5, 1300 192.7 / 187.8, 1500 195.8 / 196.1,
//   2048 218.5 / 222.8; 64 Mi 1024 341 / 329, 24 Mi 1024 137.8 / 140.3 (the most that it costs below the line);
//   8192-wide, 64 Mi 1024 tokens 342.5 / 336.1, 40 Mi 1024 227.0 / 227.2, 48 Mi 1150 280.8 / 281.7, 1500 292 / 297;
//   14336-wide, 24 Mi 64 tokens 154.3 / 149.8, 1024 181.1 / 178.8, 30 Mi 1300 201 / 203, 40 Mi 2048 309 / 327, 50 Mi 1024 310 / 314.
// (At 1300 tokens 4096-wide rows would still gain, at 1150 8192-wide ones no longer: the line keeps to what both gain from.)
bool update_requests_ahead(int64_t in, int64_t tokens) { return tokens <= (in <= 8192 ? 1024 : 768); }

// A group up to 1024 tokens whatever the widths of its segments.  Planner chunks of a block in us, without / with: 4096-wide under
// 256 MiB 300 tokens 1062 / 1032, 1024 tokens 1110 / 1105; under 128 MiB 1184 / 1165; 2048-wide 1024 tokens 352 / 340; 3072-wide 622 / 612; 4096-wide
// with 11008 1009 / 997; groups of 14336-wide segments at 1024 tokens 179.8 / 180.4, 333.8 / 328.8, 637 / 629.
bool group_requests_ahead(int64_t tokens) { return tokens <= 1024; }

int64_t countable_run(int64_t in, int32_t S, int64_t bm, int64_t bn, int threads) {
  const int64_t tiles = kMaxLaunchThreads / threads / 8 * 8 / S;             // the grid is a multiple of the 8 XCDs
  const int64_t rows = tiles / ceil_div(in, bn) * bm - 8;      // a run of whole rows touches one more; the first tile may begin 7 earlier
  return rows <= 0 ? 0 : rows <= INT64_MAX / in ? rows * in : INT64_MAX;
}

// A row group as one workgroup or as four.  A part of 16 rows evens out the device and spreads the rows that many tokens
// name; what it repeats is the pass over the ids.  Times in us, one / four parts, of the update, the gradient, the gradient
// added to g; ids heavy-tailed as in text unless said otherwise:
//   The update takes four from 448 columns on, where 26 bytes per element outweigh the pass: 128 Mi elements of 128256 x
//   4096, 4096 tokens 665 / 631; 50257 x 768 227 / 199; 300000 rows, 64 and 4096 uniform ids: 512 wide 510 / 463 and 510 /
//   473, 448 wide 448 / 390 and 445 / 429, 384 wide 554 / 517 and 563 / 600, 320 wide 463 / 460 and 481 / 572, 93 wide 264 / 326.
//   Any call takes four when one would leave compute units without a group: 8000 x 512 (125 groups) 53 / 45, 42 / 36,
//   33 / 35; 2000 x 64, 8192 tokens 31 / 15, 27 / 14, 28 / 14; 300 x 4096, 8192 tokens 653 / 311, 612 / 304, 628 / 308.
//   The gradient also where two groups a compute unit meet eight or more tokens each: 32 Mi of 32000 x 4096 111 / 67, 77 / 48;
//   4000 x 8192 340 / 162, 345 / 163; 32000 x 1024 107 / 85, 64 / 62 (uniform ids 36 / 57, 28 / 50).  Else one: 128 Mi of 128256 x
//   4096 179 / 244, 64 / 140; 50257 x 768 65 / 90, 41 / 72; 111484 x 1137, 4 tokens 19 / 26, 6 / 9.
// Where a launch cannot count the threads of four parts (2^21 row groups, 128 Mi narrow rows) it is one; the sums are the
// same either way.
int embed_parts(bool update, int64_t groups, int64_t rows, int64_t in, int64_t T, int compute_units) {
  const int64_t cus = compute_units > 0 ? compute_units : kDefaultComputeUnits, most = kMaxLaunchThreads / kEmbedThreads;
  if (groups > most) return 0;
  if (groups > most / 4) return 1;
  if (groups <= cus) return 4;
  return update ? (in >= 448 ? 4 : 1) : groups <= cus * 9 / 4 && T >= rows / 8 ? 4 : 1;
}

Split pick_split(int32_t kind, int32_t dtype, int64_t out, int64_t in, int64_t T, int64_t begin,
                 int64_t end, int32_t forced, bool mfma, int compute_units) {
  (void)out; (void)dtype;
  if (kind != 0) return {1, T};                       // only linear layers are ever split
  const int64_t bk = mfma ? kMainTileK : kOtherTileK;
  int64_t S = forced;
  if (S <= 0 && mfma && takes_small_tiles(in, T, begin, end, compute_units)) {
    // Small tiles: a workgroup needs about 0.2 us per 32 tokens while no more than 1.6 of them share a
    // compute unit, in proportion longer beyond; a split costs 4 us for the reduction's launch and 8
    // bytes per element and slab at 5 TB/s.  The cheapest S up to 8 with at least 512 tokens per slab is within
    // 15 % of the best of 1 - 32 slabs in 30 measured cases (16 - 576 tiles, 1024 - 8192 tokens), e.g. 80 tiles,
    // 4096 tokens: 16 us with 5 or 6 slabs against 27 with one; 272 tiles, 2048 tokens: 19 with one, 21 with two.
    // In a long slab it needs 0.27 us per 32 (one slab, 256 tiles: 14 us at 2100 tokens, 16 at 2500, 26 at 3000, 34 at 4096; with rows
    // that are not whole 128-byte lines 20, 25, 30): the fused call on 260 tiles at 3000 tokens takes 34 us with one slab, 27
    // with two, 30 on the large tiles.
    const double tiles = (double)small_tiles(in, begin, end), elems = (double)(end - begin);
    const double room = 1.6 * (compute_units > 0 ? compute_units : kDefaultComputeUnits);
    const int64_t long_slab = in % 64 == 0 ? 2688 : 2304;
    double best = 0.0;
    for (int64_t k = 1; k <= 8 && (k == 1 || T / k >= 512); ++k) {
      const double crowd = tiles * (double)k / room, per32 = tiles <= room && T / k > long_slab ? 0.27 : 0.2;
      const double cost = per32 * (double)T / 32.0 / (double)k * (crowd > 1.0 ? crowd : 1.0) +
                          (k > 1 ? 4.0 + (double)k * elems * 8.0 / 5e6 : 0.0);
      if (k == 1 || cost < best) {
        best = cost;
        S = k;
      }
    }
  }
  if (S <= 0 && mfma) {
    WgradProblem tmp{};                               // the large tiles hold the body rows
    tmp.begin = begin;
    tmp.end = end;
    tmp.in = in;
    const RowSplit rs = split_rows(tmp);
    const int64_t rows = rs.rb1 > rs.rb0 ? rs.rb1 - rs.rb0 : 1;
    const int64_t tiles = ceil_div(rows, kMainTileM) * ceil_div(in, kMainTileN);
    const int64_t slots = compute_units > 0 ? compute_units : kDefaultComputeUnits;   // resident workgroups
    S = 1;
    if (tiles <= slots / 4) {
      // Splitting pays only when the 256 x 256 tiles fill at most a quarter of the compute units.
      // A slab costs its tokens' share of the loop, every further slab 8 bytes per element of
      // partial traffic plus one more set-up and epilogue per tile: time ~ a T / S + b S tiles,
      // least at S = sqrt(a T / (b tiles)).  a / b = 1 / 12 fits the measured grid (16 - 192
      // tiles x 1024 - 8192 tokens x 1 - 16 slabs, plain and fused call, in = 4096); more than 8
      // slabs never won, and from 128 tiles on one slab is best.
      while ((S + 1) * (S + 1) * 12 * tiles <= T && S < 8) ++S;
      if (S > slots / tiles) S = slots / tiles;
      if (S > T / 256) S = T / 256 > 0 ? T / 256 : 1;    // never slabs of fewer than 256 tokens
    }
  }
  if (S <= 0) S = 1;                                  // fp32 and ragged layers are split only on request
  int64_t kslab = ceil_div(ceil_div(T, S), bk) * bk;
  S = ceil_div(T, kslab);                             // no empty slab
  return {(int32_t)S, kslab};
}

}  // namespace chunkft
