// What the gradient kernels without an edge-row path share: a grid of tiles over the rows that a chunk
// touches, with every element masked by the chunk's range as it leaves.
#ifndef CHUNKFT_TILES_H
#define CHUNKFT_TILES_H

#include "device.h"
#include "internal.h"
#include "launch.h"

namespace chunkft {

struct TileGrid {
  WgradProblem p;
  int64_t r0;                  // first row of the grid
  int32_t tiles_m, tiles_n, n_items, group_m;
  Sinks s;
};

// The grid of BM x BN tiles from a multiple of row_step on.  False if its items cannot be counted in 32 bits.
template <int BM, int BN>
bool fill_grid(TileGrid& q, const WgradProblem& p, const Sinks& s, int64_t row_step) {
  q = TileGrid{};
  q.p = p;
  q.s = s;
  q.r0 = p.begin / p.in / row_step * row_step;
  const int64_t rows = (p.end - 1) / p.in - q.r0 + 1;
  const int64_t tiles_m = ceil_div(rows, BM), tiles_n = ceil_div(p.in, BN);
  if (tiles_m > 0x3fffffff || tiles_n > 0x3fffffff || tiles_m * tiles_n > 0x3fffffff / p.S) return false;
  q.tiles_m = (int32_t)tiles_m;
  q.tiles_n = (int32_t)tiles_n;
  q.n_items = (int32_t)(tiles_m * tiles_n * p.S);
  q.group_m = 8;
  return true;
}

// Which tile and which tokens a workgroup takes.
struct Place {
  int64_t row0, col0;          // first row and column that this tile emits
  int64_t row_b, col_b;        // first row and column that it loads
  int64_t k_begin, k_end;      // tokens of its slab
  int slab;
};

template <int BM, int BN>
__device__ __forceinline__ Place place_of(const TileGrid& q, int item) {
  const WgradProblem& p = q.p;
  Place w;
  const int n_tiles = q.tiles_m * q.tiles_n;
  w.slab = item / n_tiles;
  const int tile = item - w.slab * n_tiles;
  // tile order inside an XCD's run of items as in the bf16 kernel: groups of tile rows
  const int per_group = q.group_m * q.tiles_n;
  const int first_m = tile / per_group * q.group_m;
  const int gsz = (q.tiles_m - first_m < q.group_m) ? q.tiles_m - first_m : q.group_m;
  const int in_grp = tile % per_group;
  w.row0 = q.r0 + (int64_t)(first_m + in_grp % gsz) * BM;
  w.col0 = (int64_t)(in_grp / gsz) * BN;
  // A tile that would reach past the tensor is moved back inside it (the rows and columns it then shares
  // with its neighbour are not emitted); where the tensor is smaller than a tile the lanes past its end
  // re-read the last row or column.
  w.row_b = (w.row0 + BM > p.out && p.out >= BM) ? p.out - BM : w.row0;
  w.col_b = (w.col0 + BN > p.in && p.in >= BN) ? p.in - BN : w.col0;
  w.k_begin = (int64_t)w.slab * p.kslab;
  w.k_end = (w.k_begin + p.kslab < p.T) ? w.k_begin + p.kslab : p.T;
  return w;
}

// Sends ROWS staged rows of BN columns (row pitch PITCH; the sum of PARTS such areas, in order) to their
// destination: four columns per lane, up to four groups of them per trip so that their state loads travel
// together.  row_of maps a staged row to its row of the tile.
template <int MODE, int ROWS, int BN, int PITCH, int NT, int PARTS, class RowOf>
__device__ __forceinline__ void emit_rows(const TileGrid& q, const Place& w, const float* staged, RowOf&& row_of) {
  const WgradProblem& p = q.p;
  const int64_t E = p.end - p.begin;
  float* const g_dst = MODE == EMIT_PARTIAL ? q.s.ws + (int64_t)w.slab * q.s.ws_pitch : q.s.g;
  constexpr int LPR = BN / 4, GROUPS = ROWS * LPR;
  constexpr int STEP = GROUPS < NT ? 1 : (GROUPS / NT < 4 ? GROUPS / NT : 4);
  static_assert(GROUPS < NT || GROUPS % (NT * STEP) == 0, "whole trips");
  for (int o = threadIdx.x; o < GROUPS; o += NT * STEP) {
    Vec4Sink d[STEP];
    State4 st[STEP];
    bool whole[STEP], some[STEP];
    int64_t flat[STEP];
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
      const int rr = (o + u * NT) / LPR, cc = (o + u * NT) % LPR * 4;
      const int64_t row = w.row_b + row_of(rr), col = w.col_b + cc;
      flat[u] = row * p.in + col;
      some[u] = row >= w.row0 && row < p.out && flat[u] < p.end && flat[u] + 4 > p.begin && col < p.in && col + 4 > w.col0;
      whole[u] = some[u] && flat[u] >= p.begin && flat[u] + 4 <= p.end && col >= w.col0 && col + 4 <= p.in;
      const int64_t i = flat[u] - p.begin;
      d[u].g = g_dst + i;
      d[u].master = q.s.master + i;
      d[u].m = q.s.m + i;
      d[u].v = q.s.v + i;
      d[u].W = q.s.w_kind == W_BF16 ? (void*)((unsigned short*)q.s.W + flat[u]) : (void*)((float*)q.s.W + flat[u]);
      if (whole[u]) st[u] = load_state4<MODE>(d[u]);
    }
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
      if (!some[u]) continue;
      const int rr = (o + u * NT) / LPR, cc = (o + u * NT) % LPR * 4;
      const float* src = staged + rr * PITCH + cc;
      float4 val = *(const float4*)src;
#pragma unroll
      for (int k = 1; k < PARTS; ++k) {
        const float4 x = *(const float4*)(src + k * (ROWS * PITCH));
        val.x += x.x; val.y += x.y; val.z += x.z; val.w += x.w;
      }
      if (whole[u]) {
        finish4<MODE>(d[u], q.s.w_kind, q.s.c, f32x4_u{val.x, val.y, val.z, val.w}, st[u]);
      } else {
        const float e4[4] = {val.x, val.y, val.z, val.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t col = w.col_b + cc + e, f = flat[u] + e;
          if (col >= w.col0 && col < p.in && f >= p.begin && f < p.end)
            emit<MODE>(q.s, E, w.slab, f - p.begin, f, e4[e]);
        }
      }
    }
  }
}

}  // namespace chunkft
#endif
