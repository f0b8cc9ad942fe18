// Tile schedule of the fused loss-head projection: plain constexpr integer
// functions (no HIP types), so that the same definitions compile for the GPU
// and, in the tests, with the host C++ compiler.
#pragma once

#include "attn_sched.h"

namespace cattn {

constexpr int kLmhTileV = 256;  // vocabulary rows per output tile
constexpr int kLmhTileM = 256;  // tokens per output tile
constexpr int kLmhKC = 32;      // K chunk per ring slot
constexpr int kLmhPartW = 64;   // vocabulary entries per partial statistic

constexpr int lmh_vtiles(int N) { return (N + kLmhTileV - 1) / kLmhTileV; }
constexpr int lmh_mtiles(int M) { return (M + kLmhTileM - 1) / kLmhTileM; }

// Output tiles whose vocabulary tile index is congruent to x modulo kXcdGroup:
// the tiles of chiplet x (work groups are dealt to the chiplets round-robin).
constexpr int lmh_xcd_vtiles(int x, int n_vt) { return x < n_vt ? (n_vt - x + kXcdGroup - 1) / kXcdGroup : 0; }
constexpr int lmh_xcd_tiles(int x, int n_vt, int n_mt) { return lmh_xcd_vtiles(x, n_vt) * n_mt; }

// The l-th tile (0 <= l < lmh_xcd_tiles) of chiplet x, as (vocabulary tile,
// token tile) packed into vt * 65536 + mt.  A chiplet walks its vocabulary
// tiles in bands of 8 with the token tiles inside and the vocabulary index
// fastest, so that the tiles it runs at once share a few W and X row blocks
// (its L2 holds them).
constexpr int lmh_xcd_tile(int x, int l, int n_vt, int n_mt) {
  const int nv = lmh_xcd_vtiles(x, n_vt);
  const int vb = l / (8 * n_mt);
  const int g = imin(8, nv - 8 * vb);
  const int rem = l - vb * 8 * n_mt;
  const int mt = rem / g;
  const int vt = x + kXcdGroup * (8 * vb + rem % g);
  return vt * 65536 + mt;
}

// Work items of chiplet x for per_xcd work groups.  Whole tiles fill as many
// complete rounds of the work groups as there are; the R < per_xcd tiles left
// over would occupy only R of them for another whole tile's time, so each is
// cut into f parts (the largest f of 8, 4, 2, 1 with R f <= per_xcd): halves
// of the vocabulary first, then halves and quarters of the tokens.  A wave
// keeps its place in the tile, so that 8 / f of the eight waves have work, each
// as much as in a whole tile, and all of them copy as many rows: a part costs
// about 0.4 of a tile whatever f > 2.  1024 x 50304 x 1600 (788 tiles on 256 work groups): 195 us
// with four rounds of whole tiles, 178 with three and a round of parts; 2944 x
// 10496 x 704 75.5 / 68.2, 128 x 18432 x 1408 30.3 / 26.8.
constexpr int lmh_cut(int tiles, int per_xcd) {
  const int rest = tiles % per_xcd;
  int f = 1;
  while (rest > 0 && f < 8 && rest * f * 2 <= per_xcd) f *= 2;
  return f;
}
constexpr int lmh_xcd_items(int tiles, int per_xcd) {
  const int rest = tiles % per_xcd;
  return tiles - rest + rest * lmh_cut(tiles, per_xcd);
}
// Item i: rows v0 .. v0 + v_ext - 1 of the vocabulary, m0 .. m0 + m_ext - 1 of
// the tokens (some may lie past the end).
struct LmhItem {
  int v0, m0, v_ext, m_ext;
};
constexpr LmhItem lmh_xcd_item(int x, int i, int n_vt, int n_mt, int per_xcd) {
  const int tiles = lmh_xcd_tiles(x, n_vt, n_mt), whole = tiles - tiles % per_xcd;
  const int f = i < whole ? 1 : lmh_cut(tiles, per_xcd);
  const int l = i < whole ? i : whole + (i - whole) / f;
  const int part = i < whole ? 0 : (i - whole) % f;
  const int tile = lmh_xcd_tile(x, l, n_vt, n_mt);
  const int fv = f > 1 ? 2 : 1, v_ext = kLmhTileV / fv, m_ext = kLmhTileM / (f / fv);
  return LmhItem{(tile >> 16) * kLmhTileV + part % fv * v_ext, (tile & 0xffff) * kLmhTileM + part / fv * m_ext, v_ext,
                 m_ext};
}

// Persistent grid: work group b runs on chiplet b % kXcdGroup and takes that
// chiplet's items b / kXcdGroup, b / kXcdGroup + per_xcd, ... where per_xcd is
// the number of work groups per chiplet (the grid has kXcdGroup * per_xcd).
constexpr int lmh_grid(int n_wg_per_xcd) { return kXcdGroup * n_wg_per_xcd; }

}  // namespace cattn
