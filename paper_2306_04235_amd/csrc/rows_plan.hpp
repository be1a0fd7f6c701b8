// rows_plan.hpp -- rows per block and LDS layout of the row-wise decoder's
// launches (decode_rows.hip): plain host arithmetic, no device code.
#pragma once

namespace mnmt {

constexpr int kRowsMaxLds = 160 * 1024;
constexpr int kVtStride = 17;  // dwords per column of the transposed values (odd: no bank conflicts)
constexpr int kVtBytes = 64 * kVtStride * 4;

// Waves of a block: they divide the 16-column tiles of every linear layer.
constexpr int rows_waves(int d) { return d == 64 ? 4 : d == 128 ? 8 : d == 384 ? 12 : 16; }

// LDS layout, sized by the host for the launch (byte offsets, 16-aligned).
struct RowsLds {
  int ln, a, hist, act, p, total;  // LayerNorm constants, int8 input rows, cache-row history, q|k|v rows, the waves'
                                   // attention scratch; the hidden rows lie over the last two
  int np;                          // softmax weights per wave
};

struct RowsSizes {
  int R, d, h, F, T, S;  // rows, widths and heads, cache positions, source positions
  int t;                 // position of the step; < 0: any below T
};

struct RowsPlan {
  int rows, blocks;  // rows per block
  RowsLds lds;
};

inline RowsLds rows_lds(const RowsSizes& g, int RB) {
  auto align16 = [](int v) { return (v + 15) / 16 * 16; };
  RowsLds l{};
  const int own = g.t < 0 ? g.T : g.t + 1, keys = own > g.S ? own : g.S, w = rows_waves(g.d);
  l.np = (keys + 63) / 64 * 64;
  l.ln = align16(RB * (g.d + 4) * 4);
  l.a = l.ln + 24 * g.d;
  l.hist = align16(l.a + RB * (g.d + 16));
  l.act = align16(l.hist + RB * ((g.T + 63) / 64 * 64));
  l.p = align16(l.act + RB * (3 * g.d + 16));
  const int att = l.p + (RB * g.h < w ? RB * g.h : w) * (l.np * 4 + kVtBytes), hid = l.act + RB * (g.F + 16);
  l.total = att > hid ? att : hid;
  return l;
}

// Rows per block: the grid reaches 256 blocks (one per CU) with as few rows
// per block as possible, up to the 16 rows of a tile, the waves of a block
// (one LayerNorm row each) and the LDS of a CU; past that, the fewest rounds
// of 256 blocks, evenly filled (4096 rows of the base model: two rounds of 8
// rows against a full and a nearly empty one of 11).
inline RowsPlan rows_plan(const RowsSizes& g) {
  int most = rows_waves(g.d);
  while (most > 1 && rows_lds(g, most).total > kRowsMaxLds) --most;
  const int rounds = (g.R + 256 * most - 1) / (256 * most);
  RowsPlan p{};
  p.rows = (g.R + 256 * rounds - 1) / (256 * rounds);
  p.blocks = (g.R + p.rows - 1) / p.rows;
  p.lds = rows_lds(g, p.rows);
  return p;
}

}  // namespace mnmt
