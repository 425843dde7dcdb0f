// Host-side walk of the preprocessing kernels' tiles through their index functions:
// the float and 8-bit kernels on 16 x 64 and 8 x 32 tiles, the matrix kernel on 8 x
// 64 and 8 x 32.  Every access inside its array, every cell made once, every pixel
// owned once, and the launch grid of any number of tiles.
#include <cstdio>
#include <vector>

#include "dsgm_geom.h"

namespace g = dsgm::geom;
namespace pre = dsgm::geom::pre;
static int bad = 0;
#define CHECK(c, ...)               \
  do {                              \
    if (!(c) && bad++ < 10) {       \
      std::printf("FAIL %s: ", #c); \
      std::printf(__VA_ARGS__);     \
      std::printf("\n");            \
    }                               \
  } while (0)

using Marks = std::vector<int>;
static void once(const Marks& v, const char* what) {
  for (size_t i = 0; i < v.size(); ++i) CHECK(v[i] == 1, "%s %zu made %d times", what, i, v[i]);
}
static void mark(Marks& v, int i, const char* what) {
  CHECK(i >= 0 && size_t(i) < v.size(), "%s %d outside", what, i);
  if (i >= 0 && size_t(i) < v.size()) ++v[size_t(i)];
}

// the cells of one tile in the float kernel and the 8-bit single-precision kernel
template <int RG, bool MED, typename Tile>
static void cells() {
  using G = pre::Geo<RG, MED, Tile>;
  Marks raw(G::RAW_N, 0), hb(G::HB_N, 0), gb(G::GB_N, 0), gb8(G::GB_N, 0);
  for (int tid = 0; tid < pre::NT; ++tid) {
    for (int l = 0; l < G::LOADS; ++l)
      if (G::raw_active(tid, l)) mark(raw, G::raw_cell(tid, l), "raw cell");
    // a lane's pairs of a round are adjacent in one row, from one window
    for (int rd = 0; rd < G::ROW_ROUNDS; ++rd) {
      const int p0 = G::row_pair(tid, rd * G::ROW_SEG);
      if (!G::row_active(tid, rd * G::ROW_SEG)) continue;
      const int w0 = G::row_window(p0), outs = 2 * G::ROW_SEG;
      CHECK(w0 / G::RAW_W == (2 * p0) / G::HB_W && w0 % G::RAW_W == (2 * p0) % G::HB_W, "window %d", w0);
      CHECK(w0 % G::RAW_W + outs + 2 * RG - 1 < G::RAW_W, "window %d leaves its row", w0);
      CHECK((2 * p0) % G::HB_W + outs <= G::HB_W, "pairs %d leave their row", p0);
      for (int o = 0; o < outs; ++o) mark(hb, 2 * p0 + o, "row output");
    }
    if (G::col_active(tid, 0)) {
      const int c0 = 2 * G::col_pair(tid, 0);
      CHECK(c0 + (G::COL_IT + 2 * RG - 1) * G::HB_W + 1 < G::HB_N, "column input of %d", c0);
      for (int it = 0; it < G::COL_IT; ++it) {
        CHECK(G::col_active(tid, it) && 2 * G::col_pair(tid, it) == c0 + it * G::GB_W, "column pair %d", it);
        for (int c = 0; c < 2; ++c) mark(gb, c0 + it * G::GB_W + c, "column output");
      }
    }
    for (int it = 0; it < G::GB_IT; ++it) {
      if (!G::gb_active(tid, it)) continue;
      const int cell = G::gb_cell(tid, it);
      mark(gb8, cell, "blurred cell");
      CHECK(G::blur_window(cell) + 2 * RG * G::RAW_W + 2 * RG < G::RAW_N, "window of cell %d", cell);
    }
  }
  once(raw, "raw cell");
  if (RG > 0) {
    once(hb, "row output");
    once(gb, "column output");
    once(gb8, "blurred cell");
  }
}

// the tiles of a frame: sources, medians, owners
template <int RG, bool MED, typename Tile>
static void frame(int64_t H, int64_t W, int64_t rs) {
  using G = pre::Geo<RG, MED, Tile>;
  const int64_t nx = (W + G::TW - 1) / G::TW, ny = (H + G::TH - 1) / G::TH;
  Marks owner(size_t(H * W), 0);
  for (int64_t b = 0; b < nx * ny; ++b) {
    const int64_t tile = g::tile_of(b, nx * ny), y0 = tile / nx * G::TH, x0 = tile % nx * G::TW;
    for (int tid = 0; tid < pre::NT; ++tid) {
      for (int l = 0; l < G::LOADS; ++l) {
        if (!G::raw_active(tid, l)) continue;
        const int64_t o = G::raw_source(G::raw_cell(tid, l), y0, x0, H, W, rs);
        CHECK(o >= 0 && o < (H - 1) * rs + W, "source %lld", (long long)o);
      }
      const int64_t gy = y0 + G::lane_row(tid), gx = x0 + G::lane_col(tid);
      for (int d = 0; d < 3; ++d) {
        const int r = G::med_row(gy, d, y0, H);
        CHECK(!MED || (r >= 0 && r < G::GB_H), "median row %d", r);
      }
      for (int d = 0; d < G::PX + 2; ++d) {
        const int c = G::med_col(gx, d, x0, W);
        CHECK(!MED || (c >= 0 && c < G::GB_W), "median column %d", c);
      }
      for (int q = 0; q < G::PX; ++q)
        if (gy < H && gx + q < W) mark(owner, int(gy * W + gx + q), "pixel");
    }
  }
  once(owner, "pixel");
}

// the matrix kernel's tile
template <int RG, bool MED, typename Tile>
static void matrix() {
  using E = pre::Geo8<RG, MED, Tile>;
  using G = typename E::G;
  constexpr int RAW = G::RAW_H * E::RP, GB = G::GB_H * E::GBP;
  Marks slot(size_t(RAW), 0);
  for (int tid = 0; tid < pre::NT; ++tid)
    for (int l = 0; l < E::LD; ++l)
      if (E::staged(tid, l)) {
        CHECK(E::stage_cell(tid, l) < E::CELLS, "staged dword %d", E::stage_cell(tid, l));
        mark(slot, E::stage_slot(E::stage_cell(tid, l)), "slot");
      }
  for (int r = 0; r < G::RAW_H; ++r)
    for (int c = 0; c < E::RP; ++c)
      CHECK(slot[size_t(r * E::RP + c)] == (c < E::DW ? 1 : 0), "slot (%d, %d)", r, c);
  auto read = [&](int i, int n) { CHECK(i >= 0 && i + n <= RAW, "raw dwords %d + %d", i, n); };
  auto in_row = [&](int i, int row) { CHECK(i / E::RP == row, "dword %d not in row %d", i, row); };
  Marks made(size_t(GB), 0), quad(size_t(GB), 0);
  for (int grp = 0; grp < E::GROUPS; ++grp)
    for (int m = 0; m < 16; ++m)
      for (int rgrp = 0; rgrp < 4; ++rgrp) {
        const int win = grp * 16 + m, wr = E::win_row(win), wc = E::win_col(win);
        for (int st = 0; st < E::SETS; ++st) {
          read(E::win_src(wr, wc, 4 * st + rgrp), 4);
          in_row(E::win_src(wr, wc, 4 * st + rgrp) + 3, wr + (4 * st + rgrp < E::N ? 4 * st + rgrp : E::N - 1));
        }
        const bool mine = E::takes(win, rgrp);
        // the undecided cells' own windows (a lane without any: the window's first)
        for (int i = 0; i < (mine ? 4 : 1); ++i) {
          const int col = mine ? wc + 4 * rgrp + i : wc;
          for (int y = 0; y < E::N; ++y) {
            read(E::cell_src(wr, col) + y * E::RP, E::N > 5 ? 3 : 2);
            in_row(E::cell_src(wr, col) + y * E::RP + (E::N > 5 ? 2 : 1), wr + y);
          }
          if (mine && col < G::GB_W)
            CHECK(col + E::N - 1 < 4 * E::DW, "cell %d reads beyond the staged columns", col);
        }
        if (mine)
          for (int i = 0; i < 4; ++i) mark(made, E::win_dst(wr, wc, rgrp) + i, "cell");
      }
  for (int c = 0; c < E::QUADS; ++c) {
    for (int y = 0; y < E::N; ++y) {
      read(E::quad_src(c) + y * E::RP, (E::N + 6) / 4);
      in_row(E::quad_src(c) + y * E::RP + (E::N + 6) / 4 - 1, c / E::QR + y);
    }
    CHECK(E::quad_dst(c) % 4 == 0, "unaligned store %d", E::quad_dst(c));
    for (int i = 0; i < 4; ++i) mark(quad, E::quad_dst(c) + i, "quad cell");
  }
  for (int r = 0; r < G::GB_H; ++r)
    for (int c = 0; c < E::GBP; ++c) {
      const size_t i = size_t(r * E::GBP + c);
      CHECK(c < G::GB_W ? made[i] == 1 : made[i] <= 1, "cell (%d, %d) made %d times", r, c, made[i]);
      CHECK(c < G::GB_W ? quad[i] == 1 : quad[i] <= 1, "cell (%d, %d) summed %d times", r, c, quad[i]);
    }
}

// the staged bytes' sources at the corners of a frame of any size
template <int RG, bool MED, typename Tile>
static void sources(int64_t H, int64_t W, int64_t rs) {
  using E = pre::Geo8<RG, MED, Tile>;
  using G = typename E::G;
  const int64_t nx = (W + G::TW - 1) / G::TW, ny = (H + G::TH - 1) / G::TH;
  for (const int64_t ty : {int64_t(0), ny / 2, ny - 1})
    for (const int64_t tx : {int64_t(0), nx / 2, nx - 1})
      for (int i = 0; i < E::CELLS; ++i)
        for (int b = 0; b < 4; ++b) {
          const int64_t y0 = ty * G::TH, x0 = tx * G::TW;
          const int64_t o = E::stage_source(i, b, y0, x0, H, W, rs);
          CHECK(o >= 0 && o < (H - 1) * rs + W && o < (int64_t(1) << 31), "source %lld", (long long)o);
          const int64_t x = x0 - G::R + 4 * (i % E::DW) + b;  // clamped to the nearest column
          CHECK(o % rs == (x < 0 ? 0 : x >= W ? W - 1 : x), "column %lld from %lld", (long long)x, (long long)(o % rs));
          if (E::inner(x0, W))
            CHECK(o == E::stage_source(i, 0, y0, x0, H, W, rs) + b, "inner dword %d", i);
        }
}

template <int RG, bool MED>
static void all() {
  const int64_t shapes[][3] = {{1, 1, 1}, {8, 32, 32}, {16, 64, 64}, {9, 33, 40}, {37, 150, 150}, {70, 99, 99}};
  cells<RG, MED, pre::Big>();
  cells<RG, MED, pre::Small>();
  for (const auto& s : shapes) {
    frame<RG, MED, pre::Big>(s[0], s[1], s[2]);
    frame<RG, MED, pre::Small>(s[0], s[1], s[2]);
    frame<RG, MED, pre::Wide>(s[0], s[1], s[2]);
  }
  if constexpr (RG > 0) {
    matrix<RG, MED, pre::Wide>();
    matrix<RG, MED, pre::Small>();
    const int64_t M = (int64_t(1) << 31) - 1;
    const int64_t big[][3] = {{1, 1, 1}, {5, 3, 3}, {37, 150, 160}, {1, M, M}, {M, 1, 1}, {2, M / 2, M / 2}};
    for (const auto& s : big) {
      sources<RG, MED, pre::Wide>(s[0], s[1], s[2]);
      sources<RG, MED, pre::Small>(s[0], s[1], s[2]);
    }
  }
}

// every tile has one workgroup of the grid, and no dimension reaches 2^32 lanes
static void grids() {
  for (const int64_t n : {int64_t(1), int64_t(300), pre::GRID_X - 1, pre::GRID_X, pre::GRID_X + 1, 3 * pre::GRID_X + 7,
                          (int64_t(1) << 28), (int64_t(1) << 31) - 1}) {
    const int64_t x = pre::grid_x(n), y = pre::grid_y(n);
    CHECK(x * pre::NT < (int64_t(1) << 32) && y < 65536 && x * y >= n && x * (y - 1) < n, "grid of %lld", (long long)n);
    CHECK(pre::workgroup(x - 1, y - 1, x) == x * y - 1 && pre::workgroup(0, y - 1, x) < n, "last row");
    for (const int64_t b : {int64_t(0), n / 2, n - 1})
      CHECK(g::tile_of(b, n) >= 0 && g::tile_of(b, n) < n, "tile of %lld", (long long)b);
  }
}

int main() {
  all<0, true>();
  all<0, false>();
  all<1, true>();
  all<1, false>();
  all<2, true>();
  all<2, false>();
  all<3, true>();
  all<3, false>();
  grids();
  std::printf(bad ? "%d failures\n" : "OK\n", bad);
  return bad != 0;
}
