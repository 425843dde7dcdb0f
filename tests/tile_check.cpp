// Host-side check of the 8 x 32 preprocessing tiles (geometry_check.cpp walks the
// 16 x 64 ones): every lane of every tile through the kernel's index functions.
#include <cstdio>
#include <vector>

#include "dsgm_geom.h"

namespace g = dsgm::geom;
static int bad = 0;
#define CHECK(c, ...)                    \
  do {                                   \
    if (!(c) && bad++ < 10) {            \
      std::printf("FAIL %s: ", #c);      \
      std::printf(__VA_ARGS__);          \
      std::printf("\n");                 \
    }                                    \
  } while (0)

template <int RG, bool MED>
static void check(int64_t H, int64_t W, int64_t rs) {
  using G = g::pre::Geo<RG, MED, g::pre::Small>;
  const int64_t tx_n = (W + G::TW - 1) / G::TW, ty_n = (H + G::TH - 1) / G::TH;
  std::vector<int> owner(size_t(H * W), 0);
  for (int64_t tile = 0; tile < tx_n * ty_n; ++tile) {
    const int64_t y0 = tile / tx_n * G::TH, x0 = tile % tx_n * G::TW;
    std::vector<int> raw(G::RAW_N, 0), hb(G::HB_N, 0), gb(G::GB_N, 0);
    for (int tid = 0; tid < g::pre::NT; ++tid) {
      for (int l = 0; l < G::LOADS; ++l) {
        if (!G::raw_active(tid, l)) continue;
        const int i = G::raw_cell(tid, l);
        CHECK(i < G::RAW_N, "raw cell %d", i);
        if (i < G::RAW_N) ++raw[size_t(i)];
        const int64_t o = G::raw_source(i, y0, x0, H, W, rs);
        CHECK(o >= 0 && o < (H - 1) * rs + W, "source %lld", (long long)o);
      }
      for (int it = 0; it < G::ROW_IT; ++it) {
        if (!G::row_active(tid, it)) continue;
        const int pi = G::row_pair(tid, it), w0 = G::row_window(pi);
        CHECK(2 * pi + 1 < G::HB_N && w0 + 2 * RG + 1 < G::RAW_N, "row pair %d", pi);
        CHECK(w0 / G::RAW_W == 2 * pi / G::HB_W && w0 % G::RAW_W == 2 * pi % G::HB_W, "window %d", w0);
        ++hb[size_t(2 * pi)];
        ++hb[size_t(2 * pi + 1)];
      }
      for (int it = 0; it < G::COL_IT; ++it) {
        if (!G::col_active(tid, it)) continue;
        const int pi = G::col_pair(tid, it);
        CHECK(2 * pi + 1 < G::GB_N && 2 * pi + 2 * RG * G::HB_W + 1 < G::HB_N, "col pair %d", pi);
        ++gb[size_t(2 * pi)];
        ++gb[size_t(2 * pi + 1)];
      }
      const int64_t gy = y0 + G::lane_row(tid), gx = x0 + G::lane_col(tid);
      for (int d = 0; d < 3; ++d) {
        const int r = G::med_row(gy, d, y0, H), c = G::med_col(gx, d, x0, W);
        CHECK(!MED || (r >= 0 && r < G::GB_H && c >= 0 && c < G::GB_W), "median (%d, %d)", r, c);
      }
      if (gy < H && gx < W) ++owner[size_t(gy * W + gx)];
    }
    for (int v : raw) CHECK(v == 1, "raw cell staged %d times", v);
    for (int v : hb) CHECK(v == 1, "row output made %d times", v);
    for (int v : gb) CHECK(v == 1, "column output made %d times", v);
  }
  for (int v : owner) CHECK(v == 1, "pixel owned %d times", v);
}

int main() {
  const int64_t shapes[][3] = {{1, 1, 1}, {8, 32, 32}, {9, 33, 40}, {37, 150, 150}, {240, 320, 320}};
  for (const auto& s : shapes) {
    check<0, true>(s[0], s[1], s[2]);
    check<1, true>(s[0], s[1], s[2]);
    check<2, true>(s[0], s[1], s[2]);
    check<3, true>(s[0], s[1], s[2]);
    check<1, false>(s[0], s[1], s[2]);
    check<2, false>(s[0], s[1], s[2]);
    check<3, false>(s[0], s[1], s[2]);
  }
  std::printf(bad ? "%d failures\n" : "OK\n", bad);
  return bad != 0;
}
