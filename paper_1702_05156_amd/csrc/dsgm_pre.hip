// dsgm_pre.hip -- the forward with the paper's frame preprocessing fused in
// (internal).
//
// Sec. 2.1 and the preprocessing of Sec. 3.1.1 / 3.3.1: every frame is blurred
// with a separable kernel (along rows, then along columns; a sampled,
// normalised Gaussian by default) and then median-filtered over 3 x 3
// neighbourhoods, borders clamped to the nearest valid row and column; the
// background update of Sec. 2.2-2.3 then runs on the filtered frame.  Here all
// three happen in one pass over the sequence: the filtered frame never goes
// to memory unless the caller asks for it.
//
// Decomposition: a workgroup of 256 lanes owns a TH x TW = 16 x 64 tile of
// pixels (8 x 32 for small frames) for all T frames, each lane four (one)
// horizontally adjacent pixels of one row, with their model state in registers.  Per frame the workgroup stages
// the tile plus a halo of R = RG (+1 with the median) rows and columns of the
// raw frame in LDS (indices clamped to the frame), runs the row pass and the
// column pass of the blur in LDS, then each lane takes the median of its
// pixels' 3 x 3 neighbourhoods and updates its models.  The next frame's tile
// is loaded into registers while the current one is filtered, so its HBM
// latency overlaps the arithmetic.  Tiles are dealt so that each XCD gets a
// contiguous range of them: neighbouring tiles, whose halos overlap, run on
// the same L2.
//
// The kernel is bound by vector issue, then by LDS: a lane's blur outputs are
// adjacent (six in one row, two columns of three rows), so that it reads every
// value of its windows once; the medians are plain min/max instructions.  With
// these and the update under lane masks 1080 x 1920 frames, 5 taps and median,
// went from 469 to 416 us (FP64, 50 frames) and 260 to 227 us (BF16/FP32).
//
// Median of nine: sort each of the three columns of the neighbourhood; the
// median is then the median of (largest column minimum, median of the column
// medians, smallest column maximum).  Four adjacent pixels share their column
// sorts (six columns).  All selections are exact.
//
// The blur sums run from 0 in index order with every product and sum rounded
// (no contraction) for FP64 state, the order the oracle uses.
#include <type_traits>

#include "dsgm_ext.h"
#include "dsgm_fwd_impl.h"

namespace dsgm {

namespace pre {

using fwd::fill_table;
using fwd::make_consts;

// tile shapes and every tile cell index: dsgm_geom.h
using geom::pre::NT;
using geom::pre::Geo;

// min and max of finite values (a zero's sign may differ from a sort's when +0
// and -0 tie, which leaves every value unchanged).  The instructions themselves:
// the builtins add a canonicalising max per value read from LDS, 9 of 30
// instructions per pixel with FP64 state.
__device__ __forceinline__ double mn(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double mx(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// The medians of PX horizontally adjacent pixels from the three rows of their
// PX + 2 columns: each column sorted once, then per pixel the median of (the
// largest column minimum, the median of the column medians, the smallest
// column maximum).  FP64: two pixels share the pairs of the columns they have
// in common.  FP32: the three-operand instructions, 8.5 per pixel.
template <int PX>
__device__ __forceinline__ void medians(const double (&p)[3][PX + 2], double (&xs)[PX]) {
  double lo[PX + 2], md[PX + 2], hi[PX + 2];
#pragma unroll
  for (int d = 0; d < PX + 2; ++d) {
    const double l01 = mn(p[0][d], p[1][d]), h01 = mx(p[0][d], p[1][d]);
    lo[d] = mn(l01, p[2][d]);
    const double h = mx(l01, p[2][d]);
    hi[d] = mx(h01, h);
    md[d] = mn(h01, h);
  }
#pragma unroll
  for (int q0 = 0; q0 < PX; q0 += 2) {  // pixels q0, q0 + 1 have columns q0 + 1, q0 + 2 in common
    const double l = mx(lo[q0 + 1], lo[q0 + 2]), h = mn(hi[q0 + 1], hi[q0 + 2]);
    const double ml = mn(md[q0 + 1], md[q0 + 2]), mh = mx(md[q0 + 1], md[q0 + 2]);
#pragma unroll
    for (int q = q0; q < q0 + 2 && q < PX; ++q) {
      const int o = q == q0 ? q0 : q0 + 3;  // the pixel's other column
      const double a = mx(l, lo[o]), c = mn(h, hi[o]), b = mx(ml, mn(mh, md[o]));
      xs[q] = mx(mn(a, b), mn(mx(a, b), c));
    }
  }
}
__device__ __forceinline__ float min3(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float med3(float a, float b, float c) {
  float r;
  asm("v_med3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
template <int PX>
__device__ __forceinline__ void medians(const float (&p)[3][PX + 2], float (&xs)[PX]) {
  float lo[PX + 2], md[PX + 2], hi[PX + 2];
#pragma unroll
  for (int d = 0; d < PX + 2; ++d) {
    lo[d] = min3(p[0][d], p[1][d], p[2][d]);
    md[d] = med3(p[0][d], p[1][d], p[2][d]);
    hi[d] = max3(p[0][d], p[1][d], p[2][d]);
  }
#pragma unroll
  for (int q = 0; q < PX; ++q)
    xs[q] = med3(max3(lo[q], lo[q + 1], lo[q + 2]), med3(md[q], md[q + 1], md[q + 2]),
                 min3(hi[q], hi[q + 1], hi[q + 2]));
}

// blur sum over n taps from 0 in index order (no contraction for double)
template <typename Acc>
__device__ __forceinline__ Acc tap(Acc acc, Acc w, Acc x) { return acc + w * x; }
template <>
__device__ __forceinline__ float tap<float>(float acc, float w, float x) {
  return __builtin_fmaf(w, x, acc);
}

// Frames of fewer 16 x 64 tiles than this (two per CU) are cut into 8 x 32 tiles
// of one pixel per lane: with few workgroups the chain of a tile's frames bounds
// the call, and a quarter of the pixels per lane shortens it.  16 x 64 against
// 8 x 32 tiles, 5 taps and median: FP64 500 x 240 x 320 (75 tiles) 796 / 518 us,
// 100 x 480 x 640 (300) 217 / 171 us, 50 x 720 x 1280 (900) 220 / 230 us,
// 50 x 1080 x 1920 (2,040) 419 / 478 us; BF16/FP32 632 / 365, 150 / 104,
// 116 / 132 and 230 / 285 us.
constexpr int64_t SMALL_BELOW = 512;

// Waves per SIMD the kernel is compiled for: 3 with FP64 state and four pixels per
// lane (7 taps and median took 169 VGPRs by themselves and ran at 2: one frame of 1920 x
// 2560 95.0 us, 78.9 at 3), else the compiler's choice.
template <typename Acc, typename Tile>
constexpr int pre_waves() {
  return sizeof(Acc) == 8 && Tile::px == 4 ? 3 : 1;
}

template <typename In, typename Acc, typename Io, int RG, bool MED, bool PRINTED, typename Tile>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(pre_waves<Acc, Tile>())))
pre_kernel(const PreArgs a) {
  using G = Geo<RG, MED, Tile>;
  constexpr int TH = G::TH, TW = G::TW, PX = G::PX;
  // raw, row-blurred and blurred tiles each have their own storage, so a frame
  // needs three barriers: the next frame's raw tile can be staged while slow
  // lanes still read this frame's blurred tile (without a blur the raw tile is
  // the blurred tile and a fourth barrier guards it)
  __shared__ alignas(16) Acc buf_raw[G::RAW_N];
  __shared__ alignas(16) Acc buf_hb[RG > 0 ? G::HB_N : 1];
  __shared__ alignas(16) Acc buf_gb[RG > 0 ? G::GB_N : 1];
  __shared__ TableEntry<Acc> tbl[TABLE_SIZE];
  // FP32 state and small tiles map their tile before the table is built, FP64 state on
  // large tiles after it (before / after: 1 x 1920 x 2560, 7 taps and median, FP32 50.0 /
  // 54.7 us, FP32 arrays with FP64 state 85.6 / 77.6; FP64 500 x 240 x 320, 5 taps and
  // median 522 / 532)
  constexpr bool MAP_FIRST = sizeof(Acc) == 4 || PX == 1;
  int64_t tile = 0;
  if constexpr (MAP_FIRST) {
    tile = tile_here(a);
    if (tile < 0) return;
  }
  fill_table<Acc>(tbl, a.weight_rule, a.age_max, a.var_init);  // ends with a barrier
  const StepConsts<Acc> k =
      make_consts<Acc>(a.theta_s, a.theta_d, a.var_init, a.var_floor, a.mask_floor);

  Acc wt[2 * RG + 1];
#pragma unroll
  for (int i = 0; i < 2 * RG + 1; ++i) wt[i] = Acc(a.w[i]);

  if constexpr (!MAP_FIRST) {
    tile = tile_here(a);
    if (tile < 0) return;
  }
  const int64_t y0 = (tile / a.tiles_x) * TH, x0 = (tile % a.tiles_x) * TW;
  const int tid = threadIdx.x;
  const int ty = G::lane_row(tid), tx = G::lane_col(tid);  // this lane's row and first column
  const int64_t gy = y0 + ty;

  // this lane's raw-tile elements: LDS slot and frame offset (both fixed per frame)
  uint32_t roff[G::LOADS];
#pragma unroll
  for (int l = 0; l < G::LOADS; ++l) {
    const int i = G::raw_cell(tid, l);
    roff[l] = i < G::RAW_N ? uint32_t(G::raw_source(i, y0, x0, a.H, a.W, a.row_stride))
                           : 0u;  // < 2^31 (host check)
  }
  // the median's rows and columns in the blurred tile, clamped to the frame
  int gr[3], gc[PX + 2];
#pragma unroll
  for (int d = 0; d < 3; ++d) gr[d] = G::med_row(gy, d, y0, a.H);
#pragma unroll
  for (int d = 0; d < PX + 2; ++d) gc[d] = G::med_col(x0 + tx, d, x0, a.W);
  // a tile inside the frame clamps nothing: its medians' columns are adjacent
  const bool inside = y0 > 0 && y0 + TH < a.H && x0 > 0 && x0 + TW < a.W;

  bool valid[PX];
  bool all_valid = gy < a.H;
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    valid[q] = gy < a.H && x0 + tx + q < a.W;
    all_valid = all_valid && valid[q];
  }
  const int64_t pix = gy * a.W + x0 + tx;          // state index of pixel 0
  const int64_t foff = gy * a.row_stride + x0 + tx; // frame offset of pixel 0
  const bool vec_ok = all_valid && (a.row_stride % PX) == 0 && (a.frame_stride % PX) == 0 &&
                      (a.W % PX) == 0;

  Model<Acc> s[PX];
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    if (valid[q]) {
      s[q].mA = static_cast<const Acc*>(a.mean_a)[pix + q];
      s[q].vA = static_cast<const Acc*>(a.var_a)[pix + q];
      s[q].mC = static_cast<const Acc*>(a.mean_c)[pix + q];
      s[q].vC = static_cast<const Acc*>(a.var_c)[pix + q];
      s[q].aA = a.age_a[pix + q];
      s[q].aC = a.age_c[pix + q];
    } else {
      s[q].mA = s[q].vA = s[q].mC = s[q].vC = Acc(0);
      s[q].aA = s[q].aC = 1;
    }
  }

  // the start of this lane's raw window in each round of the row pass, and its
  // first cell of the column pass: the same every frame
  uint32_t row_src[G::ROW_ROUNDS];
#pragma unroll
  for (int rd = 0; rd < G::ROW_ROUNDS; ++rd)
    row_src[rd] = uint32_t(G::row_window(G::row_pair(tid, rd * G::ROW_SEG)));
  const int col_src = 2 * G::col_pair(tid, 0);

  const In* frames = static_cast<const In*>(a.frames);
  In nxt[G::LOADS];
  auto load_frame = [&](int64_t t) {
    const In* f = frames + t * a.frame_stride;
#pragma unroll
    for (int l = 0; l < G::LOADS; ++l)
      if (G::raw_active(tid, l)) nxt[l] = f[roff[l]];
  };
  if (a.T > 0) load_frame(0);

  for (int64_t t = 0; t < a.T; ++t) {
    // 1. stage the raw tile, then start loading the next frame's
#pragma unroll
    for (int l = 0; l < G::LOADS; ++l)
      if (G::raw_active(tid, l)) buf_raw[G::raw_cell(tid, l)] = to_acc<In, Acc>(nxt[l]);
    __syncthreads();
    if (t + 1 < a.T) load_frame(t + 1);
    if (t == 0) {  // the state has arrived (one frame of 1920 x 2560, FP64: 102 us with
                   // the ages converted as they are loaded, pixel by pixel)
#pragma unroll
      for (int q = 0; q < PX; ++q) convert_ages(s[q]);
    }

    const Acc* gbp;  // the blurred tile, GB_H x GB_W
    if constexpr (RG > 0) {
      // 2. row pass: hb[r][v] = sum_j w_j raw[r][v + j], v in [0, HB_W).  A
      // lane makes ROW_SEG adjacent output pairs of one row from one window
      static_assert(G::HB_W % 2 == 0 && G::GB_W % 2 == 0, "output pairs stay in one row");
      constexpr int NO = 2 * G::ROW_SEG;
#pragma unroll
      for (int rd = 0; rd < G::ROW_ROUNDS; ++rd) {
        if (G::row_active(tid, rd * G::ROW_SEG)) {
          const Acc* src = buf_raw + row_src[rd];
          Acc* dst = buf_hb + 2 * G::row_pair(tid, rd * G::ROW_SEG);
          Acc win[NO + 2 * RG];
#pragma unroll
          for (int j = 0; j < NO + 2 * RG; ++j) win[j] = src[j];
#pragma unroll
          for (int o = 0; o < NO; ++o) {
            Acc sum = Acc(0);
#pragma unroll
            for (int j = 0; j < 2 * RG + 1; ++j) sum = tap(sum, wt[j], win[o + j]);
            dst[o] = sum;
          }
        }
      }
      __syncthreads();
      // 3. column pass: gb[r][v] = sum_i w_i hb[r + i][v], r in [0, GB_H); the
      // two tiles have the same width, so gb's row-major index is hb's.  A lane
      // makes COL_IT output pairs of one column pair, reading each row once
      static_assert(G::HB_W == G::GB_W, "row-blurred and blurred tiles share a width");
      if (G::col_active(tid, 0)) {
        const Acc* src = buf_hb + col_src;
        Acc* dst = buf_gb + col_src;
        Acc in[G::COL_IT + 2 * RG][2];
#pragma unroll
        for (int j = 0; j < G::COL_IT + 2 * RG; ++j) {
          in[j][0] = src[j * G::HB_W];
          in[j][1] = src[j * G::HB_W + 1];
        }
#pragma unroll
        for (int o = 0; o < G::COL_IT; ++o)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            Acc sum = Acc(0);
#pragma unroll
            for (int j = 0; j < 2 * RG + 1; ++j) sum = tap(sum, wt[j], in[o + j][c]);
            dst[o * G::GB_W + c] = sum;
          }
      }
      __syncthreads();
      gbp = buf_gb;
    } else {
      gbp = buf_raw;  // no blur: the raw tile (R = RM) is the blurred tile
    }

    // 4. median of each pixel's 3 x 3 neighbourhood, then the model update
    Acc xs[PX];
    if constexpr (MED) {
      Acc p[3][PX + 2];
      if (inside) {
        const Acc* nb = gbp + ty * G::GB_W + tx;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int d = 0; d < PX + 2; ++d) p[r][d] = nb[r * G::GB_W + d];
      } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int d = 0; d < PX + 2; ++d) p[r][d] = gbp[gr[r] * G::GB_W + gc[d]];
      }
      medians<PX>(p, xs);
    } else {
#pragma unroll
      for (int q = 0; q < PX; ++q) xs[q] = gbp[gr[1] * G::GB_W + gc[q + 1]];
    }

    StepRecord<Acc> rec[PX];
    uint64_t any = 0;
#pragma unroll
    for (int q = 0; q < PX; ++q) {
      rec[q] = step_core<Acc>(s[q], xs[q], k, tbl);
      any |= rec[q].swap_lanes;
    }
    if (any != 0) {
#pragma unroll
      for (int q = 0; q < PX; ++q) exchange<Acc>(s[q], xs[q], k, rec[q]);
    }
    uint64_t back[PX];  // lanes whose pixel q is background
#pragma unroll
    for (int q = 0; q < PX; ++q) {
      const bool b = bg_from<Acc, PRINTED>(rec[q].qd, s[q], xs[q], k);
      back[q] = __builtin_amdgcn_ballot_w64(b);
      rec[q].fg = !b;
    }
    using Mask = Vec<uint8_t, PX>;
    const auto mk = __builtin_bit_cast(
        Mask, typename fwd::Raw<PX>::type(mask_bytes<PX>(back)));
    // this frame's outputs, the optional ones formed under their uniform branches,
    // all of them inside one test for whole vectors (24 x 1080 x 1920, FP32 state,
    // bg and filtered frames: 165 us; with the test in each output's store 202)
    const int64_t o = t * a.frame_stride + foff;
    // FP64 state on large tiles without the median: the codes are formed in every
    // call.  The code compiled around them runs faster (5 taps, 24 x 721 x 1279 88
    // against 97 us, FP32 arrays with bg 92 / 109; its registers or wavefronts are not
    // why: held to 3 wavefronts a SIMD the other form stays at 96).  With the median
    // it is slower (116 / 110).
    constexpr bool CODES_FIRST = sizeof(Acc) == 8 && !MED && PX == 4;
    Vec<uint8_t, PX> cd;
    if constexpr (CODES_FIRST) {
#pragma unroll
      for (int q = 0; q < PX; ++q) cd.v[q] = uint8_t(code_of<Acc>(rec[q]));
    }
    auto outputs = [&](auto store) {
      store(a.masks, [&](int q) { return mk.v[q]; });
      if (a.bg) store(static_cast<Io*>(a.bg), [&](int q) { return Io(s[q].mA); });
      if (a.filtered) store(static_cast<Io*>(a.filtered), [&](int q) { return Io(xs[q]); });
      if (a.codes)
        store(a.codes, [&](int q) { return CODES_FIRST ? cd.v[q] : uint8_t(code_of<Acc>(rec[q])); });
    };
    if (vec_ok) {
      outputs([&](auto* out, auto value) {
        using X = std::remove_pointer_t<decltype(out)>;
        Vec<X, PX> v;
#pragma unroll
        for (int q = 0; q < PX; ++q) v.v[q] = value(q);
        *reinterpret_cast<Vec<X, PX>*>(out + o) = v;
      });
    } else {
      outputs([&](auto* out, auto value) {
#pragma unroll
        for (int q = 0; q < PX; ++q)
          if (valid[q]) out[o + q] = value(q);
      });
    }
    if constexpr (RG == 0) __syncthreads();  // the next frame overwrites the raw tile
  }

#pragma unroll
  for (int q = 0; q < PX; ++q) {
    if (!valid[q]) continue;
    static_cast<Acc*>(a.mean_a)[pix + q] = s[q].mA;
    static_cast<Acc*>(a.var_a)[pix + q] = s[q].vA;
    static_cast<Acc*>(a.mean_c)[pix + q] = s[q].mC;
    static_cast<Acc*>(a.var_c)[pix + q] = s[q].vC;
    a.age_a[pix + q] = age_out<Acc>(s[q].aA);
    a.age_c[pix + q] = age_out<Acc>(s[q].aC);
  }
}

template <typename In, typename Acc, typename Io, bool MED, bool PRINTED, typename Tile>
hipError_t launch_tile(PreArgs a, int rg, hipStream_t stream) {
  a.tiles_x = (a.W + Tile::tw - 1) / Tile::tw;
  a.tiles_y = (a.H + Tile::th - 1) / Tile::th;
  const dim3 grid = tile_grid(a), block{NT, 1, 1};
  // One frame with FP64 state and no median fits 4 wavefronts a SIMD, whose requests
  // then come in one burst: LDS that nothing uses holds it to 3 workgroups a CU (5 taps,
  // 1920 x 2560, 4 / 3: FP64 85.9 / 77.9 us, FP32 arrays 86.6 / 76.7; four frames are
  // faster at 4, 4 x 721 x 1279 29.3 / 33.7)
  const uint32_t lds = sizeof(Acc) == 8 && !MED && Tile::px == 4 && a.T == 1 ? 12 * 1024 : 0;
  switch (rg) {
    case 0: hipLaunchKernelGGL((pre_kernel<In, Acc, Io, 0, MED, PRINTED, Tile>), grid, block, lds, stream, a); break;
    case 1: hipLaunchKernelGGL((pre_kernel<In, Acc, Io, 1, MED, PRINTED, Tile>), grid, block, lds, stream, a); break;
    case 2: hipLaunchKernelGGL((pre_kernel<In, Acc, Io, 2, MED, PRINTED, Tile>), grid, block, lds, stream, a); break;
    case 3: hipLaunchKernelGGL((pre_kernel<In, Acc, Io, 3, MED, PRINTED, Tile>), grid, block, lds, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename In, typename Acc, typename Io, bool MED, bool PRINTED>
hipError_t launch_rg(const PreArgs& a, int rg, hipStream_t stream) {
  using geom::pre::Big;
  using geom::pre::Small;
  if (a.tiles_x * a.tiles_y < SMALL_BELOW)  // tiles of 16 x 64 (the caller's count)
    return launch_tile<In, Acc, Io, MED, PRINTED, Small>(a, rg, stream);
  return launch_tile<In, Acc, Io, MED, PRINTED, Big>(a, rg, stream);
}

template <typename In, typename Acc, typename Io>
hipError_t launch_t(const PreArgs& a, int rg, bool median, hipStream_t stream) {
  const bool printed = a.mask_rule != 0;
  if (median)
    return printed ? launch_rg<In, Acc, Io, true, true>(a, rg, stream)
                   : launch_rg<In, Acc, Io, true, false>(a, rg, stream);
  return printed ? launch_rg<In, Acc, Io, false, true>(a, rg, stream)
                 : launch_rg<In, Acc, Io, false, false>(a, rg, stream);
}

}  // namespace pre

hipError_t launch_pre(const PreArgs& a, int in_dtype, int acc, int rg, bool median,
                      hipStream_t stream) {
  if (acc == 0) {
    if (in_dtype == 0) return pre::launch_t<double, double, double>(a, rg, median, stream);
    if (in_dtype == 1) return pre::launch_t<float, double, double>(a, rg, median, stream);
    if (in_dtype == 2) return pre::launch_t<bf16_t, double, double>(a, rg, median, stream);
  } else if (acc == 1) {
    if (in_dtype == 1) return pre::launch_t<float, float, float>(a, rg, median, stream);
    if (in_dtype == 2) return pre::launch_t<bf16_t, float, float>(a, rg, median, stream);
  } else if (acc == 2) {
    if (in_dtype == 1) return pre::launch_t<float, double, float>(a, rg, median, stream);
    if (in_dtype == 2) return pre::launch_t<bf16_t, double, float>(a, rg, median, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace dsgm
