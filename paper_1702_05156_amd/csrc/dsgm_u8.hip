// dsgm_u8.hip -- the 8-bit as-run model of the appendix (internal).
//
// The appendix's inner update reads 8-bit frames and keeps each model's mean
// and variance in 8-bit images: the arithmetic is double precision, and every
// value written back is converted to an integer, the fraction dropped (here
// also limited to [0, 255], where the conversion has no defined result).  The
// tests, the swap and the mask then see the stored values.  This kernel runs
// that model time-fused like fwd_kernel: one lane owns P adjacent pixels of a
// row for all T frames with their models in registers (as the stored
// integers), and per frame reads P frame bytes and writes P mask bytes.
// The state is 6 bytes per pixel instead of 68, which is what a T = 1
// streaming caller moves per frame; such calls run u8_step_kernel below.
#include <cmath>

#include "dsgm_ext.h"
#include "dsgm_fwd_impl.h"

namespace dsgm {

namespace u8 {

using fwd::fill_table;
using fwd::ld_stream;
using fwd::make_consts;
using fwd::st_stream;

// the storage rule of an 8-bit image: drop the fraction, limit to [0, 255]
__device__ __forceinline__ double stored(double v) {
  return __builtin_fmin(255.0, __builtin_fmax(0.0, __builtin_trunc(v)));
}

// One pixel's models as the integers the images hold, with the thresholds of
// their match tests; ages are table offsets (age_in<double>).
struct Model8 {
  uint32_t mA, vA, tA, mC, vC, tC;
  int aA, aC;
};

// The step's tables.  All squared distances of 8-bit values are integers up to
// 65025, so each double-precision test is an integer comparison with the
// number of distances that pass it:
//   match       q < max(ts*v, ts*vf)          <=>  q < match[v]
//   background  q <= max(td*ref, td*mf)       <=>  q < back[ref]
// (two comparisons of the real-valued step are one with the larger threshold;
// fmax drops a NaN, and a NaN threshold passes nothing, as the comparisons do).
struct Tables8 {
  TableEntry<double> e[TABLE_SIZE];
  uint32_t match[256], back[256];
};

__device__ __forceinline__ uint32_t passing(double n) {
  return n > 0.0 ? uint32_t(__builtin_fmin(n, 65026.0)) : 0u;  // NaN: 0
}

// fills the tables and ends with a barrier
__device__ __forceinline__ void fill_tables(Tables8& t, const StepConsts<double>& k,
                                            int weight_rule, int age_max, double var_init) {
  for (int v = threadIdx.x; v < 256; v += blockDim.x) {
    t.match[v] = passing(__builtin_ceil(__builtin_fmax(k.theta_s * double(v), k.ts_vf)));
    t.back[v] = passing(__builtin_floor(__builtin_fmax(k.theta_d * double(v), k.td_mf)) + 1.0);
  }
  fill_table<double>(t.e, weight_rule, age_max, var_init);
}

// What a step decided (masks of lanes).
struct Record8 {
  uint64_t hit_a, swap;
  bool hit_c;  // of the lanes whose A failed
};

// Match tests and update of the matched model (or the reset of C) for one frame
// of one pixel, on the stored integers; the exchange is left to exchange8().
// The tests are integer comparisons; the blends are evaluated in double
// precision in the order of the real-valued step, and each result is written
// back by dropping its fraction.  A blended mean lies in [0, 255] and a
// blended variance is not negative (the weights are not, and sum to 1 within a
// rounding), so the conversion itself is the storage rule but for the
// variance's upper limit.  Values move under lane masks (update_in_place says
// why).  CARRY: the new variance's threshold is looked up and kept.  Bound by
// vector issue; one 1920 x 2560 frame per call took 20.0 us with the
// real-valued step and the storage rule on all four values, 17.4 us with this
// one, and 15.9 us with 32-bit lane-group divisions.
template <bool CARRY>
__device__ __forceinline__ Record8 step8(Model8& s, const uint32_t x, const uint32_t var_init,
                                         const Tables8& t) {
  const int dA = int(x) - int(s.mA), dC = int(x) - int(s.mC);
  Record8 r;
  r.hit_a = __builtin_amdgcn_ballot_w64(uint32_t(__mul24(dA, dA)) < s.tA);
  const bool hitC = uint32_t(__mul24(dC, dC)) < s.tC;
  int idx = hitC ? s.aC : reset_age<double>();
  uint32_t m = s.mC, v = s.vC;
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_mov_b32 %[i], %[aA]\n\t"
      "v_mov_b32 %[m], %[mA]\n\t"
      "v_mov_b32 %[v], %[vA]\n\t"
      "s_mov_b64 exec, %[all]"
      : [i] "+&v"(idx), [m] "+&v"(m), [v] "+&v"(v), [all] "=&s"(all)
      : [aA] "v"(s.aA), [mA] "v"(s.mA), [vA] "v"(s.vA), [h] "s"(r.hit_a));
  const TableEntry<double>& e = *reinterpret_cast<const TableEntry<double>*>(
      reinterpret_cast<const char*>(t.e) + idx);
  const double u = e.u, w = e.w, xd = double(x);
  const int next = e.next;
  const double mn = blend(u, double(m), w, xd);
  const double d = mn - xd;
  const uint32_t vb = uint32_t(blend(u, double(v), w, d * d));
  const uint32_t mi = uint32_t(mn);
  uint32_t vi = vb < 255u ? vb : 255u;
  vi = idx == reset_age<double>() ? var_init : vi;  // a reset: (x, var_init, 1)
  if constexpr (CARRY) {
    const uint32_t tn = t.match[vi];
    asm("s_mov_b64 %[all], exec\n\t"
        "s_mov_b64 exec, %[h]\n\t"
        "v_mov_b32 %[mA], %[m]\n\t"
        "v_mov_b32 %[vA], %[v]\n\t"
        "v_mov_b32 %[tA], %[t]\n\t"
        "v_mov_b32 %[aA], %[n]\n\t"
        "s_andn2_b64 exec, %[all], %[h]\n\t"
        "v_mov_b32 %[mC], %[m]\n\t"
        "v_mov_b32 %[vC], %[v]\n\t"
        "v_mov_b32 %[tC], %[t]\n\t"
        "v_mov_b32 %[aC], %[n]\n\t"
        "s_mov_b64 exec, %[all]"
        : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [tA] "+&v"(s.tA), [aA] "+&v"(s.aA), [mC] "+&v"(s.mC),
          [vC] "+&v"(s.vC), [tC] "+&v"(s.tC), [aC] "+&v"(s.aC), [all] "=&s"(all)
        : [m] "v"(mi), [v] "v"(vi), [t] "v"(tn), [n] "v"(next), [h] "s"(r.hit_a)
        : "scc");
  } else {
    asm("s_mov_b64 %[all], exec\n\t"
        "s_mov_b64 exec, %[h]\n\t"
        "v_mov_b32 %[mA], %[m]\n\t"
        "v_mov_b32 %[vA], %[v]\n\t"
        "v_mov_b32 %[aA], %[n]\n\t"
        "s_andn2_b64 exec, %[all], %[h]\n\t"
        "v_mov_b32 %[mC], %[m]\n\t"
        "v_mov_b32 %[vC], %[v]\n\t"
        "v_mov_b32 %[aC], %[n]\n\t"
        "s_mov_b64 exec, %[all]"
        : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [aA] "+&v"(s.aA), [mC] "+&v"(s.mC), [vC] "+&v"(s.vC),
          [aC] "+&v"(s.aC), [all] "=&s"(all)
        : [m] "v"(mi), [v] "v"(vi), [n] "v"(next), [h] "s"(r.hit_a)
        : "scc");
  }
  r.hit_c = hitC && !__builtin_amdgcn_inverse_ballot_w64(r.hit_a);
  r.swap = __builtin_amdgcn_ballot_w64(s.aC > s.aA);
  return r;
}

// the exchange in the lanes of `swap`: A <- C, C <- (x, var_init, 1)
template <bool CARRY>
__device__ __forceinline__ void exchange8(Model8& s, const uint32_t x, const uint32_t var_init,
                                          const uint64_t swap, const Tables8& t) {
  const uint32_t ti = CARRY ? t.match[var_init] : 0u;
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_mov_b32 %[mA], %[mC]\n\t"
      "v_mov_b32 %[vA], %[vC]\n\t"
      "v_mov_b32 %[tA], %[tC]\n\t"
      "v_mov_b32 %[aA], %[aC]\n\t"
      "v_mov_b32 %[mC], %[x]\n\t"
      "v_mov_b32 %[vC], %[v]\n\t"
      "v_mov_b32 %[tC], %[t]\n\t"
      "v_mov_b32 %[aC], %[one]\n\t"
      "s_mov_b64 exec, %[all]"
      : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [tA] "+&v"(s.tA), [aA] "+&v"(s.aA), [mC] "+&v"(s.mC),
        [vC] "+&v"(s.vC), [tC] "+&v"(s.tC), [aC] "+&v"(s.aC), [all] "=&s"(all)
      : [x] "v"(x), [v] "v"(var_init), [t] "v"(ti), [h] "s"(swap),
        [one] "n"(int(sizeof(TableEntry<double>))));
}

// The frame of a lane's P pixels: steps, exchanges and background tests; the
// mask bytes, and with CODES the decision codes.
template <int P, bool CARRY, bool CODES, bool PRINTED>
__device__ __forceinline__ uint32_t frame8(Model8 (&s)[P], const uint32_t (&x)[P],
                                           const uint32_t var_init, const Tables8& t,
                                           Vec<uint8_t, P>& codes) {
  Record8 r[P];
  uint64_t any = 0, back[P];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    r[q] = step8<CARRY>(s[q], x[q], var_init, t);
    any |= r[q].swap;
  }
  if (any != 0) {
#pragma unroll
    for (int q = 0; q < P; ++q) exchange8<CARRY>(s[q], x[q], var_init, r[q].swap, t);
  }
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int d = int(x[q]) - int(s[q].mA);
    const bool b = uint32_t(__mul24(d, d)) < t.back[PRINTED ? x[q] : s[q].vA];
    back[q] = __builtin_amdgcn_ballot_w64(b);
    if (CODES) {
      const bool hitA = __builtin_amdgcn_inverse_ballot_w64(r[q].hit_a);
      codes.v[q] = uint8_t((hitA ? CODE_HIT_A : (r[q].hit_c ? CODE_HIT_C : CODE_RESET)) |
                           (__builtin_amdgcn_inverse_ballot_w64(r[q].swap) ? CODE_SWAP : 0u) |
                           (b ? 0u : CODE_FG));
    }
  }
  return mask_bytes<P>(back);
}

// P bytes of each state plane <-> a lane's models
template <int P>
struct Planes8 {
  Vec<uint8_t, P> mA, vA, mC, vC, aA, aC;
};
template <int P>
__device__ __forceinline__ void unpack8(const Planes8<P>& b, const Tables8& t, Model8 (&s)[P]) {
#pragma unroll
  for (int q = 0; q < P; ++q) {
    s[q].mA = b.mA.v[q];
    s[q].vA = b.vA.v[q];
    s[q].mC = b.mC.v[q];
    s[q].vC = b.vC.v[q];
    s[q].aA = age_in<double>(b.aA.v[q]);
    s[q].aC = age_in<double>(b.aC.v[q]);
    s[q].tA = t.match[s[q].vA];
    s[q].tC = t.match[s[q].vC];
  }
}
template <int P>
__device__ __forceinline__ Planes8<P> pack8(const Model8 (&s)[P]) {
  Planes8<P> b;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    b.mA.v[q] = uint8_t(s[q].mA);
    b.vA.v[q] = uint8_t(s[q].vA);
    b.mC.v[q] = uint8_t(s[q].mC);
    b.vC.v[q] = uint8_t(s[q].vC);
    b.aA.v[q] = age_out<double>(s[q].aA);
    b.aC.v[q] = age_out<double>(s[q].aC);
  }
  return b;
}
template <int P>
__device__ __forceinline__ Planes8<P> load8(const FwdArgs& a, int64_t pix) {
  using V = Vec<uint8_t, P>;
  Planes8<P> b;
  b.mA = *reinterpret_cast<const V*>(static_cast<const uint8_t*>(a.mean_a) + pix);
  b.vA = *reinterpret_cast<const V*>(static_cast<const uint8_t*>(a.var_a) + pix);
  b.mC = *reinterpret_cast<const V*>(static_cast<const uint8_t*>(a.mean_c) + pix);
  b.vC = *reinterpret_cast<const V*>(static_cast<const uint8_t*>(a.var_c) + pix);
  b.aA = *reinterpret_cast<const V*>(a.age_a + pix);
  b.aC = *reinterpret_cast<const V*>(a.age_c + pix);
  return b;
}
template <int P>
__device__ __forceinline__ void store8(const FwdArgs& a, int64_t pix, const Planes8<P>& b) {
  using V = Vec<uint8_t, P>;
  *reinterpret_cast<V*>(static_cast<uint8_t*>(a.mean_a) + pix) = b.mA;
  *reinterpret_cast<V*>(static_cast<uint8_t*>(a.var_a) + pix) = b.vA;
  *reinterpret_cast<V*>(static_cast<uint8_t*>(a.mean_c) + pix) = b.mC;
  *reinterpret_cast<V*>(static_cast<uint8_t*>(a.var_c) + pix) = b.vC;
  *reinterpret_cast<V*>(a.age_a + pix) = b.aA;
  *reinterpret_cast<V*>(a.age_c + pix) = b.aC;
}

template <int P, bool CODES, bool PRINTED>
__global__ void __launch_bounds__(256) u8_kernel(const FwdArgs a) {
  __shared__ Tables8 tbl;
  const StepConsts<double> k =
      make_consts<double>(a.theta_s, a.theta_d, a.var_init, a.var_floor, a.mask_floor);
  fill_tables(tbl, k, a.weight_rule, a.age_max, a.var_init);  // var_init already stored
  const uint32_t var_init = uint32_t(a.var_init);

  const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= a.ngroups) return;  // no barrier follows
  const geom::Group G = geom::group_of(g, a.groups_per_row, P, a.W, a.row_stride);
  const int64_t pix = G.soff, foff = G.foff;

  Model8 s[P];
  unpack8<P>(load8<P>(a, pix), tbl, s);

  const uint8_t* frames = static_cast<const uint8_t*>(a.frames);
  constexpr int U = 8;  // frames in flight
  auto frame_at = [&](int64_t t) { return ld_stream<uint8_t, P>(frames + t * a.frame_stride + foff); };
  auto do_frame = [&](const Vec<uint8_t, P>& xv, int64_t t) {
    uint32_t xs[P];
#pragma unroll
    for (int q = 0; q < P; ++q) xs[q] = xv.v[q];
    Vec<uint8_t, P> cd;
    const auto mk = typename fwd::Raw<P>::type(
        frame8<P, true, CODES, PRINTED>(s, xs, var_init, tbl, cd));
    const int64_t o = t * a.frame_stride + foff;
    st_stream<uint8_t, P>(a.masks + o, __builtin_bit_cast(Vec<uint8_t, P>, mk));
    if (CODES) *reinterpret_cast<Vec<uint8_t, P>*>(a.codes + o) = cd;
  };
  const int64_t T = a.T;
  int64_t t = 0;
  for (; t + U <= T; t += U) {
    Vec<uint8_t, P> xb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) xb[u] = frame_at(t + u);
#pragma unroll
    for (int u = 0; u < U; ++u) do_frame(xb[u], t + u);
  }
  for (; t < T; ++t) do_frame(frame_at(t), t);
  store8<P>(a, pix, pack8<P>(s));
}

// One frame per call (T = 1, the streaming step): a persistent grid whose
// lanes walk pixel groups, each lane loading the next group's frame and state
// bytes before it updates the current group, so the loads of one group overlap
// the arithmetic of the previous one (with one frame per launch there is no
// frame loop to hide them behind).  The table is built once per workgroup,
// while the first group's bytes are on their way.  Bounded to 128 VGPRs, so
// that the whole persistent grid (four workgroups per CU) is resident at once.
template <int P, bool CODES, bool PRINTED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
u8_step_kernel(const FwdArgs a) {
  __shared__ Tables8 tbl;
  using V = Vec<uint8_t, P>;
  const uint8_t* frame = static_cast<const uint8_t*>(a.frames);
  struct Bytes {
    V x;
    Planes8<P> p;
    uint32_t pix, foff;  // < 2^31 (host check)
  };
  // group g: row h, first column w (pixel index h*W + w, frame offset h*row_stride + w)
  auto load = [&](int64_t g, Bytes& b) {
    const geom::Group G = geom::group_of(g, a.groups_per_row, P, a.W, a.row_stride);
    b.pix = uint32_t(G.soff);
    b.foff = uint32_t(G.foff);
    b.x = ld_stream<uint8_t, P>(frame + b.foff);
    b.p = load8<P>(a, b.pix);
  };
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  Bytes cur, nxt;
  // the first group's bytes are requested before the tables are built, so their
  // latency overlaps the table's divisions and its barrier
  if (g < a.ngroups) load(g, cur);
  const StepConsts<double> k =
      make_consts<double>(a.theta_s, a.theta_d, a.var_init, a.var_floor, a.mask_floor);
  fill_tables(tbl, k, a.weight_rule, a.age_max, a.var_init);
  const uint32_t var_init = uint32_t(a.var_init);
  if (g >= a.ngroups) return;  // no barrier follows
  for (; g < a.ngroups; g += stride) {
    const bool more = g + stride < a.ngroups;
    if (more) load(g + stride, nxt);
    Model8 s[P];
    uint32_t xs[P];
    unpack8<P>(cur.p, tbl, s);
#pragma unroll
    for (int q = 0; q < P; ++q) xs[q] = cur.x.v[q];
    V cd;
    const auto mk = typename fwd::Raw<P>::type(
        frame8<P, false, CODES, PRINTED>(s, xs, var_init, tbl, cd));
    st_stream<uint8_t, P>(a.masks + cur.foff, __builtin_bit_cast(V, mk));
    if (CODES) *reinterpret_cast<V*>(a.codes + cur.foff) = cd;
    store8<P>(a, cur.pix, pack8<P>(s));
    if (more) cur = nxt;
  }
}

// persistent grid of the one-frame kernel: four 256-lane workgroups per CU
// (measured against eight and sixteen on 1920 x 2560 frames, with the
// real-valued step: 22.1 us per frame against 22.7 and 23.2; a grid of one group
// per lane took 23.7)
constexpr int64_t kStepGrid = 1024;

template <int P, bool CODES, bool PRINTED>
hipError_t launch_step(const FwdArgs& a, int block, hipStream_t stream) {
  const int64_t need = (a.ngroups + block - 1) / block;
  const dim3 grid{uint32_t(need < kStepGrid ? need : kStepGrid), 1, 1}, blk{uint32_t(block), 1, 1};
  hipLaunchKernelGGL((u8_step_kernel<P, CODES, PRINTED>), grid, blk, 0, stream, a);
  return hipGetLastError();
}

template <int P>
hipError_t launch_p(const FwdArgs& a, int flags, int block, hipStream_t stream) {
  const dim3 grid{uint32_t((a.ngroups + block - 1) / block), 1, 1}, blk{uint32_t(block), 1, 1};
  const bool codes = (flags & FWD_CODES) != 0, printed = (flags & FWD_PRINTED) != 0;
  if (a.T == 1) {
    if (codes && printed) return launch_step<P, true, true>(a, block, stream);
    if (codes) return launch_step<P, true, false>(a, block, stream);
    if (printed) return launch_step<P, false, true>(a, block, stream);
    return launch_step<P, false, false>(a, block, stream);
  }
  if (codes && printed) hipLaunchKernelGGL((u8_kernel<P, true, true>), grid, blk, 0, stream, a);
  else if (codes) hipLaunchKernelGGL((u8_kernel<P, true, false>), grid, blk, 0, stream, a);
  else if (printed) hipLaunchKernelGGL((u8_kernel<P, false, true>), grid, blk, 0, stream, a);
  else hipLaunchKernelGGL((u8_kernel<P, false, false>), grid, blk, 0, stream, a);
  return hipGetLastError();
}

__global__ void __launch_bounds__(256) u8_init_kernel(const FwdArgs a) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.H * a.W) return;
  const int64_t h = i / a.W, w = i - h * a.W;
  const uint8_t x = static_cast<const uint8_t*>(a.frames)[h * a.row_stride + w];
  const uint8_t v = uint8_t(stored(a.var_init));
  static_cast<uint8_t*>(a.mean_a)[i] = x;
  static_cast<uint8_t*>(a.mean_c)[i] = x;
  static_cast<uint8_t*>(a.var_a)[i] = v;
  static_cast<uint8_t*>(a.var_c)[i] = v;
  a.age_a[i] = 1;
  a.age_c[i] = 1;
}

// The appendix's preprocessing as it runs on 8-bit frames, fused into the
// 8-bit update (one pass over the sequence, like pre_kernel): a workgroup owns
// a 16 x 64 tile (8 x 32 on small frames) for all frames, each lane four (one)
// adjacent pixels of one row with their models in registers.  Per frame it stages the tile's raw bytes
// plus a halo of RG + 1 rows and columns in LDS (indices clamped to the frame),
// computes every blurred byte of the tile and of the median's halo with the
// two-dimensional single-precision sum of the appendix's blur (window rows
// outer, columns inner, weights float(w_i * w_j), every product and sum
// rounded, no fused multiply-add), drops its fraction (limited to 255), takes
// each pixel's median of the nine blurred bytes around it and runs the 8-bit
// update on it.  Two barriers per frame: after the raw bytes are staged and
// after the blurred bytes are written; the next frame's bytes are loaded into
// registers while the current one is filtered.  All tile cell indices come
// from geom::pre::Geo.  Runs the calls with decision codes, without a blur, and
// those for which the matrix kernel does not pay (matrix_pays()).
template <int RG, bool MED, bool PRINTED, typename Tile>
__global__ void __launch_bounds__(geom::pre::NT) pre_u8_kernel(const PreArgs a) {
  using G = geom::pre::Geo<RG, MED, Tile>;
  constexpr int PX = G::PX, TH = G::TH, TW = G::TW;
  constexpr int N = 2 * RG + 1;  // taps per window row
  __shared__ float buf_raw[G::RAW_N];
  __shared__ float buf_gb[RG > 0 ? G::GB_N : 1];
  __shared__ Tables8 tbl;
  const int64_t tile = tile_here(a);
  if (tile < 0) return;
  const StepConsts<double> k =
      make_consts<double>(a.theta_s, a.theta_d, a.var_init, a.var_floor, a.mask_floor);
  fill_tables(tbl, k, a.weight_rule, a.age_max, a.var_init);  // var_init already stored
  const uint32_t var_init = uint32_t(a.var_init);
  float w2[N * N];  // the window's weights, row-major, rounded once
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) w2[i * N + j] = float(a.w[i] * a.w[j]);

  const int64_t y0 = (tile / a.tiles_x) * TH, x0 = (tile % a.tiles_x) * TW;
  const int tid = threadIdx.x;
  const int ty = G::lane_row(tid), tx = G::lane_col(tid);
  const int64_t gy = y0 + ty;

  uint32_t roff[G::LOADS];  // frame offsets of this lane's raw cells (fixed per frame)
#pragma unroll
  for (int l = 0; l < G::LOADS; ++l) {
    const int i = G::raw_cell(tid, l);
    roff[l] = i < G::RAW_N ? uint32_t(G::raw_source(i, y0, x0, a.H, a.W, a.row_stride)) : 0u;
  }
  int gr[3], gc[PX + 2];
#pragma unroll
  for (int d = 0; d < 3; ++d) gr[d] = G::med_row(gy, d, y0, a.H);
#pragma unroll
  for (int d = 0; d < PX + 2; ++d) gc[d] = G::med_col(x0 + tx, d, x0, a.W);

  bool valid[PX];
  bool all_valid = gy < a.H;
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    valid[q] = gy < a.H && x0 + tx + q < a.W;
    all_valid = all_valid && valid[q];
  }
  const int64_t pix = gy * a.W + x0 + tx;
  const int64_t foff = gy * a.row_stride + x0 + tx;
  const bool vec_ok = all_valid && (a.row_stride % PX) == 0 && (a.frame_stride % PX) == 0 &&
                      (a.W % PX) == 0;

  const uint8_t* const planes_in[4] = {static_cast<const uint8_t*>(a.mean_a),
                                       static_cast<const uint8_t*>(a.var_a),
                                       static_cast<const uint8_t*>(a.mean_c),
                                       static_cast<const uint8_t*>(a.var_c)};
  Model8 s[PX];
  {
    Planes8<PX> b;
#pragma unroll
    for (int q = 0; q < PX; ++q) {
      b.mA.v[q] = valid[q] ? planes_in[0][pix + q] : uint8_t(0);
      b.vA.v[q] = valid[q] ? planes_in[1][pix + q] : uint8_t(0);
      b.mC.v[q] = valid[q] ? planes_in[2][pix + q] : uint8_t(0);
      b.vC.v[q] = valid[q] ? planes_in[3][pix + q] : uint8_t(0);
      b.aA.v[q] = valid[q] ? a.age_a[pix + q] : uint8_t(1);
      b.aC.v[q] = valid[q] ? a.age_c[pix + q] : uint8_t(1);
    }
    unpack8<PX>(b, tbl, s);
  }

  const uint8_t* frames = static_cast<const uint8_t*>(a.frames);
  uint8_t nxt[G::LOADS];
  auto load_frame = [&](int64_t t) {
    const uint8_t* f = frames + t * a.frame_stride;
#pragma unroll
    for (int l = 0; l < G::LOADS; ++l)
      if (G::raw_active(tid, l)) nxt[l] = f[roff[l]];
  };
  if (a.T > 0) load_frame(0);

  for (int64_t t = 0; t < a.T; ++t) {
    // 1. stage the raw bytes, then start loading the next frame's
#pragma unroll
    for (int l = 0; l < G::LOADS; ++l)
      if (G::raw_active(tid, l)) buf_raw[G::raw_cell(tid, l)] = float(nxt[l]);
    __syncthreads();
    if (t + 1 < a.T) load_frame(t + 1);

    const float* gbp;
    if constexpr (RG > 0) {
      // 2. the blurred bytes of the tile and the median's halo
#pragma unroll
      for (int it = 0; it < G::GB_IT; ++it) {
        if (G::gb_active(tid, it)) {
          const int cell = G::gb_cell(tid, it);
          const float* win = buf_raw + G::blur_window(cell);
          float blur = 0.0f;
#pragma unroll
          for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) {
              const float prod = win[i * G::RAW_W + j] * w2[i * N + j];
              blur = blur + prod;
            }
          buf_gb[cell] = __builtin_fminf(255.0f, __builtin_fmaxf(0.0f, __builtin_truncf(blur)));
        }
      }
      __syncthreads();
      gbp = buf_gb;
    } else {
      gbp = buf_raw;  // no blur: the raw bytes are the blurred ones (R = RM)
    }
    constexpr int GW = RG > 0 ? G::GB_W : G::RAW_W;

    // 3. each pixel's median of the nine blurred bytes (exact in single
    // precision: the values are integers), then the 8-bit update
    uint32_t xs[PX];
    if constexpr (MED) {
      float lo[PX + 2], md[PX + 2], hi[PX + 2];
#pragma unroll
      for (int d = 0; d < PX + 2; ++d) {
        const float p0 = gbp[gr[0] * GW + gc[d]];
        const float p1 = gbp[gr[1] * GW + gc[d]];
        const float p2 = gbp[gr[2] * GW + gc[d]];
        const float l01 = __builtin_fminf(p0, p1), h01 = __builtin_fmaxf(p0, p1);
        lo[d] = __builtin_fminf(l01, p2);
        const float h = __builtin_fmaxf(l01, p2);
        hi[d] = __builtin_fmaxf(h01, h);
        md[d] = __builtin_fminf(h01, h);
      }
#pragma unroll
      for (int q = 0; q < PX; ++q) {
        const float a0 = __builtin_fmaxf(__builtin_fmaxf(lo[q], lo[q + 1]), lo[q + 2]);
        const float b0 = __builtin_fmaxf(__builtin_fminf(md[q], md[q + 1]),
                                         __builtin_fminf(__builtin_fmaxf(md[q], md[q + 1]), md[q + 2]));
        const float c0 = __builtin_fminf(__builtin_fminf(hi[q], hi[q + 1]), hi[q + 2]);
        xs[q] = uint32_t(__builtin_fmaxf(__builtin_fminf(a0, b0),
                                       __builtin_fminf(__builtin_fmaxf(a0, b0), c0)));
      }
    } else {
#pragma unroll
      for (int q = 0; q < PX; ++q) xs[q] = uint32_t(gbp[gr[1] * GW + gc[q + 1]]);
    }

    Vec<uint8_t, PX> mk, cd, fv;
    mk = __builtin_bit_cast(decltype(mk), typename fwd::Raw<PX>::type(
                                              frame8<PX, true, true, PRINTED>(s, xs, var_init, tbl, cd)));
#pragma unroll
    for (int q = 0; q < PX; ++q) fv.v[q] = uint8_t(xs[q]);
    uint8_t* const filt = static_cast<uint8_t*>(a.filtered);
    const int64_t o = t * a.frame_stride + foff;
    if (vec_ok) {
      *reinterpret_cast<Vec<uint8_t, PX>*>(a.masks + o) = mk;
      if (filt) *reinterpret_cast<Vec<uint8_t, PX>*>(filt + o) = fv;
      if (a.codes) *reinterpret_cast<Vec<uint8_t, PX>*>(a.codes + o) = cd;
    } else {
#pragma unroll
      for (int q = 0; q < PX; ++q) {
        if (!valid[q]) continue;
        a.masks[o + q] = mk.v[q];
        if (filt) filt[o + q] = fv.v[q];
        if (a.codes) a.codes[o + q] = cd.v[q];
      }
    }
    if constexpr (RG == 0) __syncthreads();  // the next frame overwrites the raw bytes
  }

#pragma unroll
  for (int q = 0; q < PX; ++q) {
    if (!valid[q]) continue;
    const Planes8<PX> b = pack8<PX>(s);
    static_cast<uint8_t*>(a.mean_a)[pix + q] = b.mA.v[q];
    static_cast<uint8_t*>(a.var_a)[pix + q] = b.vA.v[q];
    static_cast<uint8_t*>(a.mean_c)[pix + q] = b.mC.v[q];
    static_cast<uint8_t*>(a.var_c)[pix + q] = b.vC.v[q];
    a.age_a[pix + q] = b.aA.v[q];
    a.age_c[pix + q] = b.aC.v[q];
  }
}

// ------------------------------------------------- the blur on matrix cores
// The appendix's blurred byte is the integer part of a sum of N x N rounded
// products, added one by one in single precision (50 vector instructions and 25
// LDS reads a pixel for 5 taps, which bounded pre_u8_kernel).  Here the same sum
// is first formed exactly in fixed point by the matrix cores: the weights are
// rounded to multiples of 2^-24, split into three signed bytes, and the window
// sums are products of 8-bit matrices with 32-bit sums.  How far the
// single-precision result can lie from that sum is known (the weights' rounding
// and the bound on the rounding of every product and addition, blur_weights()), so
// its integer part is known too unless an integer lies that near the sum; those
// cells (about one in 3,000 on noisy frames) are evaluated in single precision, in
// the appendix's order, one by one while their wavefront waits.
//
// Without noise many sums are integers (a ramp of one level a pixel: 99 % of the
// cells are undecided; a flat area: all).  A workgroup that finds DENSE8 lanes or
// more with undecided cells therefore forms all its sums in single precision, four
// adjacent cells a lane, until a later look (every 16th frame) finds fewer; its
// first frame it forms so too.  The way does not change a byte.  50 x 1080 x 1920
// on MI355X, 3 / 5 / 7 taps: ramp 552 / 769 / 1,790 us with every undecided cell
// by itself, 319 / 436 / 635 us so; pre_u8_kernel below 330 / 452 / 665 us; flat
// frames 312 / 435 / 634 us; noise 308 / 333 / 491 and 293 / 333 / 484 us.
// Limits of 2, 4, 12 and 32 lanes (a look every 8th frame): noise with flat squares
// on 5 % of the frame 422 / 419 / 419 / 412 us, on 30 % 479 / 484 / 499 / 534 us, a
// smooth pattern (4 % undecided) 441 / 441 / 491 / 606 us.  A look every 8th and
// every 16th frame, with the compiler told that both are rare: noise, 100 x 1920 x
// 2560, 5 taps 1,515 and 1,494 us, 7 taps 2,174 and 2,138 us.  Slowest against
// pre_u8_kernel is what a look can't foretell: flat squares on 30 % of the frame, at
// other places in every frame (483 / 452 us; 7 taps 822 / 665 us).
//
// One matrix product covers 16 windows of 16 bytes in four rows: column n of B
// is a window (lane n % 16 holds 16 bytes of row lane / 16), row m of A the
// weights of the window's output m, a diagonal band, so that a product gives OW
// adjacent blurred cells of each of 16 windows.  Rows beyond the fourth are a
// second product.  Each wavefront takes every fourth group of 16 windows.
//
// Tiles are 8 x 64 pixels, two per lane: a wavefront has one group of windows a
// frame (60 of the 64 windows are used with 5 taps) and four workgroups fit a
// CU; 16 x 64 tiles, four pixels per lane, needed 192 registers (1,047 against
// 908 us for 50 frames of 1920 x 2560).  Frames of fewer 16 x 64 tiles than
// SMALL8_BELOW take 8 x 32 tiles, one pixel per lane (8 x 64 / 8 x 32 tiles):
// 500 x 240 x 320 (75) 722 / 571 us, 100 x 360 x 480 (184) 160 / 125 us,
// 100 x 480 x 640 (300) 166 / 205 us, 50 x 1080 x 1920 (2,040) 337 / 450 us.
// Bound by vector issue (83 instructions a pixel on noisy frames, half of them the
// 8-bit update).  pre_u8_kernel, which sums the windows in single precision, takes
// 600, 140, 278 and 460 us.
constexpr int64_t SMALL8_BELOW = 256;
constexpr uint32_t DENSE8 = 4;

typedef int32_t V4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t min3u(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_min3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ uint32_t med3u(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ uint32_t max3u(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_max3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// A call's window weights, prepared on the host (blur_weights()): row-major, the
// sums' bound in units of 2^-24 (the single-precision sum lies at most `above`
// above the fixed-point one and width - above below it; 0: the weights don't fit),
// 128 times the fixed-point weights' sum, and the fixed-point weights' three
// signed bytes, each window row from byte 16 of a row of zeros.
struct Blur8 {
  float w[49];
  uint32_t above, width, centre128;
  uint32_t digits[3][8][9];
};

template <int RG, bool MED, bool PRINTED, typename Tile>
__global__ void __launch_bounds__(geom::pre::NT)
    __attribute__((amdgpu_waves_per_eu(RG == 1 ? 5 : 4)))  // 3 taps, noise: 291 us at 5, 330 at 4
    pre_u8_mfma_kernel(const PreArgs a, const Blur8 f) {
  using E = geom::pre::Geo8<RG, MED, Tile>;
  using G = typename E::G;
  constexpr int N = E::N, PX = G::PX, TH = G::TH, TW = G::TW, NT = geom::pre::NT;
  __shared__ alignas(16) uint32_t raw[G::RAW_H * E::RP];   // bytes with the top bit flipped
  __shared__ alignas(16) uint32_t gb[G::GB_H * E::GBP];    // blurred bytes, one to a dword
  __shared__ Tables8 tbl;
  __shared__ uint32_t undecided[NT / 64];  // lanes with undecided cells, by wavefront
  const int64_t tile = tile_here(a);
  if (tile < 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool fixed = f.width != 0;  // the weights fit the fixed point
  const int64_t y0 = (tile / a.tiles_x) * TH, x0 = (tile % a.tiles_x) * TW;
  const int ty = G::lane_row(tid), tx = G::lane_col(tid);
  const int64_t gy = y0 + ty;

  // this lane's staged dwords: frame row offset, first column, LDS index.  Where
  // no column of the tile leaves the frame a dword is one (unaligned) load.
  const bool inner = E::inner(x0, a.W);
  uint32_t off[E::LD][4], slot[E::LD];  // the four bytes' frame offsets (< 2^31, host check)
#pragma unroll
  for (int l = 0; l < E::LD; ++l) {
    const int i = E::staged(tid, l) ? E::stage_cell(tid, l) : 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      off[l][b] = uint32_t(E::stage_source(i, b, y0, x0, a.H, a.W, a.row_stride));
    slot[l] = uint32_t(E::stage_slot(i));
  }
  // the median's rows and columns in the blurred tile, clamped to the frame
  int gr[3], gc[PX + 2];
#pragma unroll
  for (int d = 0; d < 3; ++d) gr[d] = G::med_row(gy, d, y0, a.H);
#pragma unroll
  for (int d = 0; d < PX + 2; ++d) gc[d] = G::med_col(x0 + tx, d, x0, a.W);
  const bool inside = y0 > 0 && y0 + TH < a.H && x0 > 0 && x0 + TW < a.W;

  bool valid[PX];
  bool all_valid = gy < a.H;
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    valid[q] = gy < a.H && x0 + tx + q < a.W;
    all_valid = all_valid && valid[q];
  }
  const int64_t pix = gy * a.W + x0 + tx;
  const int64_t foff = gy * a.row_stride + x0 + tx;
  const bool vec_ok = all_valid && (a.row_stride % PX) == 0 && (a.frame_stride % PX) == 0 &&
                      (a.W % PX) == 0;

  uint8_t* const planes[4] = {static_cast<uint8_t*>(a.mean_a), static_cast<uint8_t*>(a.var_a),
                              static_cast<uint8_t*>(a.mean_c), static_cast<uint8_t*>(a.var_c)};
  // the state and the first frame are requested before the tables are built
  Planes8<PX> first;
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    first.mA.v[q] = valid[q] ? planes[0][pix + q] : uint8_t(0);
    first.vA.v[q] = valid[q] ? planes[1][pix + q] : uint8_t(0);
    first.mC.v[q] = valid[q] ? planes[2][pix + q] : uint8_t(0);
    first.vC.v[q] = valid[q] ? planes[3][pix + q] : uint8_t(0);
    first.aA.v[q] = valid[q] ? a.age_a[pix + q] : uint8_t(1);
    first.aC.v[q] = valid[q] ? a.age_c[pix + q] : uint8_t(1);
  }

  const uint8_t* frames = static_cast<const uint8_t*>(a.frames);
  uint32_t nxt[E::LD];
  auto load_frame = [&](int64_t t) {
    const uint8_t* x = frames + t * a.frame_stride;
    typedef uint32_t U1 __attribute__((aligned(1)));
    if (inner) {
#pragma unroll
      for (int l = 0; l < E::LD; ++l) nxt[l] = *reinterpret_cast<const U1*>(x + off[l][0]);
    } else {
#pragma unroll
      for (int l = 0; l < E::LD; ++l) {
        nxt[l] = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) nxt[l] |= uint32_t(x[off[l][b]]) << (8 * b);
      }
    }
  };
  if (a.T > 0) load_frame(0);

  // A: output m = lane % 16, row group lane / 16, byte j: the weight's digit of
  // window row dy, window column j - m: bytes 16 - m .. 31 - m of the row (row N
  // is zero, for lanes without an output)
  const int m = lane & 15, rgrp = lane >> 4;
  V4 A[E::SETS][3];
#pragma unroll
  for (int st = 0; st < E::SETS; ++st)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t* row = f.digits[q][m < E::OW ? 4 * st + rgrp : N] + (16 - m) / 4;
#pragma unroll
      for (int dw = 0; dw < 4; ++dw)
        A[st][q][dw] = int32_t(__builtin_amdgcn_alignbyte(row[dw + 1], row[dw], uint32_t(-m) & 3u));
    }
  // (columns past the staged ones: cells that no lane takes, but sums that count)
  for (int i = tid; i < G::RAW_H * E::RP; i += NT) raw[i] = 0x80808080u;
  const StepConsts<double> k =
      make_consts<double>(a.theta_s, a.theta_d, a.var_init, a.var_floor, a.mask_floor);
  fill_tables(tbl, k, a.weight_rule, a.age_max, a.var_init);  // ends with a barrier
  const uint32_t var_init = uint32_t(a.var_init);
  // the bytes are staged less 128: the sum gets 128 times the weights back
  // and the sum's upper end is what is formed: its integer part is the result's
  // unless the integer lies less than `width` below it
  const int32_t centre = int32_t(f.above + f.centre128);
  const uint32_t width8 = f.width << 8;  // compared with the fraction in the top 24 bits
  const float near = float(f.width) * 0x1p-24f;
  Model8 s[PX];
  unpack8<PX>(first, tbl, s);

  bool plain = true;
  for (int64_t t = 0; t < a.T; ++t) {
    // 1. stage the raw bytes, then start loading the next frame's
#pragma unroll
    for (int l = 0; l < E::LD; ++l)
      if (E::staged(tid, l)) raw[slot[l]] = nxt[l] ^ 0x80808080u;
    __syncthreads();
    if (t + 1 < a.T) load_frame(t + 1);

    // 2. the blurred bytes of the tile and the median's halo
    const bool look = fixed && (t == 0 || (t & 15) == 15);  // this frame decides the next ones' way
    uint32_t n_undecided = 0;
    if (__builtin_expect(plain, RG == 1)) {
      // every sum in the appendix's order, four adjacent cells a lane
#pragma unroll 1
      for (int c = tid; c < E::QUADS; c += NT) {
        const uint32_t* src = raw + E::quad_src(c);
        float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int y = 0; y < N; ++y) {
          float v[N + 3];
#pragma unroll
          for (int x = 0; x < N + 3; ++x)
            v[x] = float(((src[y * E::RP + x / 4] ^ 0x80808080u) >> (8 * (x & 3))) & 0xFFu);
#pragma unroll
          for (int x = 0; x < N; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float prod = v[x + i] * f.w[y * N + x];
              sum[i] = sum[i] + prod;
            }
        }
        Vec<uint32_t, 4> out;
        bool any = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          out.v[i] = uint32_t(__builtin_fminf(255.0f, __builtin_fmaxf(0.0f, sum[i])));
          any |= __builtin_fabsf(sum[i] - __builtin_rintf(sum[i])) < near && sum[i] > 0.5f;
        }
        n_undecided += uint32_t(__builtin_popcountll(__builtin_amdgcn_ballot_w64(any)));
        *reinterpret_cast<Vec<uint32_t, 4>*>(gb + E::quad_dst(c)) = out;
      }
    } else {
      for (int grp = wave; grp < E::GROUPS; grp += NT / 64) {
        const int win = grp * 16 + m, wr = E::win_row(win), wc = E::win_col(win);
        V4 acc[3] = {V4{centre, centre, centre, centre}, V4{0, 0, 0, 0}, V4{0, 0, 0, 0}};
#pragma unroll
        for (int st = 0; st < E::SETS; ++st) {
          const uint32_t* src = raw + E::win_src(wr, wc, 4 * st + rgrp);
          const V4 B = {int32_t(src[0]), int32_t(src[1]), int32_t(src[2]), int32_t(src[3])};
#pragma unroll
          for (int q = 0; q < 3; ++q)
            acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[st][q], B, acc[q], 0, 0, 0);
        }
        // this lane has outputs 4*rgrp .. + 3 of its window
        uint32_t out[4], frac[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t sum =
              (((uint32_t(acc[2][i]) << 8) + uint32_t(acc[1][i])) << 8) + uint32_t(acc[0][i]);
          out[i] = sum >> 24;
          frac[i] = sum << 8;
        }
        const bool mine = E::takes(win, rgrp);
        const uint32_t low = frac[0] < frac[1] ? frac[0] : frac[1];
        if (__builtin_amdgcn_ballot_w64(mine && min3u(low, frac[2], frac[3]) < width8) != 0) {
          // an integer (not zero: the sum is not negative) lies too near one of the
          // sums: the undecided cells are evaluated in the appendix's order
          uint32_t todo = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            todo |= mine && frac[i] < width8 && out[i] != 0 ? 1u << i : 0u;
          if (__builtin_expect(look, 0))
            n_undecided += uint32_t(__builtin_popcountll(__builtin_amdgcn_ballot_w64(todo != 0)));
          while (__builtin_amdgcn_ballot_w64(todo != 0) != 0) {
            const int i = todo != 0 ? __builtin_ctz(todo) : 0;
            // (a lane that is done reads its window's first columns)
            const int col = todo != 0 ? wc + 4 * rgrp + i : wc, sh = col & 3;
            const uint32_t* src = raw + E::cell_src(wr, col);
            // a window row's N bytes lie in at most three dwords
            uint32_t d[N][3];
#pragma unroll
            for (int y = 0; y < N; ++y)
#pragma unroll
              for (int q = 0; q < (N > 5 ? 3 : 2); ++q) d[y][q] = src[y * E::RP + q] ^ 0x80808080u;
            float blur = 0.0f;
#pragma unroll
            for (int y = 0; y < N; ++y) {
              const uint32_t b0 = __builtin_amdgcn_alignbyte(d[y][1], d[y][0], sh);
              const uint32_t b1 = N > 5 ? __builtin_amdgcn_alignbyte(d[y][2], d[y][1], sh)
                                        : d[y][1] >> (8 * sh);
#pragma unroll
              for (int x = 0; x < N; ++x) {
                const uint32_t byte = ((x < 4 ? b0 : b1) >> (8 * (x & 3))) & 0xFFu;
                const float prod = float(byte) * f.w[y * N + x];
                blur = blur + prod;
              }
            }
            const uint32_t v = uint32_t(__builtin_fminf(255.0f, blur));
#pragma unroll
            for (int q = 0; q < 4; ++q) out[q] = todo != 0 && q == i ? v : out[q];
            todo &= todo - 1;
          }
        }
        if (mine) {
          uint32_t* dst = gb + E::win_dst(wr, wc, rgrp);
          *reinterpret_cast<Vec<uint32_t, 4>*>(dst) = Vec<uint32_t, 4>{{out[0], out[1], out[2], out[3]}};
        }
      }
    }
    if (__builtin_expect(look, 0)) {  // (uniform, as the test of the lane is not)
      if (lane == 0) undecided[wave] = n_undecided;
    }
    __syncthreads();
    if (__builtin_expect(look, 0)) {
      const uint32_t n = undecided[0] + undecided[1] + undecided[2] + undecided[3];
      plain = __builtin_amdgcn_readfirstlane(n) >= DENSE8;
    }

    // 3. each pixel's median of the nine blurred bytes, then the 8-bit update
    uint32_t xs[PX];
    if constexpr (MED) {
      uint32_t p[3][PX + 2];
      if (inside) {
        const uint32_t* nb = gb + ty * E::GBP + tx;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int d = 0; d < PX + 2; ++d) p[r][d] = nb[r * E::GBP + d];
      } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int d = 0; d < PX + 2; ++d) p[r][d] = gb[gr[r] * E::GBP + gc[d]];
      }
      uint32_t lo[PX + 2], md[PX + 2], hi[PX + 2];
#pragma unroll
      for (int d = 0; d < PX + 2; ++d) {
        lo[d] = min3u(p[0][d], p[1][d], p[2][d]);
        md[d] = med3u(p[0][d], p[1][d], p[2][d]);
        hi[d] = max3u(p[0][d], p[1][d], p[2][d]);
      }
#pragma unroll
      for (int q = 0; q < PX; ++q)
        xs[q] = med3u(max3u(lo[q], lo[q + 1], lo[q + 2]), med3u(md[q], md[q + 1], md[q + 2]),
                      min3u(hi[q], hi[q + 1], hi[q + 2]));
    } else {
#pragma unroll
      for (int q = 0; q < PX; ++q) xs[q] = gb[gr[1] * E::GBP + gc[q + 1]];
    }

    using Bytes = Vec<uint8_t, PX>;
    Bytes none, fv;
    const Bytes mk = __builtin_bit_cast(
        Bytes, typename fwd::Raw<PX>::type(frame8<PX, true, false, PRINTED>(s, xs, var_init, tbl, none)));
    const int64_t o = t * a.frame_stride + foff;
    auto put = [&](uint8_t* out, const Bytes& v) {
      if (vec_ok) {
        *reinterpret_cast<Bytes*>(out + o) = v;
      } else {
#pragma unroll
        for (int q = 0; q < PX; ++q)
          if (valid[q]) out[o + q] = v.v[q];
      }
    };
    put(a.masks, mk);
    if (a.filtered) {
#pragma unroll
      for (int q = 0; q < PX; ++q) fv.v[q] = uint8_t(xs[q]);
      put(static_cast<uint8_t*>(a.filtered), fv);
    }
  }

  const Planes8<PX> b = pack8<PX>(s);
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    if (!valid[q]) continue;
    planes[0][pix + q] = b.mA.v[q];
    planes[1][pix + q] = b.vA.v[q];
    planes[2][pix + q] = b.mC.v[q];
    planes[3][pix + q] = b.vC.v[q];
    a.age_a[pix + q] = b.aA.v[q];
    a.age_c[pix + q] = b.aC.v[q];
  }
}

// Half an ulp of a single-precision value up to v, in units of 2^-24.
double half_ulp24(double v) {
  int e;
  std::frexp(v, &e);  // v in [2^(e-1), 2^e)
  return std::ldexp(1.0, e - 1);
}

// The window weights float(w_i * w_j), and, if they fit the fixed-point form,
// their digits and how far the appendix's single-precision sum can lie above the
// fixed-point one and from its lowest to its highest: the weights' rounding at all
// pixels whose weight was rounded down (up), and half an ulp of every product and
// of every partial sum, which are largest with all pixels at 255 (the rounding of
// a sum grows with it).
Blur8 blur_weights(const double* w, int n) {
  Blur8 f{};
  bool fits = true;
  double total = 0.0, down = 0.0, up = 0.0, chain = 0.0;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      f.w[i * n + j] = float(w[i] * w[j]);
      const double v = double(f.w[i * n + j]);
      fits = fits && v >= 0.0 && v <= 0.49;  // three signed bytes of 2^-24
      if (!fits) continue;
      const double fixed = std::rint(v * 16777216.0), off = v * 16777216.0 - fixed;
      (off > 0.0 ? down : up) += std::fabs(off);
      total += v;
      if (v > 0.0) chain += half_ulp24(255.001 * v);
      if (total > v) chain += half_ulp24(255.001 * total);  // the first sum is the product itself
      int32_t rest = int32_t(fixed);
      f.centre128 += 128u * uint32_t(rest);
      for (int q = 0; q < 3; ++q) {
        const int8_t d = int8_t(rest);  // the low byte, signed
        rest = (rest - d) / 256;
        reinterpret_cast<int8_t*>(f.digits[q][i])[16 + j] = d;
      }
    }
  const double above = std::ceil(255.0 * down + 1.0001 * chain) + 1.0;
  const double width = above + std::ceil(255.0 * up + 1.0001 * chain) + 1.0;
  // 255 * total + above stays below 256
  if (fits && total <= 1.003 && width < double(1u << 20)) {
    f.above = uint32_t(above);
    f.width = uint32_t(width);
  }
  return f;
}

template <int RG, bool MED, bool PRINTED>
hipError_t launch_pre_mfma(PreArgs a, const Blur8& f, hipStream_t stream) {
  using geom::pre::Small;
  using geom::pre::Wide;
  auto go = [&](auto tile, auto kernel) {
    using Tile = decltype(tile);
    a.tiles_x = (a.W + Tile::tw - 1) / Tile::tw;
    a.tiles_y = (a.H + Tile::th - 1) / Tile::th;
    hipLaunchKernelGGL(kernel, tile_grid(a), dim3(geom::pre::NT), 0, stream, a, f);
    return hipGetLastError();
  };
  if constexpr (MED) {  // (matrix_pays() sends no small frames without it)
    if (a.tiles_x * a.tiles_y < SMALL8_BELOW)  // tiles of 16 x 64 (the caller's count)
      return go(Small{}, pre_u8_mfma_kernel<RG, MED, PRINTED, Small>);
  }
  return go(Wide{}, pre_u8_mfma_kernel<RG, MED, PRINTED, Wide>);
}

// Whether a call runs the matrix kernel, by taps, call length and frame size (tiles of
// 16 x 64).  Its set-up, and on large frames its tiles of half the size, have to be
// paid for by the blur.  pre_u8_kernel / pre_u8_mfma_kernel, us.  With the median: T x
// 1080 x 1920, 5 taps T = 1 23.4 / 25.2, 2 32.5 / 32.0, 4 50.1 / 44.0; 7 taps 4 66.8 /
// 63.3, 6 91.7 / 81.8; 3 taps 2 27.3 / 26.3; without noise 5 taps 4 49.7 / 50.8, 7 taps 8
// 117.8 / 120.9; 600 x 800 (494 tiles) 7 taps 1 10.0 / 11.0, a smooth pattern 4 21.7 /
// 27.0; 480 x 640 (300) 5 taps 1 8.5 / 7.7, 7 taps 4 21.3 / 18.5.  Weights that don't
// fit the fixed point, summed in single precision throughout: 5 taps 6 x 1080 x 1920
// 67.9 / 68.2, 32 294 / 285, 500 x 240 x 320 1,225 / 739.  Without the median, whose halo
// makes most of the windows, three and five taps are too little: 50 x 1080 x 1920 194 /
// 228 and 280 / 276 (without noise 263 / 350), 100 x 480 x 640 84 / 132 and 108 / 142, 100
// x 70 x 99 67 / 98 and 85 / 125; seven taps 50 x 1080 x 1920 430 / 329 (440 / 503), 4
// 47 / 45 (47 / 55), 50 x 600 x 800 121 / 101, 100 x 480 x 640 148 / 169.
bool matrix_pays(int rg, bool median, bool fits, int64_t T, int64_t tiles) {
  constexpr int64_t LARGE8 = 400;
  if (!median) return rg == 3 && fits && T >= 8 && tiles >= LARGE8;
  return tiles < LARGE8 || T >= (rg == 1 ? 1 : !fits ? 16 : rg == 2 ? 3 : 5);
}

// The single-precision kernel on 16 x 64 tiles, on small frames 8 x 32: there the
// chain of a tile's frames bounds the call (16 x 64 / 8 x 32, median only 24 x 240 x
// 320 34.4 / 18.5 us, 5 taps with codes 65.7 / 33.8; 1 x 70 x 99 5.9 / 4.0).  Without
// the median a tile's halo is narrow, and frames below MIDDLE8 tiles, and calls of four
// frames and more at any size, take 8 x 32: 3 / 5 taps 1 x 480 x 640 7.1 / 5.3 and 7.7 /
// 5.6 us, 50 x 800 x 1300 167 / 112 and 225 / 152 us, 50 x 1080 x 1920 215 /
// 194 and 297 / 280, 4 x 1080 x 1920 29.7 / 27.9 and 35.9 / 34.6 (one frame 17.8 / 17.7
// and 17.3 / 20.3; without the blur 50 x 1080 x 1920 179 / 200).
template <int RG, bool MED, bool PRINTED>
hipError_t launch_pre_plain(PreArgs a, hipStream_t stream) {
  auto go = [&](auto tile, auto kernel) {
    using Tile = decltype(tile);
    a.tiles_x = (a.W + Tile::tw - 1) / Tile::tw;
    a.tiles_y = (a.H + Tile::th - 1) / Tile::th;
    hipLaunchKernelGGL(kernel, tile_grid(a), dim3(geom::pre::NT), 0, stream, a);
    return hipGetLastError();
  };
  constexpr int64_t MIDDLE8 = 512;
  const int64_t tiles = a.tiles_x * a.tiles_y;
  if (tiles < SMALL8_BELOW || (RG > 0 && !MED && (a.T >= 4 || tiles < MIDDLE8)))
    return go(geom::pre::Small{}, pre_u8_kernel<RG, MED, PRINTED, geom::pre::Small>);
  return go(geom::pre::Big{}, pre_u8_kernel<RG, MED, PRINTED, geom::pre::Big>);
}

template <bool MED, bool PRINTED>
hipError_t launch_pre_rg(const PreArgs& a, int rg, hipStream_t stream) {
  // (decision codes, a debug output, exist on pre_u8_kernel only)
  bool matrix = rg > 0 && !a.codes;
  Blur8 f;
  if (matrix) {
    f = blur_weights(a.w, 2 * rg + 1);
    matrix = matrix_pays(rg, MED, f.width != 0, a.T, a.tiles_x * a.tiles_y);
  }
  switch (rg) {
    case 0: return launch_pre_plain<0, MED, PRINTED>(a, stream);
    case 1:
      if constexpr (MED) {
        if (matrix) return launch_pre_mfma<1, MED, PRINTED>(a, f, stream);
      }
      return launch_pre_plain<1, MED, PRINTED>(a, stream);
    case 2:
      if constexpr (MED) {
        if (matrix) return launch_pre_mfma<2, MED, PRINTED>(a, f, stream);
      }
      return launch_pre_plain<2, MED, PRINTED>(a, stream);
    case 3: return matrix ? launch_pre_mfma<3, MED, PRINTED>(a, f, stream)
                          : launch_pre_plain<3, MED, PRINTED>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace u8

hipError_t launch_fwd_u8(const FwdArgs& a, int P, int flags, int block, hipStream_t stream) {
  if (flags & (FWD_BG | FWD_CKPT)) return hipErrorInvalidValue;
  if (P == 4) return u8::launch_p<4>(a, flags, block, stream);
  if (P == 2) return u8::launch_p<2>(a, flags, block, stream);
  if (P == 1) return u8::launch_p<1>(a, flags, block, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_pre_u8(const PreArgs& a, int rg, bool median, hipStream_t stream) {
  const bool printed = a.mask_rule != 0;
  if (median)
    return printed ? u8::launch_pre_rg<true, true>(a, rg, stream)
                   : u8::launch_pre_rg<true, false>(a, rg, stream);
  return printed ? u8::launch_pre_rg<false, true>(a, rg, stream)
                 : u8::launch_pre_rg<false, false>(a, rg, stream);
}

hipError_t launch_init_u8(const FwdArgs& a, hipStream_t stream) {
  const int64_t n = a.H * a.W;
  hipLaunchKernelGGL(u8::u8_init_kernel, dim3(uint32_t((n + 255) / 256)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace dsgm
