// dsgm_device.h -- device-side pieces shared by the DSGM kernels (internal).
//
// One step of the Dual-Mode Single Gaussian Model for one pixel (Henderson &
// Vertescher, arXiv:1702.05156, Sec. 2.2-2.3 and the appendix's inner update),
// written for 64-wide wavefronts, the selected model updated in place under lane masks:
//
//   match tests   hitA = (x-mA)^2 < ts*max(vA, vf); hitC = (x-mC)^2 < ts*max(vC, vf)
//                 (evaluated as two comparisons, see step_core())
//                 (C only counts when A failed: the table index below gives A priority)
//   update        the matched model (A if hitA, else C) is blended with x using the
//                 weights of its age (Sec. 2.2): m' = u*m + w*x, V = (m'-x)^2,
//                 v' = u*v + w*V, age' = min(age+1, age_max)
//   reset         neither matched: C = (x, var_init, 1).  This is the same update
//                 with the table slot RESET_SLOT, whose weights are u = 0, w = 1,
//                 whose variance offset is var_init and whose next age is 1:
//                 0*m + 1*x = x, (x-x)^2 = 0, 0*v + 1*0 + var_init = var_init, all
//                 exact in IEEE arithmetic, so no extra select is needed.
//   exchange      if hitA the result goes to A, else to C
//   swap          C older than A: A = C, C = (x, var_init, 1) (rare: a branch
//                 that the whole wavefront skips when no lane swaps)
//   mask          background iff (mA-x)^2 <= td*max(mf, ref), ref = vA or x
//
// With Acc = double every product and sum is rounded on its own (the library is
// built with -ffp-contract=off), so results are bit-identical to a scalar FP64
// evaluation in the paper's order.  With Acc = float the two blends use fused
// multiply-adds.  With Acc = f32x2 (compensated single precision, see
// dsgm_f32x2.h) the step has its own form, step_core_x2().
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dsgm_f32x2.h"

namespace dsgm {

constexpr int RESET_SLOT = 256;  // table slot used by the candidate reset
constexpr int TABLE_SIZE = 257;  // ages 0..255 plus the reset slot

enum : unsigned { CODE_HIT_A = 1, CODE_HIT_C = 2, CODE_RESET = 4, CODE_SWAP = 8, CODE_FG = 16 };

// Per-age update constants.  `r` is added to the blended variance (0 except in
// the reset slot); `next` is the age after the update.
template <typename Acc>
struct alignas(4 * sizeof(Acc)) TableEntry {
  Acc u, w, r;
  int32_t next;
};

// Ages are held in registers (and in `next`) as byte offsets of their table
// entries, so that an entry's LDS address needs no shift per frame; they order
// as the ages do.  Loads and stores of the state convert.
template <typename Acc>
__device__ __forceinline__ int age_in(int age) {
  return age * int(sizeof(TableEntry<Acc>));
}
template <typename Acc>
__device__ __forceinline__ uint8_t age_out(int offset) {
  return uint8_t(uint32_t(offset) / uint32_t(sizeof(TableEntry<Acc>)));
}
template <typename Acc>
__device__ __forceinline__ int reset_age() {
  return age_in<Acc>(RESET_SLOT);
}
template <typename Acc>
__device__ __forceinline__ TableEntry<Acc> entry_at(const TableEntry<Acc>* __restrict__ tbl,
                                                    int offset) {
  return *reinterpret_cast<const TableEntry<Acc>*>(reinterpret_cast<const char*>(tbl) + offset);
}

template <typename Acc>
struct StepConsts {
  Acc theta_s, theta_d, var_init;
  Acc ts_vf;  // theta_s * var_floor
  Acc td_mf;  // theta_d * mask_floor
};

// Fill one table slot.  w = 1/(a+1) (Sec. 2.2) or 1/a (appendix), u = 1 - w,
// both rounded in the accumulation type; age 0 (never valid) maps to w = 1.
template <typename Acc>
__device__ inline TableEntry<Acc> make_entry(int i, int weight_rule, int age_max, Acc var_init) {
  if constexpr (is_f32x2<Acc>::value) {
    // the FP64 weights, each split into the nearest pair
    const TableEntry<double> d = make_entry<double>(i, weight_rule, age_max, double(var_init));
    TableEntry<f32x2> e;
    e.u = f32x2(d.u);
    e.w = f32x2(d.w);
    e.r = i == RESET_SLOT ? var_init : f32x2(0.f);
    static_assert(sizeof(TableEntry<f32x2>) == sizeof(TableEntry<double>), "one age unit");
    e.next = d.next;
    return e;
  } else {
    TableEntry<Acc> e;
    if (i == RESET_SLOT) {
      e.u = Acc(0);
      e.w = Acc(1);
      e.r = var_init;
      e.next = age_in<Acc>(1);
      return e;
    }
    const Acc one = Acc(1);
    Acc w;
    if (weight_rule == 1)
      w = i == 0 ? one : one / Acc(i);
    else
      w = one / (Acc(i) + one);
    e.w = w;
    e.u = one - w;
    e.r = Acc(0);
    e.next = age_in<Acc>(i + 1 < age_max ? i + 1 : age_max);
    return e;
  }
}

// The per-launch constants of the step.  The floor products are rounded once
// in the accumulation type (for f32x2: formed in FP64 and split), identically
// in the forward and the adjoint's replay, so both take the same decisions.
template <typename Acc>
__device__ __forceinline__ StepConsts<Acc> step_consts(double theta_s, double theta_d,
                                                       double var_init, double var_floor,
                                                       double mask_floor) {
  StepConsts<Acc> k;
  if constexpr (is_f32x2<Acc>::value) {
    k.theta_s = f32x2(theta_s);
    k.theta_d = f32x2(theta_d);
    k.var_init = f32x2(var_init);
    k.ts_vf = f32x2(theta_s * var_floor);
    k.td_mf = f32x2(theta_d * mask_floor);
  } else {
    k.theta_s = Acc(theta_s);
    k.theta_d = Acc(theta_d);
    k.var_init = Acc(var_init);
    k.ts_vf = k.theta_s * Acc(var_floor);
    k.td_mf = k.theta_d * Acc(mask_floor);
  }
  return k;
}

__device__ __forceinline__ double larger(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ float larger(float a, float b) { return __builtin_fmaxf(a, b); }

// blend u*a + w*b
__device__ __forceinline__ double blend(double u, double a, double w, double b) {
  return u * a + w * b;  // two roundings and a rounded sum (no contraction)
}
__device__ __forceinline__ float blend(float u, float a, float w, float b) {
  return __builtin_fmaf(u, a, w * b);
}

template <typename Acc>
struct Model {
  Acc mA, vA, mC, vC;
  int aA, aC;  // ages as table offsets (age_in)
};

// Converts ages that were loaded as bytes, at this point and no earlier
// (volatile): the conversion waits for the loads, so a kernel requests its
// first frames before it.
template <typename Acc>
__device__ __forceinline__ void convert_ages(Model<Acc>& s) {
  asm volatile("" : "+v"(s.aA), "+v"(s.aC));
  s.aA = age_in<Acc>(s.aA);
  s.aC = age_in<Acc>(s.aC);
}

// What one step decided, for the reverse sweep: the table offset used (of the
// matched model's age, or of RESET_SLOT), whether A matched, whether C was promoted,
// and d = (updated mean) - x of the blend.
template <typename Acc>
struct StepRecord {
  Acc d;
  int idx;
  bool hitA, hitC, swap, fg;
  uint64_t swap_lanes;  // the lanes whose C is to be promoted
  Acc qd;               // (mA - x)^2 of the background test
  Acc qC, V;            // f32x2 only: C's test distance and the update's d*d
};

// The condition as a lane mask in a pair of scalar registers other than VCC.
// The empty asm only fixes where the mask lives: the selects on it are then
// encoded with an explicit mask register instead of the short form that reads
// VCC, whose back-to-back use stalls a gfx950 SIMD: a compare and four selects
// of 64 lanes took 72 cycles with VCC against 19 with another register pair
// (two selects 18.5 against 11.0; 8 waves per SIMD; at 2 waves 44 against
// 13.5).  Every 64-bit select is such a pair.
__device__ __forceinline__ bool lane_mask(bool c) {
  uint64_t m = __builtin_amdgcn_ballot_w64(c);
  asm("" : "+s"(m));
  return __builtin_amdgcn_inverse_ballot_w64(m);
}

// The step in compensated single precision.  The frames are floats, so x is
// exact (x.lo = 0).  Same decisions and order as step_core() below, in the
// algebraically equal forms that need fewer pair operations:
//   m' = u*m + w*x = m + w*(x - m)     (u = 1 - w)
//   d  = m' - x    = -u*(x - m)
// with x - m taken from the match test, and the reset written as a select of
// (x, var_init) so that it stays exact.
__device__ __forceinline__ StepRecord<f32x2> step_core_x2(Model<f32x2>& s, const f32x2 xx,
                                                          const StepConsts<f32x2>& k,
                                                          const TableEntry<f32x2>* __restrict__ tbl) {
  using namespace x2;
  const float x = xx.hi;
  const f32x2 dA = sub(x, s.mA);
  const f32x2 qA = sqr(dA);
  const f32x2 dC = sub(x, s.mC);
  const f32x2 qC = sqr(dC);
  // both comparisons of each test are evaluated (no short circuit)
  const bool hA0 = lt(qA, mul(k.theta_s, s.vA)), hA1 = lt(qA, k.ts_vf);
  const bool hC0 = lt(qC, mul(k.theta_s, s.vC)), hC1 = lt(qC, k.ts_vf);
  const bool hitA = hA0 | hA1;
  const bool hitC = hC0 | hC1;
  const bool reset = !hitA && !hitC;

  const int idx = hitA ? s.aA : (hitC ? s.aC : reset_age<f32x2>());
  const f32x2 m = sel(hitA, s.mA, s.mC);
  const f32x2 v = sel(hitA, s.vA, s.vC);
  const f32x2 d0 = sel(hitA, dA, dC);
  const TableEntry<f32x2> e = entry_at(tbl, idx);

  const f32x2 d = mul(f32x2(-e.u.hi, -e.u.lo), d0);  // 0 in the reset slot (u = 0)
  const f32x2 V = sqr(d);
  const f32x2 mn = sel(reset, f32x2(x), add(m, mul(e.w, d0)));
  const f32x2 vn = sel(reset, k.var_init, add(mul(e.u, v), mul(e.w, V)));
  const int an = e.next;

  s.mA = sel(hitA, mn, s.mA);
  s.vA = sel(hitA, vn, s.vA);
  s.aA = hitA ? an : s.aA;
  s.mC = sel(hitA, s.mC, mn);
  s.vC = sel(hitA, s.vC, vn);
  s.aC = hitA ? s.aC : an;

  StepRecord<f32x2> r;
  r.d = d;
  r.idx = idx;
  r.hitA = hitA;
  r.hitC = hitC && !hitA;
  r.swap_lanes = __builtin_amdgcn_ballot_w64(s.aC > s.aA);
  r.swap = __builtin_amdgcn_inverse_ballot_w64(r.swap_lanes);
  r.fg = false;
  r.qd = sel(hitA, V, qA);
  r.qC = qC;
  r.V = V;
  return r;
}

// The matched model's update in place.  `hit_a` is the mask of the lanes whose
// A matched; the other lanes update C (or reset it, by the table entry of the
// reset slot).  Both halves run under their own lane mask and write the
// model's registers directly, instead of selecting the matched model, updating
// it and selecting it back into A or C: ten selects per pixel (eighteen with
// double state) against none.  The time-fused kernels are bound by vector issue
// (a select costs 4 cycles of a SIMD, a move under a mask 2), so the updates of
// both models cost less than the selects around one.  Returned: d = (updated
// mean) - x of the blend; with QD, qa becomes the background test's squared
// distance d*d in the lanes that updated A.  The arithmetic and its order are
// those of  m' = u*m + w*x, V = (m' - x)^2, v' = u*v + w*V + r.  r enters by
// the fused w*V + r, which is the rounded product where r is zero and exactly
// r in the reset slot (w = 1, V = 0, u = 0).
template <bool QD>
__device__ __forceinline__ double update_in_place(Model<double>& s, const double x,
                                                  const TableEntry<double>& e,
                                                  const uint64_t hit_a, double& qa) {
  double d, t;
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "v_mul_f64 %[t], %[w], %[x]\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_mul_f64 %[mA], %[u], %[mA]\n\t"
      "v_mul_f64 %[vA], %[u], %[vA]\n\t"
      "v_mov_b32 %[aA], %[n]\n\t"
      "v_add_f64 %[mA], %[mA], %[t]\n\t"
      "v_add_f64 %[d], %[mA], -%[x]\n\t"
      "s_andn2_b64 exec, %[all], %[h]\n\t"
      "v_mul_f64 %[mC], %[u], %[mC]\n\t"
      "v_mul_f64 %[vC], %[u], %[vC]\n\t"
      "v_mov_b32 %[aC], %[n]\n\t"
      "v_add_f64 %[mC], %[mC], %[t]\n\t"
      "v_add_f64 %[d], %[mC], -%[x]\n\t"
      "s_mov_b64 exec, %[all]\n\t"
      "v_mul_f64 %[t], %[d], %[d]\n\t"
      "v_fma_f64 %[t], %[w], %[t], %[r]\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      ".if %[qd]\n\t"
      "v_mul_f64 %[q], %[d], %[d]\n\t"
      ".endif\n\t"
      "v_add_f64 %[vA], %[vA], %[t]\n\t"
      "s_andn2_b64 exec, %[all], %[h]\n\t"
      "v_add_f64 %[vC], %[vC], %[t]\n\t"
      "s_mov_b64 exec, %[all]"
      : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [mC] "+&v"(s.mC), [vC] "+&v"(s.vC), [aA] "+&v"(s.aA),
        [aC] "+&v"(s.aC), [q] "+&v"(qa), [d] "=&v"(d), [t] "=&v"(t), [all] "=&s"(all)
      : [x] "v"(x), [u] "v"(e.u), [w] "v"(e.w), [r] "v"(e.r), [n] "v"(e.next), [h] "s"(hit_a),
        [qd] "n"(QD ? 1 : 0)
      : "scc");
  return d;
}
template <bool QD>
__device__ __forceinline__ float update_in_place(Model<float>& s, const float x,
                                                 const TableEntry<float>& e, const uint64_t hit_a,
                                                 float& qa) {
  float d, t;
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "v_mul_f32 %[t], %[w], %[x]\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_fma_f32 %[mA], %[u], %[mA], %[t]\n\t"
      "v_mov_b32 %[aA], %[n]\n\t"
      "v_sub_f32 %[d], %[mA], %[x]\n\t"
      "s_andn2_b64 exec, %[all], %[h]\n\t"
      "v_fma_f32 %[mC], %[u], %[mC], %[t]\n\t"
      "v_mov_b32 %[aC], %[n]\n\t"
      "v_sub_f32 %[d], %[mC], %[x]\n\t"
      "s_mov_b64 exec, %[all]\n\t"
      "v_mul_f32 %[t], %[d], %[d]\n\t"
      "v_fma_f32 %[t], %[w], %[t], %[r]\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      ".if %[qd]\n\t"
      "v_mul_f32 %[q], %[d], %[d]\n\t"
      ".endif\n\t"
      "v_fma_f32 %[vA], %[u], %[vA], %[t]\n\t"
      "s_andn2_b64 exec, %[all], %[h]\n\t"
      "v_fma_f32 %[vC], %[u], %[vC], %[t]\n\t"
      "s_mov_b64 exec, %[all]"
      : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [mC] "+&v"(s.mC), [vC] "+&v"(s.vC), [aA] "+&v"(s.aA),
        [aC] "+&v"(s.aC), [q] "+&v"(qa), [d] "=&v"(d), [t] "=&v"(t), [all] "=&s"(all)
      : [x] "v"(x), [u] "v"(e.u), [w] "v"(e.w), [r] "v"(e.r), [n] "v"(e.next), [h] "s"(hit_a),
        [qd] "n"(QD ? 1 : 0)
      : "scc");
  return d;
}

// The table offset of the step: A's age where A matched, else C's where C
// matched, else the reset slot's.  A's is a move under its mask: as a nested
// select it became a branch, which kept the pixels of a lane from being
// scheduled together.
template <typename Acc>
__device__ __forceinline__ int slot_of(const Model<Acc>& s, const uint64_t hit_a,
                                       const bool hit_c) {
  int idx = hit_c ? s.aC : reset_age<Acc>();
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_mov_b32 %[i], %[aA]\n\t"
      "s_mov_b64 exec, %[all]"
      : [i] "+&v"(idx), [all] "=&s"(all)
      : [aA] "v"(s.aA), [h] "s"(hit_a));
  return idx;
}

// The same update by selects: the matched model (or C, to be reset) is selected,
// updated and selected back.  More instructions than update_in_place, but fewer one
// after the other: each write of a lane mask waits for the instructions before
// it.  `idx` is the step's table offset, qa as in update_in_place.
template <typename Acc>
__device__ __forceinline__ Acc update_selected(Model<Acc>& s, const Acc x, const bool hit_a,
                                               const bool hit_c,
                                               const TableEntry<Acc>* __restrict__ tbl, int& idx,
                                               Acc& qa) {
  const bool a = lane_mask(hit_a);
  const int ic = hit_c ? s.aC : reset_age<Acc>();
  idx = a ? s.aA : ic;
  const Acc m = a ? s.mA : s.mC;
  const Acc v = a ? s.vA : s.vC;
  const TableEntry<Acc> e = entry_at(tbl, idx);
  const Acc mn = blend(e.u, m, e.w, x);
  const Acc d = mn - x;
  const Acc V = d * d;
  const Acc vn = blend(e.u, v, e.w, V) + e.r;
  s.mA = a ? mn : s.mA;
  s.vA = a ? vn : s.vA;
  s.aA = a ? e.next : s.aA;
  s.mC = a ? s.mC : mn;
  s.vC = a ? s.vC : vn;
  s.aC = a ? s.aC : e.next;
  qa = a ? V : qa;
  return d;
}

// The mask bytes of P pixels from the lane masks of their background tests:
// 255 except in byte q of the lanes of bg[q], cleared under the masks.
template <int P>
__device__ __forceinline__ uint32_t mask_bytes(const uint64_t (&bg)[P]) {
  uint32_t m;
  uint64_t all;
  static_assert(P == 1 || P == 2 || P == 4, "pixels per lane");
  if constexpr (P == 1) {
    m = __builtin_amdgcn_inverse_ballot_w64(bg[0]) ? 0u : 255u;
  } else if constexpr (P == 2) {
    asm("s_mov_b64 %[all], exec\n\t"
        "v_mov_b32 %[m], -1\n\t"
        "s_mov_b64 exec, %[a]\n\t"
        "v_mov_b32 %[m], 0xff00\n\t"
        "s_mov_b64 exec, %[b]\n\t"
        "v_and_b32 %[m], 0xff, %[m]\n\t"
        "s_mov_b64 exec, %[all]"
        : [m] "=&v"(m), [all] "=&s"(all)
        : [a] "s"(bg[0]), [b] "s"(bg[1]));
  } else {
    asm("s_mov_b64 %[all], exec\n\t"
        "v_mov_b32 %[m], -1\n\t"
        "s_mov_b64 exec, %[a]\n\t"
        "v_mov_b32 %[m], 0xffffff00\n\t"
        "s_mov_b64 exec, %[b]\n\t"
        "v_and_b32 %[m], 0xffff00ff, %[m]\n\t"
        "s_mov_b64 exec, %[c]\n\t"
        "v_and_b32 %[m], 0xff00ffff, %[m]\n\t"
        "s_mov_b64 exec, %[d]\n\t"
        "v_and_b32 %[m], 0xffffff, %[m]\n\t"
        "s_mov_b64 exec, %[all]"
        : [m] "=&v"(m), [all] "=&s"(all)
        : [a] "s"(bg[0]), [b] "s"(bg[1]), [c] "s"(bg[2]), [d] "s"(bg[3]));
  }
  return m;
}

// Match tests, update of the matched model and the exchange decision (not yet
// applied) for one frame of one pixel.  r.fg is left unset; r.qd is the
// squared distance (mA - x)^2 after the update (QD only): the update's d*d if
// A matched, else the A test's distance (x - mA is the exact negation of
// mA - x, so the square is the same number).
template <typename Acc, bool QD = true, bool SELECT = false>
__device__ __forceinline__ StepRecord<Acc> step_core(Model<Acc>& s, const Acc x,
                                                     const StepConsts<Acc>& k,
                                                     const TableEntry<Acc>* __restrict__ tbl) {
  if constexpr (is_f32x2<Acc>::value) {
    return step_core_x2(s, x, k, tbl);
  } else {
  // q < theta*max(v, f)  <=>  q < theta*v  or  q < theta*f  for theta >= 0:
  // rounding is monotone, so round(theta*max(v,f)) = max(round(theta*v),
  // round(theta*f)); the floor products are per-launch constants.
  const Acc dA = x - s.mA;
  const Acc dC = x - s.mC;
  Acc qA = dA * dA;
  const Acc qC = dC * dC;
  const Acc tA = k.theta_s * s.vA;
  const Acc tC = k.theta_s * s.vC;
  const uint64_t hit_a = __builtin_amdgcn_ballot_w64((qA < tA) | (qA < k.ts_vf));
  const bool hitC = (qC < tC) | (qC < k.ts_vf);
  StepRecord<Acc> r;
  r.hitA = __builtin_amdgcn_inverse_ballot_w64(hit_a);
  r.hitC = hitC && !r.hitA;
  if constexpr (SELECT) {
    r.d = update_selected<Acc>(s, x, r.hitA, hitC, tbl, r.idx, qA);
  } else {
    r.idx = slot_of<Acc>(s, hit_a, hitC);
    const TableEntry<Acc> e = entry_at(tbl, r.idx);
    r.d = update_in_place<QD>(s, x, e, hit_a, qA);
  }
  r.qd = qA;
  r.swap_lanes = __builtin_amdgcn_ballot_w64(s.aC > s.aA);
  r.swap = __builtin_amdgcn_inverse_ballot_w64(r.swap_lanes);
  r.fg = false;
  return r;
  }
}

// The exchange in the lanes of `swap`: C older than A makes C the new A and
// resets C to (x, var_init, 1).  Moves under the mask, as in update_in_place.
// Callers skip it as a whole when no lane of the wavefront swaps (a uniform
// branch: 0.1 % of the pixels swap); with QD, qd becomes the new A's (mA - x)^2.
template <bool QD>
__device__ __forceinline__ void swap_in_place(Model<double>& s, const double x,
                                              const StepConsts<double>& k, const uint64_t swap,
                                              double& qd) {
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_mov_b64 %[mA], %[mC]\n\t"
      "v_mov_b64 %[vA], %[vC]\n\t"
      "v_mov_b32 %[aA], %[aC]\n\t"
      "v_mov_b64 %[mC], %[x]\n\t"
      "v_mov_b64 %[vC], %[vi]\n\t"
      "v_mov_b32 %[aC], %[one]\n\t"
      ".if %[qdf]\n\t"
      "v_add_f64 %[q], %[mA], -%[x]\n\t"
      "v_mul_f64 %[q], %[q], %[q]\n\t"
      ".endif\n\t"
      "s_mov_b64 exec, %[all]"
      : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [mC] "+&v"(s.mC), [vC] "+&v"(s.vC), [aA] "+&v"(s.aA),
        [aC] "+&v"(s.aC), [q] "+&v"(qd), [all] "=&s"(all)
      : [x] "v"(x), [vi] "v"(k.var_init), [h] "s"(swap),
        [one] "n"(int(sizeof(TableEntry<double>))), [qdf] "n"(QD ? 1 : 0));
}
template <bool QD>
__device__ __forceinline__ void swap_in_place(Model<float>& s, const float x,
                                              const StepConsts<float>& k, const uint64_t swap,
                                              float& qd) {
  uint64_t all;
  asm("s_mov_b64 %[all], exec\n\t"
      "s_mov_b64 exec, %[h]\n\t"
      "v_mov_b32 %[mA], %[mC]\n\t"
      "v_mov_b32 %[vA], %[vC]\n\t"
      "v_mov_b32 %[aA], %[aC]\n\t"
      "v_mov_b32 %[mC], %[x]\n\t"
      "v_mov_b32 %[vC], %[vi]\n\t"
      "v_mov_b32 %[aC], %[one]\n\t"
      ".if %[qdf]\n\t"
      "v_sub_f32 %[q], %[mA], %[x]\n\t"
      "v_mul_f32 %[q], %[q], %[q]\n\t"
      ".endif\n\t"
      "s_mov_b64 exec, %[all]"
      : [mA] "+&v"(s.mA), [vA] "+&v"(s.vA), [mC] "+&v"(s.mC), [vC] "+&v"(s.vC), [aA] "+&v"(s.aA),
        [aC] "+&v"(s.aC), [q] "+&v"(qd), [all] "=&s"(all)
      : [x] "v"(x), [vi] "v"(k.var_init), [h] "s"(swap),
        [one] "n"(int(sizeof(TableEntry<float>))), [qdf] "n"(QD ? 1 : 0));
}

// The exchange a step decided.  Afterwards mA is the promoted C, and with f32x2
// state its distance is the update's d*d if C matched; if A matched (possible
// only from a state whose C was older than A), the untouched C's test distance.
template <typename Acc, bool QD = true>
__device__ __forceinline__ void exchange(Model<Acc>& s, const Acc x, const StepConsts<Acc>& k,
                                         StepRecord<Acc>& r) {
  if constexpr (is_f32x2<Acc>::value) {
    const bool swap = r.swap;
    s.mA = swap ? s.mC : s.mA;
    s.vA = swap ? s.vC : s.vA;
    s.aA = swap ? s.aC : s.aA;
    s.mC = swap ? x : s.mC;
    s.vC = swap ? k.var_init : s.vC;
    s.aC = swap ? age_in<Acc>(1) : s.aC;
    r.qd = x2::sel(swap, x2::sel(r.hitA, r.qC, r.V), r.qd);
  } else {
    swap_in_place<QD>(s, x, k, r.swap_lanes, r.qd);
  }
}

// The background test (and the mask, its negation) from the step's squared
// distance qd = (mA - x)^2 and the state after the exchange.
template <typename Acc, bool PRINTED>
__device__ __forceinline__ bool bg_from(const Acc qd, const Model<Acc>& s, const Acc x,
                                        const StepConsts<Acc>& k) {
  if constexpr (is_f32x2<Acc>::value) {
    using namespace x2;
    const f32x2 ref = PRINTED ? x : s.vA;
    const bool b0 = le(qd, mul(k.theta_d, ref)), b1 = le(qd, k.td_mf);
    return b0 | b1;
  } else {
    const Acc ref = PRINTED ? x : s.vA;
    // one comparison with the larger threshold (of which neither is NaN for
    // finite input; fmax drops a NaN, as the two comparisons would)
    return qd <= larger(k.theta_d * ref, k.td_mf);
  }
}
template <typename Acc, bool PRINTED>
__device__ __forceinline__ bool fg_from(const Acc qd, const Model<Acc>& s, const Acc x,
                                        const StepConsts<Acc>& k) {
  return !bg_from<Acc, PRINTED>(qd, s, x, k);
}

// One frame of one pixel without its mask (state updated in place).
template <typename Acc>
__device__ __forceinline__ StepRecord<Acc> step_rec(Model<Acc>& s, const Acc x,
                                                    const StepConsts<Acc>& k,
                                                    const TableEntry<Acc>* __restrict__ tbl) {
  StepRecord<Acc> r = step_core<Acc, false>(s, x, k, tbl);
  if (r.swap_lanes != 0) exchange<Acc, false>(s, x, k, r);
  return r;
}

// The decision code of a step (CODE_* bits).
template <typename Acc>
__device__ __forceinline__ unsigned code_of(const StepRecord<Acc>& r) {
  return (r.hitA ? CODE_HIT_A : (r.hitC ? CODE_HIT_C : CODE_RESET)) | (r.swap ? CODE_SWAP : 0u) |
         (r.fg ? CODE_FG : 0u);
}

// Adjoint of one step, decisions fixed (the chain rule through step_rec):
//   bg = mA after the step           gmA += gbg
//   swap: A <- C, C <- (x, var_init) gx += gmC, gvi += gvC, (gmC, gvC) <- (gmA, gvA), A's = 0
//   blend of the matched model M (with the reset as the slot u = 0, w = 1, d = 0):
//     gV = w*gv, gd = 2*d*gV, gmn = gm + gd, gx += w*gmn - gd, gv <- u*gv, gm <- u*gmn
//   reset slot: var_init enters the new variance with slope 1: gvi += gv
// The operation order is that of a scalar FP64 evaluation, so with Acc = double
// the per-element results are bit-identical to it.
template <typename Acc>
struct Adjoint {
  Acc gmA, gvA, gmC, gvC;
  double gvi;  // this pixel's contribution to d/d(var_init), in FP64
};


template <typename Acc, bool HAS_GBG>
__device__ __forceinline__ Acc reverse_step(Adjoint<Acc>& g, const Acc gbg, const Acc d,
                                            const int idx, const bool hitA, const bool swapped,
                                            const TableEntry<Acc>& e) {
  if (HAS_GBG) g.gmA = g.gmA + gbg;
  Acc gx = Acc(0);
  if (__builtin_amdgcn_ballot_w64(swapped) != 0) {
    const bool swap = lane_mask(swapped);
    gx = swap ? gx + g.gmC : gx;
    g.gvi = swap ? g.gvi + double(g.gvC) : g.gvi;
    g.gmC = swap ? g.gmA : g.gmC;
    g.gvC = swap ? g.gvA : g.gvC;
    g.gmA = swap ? Acc(0) : g.gmA;
    g.gvA = swap ? Acc(0) : g.gvA;
  }
  const Acc gm = hitA ? g.gmA : g.gmC;
  const Acc gv = hitA ? g.gvA : g.gvC;
  const Acc gV = e.w * gv;
  const Acc gd = (Acc(2) * d) * gV;
  const Acc gmn = gm + gd;
  gx = gx + (e.w * gmn - gd);
  const Acc gvn = e.u * gv;
  const Acc gmo = e.u * gmn;
  if (idx == reset_age<Acc>()) g.gvi += double(gv);
  g.gmA = hitA ? gmo : g.gmA;
  g.gvA = hitA ? gvn : g.gvA;
  g.gmC = hitA ? g.gmC : gmo;
  g.gvC = hitA ? g.gvC : gvn;
  return gx;
}

// ---------------------------------------------------------------- storage types
struct bf16_t {
  uint16_t bits;
};

template <typename In, typename Acc>
__device__ __forceinline__ Acc to_acc(In v) {
  return Acc(v);
}
template <>
__device__ __forceinline__ float to_acc<bf16_t, float>(bf16_t v) {
  return __uint_as_float(uint32_t(v.bits) << 16);
}
template <>
__device__ __forceinline__ double to_acc<bf16_t, double>(bf16_t v) {
  return double(__uint_as_float(uint32_t(v.bits) << 16));
}
template <>
__device__ __forceinline__ f32x2 to_acc<bf16_t, f32x2>(bf16_t v) {
  return f32x2(__uint_as_float(uint32_t(v.bits) << 16));
}

// P consecutive elements, aligned to their total size so that the compiler
// emits the widest loads and stores the alignment allows.
template <typename X, int P>
struct alignas(sizeof(X) * P) Vec {
  X v[P];
};

}  // namespace dsgm
