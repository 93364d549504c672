// Device helpers shared by the contraction kernels (gfx950 only).
#pragma once

#include <cmath>

#include "kernels.hpp"

namespace cqc {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Values the compiler cannot prove wave-uniform (loaded through pointers the
// kernel could in principle write) moved to scalar registers.
__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni(int64_t v) {
  return (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v) |
         ((int64_t)__builtin_amdgcn_readfirstlane((int32_t)(v >> 32)) << 32);
}
template <typename T> __device__ __forceinline__ T *uni(T *p) {
  return reinterpret_cast<T *>(uni((int64_t)reinterpret_cast<uintptr_t>(p)));
}
__device__ __forceinline__ double uni(double v) { return __builtin_bit_cast(double, uni(__builtin_bit_cast(int64_t, v))); }
// Global-address-space view of a pointer (a pointer that went through an
// integer is generic to the compiler, which would emit flat accesses).
template <typename T> using gptr = __attribute__((address_space(1))) T *;
template <typename T> __device__ __forceinline__ gptr<T> gbl(T *p) { return (gptr<T>)p; }
// Constant-address-space view of data that no wave writes during the kernel
// (label lists and counts, written by the preceding label-list pass): uniform
// loads through it become scalar loads, which are waited for on the scalar
// counter - not behind this wave's outstanding output stores.
template <typename T> using cptr = __attribute__((address_space(4))) const T *;
template <typename T> __device__ __forceinline__ cptr<T> cst(const T *p) { return (cptr<T>)gbl(p); }

template <typename T> struct MfmaOp;
// Accumulator layout of one 16x16 block (measured by k_selftest_mfma):
//   FP32: lane l, register r holds row 4*(l/16) + r   (4 consecutive rows)
//   FP64: lane l, register r holds row (l/16) + 4*r   (rows strided by 4)
// of column l%16, where "row" is the index contributed by the A operand.
template <> struct MfmaOp<float> {
  using V = f32x4;
  static constexpr bool kConsecutive = true;
  static __device__ __forceinline__ V run(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <> struct MfmaOp<double> {
  using V = f64x4;
  static constexpr bool kConsecutive = false;
  static __device__ __forceinline__ V run(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

__device__ __forceinline__ int row_of(const DigitMapDev &m, int s, int r) {
  int row = 0;
#pragma unroll 1
  for (int i = 0; i < m.n; ++i) {
    const int v = ((m.srcmask >> i) & 1u) ? r : s;
    const uint64_t w = i < 10 ? m.shifts[0] : m.shifts[1];
    const int sh = (int)((w >> (6 * (i < 10 ? i : i - 10))) & 63);
    row = (row << 2) | ((v >> sh) & 3);
  }
  return row;
}

__device__ inline int64_t deposit(int64_t v, const BitPos &pos, int nbits) {
  int64_t out = 0;
#pragma unroll 1
  for (int j = 0; j < nbits; ++j) {
    const uint64_t w = pos.w[0] * (j / 10 == 0) + pos.w[1] * (j / 10 == 1) + pos.w[2] * (j / 10 == 2) +
                       pos.w[3] * (j / 10 == 3) + pos.w[4] * (j / 10 == 4);
    out |= ((v >> j) & 1) << ((w >> (6 * (j % 10))) & 63);
  }
  return out;
}

// A launch whose device-side predicate is set and false does nothing.
__device__ __forceinline__ bool gated_off(const int32_t *gate, int32_t val) { return gate && *gate != val; }

// A row is live if any of its chunk flags is set.
__device__ __forceinline__ int row_live(const int32_t *flags, int nch, int row) {
  int any = 0;
  for (int c = 0; c < nch; ++c) any |= flags[(int64_t)row * nch + c];
  return any != 0;
}

// Spread consecutive logical blocks over one XCD: hardware dispatches block i
// to XCD i % 8, so logical tile t lands on XCD t / (nblocks / 8) and tiles that
// share an X row block share that XCD's L2.
__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nblocks) {
  if (nblocks % 8) return bid;
  return (bid % 8) * (nblocks / 8) + bid / 8;
}

template <typename T> __device__ __forceinline__ void load4(const T *p, T *v);
template <> __device__ __forceinline__ void load4<float>(const float *p, float *v) {
  float4 t = *reinterpret_cast<const float4 *>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ __forceinline__ void load4<double>(const double *p, double *v) {
  double2 a = reinterpret_cast<const double2 *>(p)[0];
  double2 b = reinterpret_cast<const double2 *>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}

template <typename T> __device__ __forceinline__ void store4(T *p, const T *v);
template <> __device__ __forceinline__ void store4<float>(float *p, const float *v) {
  *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ __forceinline__ void store4<double>(double *p, const double *v) {
  reinterpret_cast<double2 *>(p)[0] = make_double2(v[0], v[1]);
  reinterpret_cast<double2 *>(p)[1] = make_double2(v[2], v[3]);
}

// Gradient of the cross-entropy L = -sum_x t_x log max(p_x, 1e-30) with respect
// to p_x: -t_x / p_x above the floor, 0 at or below it (flat there).  The floor
// test is made on p widened to FP64, the division in T.
constexpr double kXentFloor = 1e-30;
// The test for FP32 p without widening: (float)1e-30 is the smallest float
// above 1e-30, so (double)p > 1e-30 exactly if p >= (float)1e-30.
constexpr float kXentFloorF = 1e-30f;
static_assert((double)kXentFloorF > kXentFloor, "the nearest float lies above the floor");
__device__ __forceinline__ bool xent_above(float p) { return p >= kXentFloorF; }
__device__ __forceinline__ bool xent_above(double p) { return p > kXentFloor; }
template <typename T>
__device__ __forceinline__ T xent_grad_of(T p, T t) {
  return xent_above(p) ? -t / p : T(0);
}
// In FP32 divided first and selected afterwards: as a conditional division the
// compiler makes one branch per output of it, which keeps the epilogues from
// being scheduled around their loads and stores.  (The FP64 division is long
// enough that the branches are the better form: 410 against 508 us for the
// small-term launches of a 52-instance FP64 training step.)
template <>
__device__ __forceinline__ float xent_grad_of<float>(float p, float t) {
  float q = -t / p;
  asm volatile("" : "+v"(q));
  return xent_above(p) ? q : 0.f;
}

// Partial-sum contribution of one output p of a cross-entropy final step
// (ContractArgs::xt): the loss term -t log max(p, 1e-30) in units of
// xent_unit, when the loss is asked for, else p itself (the mass).  FP32
// outputs take the base-2 logarithm in FP32 (one instruction) and FP64 sums of
// FP64 products; ln 2 multiplies a wave's sum once, in FP64.  Over every float
// from 2^-100 to 8 its relative error is at most 2^-23 (1.99 x 2^-24; logf 3.2 x
// 2^-24), close to p = 1 too.  Next to a float epilogue per output this is a third
// of the instructions of logf, whose rounding to FP32 it also saves.
__device__ __forceinline__ double xent_log_floor(float p) { return (double)__builtin_amdgcn_logf(fmaxf(p, kXentFloorF)); }
__device__ __forceinline__ double xent_log_floor(double p) { return log(p > kXentFloor ? p : kXentFloor); }
template <typename T> struct XentUnit { static constexpr double kLoss = 1.0; };
template <> struct XentUnit<float> { static constexpr double kLoss = 0.69314718055994530942; };
template <typename T>
__device__ __forceinline__ double xent_part(T p, T t, bool loss) {
  return loss ? -(double)t * xent_log_floor(p) : (double)p;
}
// A wave's sum of contributions as it goes into the partials.
template <typename T, int XE>
__device__ __forceinline__ double xent_total(double sum) {
  return XE == 2 ? sum * XentUnit<T>::kLoss : sum;
}

// One output p of a cross-entropy final step at element o of the output order:
// gradient to xg, p to z if set; returns the partial-sum contribution.  GLB:
// global accesses and the division of xent_grad_of.  The register kernels take
// generic accesses and a conditional division where they write outputs one by
// one (FP64, deposit order): they are bound by these scattered accesses, and
// with the other form a wave has more of them under way at a time, which is
// slower.  Sixteen FP32 instances of 18 qubits in deposit order take 128 us per
// run, 166 with GLB; in FP64, blocked, 139 against 167.  Bound by arithmetic
// instead, FP64 with the loss is faster with GLB (64 instances of 12 to 19 qubits
// in deposit order: 551 us, 606 without), and so are the deposits of the wide kernels (sixteen
// of 19 qubits, BF16X6: 104 us against 114).
template <typename T, bool GLB = false>
__device__ __forceinline__ double xent_put1(const ContractArgs &a, int64_t o, T p, bool loss) {
  if constexpr (GLB) {
    const T t = gbl(static_cast<const T *>(a.xt))[o];
    if (a.Z) gbl(static_cast<T *>(a.Z))[o] = p;
    gbl(static_cast<T *>(a.xg))[o] = xent_grad_of(p, t);
    return xent_part(p, t, loss);
  } else {
    const T t = static_cast<const T *>(a.xt)[o];
    if (a.Z) static_cast<T *>(a.Z)[o] = p;
    static_cast<T *>(a.xg)[o] = xent_above(p) ? -t / p : T(0);
    return xent_part(p, t, loss);
  }
}

// Four consecutive outputs at elements o..o+3 (o a multiple of 4): vector
// accesses; the contributions go to c[].
template <typename T>
__device__ __forceinline__ void xent_put4(const ContractArgs &a, int64_t o, const T (&v)[4], double (&c)[4],
                                          bool loss) {
  T t[4], g[4];
  load4<T>(static_cast<const T *>(a.xt) + o, t);
  if (a.Z) store4<T>(static_cast<T *>(a.Z) + o, v);
#pragma unroll
  for (int r = 0; r < 4; ++r) g[r] = xent_grad_of(v[r], t[r]);
  store4<T>(static_cast<T *>(a.xg) + o, g);
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = xent_part(v[r], t[r], loss);
}

// FP32 forms with the targets loaded ahead.  A wait for a load also waits for
// every memory access issued before it (loads and stores retire through one
// in-order counter), so a final step that loaded t next to each store would
// wait for its own earlier stores every time: the kernels load the targets of
// a whole tile before its first store instead.  Targets are read once and
// gradients written once: non-temporal accesses.
__device__ __forceinline__ f32x4 xent_t4(const ContractArgs &a, int64_t o) {
  return __builtin_nontemporal_load((gptr<const f32x4>)(gbl(static_cast<const float *>(a.xt)) + o));
}
__device__ __forceinline__ void xent_emit4(const ContractArgs &a, int64_t o, const float (&v)[4], const f32x4 &t,
                                           double (&c)[4], bool loss) {
  if (a.Z) *(gptr<f32x4>)(gbl(static_cast<float *>(a.Z)) + o) = f32x4{v[0], v[1], v[2], v[3]};
  f32x4 g;
#pragma unroll
  for (int r = 0; r < 4; ++r) g[r] = xent_grad_of(v[r], t[r]);
  __builtin_nontemporal_store(g, (gptr<f32x4>)(gbl(static_cast<float *>(a.xg)) + o));
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = xent_part(v[r], t[r], loss);
}

// Wave-wide FP64 sum in a fixed order (butterfly); every lane gets the total.
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Largest d with prefix[d] <= item (the step a work-queue item belongs to).
// The table is written before the launch and only read during it, and the
// item is the same for the whole block: the search runs on scalar loads
// through the constant address space, which wait on the scalar counter - not
// behind this wave's outstanding vector loads and output stores, as a chain
// of dependent vector loads would.
__device__ __forceinline__ int find_desc(const int64_t *prefix, int n, int64_t item) {
  using cp = const __attribute__((address_space(4))) int64_t *;
  const cp tab = (cp)(const __attribute__((address_space(1))) int64_t *)prefix;
  const int64_t it = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(item >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)item));
  int lo = 0, hi = __builtin_amdgcn_readfirstlane(n - 1);   // largest d with prefix[d] <= it
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tab[mid] <= it) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

}  // namespace cqc
