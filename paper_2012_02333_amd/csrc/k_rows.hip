// Row kernel: FP32 steps of at most two shared cuts (1, 4 or 16 terms), which
// are bound by their output bytes.
//
// What decides such a step is how its outputs reach memory: a plain copy of one
// 16-byte access per thread in address order moves 6.6 TB/s on this card, the
// same copy in larger pieces per thread 5.2 to 5.8.  So a wave here owns 64 C
// adjacent columns and writes them row by row, 1024 contiguous bytes per
// instruction at C = 4, straight from the accumulators:
//   - v_mfma_f32_4x4x1_16b_f32 multiplies 4 rows by 64 columns for one term.
//     Lane l's B operand is its own column l, so lane l's accumulators are four
//     rows of column l, and C products with the C columns a lane holds leave it
//     C consecutive outputs of each row: no staging, no LDS, no barrier.
//   - the A operand of one register is 16 blocks of four rows: with 4 terms of
//     16 rows in it, the block selector picks the term and the four rows, so 16
//     rows of 16 terms are four registers (and one load each).
// No product is wasted on padding at 4 terms, and waves of neighbouring units
// write neighbouring memory (units run over the panels of a row run first).
// The Y operands (C K registers) are loaded once per run of row tiles.
// Measured against the LDS-staged strips of two 64 x 256 tiles that this
// replaces: 389 M outputs of the cross-entropy form 785 us there, 582 here (8
// bytes each: 5.3 TB/s); 2^30 outputs of 16 terms 787 and 755 us; 2^24 outputs
// of 16 terms 15.5 and 14.8 us; 42 M outputs 128 columns wide, cross-entropy
// form, 149 us on 32 x 128 tiles and 64 here.  (Trace names with "strip" are those
// of the step class: users of the trace know it by the kernel that ran it before.)
#include <algorithm>
#include <type_traits>

#include "kdev.hpp"

namespace cqc {

// The C columns of a lane: C consecutive ones, or for FP64 outputs two pairs
// 128 columns apart (16 bytes each), so every access of a wave is contiguous.
template <typename O, int C> struct RowCols {
  static constexpr bool kPairs = sizeof(O) == 8 && C == 4;
  static __device__ __forceinline__ uint32_t col(int lane) { return (uint32_t)((kPairs ? 2 : C) * lane); }
};

// Rows may be aligned to an element only.
typedef float u2 __attribute__((ext_vector_type(2), aligned(4)));
typedef float u4 __attribute__((ext_vector_type(4), aligned(4)));
typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));

template <int C> __device__ __forceinline__ void load_cols(gptr<const char> p, bool pairs, float (&v)[C]) {
  if constexpr (C == 4) {
    if (pairs) {
      const u2 a = *(gptr<const u2>)p, b = *(gptr<const u2>)(p + 512);
      v[0] = a[0]; v[1] = a[1]; v[2] = b[0]; v[3] = b[1];
    } else {
      const u4 a = *(gptr<const u4>)p;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = a[c];
    }
  } else if constexpr (C == 2) {
    const u2 a = *(gptr<const u2>)p;
    v[0] = a[0]; v[1] = a[1];
  } else {
    v[0] = *(gptr<const float>)p;
  }
}

// Outputs are written once and not read here: non-temporal.  PLAIN (the next
// step reads them, or rows_plain_stores): ordinary stores.
template <bool PLAIN> __device__ __forceinline__ void store_d2(gptr<char> p, double a, double b) {
  if constexpr (PLAIN) *(gptr<d2>)p = d2{a, b};
  else __builtin_nontemporal_store(d2{a, b}, (gptr<d2>)p);
}
template <bool PLAIN, int C> __device__ __forceinline__ void store_cols(gptr<char> p, const float (&v)[C]) {
  if constexpr (C == 4) {
    if constexpr (PLAIN) *(gptr<u4>)p = u4{v[0], v[1], v[2], v[3]};
    else __builtin_nontemporal_store(u4{v[0], v[1], v[2], v[3]}, (gptr<u4>)p);
  } else if constexpr (C == 2) {
    if constexpr (PLAIN) *(gptr<u2>)p = u2{v[0], v[1]};
    else __builtin_nontemporal_store(u2{v[0], v[1]}, (gptr<u2>)p);
  } else {
    if constexpr (PLAIN) *(gptr<float>)p = v[0];
    else __builtin_nontemporal_store(v[0], (gptr<float>)p);
  }
}
template <bool PLAIN, int C> __device__ __forceinline__ void store_cols(gptr<char> p, const double (&v)[C]) {
  if constexpr (C == 4) {
    store_d2<PLAIN>(p, v[0], v[1]);
    store_d2<PLAIN>(p + 1024, v[2], v[3]);
  } else if constexpr (C == 2) {
    store_d2<PLAIN>(p, v[0], v[1]);
  } else {
    if constexpr (PLAIN) *(gptr<double>)p = v[0];
    else __builtin_nontemporal_store(v[0], (gptr<double>)p);
  }
}
template <int C> __device__ __forceinline__ void load_targets(gptr<const char> p, float (&v)[C]) {
  if constexpr (C == 4) {
    const u4 a = __builtin_nontemporal_load((gptr<const u4>)p);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = a[c];
  } else if constexpr (C == 2) {
    const u2 a = __builtin_nontemporal_load((gptr<const u2>)p);
    v[0] = a[0]; v[1] = a[1];
  } else {
    v[0] = __builtin_nontemporal_load((gptr<const float>)p);
  }
}

// One unit (this wave): columns n0 .. n0 + 64 C - 1 of 2^lt 16-row tiles.
// KEEP: p is written too in the cross-entropy form.  PLAIN: ordinary stores.
template <typename O, int MODE, int XE, bool KEEP, int C, int NS, bool PLAIN = false>
__device__ __forceinline__ void rows_unit(const ContractArgs &a, int lt, int64_t unit) {
  constexpr int K = 1 << (2 * NS), NV = K >= 4 ? K / 4 : 1;
  constexpr int kLogC = C == 4 ? 2 : C == 2 ? 1 : 0;
  using RC = RowCols<O, C>;
  const int lane = threadIdx.x & 63;
  const int logM = uni(a.logM), logN = uni(a.logN);
  const int lp = logN - 6 - kLogC, lr = logM - 4 - lt;   // log2 of panels and of row runs
  const int64_t batch = unit >> (lp + lr);
  if (batch >= a.nbatch) return;
  const int64_t n0 = (unit & ((int64_t(1) << lp) - 1)) << (6 + kLogC);
  const int64_t m0 = ((unit >> lp) & ((int64_t(1) << lr) - 1)) << (4 + lt);
  const int rX = (int)(batch >> (2 * a.nRY)), rY = (int)(batch & ((int64_t(1) << (2 * a.nRY)) - 1));
  // rows of the operands: lane t < K computes those of term t
  const int rx = lane < K ? row_of(a.mx, lane, rX) : 0, ry = lane < K ? row_of(a.my, lane, rY) : 0;
  // early termination: dead terms become zero operands
  uint32_t live = (1u << K) - 1u;
  const bool flags = uni(a.flagX) != nullptr;
  if (flags)
    live = (uint32_t)__ballot(lane < K && (row_live(a.flagX, a.nchX, rx) & row_live(a.flagY, a.nchY, ry)));
  const gptr<const char> Yb = gbl(reinterpret_cast<const char *>(uni(a.Y))) + 4 * n0;
  const uint32_t yc = 4u * RC::col(lane);
  float y[K][C];
#pragma unroll
  for (int t = 0; t < K; ++t) {
    const int row = __builtin_amdgcn_readlane(ry, t);
    load_cols<C>(Yb + ((int64_t)row << (logN + 2)) + yc, RC::kPairs, y[t]);
  }
  // X: lane l of register v holds row l % 16 of term 4 v + l / 16
  const gptr<const float> Xb = gbl(static_cast<const float *>(uni(a.X)));
  gptr<const float> xp[NV];
  float x[NV];
  auto masked = [&](int v, float w) {   // dead terms of the packed operand
    return !flags || ((live >> (K >= 4 ? 4 * v + (lane >> 4) : 0)) & 1u) ? w : 0.f;
  };
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int row = __shfl(rx, K >= 4 ? 4 * v + (lane >> 4) : 0, 64);
    xp[v] = Xb + ((int64_t)row << logM) + m0 + (lane & 15);
    x[v] = *xp[v];
  }
  if (flags) {
#pragma unroll
    for (int t = 0; t < K; ++t)
#pragma unroll
      for (int c = 0; c < C; ++c) y[t][c] = (live >> t) & 1u ? y[t][c] : 0.f;
  }
  const int64_t rowb = sizeof(O) * (int64_t(1) << logN);   // bytes of an output row
  const int64_t o0 = sizeof(O) * ((MODE == kModeIntermediate ? batch << (logM + logN) : 0) + (m0 << logN) + n0);
  gptr<char> Zr = gbl(static_cast<char *>(uni(a.Z))) + o0;
  gptr<const char> Tr = XE ? gbl(static_cast<const char *>(uni(a.xt))) + o0 : nullptr;
  gptr<char> Gr = XE ? gbl(static_cast<char *>(uni(a.xg))) + o0 : nullptr;
  const uint32_t zc = sizeof(O) * RC::col(lane);
  const O sc = MODE == kModeIntermediate ? O(1) : (O)uni(a.scale);
  double msum = 0.0;
  // cross-entropy form: the targets of the next two groups of four rows in flight
  float tv[XE ? 2 : 1][4][C];
  // a scalar row pointer moved on row by row; opaque, or the compiler keeps one
  // 64-bit lane address per row and buffer in registers
  auto advance = [&](auto &p) {
    p += rowb;
    asm volatile("" : "+s"(p));
  };
  auto targets = [&](int slot) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      load_targets<C>(Tr + zc, tv[XE ? slot : 0][r]);
      advance(Tr);
    }
  };
  if constexpr (XE) {
    targets(0);
    targets(1);
  }
  const int tiles = 1 << lt;
  for (int it = 0; it < tiles; ++it) {
    float xn[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (it + 1 < tiles) xp[v] += 16;   // the last tile reloads itself
      xn[v] = *xp[v];
      x[v] = masked(v, x[v]);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 acc[C];
      auto products = [&](auto G) {
        constexpr int rg = decltype(G)::value;
        auto term = [&](auto Tc) {
          constexpr int t = decltype(Tc)::value;
#pragma unroll
          for (int c = 0; c < C; ++c)
            acc[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[t / 4], y[t][c], t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[c],
                                                        4, K >= 4 ? 4 * (t % 4) + rg : rg, 0);
        };
        term(std::integral_constant<int, 0>{});
        if constexpr (K >= 4) {
          term(std::integral_constant<int, 1>{});
          term(std::integral_constant<int, 2>{});
          term(std::integral_constant<int, 3>{});
        }
        if constexpr (K == 16) {
          term(std::integral_constant<int, 4>{});
          term(std::integral_constant<int, 5>{});
          term(std::integral_constant<int, 6>{});
          term(std::integral_constant<int, 7>{});
          term(std::integral_constant<int, 8>{});
          term(std::integral_constant<int, 9>{});
          term(std::integral_constant<int, 10>{});
          term(std::integral_constant<int, 11>{});
          term(std::integral_constant<int, 12>{});
          term(std::integral_constant<int, 13>{});
          term(std::integral_constant<int, 14>{});
          term(std::integral_constant<int, 15>{});
        }
      };
      if (g == 0) products(std::integral_constant<int, 0>{});
      else if (g == 1) products(std::integral_constant<int, 1>{});
      else if (g == 2) products(std::integral_constant<int, 2>{});
      else products(std::integral_constant<int, 3>{});
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        O v[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = (O)acc[c][r] * sc;
        if constexpr (XE) {
          float gr[C];
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const float t = tv[g & 1][r][c];
            gr[c] = xent_grad_of(v[c], t);
            msum += xent_part(v[c], t, XE == 2);
          }
          if constexpr (KEEP) {
            store_cols<false, C>(Zr + zc, v);
            advance(Zr);
          }
          store_cols<false, C>(Gr + zc, gr);
          advance(Gr);
          // one row's arithmetic in registers at a time (the sum would be put
          // off, with all its operands alive)
          asm volatile("" : "+v"(msum));
          __builtin_amdgcn_sched_barrier(0);
        } else {
          store_cols<PLAIN, C>(Zr + zc, v);
          advance(Zr);
          if (MODE != kModeIntermediate) {
            if constexpr (C == 4) msum += ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
            else
#pragma unroll
              for (int c = 0; c < C; ++c) msum += (double)v[c];
          }
        }
      }
      if constexpr (XE)
        if (g < 2 || it + 1 < tiles) targets(g & 1);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v] = xn[v];
  }
  if (MODE == kModeIntermediate) {
    if (a.flagZ && lane == 0 && (unit & ((int64_t(1) << (lp + lr)) - 1)) == 0) gbl(a.flagZ)[batch] = live != 0;
  } else if (a.partials) {
    const double tot = xent_total<O, XE>(wave_sum_f64(msum));
    if (lane == 0) gbl(a.partials)[unit] = tot;
  }
}

template <typename O, int MODE, int C, int NS, bool PLAIN>
__global__ __launch_bounds__(256) void k_rows(const ContractArgs a, int lt) {
  if (gated_off(a.gate, a.gate_val)) return;
  rows_unit<O, MODE, 0, true, C, NS, PLAIN>(a, lt, (int64_t)blockIdx.x * 4 + uni((int32_t)(threadIdx.x >> 6)));
}

// Many steps of one shape class per launch: block b belongs to the step d with
// prefix[d] <= b < prefix[d + 1].  One block per four units, not persistent:
// the dispatcher keeps the blocks in address order and needs no counter.
template <int MODE, int XE, int C, int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NS == 2 ? 3 : 4))) void k_rows_table(const ContractArgs *__restrict__ descs,
                                                    const int64_t *__restrict__ prefix, int ndesc) {
  const int d = uni(find_desc(prefix, ndesc, (int64_t)blockIdx.x));
  const ContractArgs &a = descs[d];
  const int lt = rows_log_tiles(uni(a.logM), uni(a.logN), 2 * (uni(a.nRX) + uni(a.nRY)), C, NS);
  const int64_t unit = ((int64_t)blockIdx.x - uni(prefix[d])) * 4 + uni((int32_t)(threadIdx.x >> 6));
  if (XE == 0 || uni(a.Z)) rows_unit<float, MODE, XE, true, C, NS, MODE == kModeIntermediate>(a, lt, unit);
  else rows_unit<float, MODE, XE, XE == 0, C, NS>(a, lt, unit);
}

// The FP64 form (FP64 output, single calls): 16 rows by 128 columns per tile on
// v_mfma_f64_16x16x4_f64, the same products in the same order as the register
// kernel, so the same bits.  The even and odd columns of 32 sit in two products:
// a lane's pair of accumulators is 16 adjacent bytes, and one instruction
// writes 256 contiguous bytes of four rows (128 from the register kernel, which
// also loads Y again for every 64 rows).  One row tile per wave: 2^9 x 2^16 outputs
// of 16 terms took 48.8, 54.5, 55.5, 55.5 us with 1, 2, 4, 8.  2^10 x 2^12 outputs
// take 0.86 of the register kernel's time, 2^9 x 2^15 0.95, 2^9 x 2^16 0.97 (one,
// four and 16 terms alike).
template <int MODE, int NS, bool PLAIN>
__device__ __forceinline__ void rows64_unit(const ContractArgs &a, int64_t unit) {
  constexpr int K = 1 << (2 * NS), NQ = K >= 4 ? K / 4 : 1, NB = 8;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  const int logM = uni(a.logM), logN = uni(a.logN);
  const int lp = logN - 7, lr = logM - 4;
  const int64_t batch = unit >> (lp + lr);
  if (batch >= a.nbatch) return;
  const int64_t n0 = (unit & ((int64_t(1) << lp) - 1)) << 7;
  const int64_t m0 = ((unit >> lp) & ((int64_t(1) << lr) - 1)) << 4;
  const int rX = (int)(batch >> (2 * a.nRY)), rY = (int)(batch & ((int64_t(1) << (2 * a.nRY)) - 1));
  // rows of the operands: lane t < K computes those of term t, and whether it is live
  const int rx = lane < K ? row_of(a.mx, lane, rX) : 0, ry = lane < K ? row_of(a.my, lane, rY) : 0;
  uint32_t live = (1u << K) - 1u;
  if (uni(a.flagX) != nullptr)
    live = (uint32_t)__ballot(lane < K && (row_live(a.flagX, a.nchX, rx) & row_live(a.flagY, a.nchY, ry)));
  const gptr<const double> Xb = gbl(static_cast<const double *>(uni(a.X))), Yb = gbl(static_cast<const double *>(uni(a.Y)));
  double y[NQ][NB], x[NQ];
  bool ok[NQ];   // this lane's term of the quad is live
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int t = 4 * q + lg, ts = t < K ? t : 0;
    ok[q] = t < K && ((live >> ts) & 1u);
    const gptr<const double> yr = Yb + ((int64_t)__shfl(ry, ts, 64) << logN) + n0 + 2 * l16;
#pragma unroll
    for (int p = 0; p < NB / 2; ++p) {
      const d2 v = *(gptr<const d2>)(yr + 32 * p);
      y[q][2 * p] = v[0];
      y[q][2 * p + 1] = v[1];
    }
    x[q] = Xb[((int64_t)__shfl(rx, ts, 64) << logM) + m0 + l16];
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    x[q] = ok[q] ? x[q] : 0.0;
#pragma unroll
    for (int j = 0; j < NB; ++j) y[q][j] = ok[q] ? y[q][j] : 0.0;
  }
  const double sc = MODE == kModeIntermediate ? 1.0 : uni(a.scale);
  gptr<double> Z = gbl(static_cast<double *>(uni(a.Z))) + (MODE == kModeIntermediate ? batch << (logM + logN) : 0) +
                   ((m0 + lg) << logN) + n0 + 2 * l16;
  double msum = 0.0;
#pragma unroll
  for (int p = 0; p < NB / 2; ++p) {
    f64x4 e{0, 0, 0, 0}, o{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      e = MfmaOp<double>::run(x[q], y[q][2 * p], e);
      o = MfmaOp<double>::run(x[q], y[q][2 * p + 1], o);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double v0 = e[r] * sc, v1 = o[r] * sc;
      store_d2<PLAIN>((gptr<char>)(Z + ((int64_t)(4 * r) << logN) + 32 * p), v0, v1);
      if (MODE != kModeIntermediate) msum += v0 + v1;
    }
  }
  if (MODE == kModeIntermediate) {
    if (a.flagZ && lane == 0 && (unit & ((int64_t(1) << (lp + lr)) - 1)) == 0) gbl(a.flagZ)[batch] = live != 0;
  } else if (a.partials) {
    const double tot = wave_sum_f64(msum);
    if (lane == 0) gbl(a.partials)[unit] = tot;
  }
}

template <int MODE, int NS, bool PLAIN>
__global__ __launch_bounds__(256) void k_rows_f64(const ContractArgs a) {
  if (gated_off(a.gate, a.gate_val)) return;
  rows64_unit<MODE, NS, PLAIN>(a, (int64_t)blockIdx.x * 4 + uni((int32_t)(threadIdx.x >> 6)));
}

int64_t rows_units(const ContractArgs &a) {
  const int lt = rows_log_tiles(a.logM, a.logN, 2 * (a.nRX + a.nRY), a.rows, a.nS);
  return a.nbatch << (a.logM - 4 - lt + a.logN - 6 - (a.rows == 4 ? 2 : a.rows == 2 ? 1 : 0));
}

int64_t rows_f64_units(const ContractArgs &a) { return a.nbatch << (a.logM - 4 + a.logN - 7); }

template <typename O, int MODE, int C, bool PLAIN>
static Status launch_rows_p(const char *nm, const ContractArgs &a, hipStream_t s) {
  const int lt = rows_log_tiles(a.logM, a.logN, 2 * (a.nRX + a.nRY), a.rows, a.nS);
  const dim3 grid((unsigned)((rows_units(a) + 3) / 4)), block(256);
  switch (a.nS) {
    case 0: return launch(nm, k_rows<O, MODE, C, 0, PLAIN>, grid, block, 0, s, a, lt);
    case 1: return launch(nm, k_rows<O, MODE, C, 1, PLAIN>, grid, block, 0, s, a, lt);
    default: return launch(nm, k_rows<O, MODE, C, 2, PLAIN>, grid, block, 0, s, a, lt);
  }
}

template <typename O, int MODE, int C>
static Status launch_rows_c(const char *nm, const ContractArgs &a, hipStream_t s) {
  if (MODE == kModeIntermediate || rows_plain_stores(a.nS, a.logM, a.logN, sizeof(O) == 8))
    return launch_rows_p<O, MODE, C, true>(nm, a, s);
  return launch_rows_p<O, MODE, C, MODE == kModeIntermediate>(nm, a, s);
}

template <typename O, int MODE>
static Status launch_rows_m(const ContractArgs &a, hipStream_t s) {
  switch (a.rows) {
    case 4: return launch_rows_c<O, MODE, 4>(sizeof(O) == 4 ? "contract_small_strip_64x256" : "contract_small_rows_256", a, s);
    case 2: return launch_rows_c<O, MODE, 2>("contract_small_rows_128", a, s);
    default: return launch_rows_c<O, MODE, 1>("contract_small_rows_64", a, s);
  }
}

Status launch_rows(bool out_double, const ContractArgs &a, hipStream_t s) {
  const int logc = a.rows == 4 ? 2 : a.rows == 2 ? 1 : 0;
  if (a.rows < 1 || a.nS > 2 || a.logM < 4 || a.logN < 6 + logc || a.mode == kModeFinalDeposit)
    return Status::fail(CQC_ERR_INVALID_ARG, "row contraction: step shape");
  if (a.mode == kModeIntermediate) return launch_rows_m<float, kModeIntermediate>(a, s);
  return out_double ? launch_rows_m<double, kModeFinalBlocked>(a, s) : launch_rows_m<float, kModeFinalBlocked>(a, s);
}

template <int MODE, bool PLAIN>
static Status launch_rows_f64_m(const ContractArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)((rows_f64_units(a) + 3) / 4)), block(256);
  const char *nm = MODE == kModeIntermediate ? "contract_rows_f64_inter" : "contract_rows_f64";
  switch (a.nS) {
    case 0: return launch(nm, k_rows_f64<MODE, 0, PLAIN>, grid, block, 0, s, a);
    case 1: return launch(nm, k_rows_f64<MODE, 1, PLAIN>, grid, block, 0, s, a);
    default: return launch(nm, k_rows_f64<MODE, 2, PLAIN>, grid, block, 0, s, a);
  }
}

Status launch_rows_f64(const ContractArgs &a, hipStream_t s) {
  if (a.rows != 2 || a.nS > 2 || a.logM < 4 || a.logN < 7 || a.mode == kModeFinalDeposit)
    return Status::fail(CQC_ERR_INVALID_ARG, "row contraction: step shape");
  if (a.mode == kModeIntermediate) return launch_rows_f64_m<kModeIntermediate, true>(a, s);
  return rows_plain_stores(a.nS, a.logM, a.logN, true) ? launch_rows_f64_m<kModeFinalBlocked, true>(a, s)
                                                             : launch_rows_f64_m<kModeFinalBlocked, false>(a, s);
}

template <int MODE, int XE, int C>
static Status launch_rows_table_c(const char *nm, int nS, const QueueLaunch &q, hipStream_t s) {
  const dim3 grid((unsigned)q.total), block(256);
  switch (nS) {
    case 0: return launch(nm, k_rows_table<MODE, XE, C, 0>, grid, block, 0, s, q.descs, q.prefix, q.ndesc);
    case 1: return launch(nm, k_rows_table<MODE, XE, C, 1>, grid, block, 0, s, q.descs, q.prefix, q.ndesc);
    default: return launch(nm, k_rows_table<MODE, XE, C, 2>, grid, block, 0, s, q.descs, q.prefix, q.ndesc);
  }
}

template <int MODE, int XE>
static Status launch_rows_table_m(int rows, int nS, const QueueLaunch &q, hipStream_t s) {
  constexpr auto name = [](const char *plain, const char *grad, const char *loss) {
    return XE == 2 ? loss : XE ? grad : plain;
  };
  switch (rows) {
    case 4: return launch_rows_table_c<MODE, XE, 4>(
        name("contract_strip_queue", "contract_rows_256_xent", "contract_rows_256_xent_loss"), nS, q, s);
    case 2: return launch_rows_table_c<MODE, XE, 2>(
        name("contract_rows_128", "contract_rows_128_xent", "contract_rows_128_xent_loss"), nS, q, s);
    default: return launch_rows_table_c<MODE, XE, 1>(
        name("contract_rows_64", "contract_rows_64_xent", "contract_rows_64_xent_loss"), nS, q, s);
  }
}

Status launch_rows_table(int mode, int rows, int nS, const QueueLaunch &q, hipStream_t s) {
  if (mode == kModeIntermediate) return launch_rows_table_m<kModeIntermediate, 0>(rows, nS, q, s);
  if (mode != kModeFinalBlocked) return Status::fail(CQC_ERR_UNSUPPORTED, "row contraction: output mode");
  if (q.xent == 2) return launch_rows_table_m<kModeFinalBlocked, 2>(rows, nS, q, s);
  if (q.xent == 1) return launch_rows_table_m<kModeFinalBlocked, 1>(rows, nS, q, s);
  return launch_rows_table_m<kModeFinalBlocked, 0>(rows, nS, q, s);
}

}  // namespace cqc
