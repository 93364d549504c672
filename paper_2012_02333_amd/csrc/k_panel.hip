// Panel contraction kernel: FP32 steps of three shared cuts (17 to 64 terms)
// with FP32 output.  (FP64 output stays on the wide kernel: its 16-byte buffer
// stores at a scalar offset wrote wrong upper halves now and then, which the
// 8-byte stores used here do not.)
//
// Such a step is bound by the FP32 matrix cores, but only just: at 64 terms a
// 64 x 64 tile is 8192 matrix-core cycles against 16 KiB of output, so
// whatever keeps the matrix cores waiting between tiles (staging, barriers,
// an epilogue) shows in full.  Here a wave holds the 64 terms of 64 columns of
// Y in 64 registers for a whole run of X tiles, and nothing is shared between
// waves: no LDS, no barrier, no staging.
//   - v_mfma_f32_32x32x1_2b_f32: one term per product, 32 rows of X
//     (broadcast to both blocks by the A selector) times 64 columns of Y, so
//     one load instruction per operand row brings a whole operand (64
//     consecutive X columns from a scalar offset), and 32 accumulators hold 32
//     x 64 outputs.
//   - a 64-row tile is two passes over the 64 terms: rows 0..31, then 32..63.
//     Each X register is reloaded for the next tile as soon as the second pass
//     has used it (a whole pass ahead of its next use), and the stores of one
//     half run between the products of the other, so loads, stores and the
//     FP64 sum all sit in the shadow of the matrix cores.
//   - even and odd columns of the panel sit in the two blocks of the product:
//     a lane's two blocks are adjacent outputs, and one store instruction
//     writes 256 contiguous bytes of two rows without staging.
// Units are kept short (eight times as many as fit at once): the two waves of a
// SIMD do not finish together, and a launch of exactly one unit per slot lost
// 15% to its ends.
// The final step of a 30-qubit, six-cut chain (2^18 x 2^12 outputs, 64 terms)
// within a call of n = 30: 1740 us on the LDS-staged wide kernel, 1310 to 1460
// here, the call 1743 and 1390 us.  Counters: matrix cores 0.77 busy at a shader
// clock of 1.86 GHz, where the products alone would take 1130 us.  By itself on
// random operands 1380 us, 1080 us without its stores.
#include <algorithm>

#include "kdev.hpp"

namespace cqc {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x32 __attribute__((ext_vector_type(32)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

// Buffer accesses: a 64-bit base and its size in four scalar registers, one
// scalar 32-bit offset per access and one vector offset per lane.  An empty
// range drops the access.
typedef __amdgpu_buffer_rsrc_t BufRsrc;
__device__ __forceinline__ BufRsrc buf_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ float buf_load(BufRsrc r, uint32_t lane_off, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)off, 0));
}
constexpr int kBufNt = 2;   // non-temporal: read or written once
__device__ __forceinline__ f32x2 buf_load2_nt(BufRsrc r, uint32_t lane_off, uint32_t off) {
  return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)off, kBufNt));
}
template <int AUX>
__device__ __forceinline__ void buf_store2(float a, float b, BufRsrc r, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, f32x2{a, b}), r, (int)lane_off, (int)off, AUX);
}
__device__ __forceinline__ void buf_store2_nt(float a, float b, BufRsrc r, uint32_t lane_off, uint32_t off) {
  buf_store2<kBufNt>(a, b, r, lane_off, off);
}
// Stores of p: intermediates stay in the caches for the step that reads them
// (chain of 9, 9 and 12 qubits, three cuts each: 1393 us, 1460 with non-temporal
// stores of the 64 MiB intermediate).
template <int MODE>
__device__ __forceinline__ void buf_store_p(float a, float b, BufRsrc r, uint32_t lane_off, uint32_t off) {
  buf_store2<MODE == kModeIntermediate ? 0 : kBufNt>(a, b, r, lane_off, off);
}

namespace {
constexpr int kPT = 64;   // terms a wave holds; also the tile edge
}

// The terms of a batch entry, compacted in ascending label order: lane t holds
// the byte offsets of term t's X and Y rows (0 past the count).  From the
// step's label lists where it has them, else from the row flags, one label per
// lane.
struct PanelTerms {
  uint32_t lx, ly;
  int cnt;
};
__device__ __forceinline__ PanelTerms panel_terms(const ContractArgs &a, int64_t batch) {
  const int lane = threadIdx.x & 63;
  PanelTerms p;
  if (a.lists) {
    p.cnt = cst(uni(a.counts))[batch];
    const int32_t ld = uni(a.list_ld);
    const gptr<const uint32_t> l = gbl(reinterpret_cast<const uint32_t *>(uni(a.lists))) + batch * 2 * ld;
    p.lx = lane < p.cnt ? l[lane] : 0u;
    p.ly = lane < p.cnt ? l[ld + lane] : 0u;
    return p;
  }
  const int rX = (int)(batch >> (2 * a.nRY)), rY = (int)(batch & ((int64_t(1) << (2 * a.nRY)) - 1));
  const int rx = row_of(a.mx, lane, rX), ry = row_of(a.my, lane, rY);
  const int live = a.flagX ? row_live(a.flagX, a.nchX, rx) & row_live(a.flagY, a.nchY, ry) : 1;
  const unsigned long long bal = __ballot(live);
  p.cnt = __popcll(bal);
  const int pre = __popcll(bal & ((1ull << lane) - 1ull));
  const int dest = 4 * (live ? pre : p.cnt + lane - pre);   // the dead labels behind the live ones
  p.lx = (uint32_t)__builtin_amdgcn_ds_permute(dest, live ? (int)((uint32_t)rx << (a.logM + 2)) : 0);
  p.ly = (uint32_t)__builtin_amdgcn_ds_permute(dest, live ? (int)((uint32_t)ry << (a.logN + 2)) : 0);
  return p;
}
__device__ __forceinline__ uint32_t term(uint32_t l, int t) { return (uint32_t)__builtin_amdgcn_readlane((int)l, t); }

// One unit (this wave): the 64-column panel of Y at n0 against `tiles` 64-row
// tiles of X from row m_first; returns this lane's share of the FP64 sum.
// FULL: all 64 terms live.
template <int MODE, int XE, bool FULL>
__device__ __forceinline__ double panel_rows(const ContractArgs &a, const PanelTerms &pt, int64_t batch,
                                             int64_t m_first, int tiles, int64_t n0) {
  const int lane = threadIdx.x & 63;
  const int logM = uni(a.logM), logN = uni(a.logN);
  const int cnt = uni(pt.cnt);
  const BufRsrc X = buf_rsrc(uni(a.X), 4u << (logM + 2 * (uni(a.nS) + uni(a.nRX))));
  const BufRsrc Y = buf_rsrc(uni(a.Y), 4u << (logN + 2 * (uni(a.nS) + uni(a.nRY))));
  const uint32_t xl = 4u * lane;
  // lanes 0..31 hold the panel's even columns, 32..63 the odd ones
  const uint32_t yl = 4u * (lane < 32 ? 2 * lane : 2 * lane - 63);
  float y[kPT], x[kPT];
#pragma unroll
  for (int t = 0; t < kPT; ++t) y[t] = buf_load(Y, yl, term(pt.ly, t) + 4u * (uint32_t)n0);
#pragma unroll
  for (int t = 0; t < kPT; ++t) x[t] = buf_load(X, xl, term(pt.lx, t) + 4u * (uint32_t)m_first);
  if (!FULL) {
#pragma unroll
    for (int t = 0; t < kPT; ++t) y[t] = t < cnt ? y[t] : 0.f;
  }

  double msum = 0.0;
  const float sc = MODE == kModeIntermediate ? 1.f : (float)uni(a.scale);
  char *Zb = uni(static_cast<char *>(a.Z));
  if (MODE == kModeIntermediate) Zb += (batch << (logM + logN)) * 4;
  const char *Tb = XE ? uni(static_cast<const char *>(a.xt)) : nullptr;
  char *Gb = XE ? uni(static_cast<char *>(a.xg)) : nullptr;
  // the lane's two columns; lanes 32..63 write four rows further down
  const uint32_t zl = 4u * (((uint32_t)(lane >> 5) << (logN + 2)) + 2u * (lane & 31));
  // rows 32 half .. 32 half + 31 of the tile at row m, in an output buffer
  auto rows = [&](const char *base, int64_t m, int half, bool on) {
    return buf_rsrc(base + (((m + 32 * half) << logN) + n0) * 4, on ? 128u << logN : 0u);
  };
  auto row_off = [&](int r) { return (uint32_t)(4 * ((r % 4) + 8 * (r / 4))) << logN; };
  // outputs r and 16 + r of every lane of a half tile.  The cross-entropy form
  // keeps the targets of the next kTv stores in flight (a whole half tile of
  // them does not fit the registers): store r uses slot r % kTv, which is then
  // loaded for the store kTv later.
  constexpr int kTv = 8;
  f32x2 tv[XE ? kTv : 1];
  if (XE)
#pragma unroll
    for (int r = 0; r < kTv; ++r) tv[XE ? r : 0] = f32x2{0.f, 0.f};
  auto put = [&](BufRsrc Z, BufRsrc G, const f32x32 &acc, int r) {
    const float v0 = acc[r] * sc, v1 = acc[16 + r] * sc;
    if constexpr (XE) {
      const f32x2 t = tv[r % kTv];
      buf_store2_nt(v0, v1, Z, zl, row_off(r));   // dropped where p is not kept
      buf_store2_nt(xent_grad_of(v0, t[0]), xent_grad_of(v1, t[1]), G, zl, row_off(r));
      msum += xent_part(v0, t[0], XE == 2) + xent_part(v1, t[1], XE == 2);
      asm volatile("" : "+v"(msum));   // or the sum is put off, with all its operands alive
    } else {
      buf_store_p<MODE>(v0, v1, Z, zl, row_off(r));
      if (MODE != kModeIntermediate) msum += (double)v0 + (double)v1;
    }
  };
  const bool hasZ = !XE || uni(a.Z) != nullptr;
  f32x32 acc0{}, acc1{};
  for (int it = 0; it < tiles; ++it) {
    const int64_t m0 = m_first + (int64_t)it * kPT;
    const uint32_t mn = 4u * (uint32_t)(it + 1 < tiles ? m0 + kPT : m0);   // the last tile reloads itself
    int c = cnt;
    if (!FULL) asm volatile("" : "+s"(c));   // keep 64 per-term masks out of registers
    // rows 0..31 of the tile; between the products the stores of the previous
    // tile's rows 32..63 (for the first tile an empty range drops them, and
    // their sums are zero)
    {
      const BufRsrc Zp = rows(Zb, m0 - kPT, 1, hasZ && it > 0), Gp = rows(Gb, m0 - kPT, 1, it > 0);
      const BufRsrc T0 = rows(Tb, m0 - kPT, 1, it > 0), T1 = rows(Tb, m0, 0, true);
#pragma unroll
      for (int g = 0; g < kPT / 8; ++g) {
        if (FULL || g == 0 || 8 * g < c) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int t = 8 * g + i;
            const float xv = FULL || t < c ? x[t] : 0.f;
            acc0 = __builtin_amdgcn_mfma_f32_32x32x1f32(xv, y[t], t == 0 ? f32x32{} : acc0, 1, 0, 0);
          }
        }
#pragma unroll
        for (int r = 2 * g; r < 2 * g + 2; ++r) {
          put(Zp, Gp, acc1, r);
          if constexpr (XE) {
            tv[r % kTv] = r < 16 - kTv ? buf_load2_nt(T0, zl, row_off(r + kTv)) : buf_load2_nt(T1, zl, row_off(r + kTv - 16));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (!FULL) asm volatile("" : "+s"(c));   // nor the 64 masked operands
    // rows 32..63; the stores of rows 0..31, and the next tile's operands into
    // the registers this pass has just left
    {
      const BufRsrc Zc = rows(Zb, m0, 0, hasZ), Gc = rows(Gb, m0, 0, true);
      const BufRsrc T0 = rows(Tb, m0, 0, true), T1 = rows(Tb, m0, 1, true);
#pragma unroll
      for (int g = 0; g < kPT / 8; ++g) {
        if (FULL || g == 0 || 8 * g < c) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int t = 8 * g + i;
            const float xv = FULL || t < c ? x[t] : 0.f;
            acc1 = __builtin_amdgcn_mfma_f32_32x32x1f32(xv, y[t], t == 0 ? f32x32{} : acc1, 1, 1, 0);
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int t = 8 * g + i;
          x[t] = buf_load(X, xl, term(pt.lx, t) + mn);
        }
#pragma unroll
        for (int r = 2 * g; r < 2 * g + 2; ++r) {
          put(Zc, Gc, acc0, r);
          if constexpr (XE) {
            tv[r % kTv] = r < 16 - kTv ? buf_load2_nt(T0, zl, row_off(r + kTv)) : buf_load2_nt(T1, zl, row_off(r + kTv - 16));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const int64_t ml = m_first + (int64_t)(tiles - 1) * kPT;
  const BufRsrc Zl = rows(Zb, ml, 1, hasZ), Gl = rows(Gb, ml, 1, true);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    put(Zl, Gl, acc1, r);
    if constexpr (XE)
      if (r < 16 - kTv) tv[r] = buf_load2_nt(rows(Tb, ml, 1, true), zl, row_off(r + kTv));
  }
  return msum;
}

// Units of a step: (batch entry, run of row tiles, panel), panels fastest, so
// the four waves of a block share their X rows in L1 where the step has four
// panels.
template <int MODE, int XE>
__device__ __forceinline__ void panel_unit(const ContractArgs &a, int lt, int64_t unit) {
  const int lp = uni(a.logN) - 6, lc = uni(a.logM) - 6 - lt;   // log2 of panels and of row runs
  if (unit >> (lp + lc) >= a.nbatch) return;
  const int64_t n0 = (unit & ((int64_t(1) << lp) - 1)) * kPT;
  const int64_t run = (unit >> lp) & ((int64_t(1) << lc) - 1);
  const int64_t batch = unit >> (lp + lc);
  const PanelTerms pt = panel_terms(a, batch);
  const bool first = (unit & ((int64_t(1) << (lp + lc)) - 1)) == 0 && (threadIdx.x & 63) == 0;
  if (MODE == kModeIntermediate && first && a.flagZ && !a.lists) gbl(a.flagZ)[batch] = pt.cnt > 0;
  const double s = pt.cnt == kPT ? panel_rows<MODE, XE, true>(a, pt, batch, run << (lt + 6), 1 << lt, n0)
                                 : panel_rows<MODE, XE, false>(a, pt, batch, run << (lt + 6), 1 << lt, n0);
  if (MODE != kModeIntermediate && a.partials) {
    const double tot = xent_total<float, XE>(wave_sum_f64(s));
    if ((threadIdx.x & 63) == 0) gbl(a.partials)[unit] = tot;
  }
}

template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_panel(const ContractArgs a, int lt) {
  if (gated_off(a.gate, a.gate_val)) return;
  // blocks of one XCD take a contiguous range of units: they share X rows in L2
  const int64_t blk = a.xcd_remap ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
  panel_unit<MODE, 0>(a, lt, blk * 4 + uni((int32_t)(threadIdx.x >> 6)));
}

// Many steps per launch: items of four units from an atomic queue (see
// k_contract_queue).
template <int MODE, int XE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_panel_queue(const ContractArgs *__restrict__ descs, const int64_t *__restrict__ prefix, int ndesc,
                   unsigned long long *queue, int64_t total) {
  __shared__ int64_t item;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) item = (int64_t)atomicAdd(queue, 1ull);
    __syncthreads();
    const int64_t it = uni(item);
    if (it >= total) return;
    const int d = uni(find_desc(prefix, ndesc, it));
    const ContractArgs &a = descs[d];
    panel_unit<MODE, XE>(a, uni(a.panel) - 1, (it - uni(prefix[d])) * 4 + uni((int32_t)(threadIdx.x >> 6)));
  }
}

// ---------------------------------------------------------------------------
// Four and more shared cuts: the terms of a panel no longer fit the registers,
// so both operands stream.  A wave owns one 64 x 64 output tile; every term is
// one load of each operand (64 columns from a scalar row offset) and two
// products of 64 rows by 32 columns (even columns, odd columns), 128
// matrix-core cycles; kST terms of both are in flight, and the 2 x 2 waves of
// a block share their rows in L1.  No LDS and no barrier: three waves per SIMD
// cover each other's first loads and last stores.  The staged wide kernel
// spent as long staging, waiting at two barriers per 32 terms and on its
// epilogue as on its products: 88.7 M outputs of 256 terms with the
// cross-entropy epilogue 599 us there, 470 us here (two or three waves per SIMD
// alike; products alone about 300); a single 2^22-output step 45 us, 28 here.
constexpr int kST = 32;

// Waves of a block over a step's tiles: 2 x 2, or in a line where one operand
// is a single tile wide.
struct StreamShape {
  int wm, wn, tm, tn;   // log2 of waves and of block tiles, rows and columns
};
__host__ __device__ inline StreamShape stream_shape(int logM, int logN) {
  const int m = logM - 6, n = logN - 6;
  StreamShape s;
  s.wn = n < 1 ? 0 : m == 0 && n > 1 ? 2 : 1;
  s.wm = m < 2 - s.wn ? m : 2 - s.wn;
  s.tm = m - s.wm;
  s.tn = n - s.wn;
  return s;
}

template <int MODE, int XE>
__device__ __forceinline__ void stream_block(const ContractArgs &a, int64_t blk) {
  const int lane = threadIdx.x & 63, wave = uni((int32_t)(threadIdx.x >> 6));
  const int logM = uni(a.logM), logN = uni(a.logN);
  const StreamShape sh = stream_shape(logM, logN);
  const int64_t part = 4 * blk + wave;
  if (wave >> (sh.wm + sh.wn)) {
    if (MODE != kModeIntermediate && a.partials && lane == 0) gbl(a.partials)[part] = 0.0;
    return;
  }
  const int64_t tn = blk & ((int64_t(1) << sh.tn) - 1), tm = (blk >> sh.tn) & ((int64_t(1) << sh.tm) - 1);
  const int64_t batch = blk >> (sh.tn + sh.tm);
  const int64_t m0 = ((tm << sh.wm) + (wave >> sh.wn)) * kPT;
  const int64_t n0 = ((tn << sh.wn) + (wave & ((1 << sh.wn) - 1))) * kPT;
  const int cnt = cst(uni(a.counts))[batch];
  const int32_t ld = uni(a.list_ld);
  const cptr<uint32_t> offX = cst(reinterpret_cast<const uint32_t *>(uni(a.lists))) + batch * 2 * ld;
  const cptr<uint32_t> offY = offX + ld;
  const BufRsrc X = buf_rsrc(uni(a.X), 4u << (logM + 2 * (uni(a.nS) + uni(a.nRX))));
  const BufRsrc Y = buf_rsrc(uni(a.Y), 4u << (logN + 2 * (uni(a.nS) + uni(a.nRY))));
  const uint32_t xl = 4u * lane, mb = 4u * (uint32_t)m0, nb = 4u * (uint32_t)n0;
  const uint32_t yl = 4u * (lane < 32 ? 2 * lane : 2 * lane - 63);   // even columns, then odd ones
  // groups of kST terms (at least one; the lists are padded with offset 0)
  const int groups = cnt == 0 ? 1 : (cnt + kST - 1) / kST;
  float x[kST], y[kST];
#pragma unroll
  for (int t = 0; t < kST; ++t) {
    x[t] = buf_load(X, xl, offX[t] + mb);
    y[t] = buf_load(Y, yl, offY[t] + nb);
  }
  f32x32 acc0{}, acc1{};
  for (int g = 0; g + 1 < groups; ++g) {
    const cptr<uint32_t> nx = offX + (g + 1) * kST, ny = offY + (g + 1) * kST;
#pragma unroll
    for (int t = 0; t < kST; ++t) {
      acc0 = __builtin_amdgcn_mfma_f32_32x32x1f32(x[t], y[t], acc0, 0, 0, 1);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x1f32(x[t], y[t], acc1, 0, 0, 2);
      x[t] = buf_load(X, xl, nx[t] + mb);
      y[t] = buf_load(Y, yl, ny[t] + nb);
      if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the tile's outputs: 256 contiguous bytes of two rows per access
  const uint32_t zl = 4u * (((uint32_t)(lane >> 5) << (logN + 2)) + 2u * (lane & 31));
  auto rows = [&](const void *base) {
    return buf_rsrc(static_cast<const char *>(base) + ((MODE == kModeIntermediate ? batch << (logM + logN) : 0) +
                                                       (m0 << logN) + n0) * 4, base ? 256u << logN : 0u);
  };
  auto row_off = [&](int r) { return (uint32_t)(4 * (32 * (r / 16) + (r % 4) + 8 * ((r % 16) / 4))) << logN; };
  // cross-entropy form: half the targets before the last group, the others as
  // the first are used
  constexpr int kTv = 16;
  f32x2 tv[XE ? kTv : 1];
  const BufRsrc T = rows(XE ? uni(a.xt) : nullptr);
  if constexpr (XE)
#pragma unroll
    for (int r = 0; r < kTv; ++r) tv[r] = buf_load2_nt(T, zl, row_off(r));
  const int rest = cnt - (groups - 1) * kST;   // terms of the last group
#pragma unroll
  for (int t = 0; t < kST; ++t) {
    const float xv = t < rest ? x[t] : 0.f, yv = t < rest ? y[t] : 0.f;
    acc0 = __builtin_amdgcn_mfma_f32_32x32x1f32(xv, yv, acc0, 0, 0, 1);
    acc1 = __builtin_amdgcn_mfma_f32_32x32x1f32(xv, yv, acc1, 0, 0, 2);
  }
  const float sc = MODE == kModeIntermediate ? 1.f : (float)uni(a.scale);
  const BufRsrc Z = rows(uni(a.Z)), G = rows(XE ? uni(a.xg) : nullptr);
  double msum = 0.0;
#pragma unroll
  for (int r = 0; r < 32; ++r) {
    const float v0 = acc0[r] * sc, v1 = acc1[r] * sc;
    if (!XE) buf_store_p<MODE>(v0, v1, Z, zl, row_off(r));
    if constexpr (XE) {
      const f32x2 t = tv[r % kTv];
      if (r + kTv < 32) tv[r % kTv] = buf_load2_nt(T, zl, row_off(r + kTv));
      buf_store2_nt(v0, v1, Z, zl, row_off(r));   // dropped where p is not kept
      buf_store2_nt(xent_grad_of(v0, t[0]), xent_grad_of(v1, t[1]), G, zl, row_off(r));
      msum += xent_part(v0, t[0], XE == 2) + xent_part(v1, t[1], XE == 2);
      asm volatile("" : "+v"(msum));   // or the sum is put off, with all its operands alive
    } else if (MODE != kModeIntermediate) {
      msum += (double)v0 + (double)v1;
    }
  }
  if (MODE != kModeIntermediate && a.partials) {
    const double tot = xent_total<float, XE>(wave_sum_f64(msum));
    if (lane == 0) gbl(a.partials)[part] = tot;
  }
}

template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_stream(const ContractArgs a) {
  if (gated_off(a.gate, a.gate_val)) return;
  // blocks of one XCD take a contiguous range of tiles: they share operand rows in L2
  stream_block<MODE, 0>(a, a.xcd_remap ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x);
}

template <int MODE, int XE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_stream_queue(const ContractArgs *__restrict__ descs, const int64_t *__restrict__ prefix, int ndesc,
                    unsigned long long *queue, int64_t total) {
  __shared__ int64_t item;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) item = (int64_t)atomicAdd(queue, 1ull);
    __syncthreads();
    const int64_t it = uni(item);
    if (it >= total) return;
    const int d = uni(find_desc(prefix, ndesc, it));
    stream_block<MODE, XE>(descs[d], it - uni(prefix[d]));
  }
}

static int64_t stream_blocks(const ContractArgs &a) {
  const StreamShape sh = stream_shape(a.logM, a.logN);
  return a.nbatch << (sh.tm + sh.tn);
}

// Row tiles per unit (log2) of a single-step launch: about 16384 units.
static int panel_log_tiles(const ContractArgs &a) {
  const int total = a.logM + a.logN - 12 + 2 * (a.nRX + a.nRY);   // log2 of 64 x 64 tiles
  return std::max(0, std::min(total - 14, a.logM - 6));
}

int64_t panel_partials(const ContractArgs &a, bool queue) {
  if (a.nS > 3) return 4 * stream_blocks(a);
  return a.nbatch << (a.logM + a.logN - 12 - (queue ? a.panel - 1 : panel_log_tiles(a)));
}

// With up to this many row flags per label the waves read them themselves;
// beyond it the label-list pass does it once per batch entry (its launch costs
// 4 us, and a wave reads one flag per label in about 0.5 us).
constexpr int kPanelFlags = 8;

Status launch_panel(const ContractArgs &args, hipStream_t s) {
  ContractArgs a = args;
  if (a.nS < 3 || a.logM < 6 || a.logN < 6 || a.mode == kModeFinalDeposit)
    return Status::fail(CQC_ERR_INVALID_ARG, "panel contraction: step shape");
  if (a.nS > 3) {
    CQC_TRY(launch_label_list(a, s));
    const dim3 g((unsigned)stream_blocks(a)), b(256);
    return a.mode == kModeIntermediate ? launch("wide_f32_inter_stream", k_stream<kModeIntermediate>, g, b, 0, s, a)
                                       : launch("wide_f32_final_stream", k_stream<kModeFinalBlocked>, g, b, 0, s, a);
  }
  if (a.flagX && a.nchX + a.nchY > kPanelFlags) CQC_TRY(launch_label_list(a, s));
  else a.lists = nullptr;
  const int lt = panel_log_tiles(a);
  const dim3 grid((unsigned)((panel_partials(a, false) + 3) / 4)), block(256);
  if (a.mode == kModeIntermediate)
    return launch("wide_f32_inter_panel", k_panel<kModeIntermediate>, grid, block, 0, s, a, lt);
  return launch("wide_f32_final_panel", k_panel<kModeFinalBlocked>, grid, block, 0, s, a, lt);
}

Status launch_panel_queue(int mode, const QueueLaunch &q, hipStream_t s) {
  if (!q.bprefix || q.btotal < 1) return Status::fail(CQC_ERR_INVALID_ARG, "panel queue without label-list table");
  const dim3 grid(q.grid), block(256);
  CQC_TRY(launch_label_list_table(q, s));
  const char *nm = q.stream ? "wide_f32_queue_stream" : "wide_f32_queue";
  const char *nx = q.stream ? "wide_f32_queue_xent_stream" : "wide_f32_queue_xent_panel";
  if (q.stream) {
    if (mode == kModeIntermediate)
      return launch(nm, k_stream_queue<kModeIntermediate, 0>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
    if (mode != kModeFinalBlocked) return Status::fail(CQC_ERR_INVALID_ARG, "panel queue: output mode");
    if (q.xent == 2)
      return launch(nx, k_stream_queue<kModeFinalBlocked, 2>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
    if (q.xent == 1)
      return launch(nx, k_stream_queue<kModeFinalBlocked, 1>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
    return launch(nm, k_stream_queue<kModeFinalBlocked, 0>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
  }
  if (mode == kModeIntermediate)
    return launch(nm, k_panel_queue<kModeIntermediate, 0>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
  if (mode != kModeFinalBlocked) return Status::fail(CQC_ERR_INVALID_ARG, "panel queue: output mode");
  if (q.xent == 2)
    return launch(nx, k_panel_queue<kModeFinalBlocked, 2>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
  if (q.xent == 1)
    return launch(nx, k_panel_queue<kModeFinalBlocked, 1>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
  return launch(nm, k_panel_queue<kModeFinalBlocked, 0>, grid, block, 0, s, q.descs, q.prefix, q.ndesc, q.queue, q.total);
}

}  // namespace cqc
