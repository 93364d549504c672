// Kernel argument blocks and host launchers of the gfx950 kernels.
#pragma once

#include <cstdint>

#include "common.hpp"

namespace cqc {

// Row-index map of one operand, packed into scalars so the kernel never indexes
// a kernel-argument array with a runtime index (that turns into dependent
// vector loads from the argument segment).  Digit i (most significant first)
// takes source (srcmask >> i) & 1 (0: shared index s, 1: rest index r) and
// shift (shifts[i / 10] >> 6 (i % 10)) & 63.
struct DigitMapDev {
  int32_t n;
  uint32_t srcmask;
  uint64_t shifts[2];
};

// Output-bit positions of the column bits of an operand (bit j counted from
// the least significant), 6 bits each, 10 per word.
struct BitPos {
  uint64_t w[5];
};

// One pairwise contraction step (see plan.hpp), executed as a batched GEMM
//   C_b[m][n] = sum_{s live} X[rowX(s, rX)][m] * Y[rowY(s, rY)][n],  b = (rX, rY)
enum ContractMode : int32_t {
  kModeIntermediate = 0,  // Z[b][m][n] row-major, Acc dtype, row flags of Z written
  kModeFinalBlocked = 1,  // out[m * N + n] * scale
  kModeFinalDeposit = 2   // out[rowoff(m) + coloff(n)] * scale, per-bit positions
};

struct ContractArgs {
  const void *X;
  const void *Y;
  const int32_t *flagX;   // [rows][nchX] chunk flags
  const int32_t *flagY;
  int32_t nchX, nchY;
  int32_t *flagZ;
  void *Z;
  int32_t logM, logN;
  int32_t nS, nRX, nRY;
  int32_t tilesM, tilesN;
  int32_t mode;
  int32_t xcd_remap;  // 1: keep consecutive logical tiles on one XCD
  int64_t nblocks;
  double scale;
  DigitMapDev mx, my;
  BitPos posX, posY;  // deposit mode: column bit -> output bit position
  double *partials;  // [nblocks] per-block FP64 sums of the written outputs, or null
  // wide kernel only: live-label lists of every batch entry (written by the
  // label-list pass of the same step)
  int32_t *lists;    // [nbatch][2][list_ld] byte offsets of the live terms' X rows, then of
                     //   their Y rows, ascending s; padding 0
  int32_t *counts;   // [nbatch] live labels
  int32_t list_ld;   // pairs per batch entry: 4^nS rounded up to a multiple of 32
  int32_t rows;      // > 0: a small-term step that runs on the row kernel, with this many columns per lane
  int64_t nbatch;
  // device-side predicate: when gate is set, the launch does nothing unless
  // *gate == gate_val (a dynamic-definition query enqueues the kernels of
  // every depth a recursion can have, and runs only the one its pick chose)
  const int32_t *gate;
  int32_t gate_val;
  int32_t panel;     // > 0: a wide step that runs on the panel kernel (every step of a queue group
                     //   alike); in a queue launch 1 + log2 of the row tiles of a unit
  // split-BF16 wide steps of single calls: the operands already split into
  // bfloat16 parts, each part a plane of the operand's layout and size (2^xlog
  // and 2^ylog elements), or null (the wide kernel splits while staging)
  const void *Xs;
  const void *Ys;
  int32_t xlog, ylog;
  // split-BF16 intermediate steps whose result only a split step reads: the
  // parts of Z are written here, planes as above, instead of Z
  void *Zs;
  // cross-entropy form of a final step (batched launches): xt is the target t
  // in output order; every output p gets dL/dp = -t/p (0 where p <= 1e-30)
  // written to xg at its position, p itself is written only if Z is set, and
  // the partial sums add the loss terms -t log max(p, 1e-30) (kernel form with
  // the loss) or p
  const void *xt;
  void *xg;
};
// A batch keeps one of these per step in the caller's workspace, whose size its
// users may have on record.
static_assert(sizeof(ContractArgs) <= 344, "the workspaces of batches grow");

// FP64 mass partials: every wave of a final-step tile (four per block) stores
// the FP64 sum of the outputs it wrote at partials[kPartialsPerTile * tile +
// wave], so no block barrier stands between a tile's stores and the next
// tile; the final pass adds them in index order.
constexpr int kPartialsPerTile = 4;

// Workspace of the label lists of a step run by the wide kernel.
// Operands of the wide kernel are addressed with 32-bit byte offsets.
constexpr int64_t kWideMaxOperandElems = int64_t(1) << 30;
inline int32_t wide_list_ld(int nS) { return (int32_t)((((int64_t)1 << (2 * nS)) + 31) / 32 * 32); }
inline size_t wide_list_bytes(int nS, int64_t nbatch) {
  return (size_t)nbatch * (size_t)wide_list_ld(nS) * 8 + (size_t)nbatch * 4;
}

// Row flags are kept per (row, chunk of kFlagChunk columns): flag[r * nch + c]
// says whether chunk c of row r has a non-zero element; a row is live if any
// of its chunk flags is set.  Splitting rows lets the flag pass run with many
// waves instead of one per long row.
constexpr int kFlagChunk = 2048;
__host__ __device__ inline int64_t flag_chunks(int64_t cols) { return (cols + kFlagChunk - 1) / kFlagChunk; }
// Waves of the flag pass: one per chunk of a row longer than kFlagRun columns,
// or per flag_rows() shorter rows (cols is a power of two); four per block.
// Runs of 2048 columns left too few waves for small tensors (282 K doubles: 7.5
// us, against 5.2 with a block per row), runs of 512 do not.
constexpr int kFlagRun = 512;
__host__ __device__ inline int64_t flag_rows(int64_t cols) { return cols < 4 ? 64 : cols <= kFlagRun ? kFlagRun / cols : 1; }
__host__ __device__ inline int64_t flag_items(int64_t rows, int64_t cols) {
  return cols > kFlagRun ? rows * flag_chunks(cols) : (rows + flag_rows(cols) - 1) / flag_rows(cols);
}
__host__ __device__ inline int64_t flag_blocks(int64_t rows, int64_t cols) { return (flag_items(rows, cols) + 3) / 4; }

struct FlagDesc {
  const void *ptr;
  int64_t rows;
  int64_t cols;
  int32_t *flags;      // [rows][flag_chunks(cols)]
  int64_t block_start; // first block of this tensor
  void *unit;          // if non-null: a unit operand (Acc-typed 1.0) is written here
  int32_t *unit_flag;  //   and its row flag set
};

struct FlagArgs {
  FlagDesc d[CQC_MAX_SUB + 1];
  int32_t n;
  int32_t is_double;
  const int32_t *gate;   // as in ContractArgs
  int32_t gate_val;
};

// Arithmetic of a plan.  BF16X6 and BF16X3 keep every tensor in FP32 and
// split the operands into three (two) bfloat16 parts inside the wide kernel.
enum class Acc { F32, F64, BF16X6, BF16X3 };
inline bool is_split(Acc a) { return a == Acc::BF16X6 || a == Acc::BF16X3; }
// bfloat16 parts per operand of the wide kernel's form (0: FP32)
inline int split_parts(Acc a) { return a == Acc::BF16X6 ? 3 : a == Acc::BF16X3 ? 2 : 0; }

// Tile configurations of the contraction kernels: L, M, S, T select the
// register-operand kernel (FP32 and FP64), W the LDS-staged wide kernel
// (FP32 and the split forms; the only one the split forms run on) or, for
// steps that fit it (ContractArgs::panel), the panel kernel.
enum TileCfg : int32_t { kTileL = 0, kTileM = 1, kTileS = 2, kTileT = 3, kTileW = 4, kTileCount = 5 };
struct TileShape { int bm, bn; };
TileShape tile_shape(int cfg);
// Built-in rule (the autotuner's cache takes precedence where it has an entry).
// wide_ok: both operands fit the wide kernel's addressing (wide_fits).
// nbatch: batch entries of the step (the wide kernel needs enough 128 x 128
// tiles over all of them to fill the chip).
// panel: the step runs on the panel kernel where its tile is W.
// spread: a launch of its own that writes through the register kernels (deposit
// order, FP64, long sums): the tile shrinks until the step fills the chip.
int choose_tile(Acc acc, int nS, int logM, int logN, bool wide_ok, bool panel, int64_t nbatch, bool spread);
// Whether the arithmetic has a kernel with this tile configuration.
bool tile_ok(Acc acc, int cfg);
// Arithmetic a step of a plan runs in.  A split-form step runs the FP32 form
// where the split has nothing to win: an operand the wide kernel cannot take
// (one column: a matrix-vector product), or at most 16 terms (nS <= 2 shared
// cuts; such a step is bound by its output writes, and FP32 products are at
// least as accurate as the BF16 ones).
inline Acc step_acc(Acc acc, bool wide_ok, int nS) {
  return is_split(acc) && (!wide_ok || nS <= 2) ? Acc::F32 : acc;
}

Status launch_row_flags(const FlagArgs &a, int64_t total_blocks, hipStream_t s);
Status launch_mass_final(const double *partials, int64_t count, double *mass, hipStream_t s,
                         const int32_t *gate = nullptr, int32_t gate_val = 0);

// One launch over many contraction steps of the same kernel configuration:
// descs[d] in device memory, prefix[d] = first queue item of step d (items of
// step d are its tiles), queue = zeroed counter.
struct QueueLaunch {
  const ContractArgs *descs;
  const int64_t *prefix;
  int32_t ndesc;
  unsigned long long *queue;
  int64_t total;
  uint32_t grid;
  const int64_t *bprefix;  // wide kernel: bprefix[d] = first batch entry of step d over the table
  int64_t btotal;          //   and the total (one label-list block per batch entry)
  bool panel = false;      // wide steps of the panel kernels
  bool stream = false;     //   with more than three shared cuts
  int xent = 0;            // final steps of the cross-entropy form (ContractArgs::xt):
                           //   1 gradient (partials sum p), 2 gradient and loss
};
Status launch_contract_queue(Acc acc, int mode, int cfg, bool small, const QueueLaunch &q, hipStream_t s);

// Batched row flags (descriptor table in device memory, block_start = prefix)
// and per-instance mass reductions; the flag pass also zeroes `counters`.
struct MassDesc {
  const double *partials;
  int64_t count;
  double *mass;
};
Status launch_row_flags_table(const FlagDesc *descs, int32_t n, int64_t total_blocks, bool is_double,
                              unsigned long long *counters, int32_t n_counters, hipStream_t s);
Status launch_mass_table(const MassDesc *descs, int32_t n, hipStream_t s);
Status launch_contract(Acc acc, bool out_double, int cfg, const ContractArgs &a, hipStream_t s);
Status launch_contract_wide(int parts, bool out_double, const ContractArgs &a, hipStream_t s);
// The live-label lists of a step (of every step of a queue launch) of the wide
// and panel kernels.
Status launch_label_list(const ContractArgs &a, hipStream_t s);
Status launch_label_list_table(const QueueLaunch &q, hipStream_t s);
// Panel kernels (k_panel.hip): the wide steps with ContractArgs::panel set.
Status launch_panel(const ContractArgs &a, hipStream_t s);
Status launch_panel_queue(int mode, const QueueLaunch &q, hipStream_t s);
// Their waves: four per block or queue item, one FP64 partial each in a final step.
int64_t panel_partials(const ContractArgs &a, bool queue);
// Row tiles per unit (log2) of a queue launch over `tiles` 64 x 64 tiles: up to
// 2^kPanelQueueLog, so that a panel is reloaded only every eighth tile, as long
// as that leaves kPanelQueueUnits units, one per SIMD.  With eight tiles
// whatever the launch, the panels of two instances of 2^20 outputs ran on 16
// blocks: 55 us per run of that batch, 28 on the staged wide kernel before, 22
// now; sixteen of 2^19 outputs 58.7, 43.8 and 30.7 (39.2 with 512 units at
// least, 33.8 with 2048 or more).  The 256-instance training step takes 3.59 ms
// with any of them.
constexpr int kPanelQueueLog = 3;
constexpr int64_t kPanelQueueUnits = 1024;
inline int panel_queue_log_tiles(int64_t tiles) {
  int lt = 0;
  while (lt < kPanelQueueLog && tiles >> (lt + 1) >= kPanelQueueUnits) ++lt;
  return lt;
}
// Row kernel (k_rows.hip): the columns per lane (4, 2 or 1) with which a step
// runs on it, or 0.  FP32 steps of at most two shared cuts, output not in
// deposit order, whole 16-row tiles, and the widest panel (64 columns per lane
// column) of the tile shape the step was given - so a tuned narrower tile
// keeps the register kernel it was timed with.  Steps under 2^kRowsMinLog
// outputs (all batch entries) stay there too: the time is the launch's either
// way, and in a batch every kind of step is a launch (seven instances of 10 to
// 12 qubits: 83 us per training step with these steps in one launch, 86 split).
constexpr int kRowsMinLog = 14;
inline int rows_cols(Acc acc, int mode, int cfg, int nS, int logM, int logN, int log_batch) {
  if (acc != Acc::F32 || mode == kModeFinalDeposit || nS > 2 || logM < 4 || logN < 6 ||
      logM + logN + log_batch < kRowsMinLog)
    return 0;
  const int c = logN >= 8 ? 4 : logN == 7 ? 2 : 1;
  switch (cfg) {
    case kTileL: return c == 4 ? 4 : 0;
    case kTileM: return c >= 2 ? c : 0;
    case kTileS: return c == 1 || logM == 4 ? c : 0;
    default: return 0;
  }
}
// The same for the FP64 form of a single call with FP64 output: 2 (128 columns)
// or 0.  Tiles L and M only, which the tile rule gives a single call's step from
// 2^20 outputs (256 blocks); below, 16 x 64 register tiles fill the chip better.
// With 16 terms and rows of 2^18 columns or more, Y (32 MiB and up) no longer
// stays in the caches from one row tile to the next: 2^6 x 2^18 outputs took 35.5
// us here, 30 on the register kernel, which reads Y once per 64 rows (2^8 x 2^16:
// 28.8 and 30.6).
inline int rows_cols_f64(int mode, int cfg, int nS, int logM, int logN, int log_batch) {
  return (cfg == kTileL || cfg == kTileM) && mode != kModeFinalDeposit && nS <= 2 && logM >= 4 && logN >= 7 &&
         logM + logN + log_batch >= kRowsMinLog && (nS < 2 || logN <= 17 || logM <= 5) ? 2 : 0;
}
// 16-row tiles per wave (log2).  Longer runs reload Y less often, but spread
// the rows that the chip writes at one time over more memory: at most two tiles
// at 16 terms and four with fewer, as long as that leaves 2048 waves (1024 with
// fewer terms) and a run covers at most 2^18 outputs of whole rows (16 2^lt rows;
// 1 MiB in FP32: beyond that the runs of a panel get slower).  One and four terms,
// us for 1, 2 and 4 tiles: 2^12 x 2^14 outputs 50, 55, 66; 2^13 x 2^13 52, 48, 55;
// 2^14 x 2^12 57, 55, 49; 2^13 x 2^14 95, 113, 129; 2^14 x 2^14 185, 219, 249.  16
// terms, 1 and 2 tiles: 2^13 x 2^14 103, 113; 2^14 x 2^14 202, 216; 2^20 x 2^10 890,
// 753 (four: 765).
__host__ __device__ inline int rows_log_tiles(int logM, int logN, int log_batch, int rows, int nS) {
  const int waves = logM - 4 + logN - 6 - (rows == 4 ? 2 : rows == 2 ? 1 : 0) + log_batch;
  const int most = nS == 2 ? 1 : 2;
  int lt = waves - (nS == 2 ? 11 : 10);
  if (lt > most) lt = most;
  if (lt > logM - 4) lt = logM - 4;
  if (lt > 14 - logN) lt = 14 - logN;
  return lt < 0 ? 0 : lt;
}
// Whether a single call's final row kernel writes with ordinary stores: outputs
// of 64 to 256 MiB with fewer than 16 terms.  They stay in the 256 MiB last-level
// cache, so that a loop that writes one buffer again and again is faster - 2^12 x
// 2^14 FP32 outputs of one term 44 us, 50 with non-temporal stores; 2^9 x 2^16 FP64
// ones 46 and 54 - and calls on buffers in turn are little slower: 51 and 50, 55 and
// 54.  Smaller and larger outputs are faster with non-temporal stores (2^10 x 2^12:
// 8.2 and 8.7; 2^14 x 2^14: 185 and 189), rows of 2^18 columns too (2^6 x 2^18, four
// terms: 15.7 and 17.3 on buffers in turn), and with 16 terms the operands need
// that cache (2^13 x 2^11 FP64 outputs: ordinary stores 27.5 us and non-temporal ones
// 30 in one buffer, 34.6 and 29.6 on buffers in turn).
inline bool rows_plain_stores(int nS, int logM, int logN, bool f64_out) {
  const int log_bytes = logM + logN + (f64_out ? 3 : 2);
  return nS < 2 && logN <= 17 && log_bytes >= 26 && log_bytes <= 28;
}
// Waves of a step: one FP64 partial each in a final step, four per block.
int64_t rows_units(const ContractArgs &a);
int64_t rows_f64_units(const ContractArgs &a);
Status launch_rows(bool out_double, const ContractArgs &a, hipStream_t s);
Status launch_rows_f64(const ContractArgs &a, hipStream_t s);
// Many steps of equal rows and nS: prefix[d] = first block of step d.
Status launch_rows_table(int mode, int rows, int nS, const QueueLaunch &q, hipStream_t s);
// FP64 partials of a final step's launch (queue launch) with tile cfg.
inline int64_t mass_partials(int cfg, const ContractArgs &a, bool queue, bool f64) {
  if (a.rows) return f64 ? rows_f64_units(a) : rows_units(a);
  return cfg == kTileW && a.panel ? panel_partials(a, queue) : kPartialsPerTile * a.nblocks;
}
// Splits `count` floats (a multiple of 4) into `parts` bfloat16 planes of
// `plane` elements each (the same split as the wide kernel's staging).
Status launch_presplit(int parts, const float *src, void *dst, int64_t count, int64_t plane, hipStream_t s);
// Whether both operands of a step are within the wide kernel's 2^30-element addressing.
bool wide_fits(const ContractArgs &a);
Status launch_contract_wide_queue(int parts, int mode, const QueueLaunch &q, hipStream_t s);
Status launch_convert(const void *src, bool src_double, void *dst, bool dst_double,
                      int64_t count, hipStream_t s);
Status launch_selftest_mfma(void *out, hipStream_t s);

}  // namespace cqc
