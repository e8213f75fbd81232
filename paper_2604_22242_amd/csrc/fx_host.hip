// Host-side pieces shared by every entry point: error reporting, launch
// configuration resolution and workspace layout.
#include <stdarg.h>
#include <stdio.h>

#include <algorithm>

#include "fx_kernels.hpp"

namespace fx {

std::string& last_error() {
  thread_local std::string s;
  return s;
}

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  last_error() = buf;
  return code;
}

int hip_check(hipError_t e, const char* what) {
  if (e == hipSuccess) return FX_OK;
  return fail(FX_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    cached[dev] = cus;
  }
  return cached[dev];
}

int check_launch(const fx_launch* c) {
  if (!c) return FX_OK;
  if (c->block != 0 && (c->block < 64 || c->block > kMaxBlock || c->block % 64))
    return fail(FX_E_CONFIG, "block %d: need a multiple of 64 in [64, %d]", c->block, kMaxBlock);
  if (c->ept != 0 && c->ept != 1 && c->ept != 2 && c->ept != 4 && c->ept != 8)
    return fail(FX_E_CONFIG, "ept %d: need 1, 2, 4 or 8", c->ept);
  if (c->vec_bytes != 0 && c->vec_bytes != 2 && c->vec_bytes != 4 && c->vec_bytes != 8 &&
      c->vec_bytes != 16)
    return fail(FX_E_CONFIG, "vec_bytes %d: need 2, 4, 8 or 16", c->vec_bytes);
  if (c->split < 0 || c->split > 65535 * 64)
    return fail(FX_E_CONFIG, "split %d out of range", c->split);
  return FX_OK;
}

// Defaults, from launch-configuration sweeps on MI355X (C2 expression
// 8192 x 8192 in FP32, FP64 and BF16; accu at 2^28 in BF16):
//   element-wise: one tile per block, no grid-stride loop, 512 threads x one
//     16-byte vector per input (6.6 TB/s FP32 on the C2 expression);
//   full reductions: one block per CU (each block takes one ticket: tens of
//     thousands of tickets on one counter serialise); 256 threads, EPT 4 for
//     4- and 8-byte types, 512 threads, EPT 2 for half types.  With its loads
//     that deep in flight one block per CU streams faster than two, whose
//     waves spread over twice the address range: accu at 2^28 FP32 291-295
//     against 298 us, 2^27 FP64 293 against 300, 2^28 BF16 153 against 157,
//     2^22 FP32 10.9 against 12.3.  Below 2^21 elements EPT 2 is faster (more
//     blocks share the latency: 2^20 FP64 7.8 against 8.7 us), every thread
//     gets 8 vectors but at least kReduceMinBlocks blocks run (2^20 BF16: 64
//     blocks 6.4 us, 32 blocks 7.5), and an input of at most 32 KB is one
//     block, which needs no cross-block finish (2^12 FP32 2.7 against 3.9 us).
//     Expressions that divide or call functions take EPT 2 and, from 2^24
//     elements on, two blocks per CU, whose waves overlap one's arithmetic with
//     the other's loads (2^26 elements, us with one and with two: X / (1 + Y % Y)
//     FP32 107, 86, BF16 93, 62; the matrix workload's expression FP32 175, 125,
//     FP64 316, 244; five functions FP32 365, 230);
//   column sums: one block per column, 512 threads, EPT 2 for 4- and 8-byte
//     types, 256, EPT 1 for half types, fewer where the column has no work for
//     them (colsum_launch), a column split into chunks only where there are
//     fewer columns than CUs;
//   row sums: two blocks per CU, 256 threads, EPT 2 for 4- and 8-byte types,
//     512 threads, EPT 1 for half types (whose arithmetic wants the waves):
//     matrix workload FP32 118 us against 126 with four blocks per CU, FP64
//     234 against 252, BF16 97; fewer chunks where a thread would get less
//     than two columns, and at most 128, since the finish reads them all
//     (64 x 32768 BF16: 17 us with 128 chunks, 22 with 512).
static constexpr int kReduceMinBlocks = 64;
static constexpr int kReduceMinVecs = 8;  // per thread
static constexpr int64_t kReduceDeepFrom = (int64_t)1 << 21;
static constexpr int64_t kReduceOneBlockBytes = 32 << 10;
static constexpr int kRowsumBlocksPerCU = 2;
static constexpr int kRowsumMinCols = 2;
static constexpr int kRowsumMaxSplit = 128;
static constexpr int kRowsumChunksHeld = 64;
// Whether a reduction needs a workspace, and of what size, is part of the
// interface and does not follow the launch heuristics: calls that leave the
// split to the library ask for the bytes of fixed launches (launch::held: full sums
// by two blocks per CU, column sums by eight, row sums in chunks of at least 32
// columns), though they write fewer partials.
static size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }
// `parts` partial sums of each of n_out results, `counters` finish counters
static size_t held_bytes(int64_t parts, int64_t n_out, int64_t counters) {
  return parts > 1 ? round256((size_t)counters * 4) + (size_t)n_out * parts * 8 : 0;
}
static constexpr int64_t kHeldTwoFrom = (int64_t)1 << 24;

// Column sums: threads for a column of n_rows, at most `block` of them with `ept`
// vectors each.  A thread without a vector costs its share of the block's start and
// end (128 x 32768 FP32 102 us with 512 threads, 15.5 with 64; 1024 x 4096 17 and 10),
// so no more threads than take ept vectors each; with few columns, whose blocks
// do not fill the chip, than take one.  A column of half storage takes twice its 256
// threads where there are one or two whole columns per CU (8192 x 512 BF16 11.4,
// 8.4; 20000 x 400 25, 16.6; 65536 x 512 71, 45); chunked ones run as fast with 256
// (65536 x 64 13.6 and 13.9).
// With a column per CU or more chunks pay only where the columns are long and hardly
// more than one per CU (65536 x 256 BF16 31 us in 4 chunks, 38 whole; 65536 x 400 47 and
// 44, 65536 x 512 56 and 45, 12000 x 700 32 and 18): each column has a finish.
static constexpr int64_t kLongColumn = 65536;
static bool long_columns(int64_t n_rows, int64_t n_cols) {
  return n_rows >= kLongColumn && 2 * n_cols < 3 * (int64_t)device_cus();
}
static fx_launch colsum_launch(int elem, int64_t n_rows, int64_t n_cols, int block, int ept) {
  const int vec = 16 / elem;
  const int64_t cus = device_cus();
  if (elem == 2 && n_cols >= cus && n_cols <= 2 * cus && !long_columns(n_rows, n_cols)) block = 512;
  const int64_t each = (int64_t)vec * (n_cols < 4 * cus ? 1 : ept);
  int b = 64;
  while (b < block && b * each < n_rows) b *= 2;
  return fx_launch{b, (int64_t)b * vec >= n_rows ? 1 : ept, 16, 0};
}
// One thread per column up to 64 bytes of it, and up to 32 rows where there are 16
// columns per CU.
// Matrix workload, a thread against a wave per column, us:
//   2^26 elements    FP32 17 rows 255, 1340, 32 rows 529, 707
//                    FP64  9 rows 489, 3645, 16 rows 1050, 2039, 28 rows 1030, 1188,
//                          32 rows 1348, 1030
//                    BF16 17 rows 138, 2263, 32 rows 193, 1191
//   2^16 elements    FP32 17 rows (3855 columns) 4.0, 4.1, 32 rows (2048) 5.3, 3.5
//                    FP64 10 rows (6553) 4.2, 6.1, 12 rows (5461) 5.5, 5.9, 16 rows
//                          (4096) 6.7, 4.8 (6144) 6.9, 5.7 (8192) 6.9, 6.6 (65536) 8.6, 34
// (FP64 loses up to 2 us at the line's lower end and a quarter at 32 rows of a
// power of two of columns; one line serves all types.)
// (In FP32 the two meet again at 40 to 48 rows, in BF16 beyond 64.)  No other
// launch reaches 2^26 columns: a grid has fewer than 2^32 threads.
constexpr int64_t kThinColumnBytes = 64, kThinRows = 32, kThinColumnsPerCU = 16;
constexpr int kThinBlock = 256;
static bool thin_columns(int elem, int64_t n_rows, int64_t n_cols) {
  return n_rows * elem <= kThinColumnBytes ||
         (n_rows <= kThinRows && n_cols >= kThinColumnsPerCU * device_cus());
}

launch resolve(int kind, int elem, int64_t n_rows, int64_t n_cols, const fx_launch* cfg,
               bool vectors, int funcs) {
  fx_launch c = cfg ? *cfg : fx_launch{0, 0, 0, 0};
  launch L;
  const bool ew = kind == 0;
  const bool full = kind == FX_R_ACCU || kind == FX_R_NORM || kind == FX_R_DOT;
  const int vec16 = 16 / elem;  // sizing always assumes 16-byte vectors
  const int64_t n = n_rows * n_cols;
  const int64_t cus = device_cus();
  int vb = c.vec_bytes ? c.vec_bytes : 16;
  if (vb < elem) vb = elem;
  if (!vectors) vb = elem;
  L.vec_bytes = vb;
  if (ew || full) {
    L.block = c.block ? c.block : default_block(kind, elem);
    L.ept = c.ept ? c.ept : default_ept(kind, elem);
    if (full && !c.ept && (funcs > 0 || n < kReduceDeepFrom)) L.ept = 2;
    const int64_t tiles = std::max<int64_t>(1, ceil_div(n, (int64_t)L.block * L.ept * vec16));
    int64_t want = tiles;
    if (full) {
      const int64_t per_block = (int64_t)L.block * kReduceMinVecs * vec16;
      const int64_t most = funcs > 0 && n >= kHeldTwoFrom ? 2 * cus : cus;
      want = std::min<int64_t>({tiles, most, std::max<int64_t>(kReduceMinBlocks, n / per_block)});
      if (n * elem <= kReduceOneBlockBytes) want = 1;
    }
    L.split = c.split ? c.split : (int)std::min<int64_t>(want, 1 << 30);
    if (full && !c.split) {
      const int64_t t2 = std::max<int64_t>(1, ceil_div(n, (int64_t)L.block * (c.ept ? c.ept : 2) * vec16));
      L.held = held_bytes(std::min<int64_t>({t2, n < kHeldTwoFrom ? cus : 2 * cus, std::max<int64_t>(32, t2 / 4)}), 1, 1);
    }
  } else if (kind == FX_R_COLSUM) {
    const fx_launch d = colsum_launch(elem, n_rows, n_cols, default_block(kind, elem), default_ept(kind, elem));
    // (a caller's own chunks are limited to a pass of the default block each, so
    // that the workspace they need does not follow the threads' rule)
    L.block = c.block ? c.block : c.ept || c.split ? default_block(kind, elem) : d.block;
    L.ept = c.ept ? c.ept : c.block || c.split ? default_ept(kind, elem) : d.ept;
    if (!c.split && thin_columns(elem, n_rows, n_cols)) {
      L.split = 0;  // thin columns: one thread per column
      if (!c.block) L.block = kThinBlock;
    } else {
      const int64_t ncol = std::max<int64_t>(1, n_cols);
      int64_t s = c.split;
      if (s) {
        s = std::min<int64_t>(s, std::max<int64_t>(1, ceil_div(n_rows, (int64_t)L.block * vec16)));
      } else {
        // Chunks only where there are fewer columns than CUs (each column
        // combined across blocks costs its last block some microseconds: 4096 x
        // 1024 FP32 11 us whole, 16 in two chunks) and a column is at least five
        // full passes of the block long, two of half storage and with fewer than 64
        // columns (whole and in chunks: 10000 x 104 FP32 7.1 us and 12.5, FP64 11.2 and
        // 14.8; 10000 x 6 FP64 8.8 and 6.6, 20000 x 60 FP64 18.3 and 13.3, FP32 10.6 and
        // 10.8), a pass or part of one each; about a
        // block per CU, two from 64 columns on (32768 x 128 FP32 13.3 us with 8
        // chunks, 18.1 with 16; 2^22 x 1 21 us with 256, 71 with 2048).
        const int64_t pass = (int64_t)L.block * vec16;
        const int64_t target = ncol * 4 >= cus ? 2 * cus : cus;
        s = ncol >= cus || n_rows < (elem == 2 || ncol * 4 < cus ? 2 : 5) * pass * L.ept ? 1 : ceil_div(target, ncol);
        s = std::min<int64_t>(s, ceil_div(n_rows, pass));
        // Half storage does twice the arithmetic per byte and wants the waves: up
        // to 8 blocks per CU of at least two passes each, at most 64 chunks, which
        // the finish reads one after another (matrix workload BF16 2^20 x 16 34 us
        // with 64 chunks, 66 with 16; 2^20 x 64 88 with 32, 145 with 8; 65536 x 256
        // 31 with 8, 38 whole; 200000 x 255 68 with 9, 88 with 3).
        // Expressions of three functions or more likewise (262144 x 256 FP32, that expression,
        // 170 us with 8, 201 whole).
        if ((elem == 2 || funcs >= 3) && (ncol < cus || long_columns(n_rows, ncol)))
          s = std::max<int64_t>(s, std::min<int64_t>({ceil_div(8 * cus, ncol), n_rows / (2 * pass), 64}));
      }
      L.split = (int)std::max<int64_t>(1, std::min<int64_t>(s, 65535));
      if (!c.split && n_rows > 32)
        L.held = held_bytes(std::min<int64_t>({ceil_div(8 * cus, ncol), 65535, std::max<int64_t>(1, ceil_div(
            n_rows, (int64_t)(c.block ? c.block : default_block(kind, elem)) * vec16))}), n_cols, n_cols);
    }
  } else {  // FX_R_ROWSUM
    L.block = c.block ? c.block : default_block(kind, elem);
    L.ept = c.ept ? c.ept : default_ept(kind, elem);
    const int vec = vb / elem;
    const int rl = rowsum_lanes(n_rows, n_cols, vec, elem, L.block);
    const int64_t tiles = std::max<int64_t>(1, ceil_div(n_rows, (int64_t)rl * vec));
    int64_t s = c.split;
    if (!s) {
      const int64_t per_thread = (int64_t)(L.block / rl) * kRowsumMinCols;
      s = std::min<int64_t>({cus * kRowsumBlocksPerCU / tiles, kRowsumMaxSplit,
                             std::max<int64_t>(1, n_cols / per_thread)});
    }
    s = std::min<int64_t>(s, std::max<int64_t>(1, n_cols));
    L.split = (int)std::max<int64_t>(1, std::min<int64_t>(s, 65535));
    if (!c.block && !c.ept && !c.vec_bytes && !c.split) {
      const int block = elem == 2 ? 64 : 256;
      const int64_t blocks = std::max<int64_t>(1, ceil_div(n_rows, (int64_t)block * vec16));
      L.held = held_bytes(std::max<int64_t>(1, std::min<int64_t>({ceil_div(cus * 512 / block, blocks), n_cols / 32, 65535})),
                          n_rows, ceil_div(n_rows, block));
    }
  }
  return L;
}

// Interpreted tapes want other configurations than compiled expressions:
// the interpreter's per-instruction cost shifts the balance towards more,
// smaller blocks.  The element-wise defaults are, per storage width, the single
// configuration with the best geometric-mean time (over each item's best) on the
// autotuner's 20,000 random training trees, two vectors per thread for FP32 and
// FP64 from 2^20 elements on.  Those of the reductions follow the shape, from the
// sweeps given at each.  On the 2,000 held-out trees all of them together give
// 1.06x the best of 145 configurations.  Column sums keep the split heuristic when there are fewer
// columns than CUs (one block per column would leave the chip idle), and row
// sums keep it always: 512 threads on full vectors are within 2% of the best
// of 144 configurations on the trees swept since their kernel combines in the
// block (4096 x 4096 FP32, 30 instructions: 92 us; 256 threads of one row each
// in 64 chunks, the default until then: 153).  The split default
// applies only when the whole configuration is left at 0: a caller that
// sets any field and leaves split at 0 gets the library's split heuristic.
fx_launch tape_launch(int kind, int elem, int64_t n_rows, int64_t n_cols, const fx_launch* cfg) {
  fx_launch c = cfg ? *cfg : fx_launch{0, 0, 0, 0};
  const bool all_default = !c.block && !c.ept && !c.vec_bytes && !c.split;
  const bool half = elem == 2;
  const int cus = device_cus();
  fx_launch d;
  switch (kind) {
    case FX_R_ACCU: case FX_R_NORM: {
      // No block without a tile: a block with nothing to add still takes a
      // ticket, and 512 of them take 10 us (2^12 elements FP32 10.2 us with 512
      // blocks, 4.2 with one; 2^18 10.3, 7.3 with 64).  Up to 2^17 elements tiles
      // of 128 threads spread better (2^16 FP32 6.2 us against 6.8, 2^14 6.2
      // against 6.5), unless 512 threads take all in one (2^12: 4.2 against 5.4).
      const int64_t n = n_rows * n_cols, wave = 64 * (half ? 1 : 2) * (16 / elem);
      const int block = all_default && n > 8 * wave && n < ((int64_t)1 << 17) ? 128 : 512;
      const int64_t tiles = ceil_div(n, block / 64 * wave);
      d = fx_launch{block, half ? 1 : 2, 16, (int)std::max<int64_t>(1, std::min<int64_t>(tiles, 2 * cus))};
      break;
    }
    case FX_R_COLSUM:
      // 512 threads with at most two columns per CU, as above 256 (8192 x 512 FP32
      // 15.8 us with 256, 12.3; 65536 x 512 BF16 101, 59, but FP64 155, 169); fewer for
      // short columns (128 x 32768 FP32 109 us, 24)
      d = fx_launch{256, half ? 1 : 2, 16, 0};
      if (all_default) d = colsum_launch(elem, n_rows, n_cols, n_cols < cus || (n_cols <= 2 * cus && (half || n_rows < kLongColumn)) ? 512 : 256, half ? 1 : 2);
      d.split = n_cols >= cus ? 1 : 0;
      break;
    case FX_R_ROWSUM: d = fx_launch{512, half ? 1 : 2, 16, 0}; break;
    default:
      // two vectors per thread fill an interpreter pass for 4- and 8-byte
      // types; they pay off once there are enough elements to keep the chip
      // busy with fewer threads (training trees: 1.073x the best against
      // 1.096x for one vector everywhere)
      d = elem >= 4 && n_rows * n_cols >= ((int64_t)1 << 20) ? fx_launch{256, 2, 16, 0}
                                                            : fx_launch{64, 1, 16, 0};
      break;
  }
  if (!c.block) c.block = d.block;
  if (!c.ept) c.ept = d.ept;
  if (!c.vec_bytes) c.vec_bytes = d.vec_bytes;
  if (all_default) c.split = d.split;
  return c;
}


ws_layout workspace_for(int kind, int64_t n_rows, int64_t n_cols, const launch& L, int elem, int vec) {
  ws_layout W;
  const size_t parts = L.split > 1 ? L.split : 0;
  if (kind == FX_R_ACCU || kind == FX_R_NORM || kind == FX_R_DOT) {
    if (parts) W.counter_bytes = 256;
    W.partial_bytes = parts * 8;
  } else if (kind == FX_R_COLSUM) {
    if (parts) W.counter_bytes = round256((size_t)n_cols * 4);
    W.partial_bytes = (size_t)n_cols * parts * 8;
  } else if (kind == FX_R_ROWSUM) {
    const int rl = rowsum_lanes(n_rows, n_cols, vec, elem, L.block);  // one counter per row tile
    if (parts) W.counter_bytes = round256((size_t)ceil_div(n_rows, (int64_t)rl * vec) * 4);
    W.partial_bytes = (size_t)n_rows * parts * 8;
  }
  if (W.total() < L.held) W.partial_bytes = L.held - W.counter_bytes;
  return W;
}

// The workspace of a tape reduction whose launch is left to the library: the
// partials of two blocks per CU, or of kRowsumChunksHeld column chunks, so that a
// launch model's or a caller's own split of that many fits it.
size_t tape_workspace(int kind, int64_t n_rows, int64_t n_cols) {
  if (kind == FX_R_ACCU || kind == FX_R_NORM) return held_bytes(2 * device_cus(), 1, 1);
  if (kind == FX_R_ROWSUM)
    return held_bytes(std::min<int64_t>(kRowsumChunksHeld, n_cols), n_rows, ceil_div(n_rows, 256));
  return 0;
}

static int elem_size(fx_dtype dt) {
  switch (dt) {
    case FX_F32: case FX_U32: return 4;
    case FX_F64: return 8;
    case FX_BF16: case FX_F16: return 2;
  }
  return 0;
}

size_t rowsum_extra_counters(int kind, fx_dtype dt, fx_shape s, const fx_launch* cfg) {
  const int elem = elem_size(dt);
  if (kind != FX_R_ROWSUM || !elem || !cfg || (!cfg->block && !cfg->ept && !cfg->vec_bytes && !cfg->split)) return 0;
  const int64_t block = cfg->block ? cfg->block : elem == 2 ? 64 : 256;
  const fx_launch t = tape_launch(kind, elem, s.n_rows, s.n_cols, cfg);
  size_t most = 0;
  for (const fx_launch* c : {cfg, &t}) {
    const launch L = resolve(kind, elem, s.n_rows, s.n_cols, c, true);
    if (L.split > 1)
      most = std::max(most, workspace_for(kind, s.n_rows, s.n_cols, L, elem, L.vec_bytes / elem).counter_bytes);
  }
  const size_t one_per_block = round256((size_t)ceil_div(s.n_rows, block) * 4);
  return most > one_per_block ? most - one_per_block : 0;
}

}  // namespace fx

using namespace fx;

extern "C" {

const char* fx_version(void) { return "fx 0.1 (gfx950)"; }

const char* fx_last_error(void) { return last_error().c_str(); }

int fx_synchronize(void* stream) {
  return hip_check(hipStreamSynchronize(static_cast<hipStream_t>(stream)), "hipStreamSynchronize");
}

size_t fx_workspace_bytes(int kind, fx_dtype dt, fx_shape shape, const fx_launch* cfg) {
  const int elem = elem_size(dt);
  if (!elem || shape.n_rows < 0 || shape.n_cols < 0 || check_launch(cfg)) return 0;
  if (kind < FX_R_ACCU || kind > FX_R_DOT) return 0;
  launch L = resolve(kind, elem, shape.n_rows, shape.n_cols, cfg, true);
  size_t b = workspace_for(kind, shape.n_rows, shape.n_cols, L, elem, L.vec_bytes / elem).total();
  // the same call may evaluate a run-time tape, whose defaults differ:
  // enough for both
  if (kind != FX_R_DOT) {
    const fx_launch t = tape_launch(kind, elem, shape.n_rows, shape.n_cols, cfg);
    launch T = resolve(kind, elem, shape.n_rows, shape.n_cols, &t, true);
    b = std::max(b, workspace_for(kind, shape.n_rows, shape.n_cols, T, elem, T.vec_bytes / elem).total());
    if (!cfg || (!cfg->block && !cfg->ept && !cfg->vec_bytes && !cfg->split))
      b = std::max(b, tape_workspace(kind, shape.n_rows, shape.n_cols));
  }
  return b;
}

int fx_resolve_launch(int kind, fx_dtype dt, fx_shape shape, const fx_launch* cfg,
                      fx_launch* out) {
  const int elem = elem_size(dt);
  if (!elem) return fail(FX_E_DTYPE, "unknown dtype %d", (int)dt);
  if (!out || shape.n_rows < 0 || shape.n_cols < 0) return fail(FX_E_ARG, "bad arguments");
  if (kind < 0 || kind > FX_R_DOT) return fail(FX_E_ARG, "unknown kind %d", kind);
  if (int rc = check_launch(cfg)) return rc;
  launch L = resolve(kind, elem, shape.n_rows, shape.n_cols, cfg, true);
  *out = fx_launch{L.block, L.ept, L.vec_bytes, L.split};
  return FX_OK;
}

}  // extern "C"
