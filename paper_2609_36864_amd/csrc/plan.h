// Work planning of the fused lm-head kernel: how one hdl_token_logprobs call
// is cut into launches and work items, and where the caller's workspace holds
// what.  Everything here depends on the sizes only (never on the mask), so the
// workspace size is known before the call.  Host code and the kernel share
// the work-item mapping below; tests compile this header on the CPU to check
// the arithmetic over wide ranges of sizes.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace hdl {

// Fused lm-head tile geometry (see lmhead_logprob.hip).
constexpr int kTileV = 256;              // vocabulary rows per workgroup tile
constexpr int kTileN = 256;              // token rows per workgroup tile
constexpr int kGroupRT = 4;              // row tiles per per-XCD launch group
constexpr int kGroupCH = 32 / kGroupRT;  // vocabulary chunks per per-XCD launch group
constexpr int kNumXcd = 8;               // XCDs per MI355X; workgroups go round-robin
constexpr int kNumCu = 256;              // compute units
constexpr int kCountBlockRows = 4096;    // rows per block of the compaction's count pass

// How one call is cut up.  A call of n_rows rows runs in launches of at most
// rows_per_launch rows (every hidden-state byte offset of a launch must fit
// in 32 bits: the DMA takes a 64-bit base plus a 32-bit per-lane offset).
// All launches of a call share the vocabulary chunking (tpc, n_ch), so the
// partials of any launch, n_ch planes of at most n_rows rows each, fit the
// workspace sized for the first.
struct LmheadPlan {
  int64_t n_rows;           // rows of the largest launch (upper bound of its scored rows)
  int64_t rows_per_launch;  // a call is cut into launches of at most this many rows
  int64_t n_vt;             // vocabulary tiles of kTileV rows
  int64_t tpc;              // vocabulary tiles per chunk (one work item's span)
  int64_t n_ch;             // vocabulary chunks
  // workspace layout (byte offsets): compacted rows int32 [n_rows] | scored
  // count + count-pass block sums | partials fp32 [planes][n_ch][n_rows]
  size_t off_rows, off_count, off_part, bytes;
  int planes;               // partial planes: max, sum of exp, sampled logit (+ entropy)
};

// The work items of one launch: row tiles (of `rows` token rows) x vocabulary
// chunks.
struct ItemGrid {
  int64_t n_rt, n_ch, rows;
};

__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
__host__ __device__ inline size_t round_up_sz(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Largest number of rows one launch may cover (a multiple of the row tile;
// 0 when a single row tile would already exceed 4 GiB).
inline int64_t rows_per_launch(int64_t d, int esz) {
  const int64_t row_bytes = d * esz;
  return ((int64_t{1} << 32) / row_bytes) / kTileN * kTileN;
}

// Vocabulary tiles per work item for a launch of `rows` rows: long items
// amortise the per-item pipeline fill and partial write, short ones balance
// the tail across 256 CUs.  Aim for about 32 items per CU (measured: at
// 16,384 rows this runs 6 % faster than 8 items per CU; at 65,536 rows both
// give 16 tiles).  The number of chunks is then rounded up to whole chunk
// groups where that adds a third at most: with 38 chunks at V = 151,936 the last
// group's blocks held 24 items, so the runs of 32 that an XCD takes straddled
// three of them (work_item).  Whole calls, rounded against not: 65,024 rows,
// d 2048, V 151,936 (38 -> 40) 0.994, 345,722 rows, d 4096 (38 -> 40) 0.999;
// 200,000 rows, d 256, V 40,000 (12 -> 16) 0.98; 300,000 rows, d 512, V 50,257
// (13 -> 16) 1.01; but 262,144 rows, V 32,000 (9 -> 16) 1.015 at d 256 and 1024.
inline int64_t default_tpc(int64_t rows, int64_t n_vt) {
  int64_t tpc = ceil_div(rows, kTileN) * n_vt / 8192;
  if (tpc < 1) tpc = 1;
  if (tpc > 16) tpc = 16;
  const int64_t n_ch = ceil_div(n_vt, tpc);
  const int64_t whole = ceil_div(n_ch, kGroupCH) * kGroupCH;
  return n_ch > kGroupCH && 3 * whole <= 4 * n_ch ? ceil_div(n_vt, whole) : tpc;
}

// Workspace layout for launches of at most `rows` rows with n_ch chunks.
inline void layout_workspace(LmheadPlan& p, int64_t rows, int planes) {
  p.n_rows = rows;
  p.planes = planes;
  size_t off = 0;
  p.off_rows = off;
  off = round_up_sz(off + sizeof(int32_t) * static_cast<size_t>(rows), 256);
  p.off_count = off;
  off = round_up_sz(off + sizeof(int32_t) * (64 + static_cast<size_t>(ceil_div(rows, kCountBlockRows))), 256);
  p.off_part = off;
  off = round_up_sz(off + sizeof(float) * static_cast<size_t>(planes) * static_cast<size_t>(p.n_ch) *
                              static_cast<size_t>(rows), 256);
  p.bytes = off;
}

// The plan of a call over n_rows_total rows (4 partial planes: room for the
// entropy accumulator, so one workspace serves both entry points).
inline LmheadPlan make_plan(int64_t n_rows_total, int64_t vocab, int64_t d, int esz) {
  LmheadPlan p{};
  p.rows_per_launch = rows_per_launch(d, esz);
  const int64_t rows = n_rows_total < p.rows_per_launch ? n_rows_total : p.rows_per_launch;
  p.n_vt = ceil_div(vocab, kTileV);
  p.tpc = default_tpc(rows, p.n_vt);
  p.n_ch = ceil_div(p.n_vt, p.tpc);
  layout_workspace(p, rows, 4);
  return p;
}

// The plan of a call whose whole workspace must fit in `total_bytes`, with
// `planes` partial planes: the default chunking where it fits (then the
// results equal those of the default plan bit for bit), else fewer, longer
// chunks.  Returns false when not even one chunk fits.
inline bool make_plan_bounded(int64_t n_rows_total, int64_t vocab, int64_t d, int esz, int planes,
                              size_t total_bytes, LmheadPlan* out) {
  LmheadPlan p{};
  p.rows_per_launch = rows_per_launch(d, esz);
  if (p.rows_per_launch < kTileN) return false;
  const int64_t rows = n_rows_total < p.rows_per_launch ? n_rows_total : p.rows_per_launch;
  p.n_vt = ceil_div(vocab, kTileV);
  // the part of the workspace that does not depend on the chunking
  p.n_ch = 0;
  layout_workspace(p, rows, planes);
  const size_t fixed = p.off_part;
  const size_t per_chunk = sizeof(float) * static_cast<size_t>(planes) * static_cast<size_t>(rows);
  if (total_bytes < fixed + per_chunk) return false;
  const int64_t n_ch_fit = static_cast<int64_t>((total_bytes - fixed) / per_chunk);
  p.tpc = default_tpc(rows, p.n_vt);
  if (ceil_div(p.n_vt, p.tpc) > n_ch_fit) p.tpc = ceil_div(p.n_vt, n_ch_fit);   // fewer, longer chunks
  p.n_ch = ceil_div(p.n_vt, p.tpc);   // <= n_ch_fit
  layout_workspace(p, rows, planes);
  if (p.bytes > total_bytes) return false;
  *out = p;
  return true;
}

// The work items of a launch that scores n_s rows.  Tiles of kTileN rows, but
//  - of half of that up to 3 / 2 kTileN rows of bf16, where a second whole tile
//    would be mostly padding and W's stream from HBM, not the matrix work, sets
//    the pace.  Kernel times, half to whole tiles, statistics: V = 151,936,
//    130 / 200 / 256 / 300 / 384 rows: d 1024 0.98 / 0.94 / 1.01 / 0.90 / 0.96,
//    d 2048 0.84 / 0.92 / 0.96 / 0.89 / 0.99, d 5120 0.83 / 0.98 / 1.00 / 0.76 /
//    0.90 (2048: 300 rows 247 -> 218 us); V = 50,257 and 100,000: 300 rows 0.69
//    to 0.91, 384 rows 0.83 to 1.08, 256 rows 1.06 to 1.14 at V = 100,000 (two
//    rounds of workgroups become four); the gradient mode within 0.05 of these.
//    Rows that are no multiple of 128 bytes (d 1000) range from 0.80 (V =
//    100,000, 300 rows) to 1.18 (V = 151,936, 340 rows).  fp32 tiles split W's
//    values on the vector ALU for every row tile anew: 1.03 to 1.06 above 256
//    rows, 1.3 below (V = 120,000), so they stay whole;
//  - of half or a quarter where their items still run at once, one on a CU: a
//    half tile takes 0.55 of a whole one's time (fp32 0.65), so with a second
//    round of workgroups little would be gained.  Whole calls against narrower
//    tiles wherever there were fewer items than CUs (in brackets: whole tiles'
//    items): bf16, d 2048, V 4,096: 600 rows (48) 0.99, 1,100 (80) 0.80, 2,500
//    (160) 0.93, 3,500 (224) 0.90; V 32,000, 200 rows (125) 0.80; fp32, d 1024,
//    the same rows 1.0, 0.71, 0.77, 0.77 and 0.72.
__host__ __device__ inline ItemGrid item_grid(int64_t n_s, int64_t n_ch, bool bf16) {
  int64_t rows = bf16 && n_s <= kTileN / 2 * 3 ? kTileN / 2 : kTileN;
  while (rows > kTileN / 4 && ceil_div(n_s, rows / 2) * n_ch <= kNumCu) rows /= 2;
  return ItemGrid{ceil_div(n_s, rows), n_ch, rows};
}

// Workgroups of one launch over n rows (n <= plan.n_rows) with the call's
// chunking: one for every item of any n_s <= n, i.e. whole tiles, at most three
// half tiles, or up to kNumCu (which is less than a round) narrower ones.
inline int64_t launch_grid(const LmheadPlan& p, int64_t n) {
  const int64_t halves = ceil_div(n, kTileN / 2);
  int64_t tiles = ceil_div(n, kTileN);
  if (tiles < (halves < 3 ? halves : 3)) tiles = halves < 3 ? halves : 3;
  const int64_t round = kNumXcd * kGroupRT * kGroupCH;
  static_assert(kNumXcd * kGroupRT * kGroupCH >= kNumCu, "the narrow items fit the smallest grid");
  return ceil_div(tiles * p.n_ch, round) * round;
}

// Work item of workgroup b.  The items are put in an order in which any 32
// consecutive ones share hidden-state and W tiles: first the row tiles in
// groups of kGroupRT, as blocks of kGroupRT tiles x kGroupCH chunks (chunk
// groups outermost), then the last n_rt mod kGroupRT tiles together with the
// group before them (5 to 7 tiles; all of them where there is no whole
// group), side by side, chunk after chunk.  Workgroups are dealt to the XCDs round-robin, and
// run s of 32 items goes to XCD s mod 8 as that XCD's next 32 workgroups, so
// whole blocks stay on one XCD and its L2.  No workgroup stands for an empty
// place of a block, so the XCDs get equal shares whatever the number of row
// tiles.  (Blocks padded to kGroupRT tiles and dealt by the call's rows, not
// the scored ones, left half of the XCDs with half of the work at 6 row tiles
// -- 1,490 rows, d 4096: 1886 us against 1526 -- and all of it on two XCDs
// where a mask left 6 of 14: 436 us against 224.)  b past the last item gets
// rt = n_rt.
__host__ __device__ inline void work_item(int64_t b, const ItemGrid& g, int64_t* rt, int64_t* ch) {
  constexpr int64_t kRun = kGroupRT * kGroupCH;
  const int64_t j = b / kNumXcd;
  int64_t at = ((j / kRun) * kNumXcd + b % kNumXcd) * kRun + j % kRun;
  int64_t left = g.n_rt % kGroupRT;
  if (left != 0 && g.n_rt > kGroupRT) left += kGroupRT;
  const int64_t whole = g.n_rt - left;
  if (at < whole * g.n_ch) {
    const int64_t gch = at / (whole * kGroupCH);
    at -= gch * whole * kGroupCH;
    const int64_t rest = g.n_ch - gch * kGroupCH;
    const int64_t chunks = rest < kGroupCH ? rest : kGroupCH;
    const int64_t grt = at / (kGroupRT * chunks);
    at -= grt * kGroupRT * chunks;
    *rt = grt * kGroupRT + at % kGroupRT;
    *ch = gch * kGroupCH + at / kGroupRT;
    return;
  }
  at -= whole * g.n_ch;
  const bool in = at < left * g.n_ch;
  *rt = in ? whole + at % left : g.n_rt;
  *ch = in ? at / left : 0;
}

}  // namespace hdl
