// Fused lm-head log-probability kernel for gfx950 (MI355X).
//
// For every scored row n (a final hidden state h_n) and its sampled token y_n
// it computes, in one pass over the vocabulary projection W [V, d]:
//
//     z_n[v] = sum_j W[v, j] h_n[j]            (lm-head contraction, Eq. 1)
//     lse_n  = log sum_v exp(z_n[v])           (softmax normaliser)
//     log p_n(y_n) = z_n[y_n] - lse_n          (sampled-token log-likelihood)
//
// without ever storing z.  The vocabulary is cut into chunks; each work item
// (row tile x chunk) leaves a partial (max, sum of exp, captured z_y) per row,
// and merge_kernel combines the chunk partials in a fixed order.  Two more
// epilogues share the same main loop: one also accumulates the next-token
// entropy (the Entropy localization baseline), the other writes the gradient
// of log p with respect to the logits for the backward pass (the logits are
// recomputed there, given the forward pass's log-sum-exp).
//
// Work item: 256 vocabulary rows x 256 token rows per V-tile, looping over
// the V-tiles of one chunk.  Eight waves per workgroup (two per SIMD, so one
// wave's LDS reads and DMA issue overlap the other's MFMAs; the per-V-tile
// epilogue, which both reach after the same slice, does not), each owning
// 128 vocab x 64 tokens as an 8 x 4 grid of 16 x 16 MFMA blocks
// (v_mfma_f32_16x16x32_bf16) with fp32 accumulators.
// W is the MFMA "A" operand (vocabulary on the M axis) and the hidden states
// are the "B" operand (tokens on the N axis), so each lane's accumulators
// hold 4 token columns and 32 vocabulary rows each: the online max /
// sum-of-exp update of a V-tile is entirely lane-local, and lanes and waves
// are merged only once per work item.
//
// Operands stream through LDS in K-slices of 128 bytes per row (64 bf16 or
// 32 fp32) through a ring of 2 stages (128 KB; more for narrow tiles, see
// Ring): the next slice is in flight (global -> LDS DMA, no VGPR staging) while
// slice i is multiplied.  16-byte
// chunks are XOR swizzled and each lane group reads the chunk frag_chunk()
// assigns it, so that the 16-row fragment reads are bank-conflict free.
// The DMA is issued from inline assembly (wave-uniform 64-bit base +
// per-lane 32-bit offset) and waited for with explicit vmcnt counts: the
// compiler cannot see that a DMA into one stage does not alias the reads of
// another, and would otherwise wait for every outstanding DMA before each LDS
// read.
#include "tile_common.h"

#include <type_traits>

namespace hdl {
namespace {

using namespace tile;

// t of a state, moved from its own max m to a larger max mn:
//   sum exp(z - mn) * (z - mn) log2(e) = f * (t + (m - mn) log2(e) * s),  f = exp(m - mn).
// An empty state (m = -inf, s = t = 0) stays 0.
__device__ __forceinline__ float shift_t(float t, float s, float m, float mn, float f) {
  return (m == mn) ? t : (m == kNegInf ? 0.f : f * __builtin_fmaf((m - mn) * kLog2e, s, t));
}

// Combine two (max m, sum of exp(z - m) s, captured logit z, and for the
// entropy t = sum exp(z - m) * (z - m) log2(e)) states.  t is only
// meaningful when entropy is requested; otherwise it stays 0 and the
// compiler drops it.  t is kept relative to m so that the entropy
// ln s - ln(2) t / s is a sum of two non-negative terms: no cancellation
// against the size of the logits.
__device__ __forceinline__ void combine(float& m, float& s, float& z, float& t, float m2, float s2,
                                        float z2, float t2) {
  const float mn = fmaxf(m, m2);
  const float fa = (m == mn) ? 1.f : fast_exp2((m - mn) * kLog2e);
  const float fb = (m2 == mn) ? 1.f : fast_exp2((m2 - mn) * kLog2e);
  t = shift_t(t, s, m, mn, fa) + shift_t(t2, s2, m2, mn, fb);
  // (an explicit fma: a contractible s * fa + s2 * fb could be fused
  // differently in different instantiations, and log p must not depend on
  // whether the entropy is requested)
  s = __builtin_fmaf(s, fa, s2 * fb);
  m = mn;
  z = fmaxf(z, z2);
}

// Eight fp32 values as sums of three bf16 values each: the value rounded to
// bf16, the rest rounded to bf16, and what is left, which has at most 8
// significant bits (8 + 8 + 8 with signed rests cover the 24 of an fp32; both
// subtractions are exact).  Exact but for pieces below bf16's smallest
// denormal, 2^-133, which are lost; under kSplitMax on the other side that is
// less than 2^-73 of a logit.  An infinity has no such pieces; a NaN stays NaN.
struct Split3 {
  bf16x8_t p[3];
};
constexpr float kSplitMax = 0x1p60f;

__device__ __forceinline__ Split3 split3(const uint4 (&x)[2]) {
  uint32_t u[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint4& q = x[i / 2];
    f32x2_t v = {__uint_as_float(i % 2 ? q.z : q.x), __uint_as_float(i % 2 ? q.w : q.y)};
#pragma unroll
    for (int o = 0; o < 3; ++o) {
      u[o][i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
      v[0] -= __uint_as_float(u[o][i] << 16);
      v[1] -= __uint_as_float(u[o][i] & 0xffff0000u);
    }
  }
  Split3 s;
#pragma unroll
  for (int o = 0; o < 3; ++o) s.p[o] = __builtin_bit_cast(bf16x8_t, make_uint4(u[o][0], u[o][1], u[o][2], u[o][3]));
  return s;
}

// Product o of the six that the split keeps (slice_f32), the smallest first.
__device__ __forceinline__ void mul_piece(int o, const Split3& a, const Split3& b, f32x4_t& acc) {
  constexpr int kA[6] = {1, 2, 0, 1, 0, 0}, kB[6] = {1, 0, 2, 0, 1, 0};
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[kA[o]], b.p[kB[o]], acc, 0, 0, 0);
}

// The largest |x| of the eight values and m (quiet NaNs are passed over).
// (v_max3_f32 itself: fmaxf would first canonicalise every operand)
__device__ __forceinline__ float max_abs(const uint4 (&x)[2], float m) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(x[i].x), "v"(x[i].y));
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(x[i].z), "v"(x[i].w));
  }
  return m;
}

// The largest m of the four lanes l, l xor 16, l xor 32, l xor 48 (the lane
// groups of one row).
__device__ __forceinline__ float max_groups(float m) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

static_assert(kKSteps == 2, "a K-slice is two K-steps");
static_assert(kVB % 2 == 0, "the gradient epilogue pairs vocabulary blocks");

// KTAIL: d is not a multiple of the K-slice, so part of every row's last slice
// is masked out (a separate instantiation keeps that work out of the common
// case).  The tail slice runs the same schedule as the others (its W
// chunks are cleared between two waits that every slice has anyway; with two
// more barriers per row and the next slice's DMAs issued in one go, 8,192
// rows at d = 2056, V = 151,936 took 4925 us, now 4836).  EPI selects what each V-tile's logits feed:
//   kEpiStats:   online max / sum of exp and the sampled-token logit;
//   kEpiEntropy: the same plus sum exp(z - m) * (z - m) for the next-token
//                entropy H = ln s - E_p[z - m] (the Entropy localization
//                baseline);
//   kEpiGrad:    the gradient of log p with respect to the logits,
//                g (1[v == y] - exp(z - lse)), written as bf16 (backward pass;
//                lse comes from the forward pass), chunk-major (8 vocabulary
//                entries of a row, then the same 8 of the next row), with
//                zero rows up to the next multiple of 64 rows so that a
//                contraction over rows can run in whole 64-row K-slices.
constexpr int kEpiStats = 0, kEpiEntropy = 1, kEpiGrad = 2;

// Row tiles are 64 TB token rows: TB = 4 (kTileN) for whole tiles, 1 or 2 where
// no more rows are left or where the chip would idle otherwise (item_grid in
// plan.h).  The eight waves keep their split of the vocabulary (2 x 128 rows)
// and share the tokens, 16 TB each, so a row's result has the same bits in
// any of them.  A narrow tile does little matrix work per K-slice and waits
// for the slice's 32 KB of W, so it keeps more slices in flight: 4 stages of
// 32 + 8 KB (TB = 1), 3 of 32 + 16 KB (TB = 2), 2 of 32 + 32 KB (TB = 4).
// Whole calls at V = 151,936, whole tiles only -> with narrow ones: 16 rows,
// d 2048 198 -> 165 us; 96 rows 216 -> 183 (W alone, 622 MB, takes 123 us at
// the 5.05 TB/s a copy reaches); 64 rows, d 4096 378 -> 307; 512 fp32 rows x
// 4,096 words (32 items on 256 CUs before) 85 -> 40.
template <int TB>
struct Ring {
  static constexpr int kStages = TB == 1 ? 4 : TB == 2 ? 3 : 2;
  static constexpr int kRowsN = 64 * TB;                      // token rows of the tile
  static constexpr int kStageSlots = kSlots + kRowsN * kChunks;
  static constexpr int kBlocksH = TB;                         // hidden-state DMA blocks per wave
  static constexpr int kDma = kBlocksPerWave + kBlocksH;      // DMA instructions per lane per slice
  static_assert(kDma * (kStages - 1) <= 63, "vmcnt range");
};
constexpr int kLdsSlots = 10240;   // 160 KB
static_assert(Ring<1>::kStages * Ring<1>::kStageSlots <= kLdsSlots && Ring<2>::kStages * Ring<2>::kStageSlots <= kLdsSlots &&
                  Ring<4>::kStages * Ring<4>::kStageSlots <= kLdsSlots,
              "LDS ring exceeds 160 KB");

// One work item: scored rows row0 .. row0 + 64 TB - 1 (of n_s) x chunk ch.
template <bool BF16, bool KTAIL, int EPI, int TB>
__device__ __forceinline__ void run_item(const LmheadArgs& p, int64_t row0, int64_t ch, int64_t n_s, uint4* lds) {
  constexpr bool ENT = EPI == kEpiEntropy;
  constexpr bool GRAD = EPI == kEpiGrad;
  using R = Ring<TB>;
  constexpr int kEsz = BF16 ? 2 : 4;
  constexpr int kElemsPer16B = 16 / kEsz;
  constexpr int kSliceK = kElemsPer16B * kChunks;   // K elements per slice
  constexpr int kWaveRows = 16 * TB;                // token rows per wave

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int wm = wave & 1;      // which 128 vocabulary rows of the tile
  const int wn = wave >> 1;     // which kWaveRows token rows of the tile
  const int r16 = lane & 15;    // row of a 16-row fragment / column of a result block
  const int grp = lane >> 4;    // lane group: K chunk of a fragment, row quad of a result block
  const int64_t n_s_pad = (n_s + 63) / 64 * 64;   // gradient mode: rows written (row_cap % 64 == 0)

  // (32-bit: a 64-bit minimum would leave these wave-uniform values, and the
  // loop's branches on them, on the vector ALU; V < 2^31)
  const int vt0 = static_cast<int>(ch * p.tpc);
  const int vt1 = vt0 + static_cast<int>(p.tpc) < static_cast<int>(p.n_vt) ? vt0 + static_cast<int>(p.tpc)
                                                                            : static_cast<int>(p.n_vt);
  const int nk = static_cast<int>((p.d + kSliceK - 1) / kSliceK);
  const int n_iter = (vt1 - vt0) * nk;
  const int64_t d = p.d;
  const int64_t V = p.vocab;

  const char* __restrict__ wbase = static_cast<const char*>(p.w);
  const char* __restrict__ hbase = static_cast<const char*>(p.hidden);

  // ---- this lane's token columns and their sampled tokens ------------------
  int tok[TB];
  float g_lse[TB], g_up[TB];   // gradient mode: lse * log2(e) and upstream gradient
#pragma unroll
  for (int bn = 0; bn < TB; ++bn) {
    int64_t e = row0 + wn * kWaveRows + bn * 16 + r16;
    e = e < n_s ? e : n_s - 1;
    const int row = p.rows[e];
    tok[bn] = p.tokens[row];
    if (GRAD) {
      // no indicator term for a token outside [0, V): padding columns of G stay 0
      tok[bn] = (tok[bn] >= 0 && tok[bn] < V) ? tok[bn] : -1;
      g_lse[bn] = p.lse_in[row] * kLog2e;
      g_up[bn] = p.grad_in[row];
    }
  }

  float run_m[TB], run_s[TB], run_z[TB], run_t[TB];
#pragma unroll
  for (int bn = 0; bn < TB; ++bn) { run_m[bn] = kNegInf; run_s[bn] = 0.f; run_z[bn] = kNegInf; run_t[bn] = 0.f; }

  f32x4_t acc[kVB][TB];
#pragma unroll
  for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
    for (int bn = 0; bn < TB; ++bn)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[bm][bn][q] = 0.f;

  // ---- direct global -> LDS loads -----------------------------------------
  // A K-slice of one operand tile is made of 1 KB blocks of kBlockRows rows.
  // Wave w fetches blocks w*kBlocksPerWave ..; within a block lane l lands in
  // LDS slot l, i.e. row l/kChunks and physical chunk l%kChunks, so it
  // fetches the logical chunk that the read swizzle maps there.
  const int lrow = lane / kChunks;
  // logical chunk this lane fetches for DMA block `block` of a tile
  auto dma_chunk = [&](int block) { return (lane % kChunks) ^ row_xor(block * kBlockRows + lrow); };
  // (KTAIL, rows shorter than a slice: no offset points past the row)
  const int row_chunks = static_cast<int>(d * kEsz / 16);
  auto fetch_chunk = [&](int block) {
    return KTAIL && dma_chunk(block) >= row_chunks ? 0 : dma_chunk(block);
  };
  const int64_t row_bytes = d * kEsz;
  // Per-lane byte offsets (row start + 16-byte chunk) of this wave's DMA
  // blocks; a launch never spans more than 4 GiB of hidden states, and W is
  // addressed from the current V-tile's first row.
  uint32_t hoff[R::kBlocksH];
#pragma unroll
  for (int i = 0; i < R::kBlocksH; ++i) {
    int64_t e = row0 + (wave * R::kBlocksH + i) * kBlockRows + lrow;
    e = e < n_s ? e : n_s - 1;
    hoff[i] = static_cast<uint32_t>(static_cast<int64_t>(p.rows[e]) * row_bytes + fetch_chunk(wave * R::kBlocksH + i) * 16);
  }
  uint32_t woff[kBlocksPerWave];
  uint64_t wtile = 0;   // address of the current V-tile's first row (uniform)
  auto set_w = [&](int vt) {
    wtile = uniform64(reinterpret_cast<uint64_t>(wbase) + static_cast<uint64_t>(int64_t{vt} * kTileV * row_bytes));
    const int last = static_cast<int>(V - 1 - int64_t{vt} * kTileV);   // (rows past V fetch row V - 1)
#pragma unroll
    for (int i = 0; i < kBlocksPerWave; ++i) {
      const int v = (wave * kBlocksPerWave + i) * kBlockRows + lrow;
      woff[i] = static_cast<uint32_t>(v < last ? v : last) * static_cast<uint32_t>(row_bytes) +
                static_cast<uint32_t>(fetch_chunk(wave * kBlocksPerWave + i) * 16);
    }
  };
  const uint32_t lds_base = static_cast<uint32_t>(
      reinterpret_cast<size_t>((__attribute__((address_space(3))) uint4*)lds));
  auto lds_addr = [&](int stage, int op, int block) -> uint32_t {
    return __builtin_amdgcn_readfirstlane(
        lds_base + static_cast<uint32_t>((stage * R::kStageSlots + op * kSlots + block * 64) * 16));
  };
  // DMA j (0 .. R::kDma-1) of a K-slice; j < kBlocksPerWave are W blocks,
  // the rest hidden-state blocks, of the slice prep_issue() moved to.  The last
  // K-slice of rows whose length is no multiple of the slice (KTAIL) is the
  // row's last 128 bytes, so that it needs no addresses of its own; the chunks
  // that the slice before it holds as well are cleared by clear_w_tail().
  uint32_t issue_kbytes = 0;
  int issue_stage = R::kStages - 1;
  // next_issue() moves on to the next slice and ring stage (scalar work only,
  // placed early in the slice before it: counters and one branch instead of a
  // division per slice after the barrier, 1 % at 16,384 rows, d 4096); set_issue() then updates the lanes'
  // offsets where that slice starts another V-tile.  Past the work item's last
  // slice the offsets stay on one line of it, so what is fetched then (into
  // stages nothing reads any more) costs next to nothing.
  int issue_kt = -1, issue_left = n_iter;
  int issue_vt = vt0;
  auto next_stage = [](int st) { return st + 1 == R::kStages ? 0 : st + 1; };
  auto next_issue = [&]() {
    issue_stage = next_stage(issue_stage);
    const bool wrap = ++issue_kt == nk;
    issue_kt = wrap ? 0 : issue_kt;
    issue_vt += wrap ? 1 : 0;
    issue_kbytes = static_cast<uint32_t>(issue_kt) * kSliceK * kEsz;
    if (KTAIL) {
      const uint32_t tail = static_cast<uint32_t>(row_bytes) - kSliceK * kEsz;
      issue_kbytes = issue_kt > 0 && issue_kt == nk - 1 ? tail : issue_kbytes;
    }
    --issue_left;
  };
  auto set_issue = [&]() {
    if (issue_kt != 0) return;
    if (issue_left >= 0) {
      set_w(issue_vt);
    } else {   // (empty asm: keeps the two branches' stores apart)
#pragma unroll
      for (int i = 0; i < kBlocksPerWave; ++i) asm volatile("v_mov_b32 %0, 0" : "=v"(woff[i]));
#pragma unroll
      for (int i = 0; i < R::kBlocksH; ++i) asm volatile("v_mov_b32 %0, 0" : "=v"(hoff[i]));
    }
  };
  auto issue_one = [&](auto j_tag) {
    constexpr int j = decltype(j_tag)::value;
    if constexpr (j < kBlocksPerWave) {
      dma16(wtile + issue_kbytes, woff[j], lds_addr(issue_stage, 0, wave * kBlocksPerWave + j));
    } else {
      constexpr int i = j - kBlocksPerWave;
      dma16(reinterpret_cast<uint64_t>(hbase) + issue_kbytes, hoff[i], lds_addr(issue_stage, 1, wave * R::kBlocksH + i));
    }
  };

  // KTAIL: clears, in a landed last K-slice, the chunks that belong to the
  // slice before it (or, in rows shorter than a slice, to none).  Each wave
  // clears what it fetched itself, between its DMA wait and the barrier that
  // every slice has anyway.  Clearing W is enough: the hidden chunks that meet
  // the zeros are the same row's own, so an infinity or NaN in them has made
  // the row's results NaN already.  (W and not the hidden states: an infinite
  // weight must reach its own vocabulary entry only.)
  auto clear_w_tail = [&](int stage) {
#pragma unroll
    for (int i = 0; i < kBlocksPerWave; ++i) {
      const int c = dma_chunk(wave * kBlocksPerWave + i);
      if (nk == 1 ? c >= row_chunks : c < nk * kChunks - row_chunks)
        lds[stage * R::kStageSlots + (wave * kBlocksPerWave + i) * 64 + lane] = make_uint4(0, 0, 0, 0);
    }
  };

  // ---- fragment reads ------------------------------------------------------
  // Fragments start at multiples of 16 rows, so a fragment row's swizzle is
  // that of (lane mod 16): one per-lane offset per K-step, plus immediates.
  // Lane group g reads chunk 4 ks + frag_chunk(g) of the K-step (A and B
  // alike, so the K positions pair up).
  const int kchunk = frag_chunk(grp);
  const int frag_lane[kKSteps] = {(r16 * kChunks + ((0 + kchunk) ^ row_xor(r16))),
                                  (r16 * kChunks + ((4 + kchunk) ^ row_xor(r16)))};
  // the two W fragments (vocabulary blocks 2 pr, 2 pr + 1) of quarter pr of K-step ks
  auto load_a = [&](int stage, int ks, int pr, uint4 (&dst)[2]) {
    const uint4* base = &lds[stage * R::kStageSlots + frag_lane[ks]];
#pragma unroll
    for (int j = 0; j < 2; ++j) dst[j] = base[(wm * 128 + (2 * pr + j) * 16) * kChunks];
  };
  // hidden-state fragment of token block bn, K-step ks
  auto load_b = [&](int stage, int ks, int bn, uint4& dst) {
    dst = lds[stage * R::kStageSlots + kSlots + frag_lane[ks] + (wn * kWaveRows + bn * 16) * kChunks];
  };
  // the 2 x TB MFMAs of quarter pr
  auto quarter_mfma = [&](const uint4 (&a)[2], const uint4 (&b)[TB], int pr) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < TB; ++i) Mma16<true>::run(a[j], b[snake<TB>(j, i)], acc[2 * pr + j][snake<TB>(j, i)]);
  };

  // Online max / sum-of-exp update of one V-tile, then capture of the
  // sampled token's logit if this lane holds it.  MASKED: the tile runs past
  // the end of the vocabulary and rows >= V are excluded.
  auto epilogue = [&](int64_t vt, auto masked_tag) {
    constexpr bool kMasked = decltype(masked_tag)::value;
    const int64_t vbase = int64_t{vt} * kTileV + wm * 128;   // first vocab row of this wave
    const int64_t vlane = vbase + 4 * grp;          // + 16 bm + i: this lane's rows
#pragma unroll
    for (int bn = 0; bn < TB; ++bn) {
      if (kMasked) {
#pragma unroll
        for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (vlane + bm * 16 + q >= V) acc[bm][bn][q] = kNegInf;
      }
      float mx = acc[0][bn][0];
#pragma unroll
      for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
        for (int q = 0; q < 4; ++q) mx = fmaxf(mx, acc[bm][bn][q]);
      const float mnew = fmaxf(run_m[bn], mx);
      if (!kMasked || mnew != kNegInf) {
        const float mb = mnew * kLog2e;
        float s4[4], t4[4];
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          float sacc = 0.f, tacc = 0.f;
#pragma unroll
          for (int bm = 2 * g4; bm < 2 * g4 + 2; ++bm)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float zq = acc[bm][bn][q];
              const float zl = __builtin_fmaf(zq, kLog2e, -mb);   // (z - m) log2(e)
              const float e = fast_exp2(zl);
              sacc += e;
              // (masked rows hold -inf and e = 0; their product term is 0)
              if (ENT) tacc = __builtin_fmaf(e, (kMasked && zq == kNegInf) ? 0.f : zl, tacc);
            }
          s4[g4] = sacc;
          t4[g4] = tacc;
        }
        const float tile_sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        const float rescale = fast_exp2(__builtin_fmaf(run_m[bn], kLog2e, -mb));
        if (ENT)   // (before run_s changes: shift_t wants the old sum)
          run_t[bn] = shift_t(run_t[bn], run_s[bn], run_m[bn], mnew, rescale) + ((t4[0] + t4[1]) + (t4[2] + t4[3]));
        run_s[bn] = __builtin_fmaf(run_s[bn], rescale, tile_sum);
        run_m[bn] = mnew;
      }
      const int64_t o = static_cast<int64_t>(tok[bn]) - vbase;
      if (o >= 0 && o < 128 && ((static_cast<int>(o) >> 2) & 3) == grp) {
        const int code = (static_cast<int>(o) >> 4) * 4 + (static_cast<int>(o) & 3);   // 4 bm + i
        float zc = kNegInf;
#pragma unroll
        for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (code == bm * 4 + q) zc = acc[bm][bn][q];
        run_z[bn] = zc;
      }
    }
#pragma unroll
    for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
      for (int bn = 0; bn < TB; ++bn)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[bm][bn][q] = 0.f;
  };

  // Gradient mode: G = g (1[v == y] - p) for the kVB x TB blocks of this
  // wave, rounded to bf16.  In each block a lane holds 4 consecutive
  // vocabulary entries of its token row: half of an 8-entry chunk (lane
  // groups 0 and 1 hold the two halves of one chunk, groups 2 and 3 those of
  // the next).  Blocks are taken in pairs: v_permlane16_swap_b32 trades the
  // odd lane groups' halves of the first block for the even groups' halves
  // of the second, so that every lane then holds one whole chunk, chunk
  // frag_chunk(g) of the pair's four, and stores it with one 16-byte store
  // (stores of 8 bytes per lane drained about 1.6 times slower: all work
  // items reach this epilogue together, and the next K-slice's DMA wait
  // also waits for these stores).  G is stored chunk-major, so a store
  // instruction covers four runs of 256 contiguous bytes (16 token rows x one
  // chunk each).  Rows >= V hold -inf, so p = 0 and G = 0 there, which
  // zero-fills the columns up to g_cols.
  auto grad_epilogue = [&](int vt) {
    const int vbase = vt * kTileV + wm * 128;   // V < 2^31
    // G's address: uniform up to the pair of blocks, plus this byte offset
    // (64-bit addresses per token column made the kernel spill); g_ld is at
    // most one chunk's rows, so it stays far below 4 GiB
    const uint32_t lane_off =
        static_cast<uint32_t>(frag_chunk(grp) * p.g_ld + row0 + wn * kWaveRows + r16) * 16u;
#pragma unroll
    for (int bn = 0; bn < TB; ++bn) {
      const int64_t e = row0 + wn * kWaveRows + bn * 16 + r16;
      const bool live = e < n_s;   // rows n_s .. round_up(n_s, 64) - 1 are written as zeros
      const float gneg = -g_up[bn];
      // The sampled token's column gets g (1 - p), computed as g - g p (one
      // rounding); `code` is its place 4 bm + q among this lane's elements of
      // the column, -1 if the lane does not hold it.
      const int o = tok[bn] - vbase;
      const int code = (o >= 0 && o < 128 && ((o >> 2) & 3) == grp) ? (o >> 4) * 4 + (o & 3) : -1;
#pragma unroll
      for (int bp = 0; bp < kVB; bp += 2) {
        uint32_t pk[2][2];   // [block of the pair][bf16 pair]: entries v0 .. v0 + 3
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int bm = bp + h;
          float gv[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float pv = fast_exp2(__builtin_fmaf(acc[bm][bn][q], kLog2e, -g_lse[bn]));
            gv[q] = __builtin_fmaf(gneg, pv, code == bm * 4 + q ? g_up[bn] : 0.f);
          }
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{gv[r], gv[r + 1]}, bf16x2_t));
            pk[h][r / 2] = live ? w : 0u;
          }
        }
        // even lane groups keep their first-block half and receive the
        // partner's (the chunk's upper half); odd groups receive the
        // partner's second-block half (the lower half) and keep their own
        const auto s0 = __builtin_amdgcn_permlane16_swap(pk[0][0], pk[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(pk[0][1], pk[1][1], false, false);
        char* pair = reinterpret_cast<char*>(p.g_out) + static_cast<int64_t>((vbase + bp * 16) / 8) * p.g_ld * 16;
        // (the pair's 32 columns lie wholly below g_cols, a multiple of 64, or
        // wholly above).  Non-temporal: G is read back only by the two GEMMs,
        // long after it has left the L2, and these write-backs would
        // otherwise evict the tiles the next K-slices' DMAs read.
        if (e < n_s_pad && vbase + bp * 16 < p.g_cols)
          __builtin_nontemporal_store(u32x4_t{s0[0], s1[0], s0[1], s1[1]},
                                      reinterpret_cast<u32x4_t*>(pair + (lane_off + bn * 256)));
      }
    }
#pragma unroll
    for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
      for (int bn = 0; bn < TB; ++bn)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[bm][bn][q] = 0.f;
  };

  // ---- pipelined main loop over (V-tile, K-slice) ------------------------
  // A K-slice is 2 K-steps x 4 quarters; quarter pr multiplies the W
  // fragments of vocabulary blocks 2 pr, 2 pr + 1 with the TB hidden-state
  // fragments.  Each quarter first reads what the next one needs: the next
  // quarter's two W fragments (alternating buffers fa[0], fa[1]) and, during
  // K-step 0, one hidden-state fragment of K-step 1 (fb[1]).  The slice's
  // last quarter waits for the next slice's DMA and the workgroup barrier,
  // reads the next slice's first W fragments and all of its K-step-0 hidden
  // fragments (fb[0]), and issues the DMAs of the slice kStages on into the
  // stage just released, beside its first MFMAs.
  const int n_pre = n_iter < R::kStages ? n_iter : R::kStages;
  for (int sl = 0; sl < n_pre; ++sl) {
    next_issue();
    set_issue();
    unroll<R::kDma>(issue_one);
  }
  if (n_pre == R::kStages) wait_vmcnt<(R::kStages - 1) * R::kDma>();
  else wait_vmcnt<0>();
  if (n_pre < R::kStages) issue_stage = R::kStages - 1;   // (slot kStages takes stage 0)
  if (KTAIL && nk == 1) clear_w_tail(0);
  raw_barrier();

  uint4 fa[2][2], fb[2][TB];
  // One K-slice, in ring stage st.  next_tail: the slice after it is the last
  // of its rows.
  [[maybe_unused]] auto slice_bf16 = [&](int st, bool next_tail) {
    const int nst = next_stage(st);
    // K-step 0
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) {
      if (pr < 3) load_a(st, 0, pr + 1, fa[(pr + 1) & 1]);
      else load_a(st, 1, 0, fa[0]);
      if (pr < TB) load_b(st, 1, pr, fb[1][pr]);
      // keep the fragment reads for the next quarter ahead of this
      // quarter's MFMAs, so their LDS latency hides under matrix work
      __builtin_amdgcn_sched_barrier(0);
      quarter_mfma(fa[pr & 1], fb[0], pr);
    }
    // K-step 1, quarters 0-2
#pragma unroll
    for (int pr = 0; pr < 3; ++pr) {
      load_a(st, 1, pr + 1, fa[(pr + 1) & 1]);
      if (pr == 0) next_issue();
      __builtin_amdgcn_sched_barrier(0);
      quarter_mfma(fa[pr & 1], fb[1], pr);
    }
    // K-step 1, quarter 3: the slice boundary.  Every read of this slice is
    // issued: wait for the next slice, then recycle this slice's stage.  On
    // the work item's last slice this waits for nothing and the reads of the
    // "next slice" fetch stale (in-bounds, unused) LDS: keeping this path
    // unconditional leaves no control-flow join before the MFMAs.  The DMAs
    // of the slice kStages on are issued with this quarter's MFMAs.
    wait_vmcnt<(R::kStages - 2) * R::kDma>();
    if (KTAIL && next_tail) clear_w_tail(nst);
    raw_barrier();
    set_issue();
    load_a(nst, 0, 0, fa[0]);
#pragma unroll
    for (int bn = 0; bn < TB; ++bn) load_b(nst, 0, bn, fb[0][bn]);
    __builtin_amdgcn_sched_barrier(0);
    unroll<R::kDma>(issue_one);
    quarter_mfma(fa[1], fb[1], 3);
  };
  // One K-slice of fp32 operands.  v_mfma_f32_16x16x4_f32 does 157 TFLOP/s on
  // the whole chip, the bf16 form 16 times that, and an fp32 value is the sum
  // of three bf16 values exactly (split3); so each pair of 16-row fragments is
  // multiplied as the six products of pieces whose orders add up to at most 2,
  // the smallest first.  The second piece is at most 2^-8 of the value's
  // leading power and the third 2^-17, so up to 2^-24 of |w h| is left out of a
  // product (random mantissas: 2^-27 rms), and the bf16 MFMA cuts an
  // accumulator that is smaller than the products to their last place instead
  // of rounding it: a logit that is a single product is within 3 x 2^-24 of
  // itself where the fp32 MFMA is within 2^-24.  In sums, fewer roundings
  // weigh more: six per 32 products.  Distance to the 64-bit logits in
  // 2^-24 of them, rms, all products of one sign, d 8, 32, 128, 256, 512, 1024:
  // fp32 MFMA 0.81, 1.4, 2.7, 3.7, 5.0, 7.2; six products 0.53, 0.52, 1.7,
  // 2.7, 3.9, 5.0; the same to three places with the products second times
  // third piece added, for 18 % more time.  A slice's 32 K values are one
  // K-step of the bf16 MFMA: lane group g holds the chunks frag_chunk(g) and
  // 4 + frag_chunk(g) of W and hidden rows alike.  Pieces are made in
  // registers, where 6 VALU instructions per value run beside the other
  // wave's MFMAs, so HBM and LDS traffic stay those of fp32.  W fragments with
  // a value too large for the split (kSplitMax; an infinite weight would meet
  // the zero pieces of the hidden states) are multiplied by the fp32 MFMA, and
  // so are token rows with one.
  // 2,048 rows, d 1024, V 32,000: 955 -> 682 us (140 -> 197 TFLOP/s of fp32
  // products, 1.18 PFLOP/s of bf16 ones), distance of log p and lse to the
  // 64-bit results 6.1e-8 -> 5.7e-8.  Splitting a block between the MFMAs of
  // the one before it, which 12 more registers allow with a few spills, took
  // 696 us.
  [[maybe_unused]] auto slice_f32 = [&](int st, bool next_tail) {
    const int nst = next_stage(st);
    const uint4* abase = &lds[st * R::kStageSlots + wm * 128 * kChunks];
    const uint4* bbase = &lds[st * R::kStageSlots + kSlots + wn * kWaveRows * kChunks];
    auto load2 = [&](const uint4* base, int block, uint4 (&dst)[2]) {
      dst[0] = base[block * 16 * kChunks + frag_lane[0]];
      dst[1] = base[block * 16 * kChunks + frag_lane[1]];
    };
    // Hidden rows with a value too large for the split.  Which MFMA takes a
    // row's products must not depend on the other rows of the call, whose bits
    // it would change: the split sees zeros in the place of such rows, the fp32
    // MFMA zeros in the place of all others (x + 0 w = x: w is finite there).
    auto zero_rows = [&](uint4 (&b)[2], bool large) {
      // (a row is in the four lanes of one r16)
      if ((max_groups(max_abs(b, 0.f)) >= kSplitMax) == large) b[0] = b[1] = make_uint4(0, 0, 0, 0);
    };
    Split3 sb[TB];
    float bmax = 0.f;
    bool large_rows;
    uint4 ra[2];
    {
      uint4 rb[TB][2];
#pragma unroll
      for (int bn = 0; bn < TB; ++bn) load2(bbase, bn, rb[bn]);
      load2(abase, 0, ra);
      next_issue();
#pragma unroll
      for (int bn = 0; bn < TB; ++bn) bmax = max_abs(rb[bn], bmax);
      large_rows = __any(bmax >= kSplitMax);
      if (__builtin_expect(large_rows, 0)) {
#pragma unroll
        for (int bn = 0; bn < TB; ++bn) zero_rows(rb[bn], true);
      }
#pragma unroll
      for (int bn = 0; bn < TB; ++bn) {
        sb[bn] = split3(rb[bn]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int bm = 0; bm < kVB; ++bm) {
      if (__builtin_expect(__any(max_abs(ra, bmax) >= kSplitMax), 0)) {
        const bool large_w = __any(max_abs(ra, 0.f) >= kSplitMax);
        if (!large_w) {
          const Split3 sa = split3(ra);
#pragma unroll
          for (int bn = 0; bn < TB; ++bn)
#pragma unroll
            for (int o = 0; o < 6; ++o) mul_piece(o, sa, sb[bn], acc[bm][bn]);
        }
        if (large_w || large_rows) {
#pragma unroll
          for (int bn = 0; bn < TB; ++bn) {
            uint4 rb[2];
            load2(bbase, bn, rb);
            if (!large_w) zero_rows(rb, false);
            Mma16<false>::run(ra[0], rb[0], acc[bm][bn]);
            Mma16<false>::run(ra[1], rb[1], acc[bm][bn]);
          }
        }
        if (bm + 1 < kVB) load2(abase, bm + 1, ra);
      } else {
        const Split3 sa = split3(ra);
        if (bm + 1 < kVB) load2(abase, bm + 1, ra);
        __builtin_amdgcn_sched_barrier(0);
        // (the TB accumulators in turn: consecutive MFMAs are independent)
#pragma unroll
        for (int o = 0; o < 6; ++o)
#pragma unroll
          for (int bn = 0; bn < TB; ++bn) mul_piece(o, sa, sb[bn], acc[bm][bn]);
      }
    }
    wait_vmcnt<(R::kStages - 2) * R::kDma>();
    if (KTAIL && next_tail) clear_w_tail(nst);
    raw_barrier();
    set_issue();
    unroll<R::kDma>(issue_one);
  };
  auto slice_step = [&](int st, bool next_tail) {
    if constexpr (BF16) slice_bf16(st, next_tail);
    else slice_f32(st, next_tail);
  };
  int st = 0;   // ring stage of the current slice
  for (int vt = vt0; vt < vt1; ++vt) {
    if constexpr (BF16) {
      load_a(st, 0, 0, fa[0]);
#pragma unroll
      for (int bn = 0; bn < TB; ++bn) load_b(st, 0, bn, fb[0][bn]);
    }
    for (int kt = 0; kt < nk; ++kt) {
      slice_step(st, nk == 1 || kt == nk - 2);
      st = next_stage(st);
    }
    if (GRAD) {
      if ((vt + int64_t{1}) * kTileV > V) {
        // rows >= V: -inf, so that they contribute G = 0
#pragma unroll
        for (int bm = 0; bm < kVB; ++bm)
#pragma unroll
          for (int bn = 0; bn < TB; ++bn)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (int64_t{vt} * kTileV + wm * 128 + bm * 16 + 4 * grp + q >= V) acc[bm][bn][q] = kNegInf;
      }
      grad_epilogue(vt);
    } else if ((vt + int64_t{1}) * kTileV <= V) {
      epilogue(vt, std::false_type{});
    } else {
      epilogue(vt, std::true_type{});
    }
  }
  wait_vmcnt<0>();   // (dummy DMAs past the end may still be landing)
  __syncthreads();
  if (GRAD) return;

  // ---- merge the four lane groups, then the two vocabulary waves ----------
#pragma unroll
  for (int bn = 0; bn < TB; ++bn) {
#pragma unroll
    for (int x = 16; x <= 32; x <<= 1) {
      const float m2 = __shfl_xor(run_m[bn], x);
      const float s2 = __shfl_xor(run_s[bn], x);
      const float z2 = __shfl_xor(run_z[bn], x);
      const float t2 = ENT ? __shfl_xor(run_t[bn], x) : 0.f;
      combine(run_m[bn], run_s[bn], run_z[bn], run_t[bn], m2, s2, z2, t2);
    }
  }
  float* xm = reinterpret_cast<float*>(lds);
  float* xs = xm + R::kRowsN;
  float* xz = xs + R::kRowsN;
  float* xt = xz + R::kRowsN;
  if (wm == 1 && grp == 0) {
#pragma unroll
    for (int bn = 0; bn < TB; ++bn) {
      const int tcol = wn * kWaveRows + bn * 16 + r16;
      xm[tcol] = run_m[bn];
      xs[tcol] = run_s[bn];
      xz[tcol] = run_z[bn];
      if (ENT) xt[tcol] = run_t[bn];
    }
  }
  __syncthreads();
  if (wm == 0 && grp == 0) {
#pragma unroll
    for (int bn = 0; bn < TB; ++bn) {
      const int tcol = wn * kWaveRows + bn * 16 + r16;
      float m = run_m[bn], s = run_s[bn], z = run_z[bn], t = run_t[bn];
      combine(m, s, z, t, xm[tcol], xs[tcol], xz[tcol], ENT ? xt[tcol] : 0.f);
      const int64_t e = row0 + tcol;
      if (e < n_s) {
        const int64_t o = ch * p.part_stride + e;
        p.part_m[o] = m;
        p.part_s[o] = s;
        p.part_z[o] = z;
        if (ENT) p.part_t[o] = t;
      }
    }
  }
}

// Two workgroup waves per SIMD have 256 VGPRs each.  Statistics and entropy take
// 232 to 240 of them in bf16; the fp32 instantiations, whose split hidden rows
// take 48, spill 13 to 21 and the gradient ones 2, all stored before the V-tile
// loop and read back outside the K loop, once per V-tile (after its last slice,
// where a reload also waits for the DMAs in flight) or after the last one.
template <bool BF16, bool KTAIL, int EPI>
__global__ __launch_bounds__(kThreads, 1) void lmhead_logprob_kernel(LmheadArgs p) {
  __shared__ uint4 lds[kLdsSlots];   // a ring of [W | hidden] stages, see Ring

  // ---- work item: XCD-aware (row tile, vocabulary chunk), see plan.h -----
  int64_t n_s = *p.n_scored - p.row_base;
  n_s = n_s < 0 ? 0 : (n_s > p.row_cap ? p.row_cap : n_s);
  const ItemGrid items = item_grid(n_s, p.n_ch, BF16);
  int64_t rt, ch;
  work_item(blockIdx.x, items, &rt, &ch);
  if (rt >= items.n_rt) return;
  // (the divisions run on the vector ALU: back to scalar registers)
  ch = __builtin_amdgcn_readfirstlane(static_cast<int>(ch));
  const int64_t row0 = __builtin_amdgcn_readfirstlane(static_cast<int>(rt * items.rows));
  const int64_t left = __builtin_amdgcn_readfirstlane(static_cast<int>(n_s - row0 < items.rows ? n_s - row0 : items.rows));
  if (left <= Ring<1>::kRowsN) run_item<BF16, KTAIL, EPI, 1>(p, row0, ch, n_s, lds);
  else if (left <= Ring<2>::kRowsN) run_item<BF16, KTAIL, EPI, 2>(p, row0, ch, n_s, lds);
  else run_item<BF16, KTAIL, EPI, 4>(p, row0, ch, n_s, lds);
}

// Combine the chunk partials of each scored row in a fixed order and write
// log p = z_y - (m + ln s); non-finite or out-of-range tokens give NaN.
// With entropy requested (ENT), also H = ln s - E_p[z - m] = ln s - ln(2) t / s.
//
// Few rows come with many chunks (594 of one vocabulary tile each up to 3,500
// rows at V = 151,936) and are bound by the latency of the partials' loads: one
// thread per row walking all of them took 255 us for 96 rows x 594 chunks, 314 us
// for 1,554 x 594, 77 us for 3,333 x 197.  So a workgroup is 32 rows x SEG chunk
// segments: segment s takes chunks s, s + SEG, ... in order, neighbouring rows
// per load, four chunks' loads in flight, and the segments' states are then
// combined in order by the row's first thread: 247 us less for the 96-row call
// (787 -> 540 us), 312 us less for 1,554 rows.  Many rows are bound by memory and
// by the combining: one thread per row (ROWS 256, SEG 1), us against 8 segments:
// 65,024 x 40 11.8 against 8.5, 131,072 x 38 13.2 against 13.2 (with the entropy
// 14.8 against 17.3), 262,144 x 4 7.0 against 9.0, 345,722 x 40 30.2 against 48.1
// (5.5 TB/s).
constexpr int64_t kMergeManyRows = int64_t{1} << 17;

template <int ROWS, int SEG, bool ENT>
__global__ __launch_bounds__(ROWS * SEG) void merge_kernel(LmheadArgs p, float* __restrict__ logp,
                                                                 float* __restrict__ lse_out,
                                                                 float* __restrict__ entropy) {
  __shared__ float xm[SEG][ROWS], xs[SEG][ROWS], xz[SEG][ROWS], xt[ENT ? SEG : 1][ROWS];
  const int r = threadIdx.x % ROWS;
  const int seg = threadIdx.x / ROWS;
  const int64_t n_s = *p.n_scored;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * ROWS + r;
  if (static_cast<int64_t>(blockIdx.x) * ROWS >= n_s) return;   // (the whole workgroup)
  float m = kNegInf, s = 0.f, z = kNegInf, t = 0.f;
  if (e < n_s) {
    constexpr int kBatch = 4;
    for (int64_t c0 = seg; c0 < p.n_ch; c0 += kBatch * SEG) {
      float bm[kBatch], bs[kBatch], bz[kBatch], bt[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int64_t c = c0 + i * SEG;
        const int64_t o = (c < p.n_ch ? c : c0) * p.part_stride + e;
        bm[i] = p.part_m[o];
        bs[i] = p.part_s[o];
        bz[i] = p.part_z[o];
        bt[i] = ENT ? p.part_t[o] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (c0 + i * SEG < p.n_ch) combine(m, s, z, t, bm[i], bs[i], bz[i], bt[i]);
    }
  }
  xm[seg][r] = m;
  xs[seg][r] = s;
  xz[seg][r] = z;
  if (ENT) xt[seg][r] = t;
  __syncthreads();
  if (seg != 0 || e >= n_s) return;
  const int n_seg = p.n_ch < SEG ? static_cast<int>(p.n_ch) : SEG;
  for (int i = 1; i < n_seg; ++i) combine(m, s, z, t, xm[i][r], xs[i][r], xz[i][r], ENT ? xt[i][r] : 0.f);
  // (no logit above -inf, as an infinite hidden state can leave them in one
  // vocabulary tile: NaN like where some are +inf)
  const float lse = m == kNegInf ? __builtin_nanf("") : m + __builtin_amdgcn_logf(s) * 0.6931471805599453f;
  const int row = p.rows[e];
  const int y = p.tokens[row];
  float lp = z - lse;
  // The exact value is <= 0; rounding in the fp32 normaliser can leave a
  // positive residue of a few ulps when one logit dominates.  (Written so
  // that a NaN -- a non-finite hidden state -- stays NaN.)
  lp = lp > 0.f ? 0.f : lp;
  if (y < 0 || y >= p.vocab) lp = __builtin_nanf("");
  logp[row] = lp;
  if (lse_out) lse_out[row] = lse;
  if (ENT) {
    // The exact value is >= 0; clamp the rounding residue of a near one-hot
    // distribution.
    const float h = __builtin_fmaf(-0.6931471805599453f, t / s, __builtin_amdgcn_logf(s) * 0.6931471805599453f);
    entropy[row] = h < 0.f ? 0.f : h;
  }
}

}  // namespace

hipError_t launch_lmhead(const LmheadArgs& a, int64_t grid, bool bf16, hipStream_t stream) {
  if (grid <= 0) return hipSuccess;
  const dim3 g(static_cast<unsigned>(grid)), b(kThreads);
  const bool tail = (a.d % (bf16 ? 8 * kChunks : 4 * kChunks)) != 0;
  const bool ent = a.part_t != nullptr;
  const int which = (bf16 ? 4 : 0) + (tail ? 2 : 0) + (ent ? 1 : 0);
  switch (which) {
    case 0: hipLaunchKernelGGL((lmhead_logprob_kernel<false, false, kEpiStats>), g, b, 0, stream, a); break;
    case 1: hipLaunchKernelGGL((lmhead_logprob_kernel<false, false, kEpiEntropy>), g, b, 0, stream, a); break;
    case 2: hipLaunchKernelGGL((lmhead_logprob_kernel<false, true, kEpiStats>), g, b, 0, stream, a); break;
    case 3: hipLaunchKernelGGL((lmhead_logprob_kernel<false, true, kEpiEntropy>), g, b, 0, stream, a); break;
    case 4: hipLaunchKernelGGL((lmhead_logprob_kernel<true, false, kEpiStats>), g, b, 0, stream, a); break;
    case 5: hipLaunchKernelGGL((lmhead_logprob_kernel<true, false, kEpiEntropy>), g, b, 0, stream, a); break;
    case 6: hipLaunchKernelGGL((lmhead_logprob_kernel<true, true, kEpiStats>), g, b, 0, stream, a); break;
    default: hipLaunchKernelGGL((lmhead_logprob_kernel<true, true, kEpiEntropy>), g, b, 0, stream, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_lmhead_grad(const LmheadArgs& a, int64_t grid, hipStream_t stream) {
  if (grid <= 0) return hipSuccess;
  const dim3 g(static_cast<unsigned>(grid)), b(kThreads);
  if (a.d % (8 * kChunks) != 0)
    hipLaunchKernelGGL((lmhead_logprob_kernel<true, true, kEpiGrad>), g, b, 0, stream, a);
  else
    hipLaunchKernelGGL((lmhead_logprob_kernel<true, false, kEpiGrad>), g, b, 0, stream, a);
  return hipGetLastError();
}

template <int ROWS, int SEG>
static void run_merge(const LmheadArgs& a, int64_t n_rows, float* logp, float* lse, float* entropy,
                      hipStream_t stream) {
  const dim3 g(static_cast<unsigned>(ceil_div(n_rows, ROWS))), b(ROWS * SEG);
  if (entropy) hipLaunchKernelGGL((merge_kernel<ROWS, SEG, true>), g, b, 0, stream, a, logp, lse, entropy);
  else hipLaunchKernelGGL((merge_kernel<ROWS, SEG, false>), g, b, 0, stream, a, logp, lse, entropy);
}

hipError_t launch_merge(const LmheadArgs& a, int64_t n_rows, float* logp, float* lse,
                        float* entropy, hipStream_t stream) {
  if (n_rows <= 0) return hipSuccess;
  // 8 or 32 segments per row.  32 shorten the chain of loads at the cost of more
  // LDS states and more steps for the row's first thread, more so with the
  // entropy's larger states; the line is the same with it, since it decides the
  // order of the sums and log p must not depend on the entropy.  Whole calls at
  // d 64, 8 -> 32 segments, us: 512 rows 14.9 -> 15.8 at 32 chunks, 17.9 -> 18.4
  // at 64, 24.4 -> 23.9 at 96, 26.2 -> 25.0 at 120, 65 -> 55 at 594; 8,192 rows
  // 77.0 -> 77.7 at 64, 111.4 -> 111.6 at 96, 469 -> 466 at 594; with the entropy
  // 512 rows 19.1 -> 22.3 at 64, 27.7 -> 29.8 at 120, 37.7 -> 37.1 at 256, 73 ->
  // 67 at 594.
  if (n_rows >= kMergeManyRows) run_merge<256, 1>(a, n_rows, logp, lse, entropy, stream);
  else if (a.n_ch >= 96) run_merge<32, 32>(a, n_rows, logp, lse, entropy, stream);
  else run_merge<32, 8>(a, n_rows, logp, lse, entropy, stream);
  return hipGetLastError();
}

}  // namespace hdl
