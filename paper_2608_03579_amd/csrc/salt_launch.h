// Host-side choices of an apply: tokens per tile, the tiles of a batch, the K
// split of the shrink and the column blocks of the expand.  Header-only and free
// of HIP calls, so that the runtime and the host-side address checks use the
// same code.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "salt_layout.h"

namespace salt {

// Tokens per tile, from the mean size of the batch's centroid groups: short
// groups (decode batches) take 16-token tiles, groups of up to ~100 tokens 32,
// up to ~400 tokens 64, longer ones (prefill) 128 when there is a centroid
// operand, which each block stages once per tile: the larger the tile, the
// fewer times it is read.  fp32 contexts always use 16.
inline int choose_tile_tokens(int esize, int T, int n_groups, bool centroids) {
  if (esize == 4 || n_groups <= 0) return 16;
  const double mean = (double)T / n_groups;
  if (mean <= 24.0) return 16;
  if (mean <= 96.0) return 32;
  if (mean <= 384.0 || !centroids) return 64;
  return 128;
}

// Tiles of a batch from the token counts of its centroid groups, per_c[c + 1]
// for c = -1 .. C - 1 (the sorted order puts c = -1 first).  A group of n tokens
// becomes k = ceil(n / M) tiles: for tiles of up to 64 tokens of near-equal
// size, the first n mod k of them one token longer; for larger tiles
// k - 1 full tiles and the remainder (the expand of 128-token tiles splits
// its work by column chunks, not by tiles, so their sizes need not match).
// Tiles are contiguous in sorted order and cover [0, T).  rank_c (per_c's
// layout): each group's largest residual rank, which its tiles' headers carry
// (null: 0).
inline void cut_tiles(const std::vector<int>& per_c, int M, std::vector<int4>& tiles,
                      const std::vector<int>* rank_c = nullptr) {
  tiles.clear();
  int start = 0;
  for (size_t g = 0; g < per_c.size(); ++g) {
    const int n = per_c[g];
    if (n <= 0) continue;
    const int k = cdiv(n, M), base = n / k, extra = n % k;
    int p = start;
    for (int i = 0; i < k; ++i) {
      const int len = M > 64 ? imin(M, n - i * M) : base + (i < extra ? 1 : 0);
      int4 t;
      t.x = p;
      t.y = len;
      t.z = (int)g - 1;
      t.w = rank_c ? (*rank_c)[g] : 0;
      tiles.push_back(t);
      p += len;
    }
    start += n;
  }
}

// A staged batch: its three lists of tiles, one behind the other, and what the
// choice of layouts goes by.
struct BatchTiles {
  int M = 16;               // the expand's tiles, of M tokens
  int n_tiles = 0;
  int n_rtiles = 0;         // tiles of 64 tokens for the shrink (0: M <= 64, and they are the expand's)
  int n_wtiles = 0;         // tiles of 16 tokens for k_shrink_wide (0: M is 16, or no rank above 2)
  int pairs = 0, wpairs = 0;   // (shrink tile, residual rank chunk) pairs that hold a rank: 64 / M and 16 tokens
  int64_t ranks8 = 0;       // over the 16-token tiles: their rank bounds, rounded up to passes of 8
  int n_slots = 0;          // distinct slots referenced
  int total() const { return n_tiles + n_rtiles + n_wtiles; }
};

// Cuts a batch (cut_tiles) into `out`, list after list.
inline BatchTiles cut_batch(const std::vector<int>& per_c, const std::vector<int>& rank_c, int M, int r_u,
                            std::vector<int4>& out) {
  BatchTiles b;
  std::vector<int4> rt, wt;
  b.M = M;
  cut_tiles(per_c, M, out, &rank_c);
  b.n_tiles = (int)out.size();
  if (M > 64) cut_tiles(per_c, 64, rt, &rank_c);
  if (M > 16 && r_u > 2) cut_tiles(per_c, 16, wt, &rank_c);
  b.n_rtiles = (int)rt.size();
  b.n_wtiles = (int)wt.size();
  auto pairs = [](const std::vector<int4>& l) {
    int n = 0;
    for (const int4& t : l) n += std::max(1, cdiv(t.w, kRankChunk));
    return n;
  };
  const std::vector<int4>& w = M > 16 ? wt : out;
  b.pairs = pairs(M > 64 ? rt : out);
  b.wpairs = pairs(w);
  for (const int4& t : w) b.ranks8 += 8 * std::max(1, cdiv(t.w, 8));
  out.insert(out.end(), rt.begin(), rt.end());
  out.insert(out.end(), wt.begin(), wt.end());
  return b;
}

// Split-K partial floats a plan of up to T tokens holds (rows of R floats): two
// K ranges per token row for a full launch of kMaxJobs tables, or one if that
// would pass 256 MiB; small batches get up to 16 Mi floats (64 MiB, at most 64
// ranges per table), so that a decode launch can split K finely enough to fill
// the device.
inline size_t plan_partial_cap(size_t T, size_t R) {
  const size_t two = 2 * (size_t)kMaxJobs * T * R;
  const size_t small = std::min((size_t)16 << 20, 64 * (size_t)kMaxJobs * T * R);
  if (two < small) return small;
  return two * 4 <= ((size_t)256 << 20) ? two : (size_t)kMaxJobs * T * R;
}

// Largest number of tiles a batch of T tokens over C centroids can cut into.
inline int max_tiles(int T, int C) { return cdiv(T, 16) + C + 1; }

constexpr double kWorkUnit = 1e-6;   // of the work and rows that the choice of layouts goes by

// Whether the shrink of a batch with residual ranks above 2 runs k_shrink_wide's
// 16-token tiles (quad layout, rows streamed group by group, each tile's own rank
// bound) or k_shrink's, which shares the centroid operand among up to 64 tokens and
// starts sooner.  From shrink times of 529 batches in both (Llama-3.2-3B, 3.1-8B and
// odd shapes, T = 1 .. 8192, ranks 3 .. 72); in units of a million: work, tokens x
// sum of in; rows, distinct residual rows x sum of in.
//  - One rank chunk: k_shrink's (Zipf T = 512, rank 16, 3 tokens a user, r_c = 64:
//    69 us against 84; T = 8192, r_c = 64, rank 4: 290 against 473, rank 16: 437 against
//    650; T = 32 of rank 16, no centroids: 9 against 13), but where the rows
//    themselves are the traffic and little of a centroid operand is shared (no
//    centroids, T = 512 of 205 users, rank 16: 84 against 59; of 55 users: 33 against
//    37; r_c = 16, 380 users of rank 12: 82 against 66), and where few 64-token tiles
//    leave the device short of blocks: up to 48 with much work and a small r_c (T =
//    2048, r_c = 16: 173 against 137; T = 4096: 252 against 246; r_c = 64: 193 against
//    198), up to 8 where tokens share rows (T = 219 of 3 users, rank 16, r_c = 64: 38
//    against 25 with tables of 1024, 43 against 38 of 3072; r_c = 16: 26 / 16, 23 / 32).
//  - Several chunks: k_shrink_wide's where the tiles' bounds differ (a few users on
//    concatenated adapters: Zipf T = 512 108 us against 80; T = 8192 1306 against 966)
//    or cut the last chunk (rank 66: 362 against 323; rank 32: 166 against 202), and
//    the work is worth its start (T = 32: 17.7 against 19.8).
//  - fp32, whose k_shrink stages nothing: k_shrink_wide's without centroids (T = 512,
//    rank 16: 106 us against 73; r_c = 16: 67 against 79; rank 4: 13.5 against 20).
inline bool wide_shrink(const ApplyLaunch& a, const BatchTiles& b, int64_t sum_rank) {
  if (a.r_u <= 2) return false;
  double in = 0;
  for (int j = 0; j < a.n_jobs; ++j) in += kWorkUnit * a.jobs[j].in;
  const double work = a.T * in, rows = (double)sum_rank * in, share = (double)a.T / std::max(1, b.n_slots);
  if (a.esize == 4) return a.r_c == 0 && (a.r_u > 8 ? work >= 0.5 : rows >= 35);
  if (a.nq == 1) {
    if (a.r_c == 0) return work >= 12.5 && rows >= 50;
    if (a.r_c <= 32 && a.M > 16 && share < 4 && rows >= 100) return true;
    if (a.M != 64) return false;
    if (b.n_tiles <= 8 && share >= 4) return a.r_c > 32 ? a.r_u > 8 || work < 4 : a.r_u > 8 && work < 4;
    return a.r_c <= 32 && work >= 12.5 && b.n_tiles <= 48;
  }
  const int n16 = b.n_wtiles ? b.n_wtiles : b.n_tiles;
  if (b.wpairs < n16 * a.nq) return a.r_c <= 64 && work >= (a.M > 16 ? 0.6 : 1.9);
  if (a.r_c == 0) return work >= 12.5;
  return kRankChunk * a.nq - b.ranks8 / n16 >= 8 &&
         (a.r_c <= 32 ? work >= 3.75 : a.r_c <= 64 && a.nq >= 3 && work >= 12.5);
}

// Whether the expand of a batch with residual ranks above 2 runs the quad layout,
// which reads as many rows as the tile's ranks need (by fours) and takes rows from
// memory better, or the row layout, which starts sooner (8 us against 10 of a small
// launch), reads rows by eights with their loads in flight together, and is the
// faster one where many tokens share a row.  From the same batches; work: tokens x
// sum of out.
//  - ranks 3 .. 6: quad (T = 512, rank 4: 49 us against 37; T = 8192: 361 against 294);
//    7, 8: row with centroids where tokens share rows (T = 8192, r_c = 64: 398 against
//    439; T = 512, one a user: 75 against 68), 9 .. 12: quad (513 against 465).
//  - 13 .. 16, where neither reads rows in vain: by how many tokens share one (T =
//    1024, 16 a user: 73 against 83; T = 512, one a user: 129 against 118), but for a
//    few 64-token tiles of little work (T = 219 of 3 users, tables of 1024: 18 against
//    14; of 3072: 29 against 27; T = 380: 34 against 35).
//  - Several chunks: quad where tiles' bounds differ and there is work (Zipf T = 512:
//    120 us against 79; T = 32: 13.8 against 16.2) or few tokens share a row (rank 32,
//    T = 489, one a user: 163 against 142; T = 8192, 32 a user: 849 against 916).
inline bool quad_rows(const ApplyLaunch& a, const BatchTiles& b, int64_t sum_rank) {
  double out = 0;
  for (int j = 0; j < a.n_jobs; ++j) out += kWorkUnit * a.jobs[j].out;
  const double work = a.T * out, share = (double)a.T / std::max(1, b.n_slots);
  if (a.esize == 4) {
    if (a.nq == 1 && a.r_c == 0) return work >= 0.12;
    return work >= 1.9 && (share < 12 || (a.r_u <= 4 && a.r_c <= 32));
  }
  if (a.nq == 1) {
    if (a.r_u <= 6 || (a.r_u <= 8 && a.r_c == 0)) return work >= 0.1;
    if (a.r_u <= 8) return work >= 1 && share < 2;
    if (a.r_u <= 12) return work >= 0.6;
    if (a.r_c == 0) return work >= 0.75 && (b.n_tiles < 8 || sum_rank >= 1.6 * a.T);
    return work >= 0.95 && (share < 12 || (a.M == 64 && b.n_tiles <= 6 && work >= 1.5 && work < 7));
  }
  const int n16 = b.n_wtiles ? b.n_wtiles : b.n_tiles;
  if (b.wpairs < n16 * a.nq) return work >= 1.9 || (work >= 1.1 && share < 4);
  return work >= 1.25 && share < 8;
}

// Sets the layouts of launch `a`, and with them the tiles of its shrink.  a.tiles
// points at the first of the batch's lists.
inline void set_layouts(ApplyLaunch& a, const BatchTiles& b, bool wide, bool quad) {
  a.wide = wide;
  a.quad = quad;
  a.MS = a.wide ? 16 : std::min(a.M, 64);
  const int skip = a.wide && b.n_wtiles ? b.n_tiles + b.n_rtiles : (!a.wide && b.n_rtiles ? b.n_tiles : 0);
  a.stiles = a.tiles + skip;
  a.n_stiles = a.wide && b.n_wtiles ? b.n_wtiles : (!a.wide && b.n_rtiles ? b.n_rtiles : b.n_tiles);
  a.n_pairs = a.wide ? b.wpairs : b.pairs;
  a.uneven = a.r_u > 2 && a.n_pairs > a.n_stiles && a.n_pairs < a.n_stiles * a.nq;
}

// Chooses them.  `a` has its jobs and batch fields, a.tiles among them.
inline void choose_layouts(ApplyLaunch& a, const BatchTiles& b, int64_t sum_rank) {
  a.M = b.M;
  a.n_tiles = b.n_tiles;
  if (a.r_u > 2) set_layouts(a, b, wide_shrink(a, b, sum_rank), quad_rows(a, b, sum_rank));
  else set_layouts(a, b, false, quad_rank1(a.M, a.r_c, a.r_u));
}

// K ranges, expand block-chunks and work offsets of launch `a`, whose jobs (in,
// out, prefix, pointers) and batch fields (T, M, n_tiles, MS, n_stiles, C, r_c, r_u, nq, R,
// esize, partial_cap) are set.  n_groups_c: centroids the batch references;
// sum_rank: residual ranks summed over the slots it references (both for the
// byte counts that bound the partial traffic).  Returns false if the partials
// of a one-range shrink do not fit.
// shrink_round: shrink blocks one round of the device holds at once (0: unknown).
inline bool configure_launch(ApplyLaunch& a, int n_cu, int n_groups_c, int64_t sum_rank, int shrink_round = 0) {
  const int KW = waves_of(a.MS) / (a.MS / 16), CW = waves_of(a.M) / (a.M / 16);
  // blocks per launch: a few rounds of the whole device; half as many, twice as
  // long, where every block has one chunk of rows above rank 2 to stream (Zipf
  // T = 512, rank-16 LoRA: 73 -> 63 us; with chunks of uneven tiles 136 -> 140 us)
  const bool rows_only = a.wide && a.n_pairs == a.n_stiles;
  const int target = (rows_only ? 4 : 8) * std::max(1, n_cu);
  const double es = (double)a.esize;
  const double adapters = (double)n_groups_c * a.r_c + (double)sum_rank;
  int64_t sum_in = 0;
  for (int j = 0; j < a.n_jobs; ++j) sum_in += a.jobs[j].in;
  // shrink: one K-range length for the whole launch, so that blocks of every
  // table carry about the same work, sized for ~target blocks; each table's
  // split is capped so that its partials (written, then read) stay within a
  // tenth of its bytes
  const int gran = (a.wide ? kQuadStep : kStepK) * KW;
  const double pairs = a.n_pairs > 0 ? (double)a.n_pairs : (double)shrink_tiles(a) * a.nq;
  const int kc_target = std::max(gran, cdiv((int)std::ceil((double)sum_in * pairs / target), gran) * gran);
  const double part_row = 8.0 * a.T * a.R;        // bytes of one K range's partials, written and read
  std::vector<int> S(a.n_jobs), s_cap(a.n_jobs);
  for (int j = 0; j < a.n_jobs; ++j) {
    const Job& jb = a.jobs[j];
    const double bytes = es * ((double)a.T * (jb.in + 2.0 * jb.out) + adapters * (jb.in + jb.out));
    const int s_traffic = std::max(1, (int)(0.1 * bytes / part_row));
    s_cap[j] = std::max(1, std::min(s_traffic, cdiv(jb.in, gran)));
    S[j] = std::max(1, std::min(cdiv(jb.in, kc_target), s_cap[j]));
  }
  // Shrink tiles of 64 tokens (long groups, many tokens).  If one K range as
  // long as the smallest table's K already gives a round of the device's
  // blocks, K is split no finer: tables with more K take ranges of about that
  // length (blocks of equal length), and a finer split would only add partials
  // for the expand to sum.  Otherwise each block is long, so a round of the
  // device that is only partly filled costs real time: the K-range length is
  // then the one that minimises (rounds of blocks) x (the longest range); ties
  // go to the longer length (fewer partials).
  bool fills = false;
  if (a.MS >= 64 && shrink_round > 0) {
    int min_in = a.jobs[0].in;
    for (int j = 1; j < a.n_jobs; ++j) min_in = std::min(min_in, a.jobs[j].in);
    const int kc = cdiv(min_in, gran) * gran;
    int64_t blocks = 0;
    std::vector<int> Sm(a.n_jobs);
    for (int j = 0; j < a.n_jobs; ++j) {
      Sm[j] = std::max(1, std::min(cdiv(a.jobs[j].in, kc), s_cap[j]));
      blocks += (int64_t)shrink_tiles(a) * a.nq * Sm[j];
    }
    if (blocks >= shrink_round) {
      S = Sm;
      fills = true;
    }
  }
  if (a.MS >= 64 && shrink_round > 0 && !fills) {
    int max_in = 0;
    for (int j = 0; j < a.n_jobs; ++j) max_in = std::max(max_in, a.jobs[j].in);
    double best = 0.0;
    for (int kc = gran; kc < max_in + gran; kc += gran) {
      int64_t blocks = 0;
      int longest = 0;
      for (int j = 0; j < a.n_jobs; ++j) {
        const int sj = std::max(1, std::min(cdiv(a.jobs[j].in, kc), s_cap[j]));
        blocks += (int64_t)shrink_tiles(a) * a.nq * sj;
        longest = std::max(longest, cdiv(cdiv(a.jobs[j].in, sj), gran) * gran);
      }
      const double est = (double)((blocks + shrink_round - 1) / shrink_round) * longest;
      if (best == 0.0 || est <= best) {
        best = est;
        for (int j = 0; j < a.n_jobs; ++j) S[j] = std::max(1, std::min(cdiv(a.jobs[j].in, kc), s_cap[j]));
      }
    }
  }
  // partials must fit, and each table's region stays below kMaxBufferBytes:
  // shrink the largest split until they do
  auto total = [&]() {
    int64_t t = 0;
    for (int j = 0; j < a.n_jobs; ++j) t += (int64_t)S[j] * a.T * a.R;
    return t;
  };
  auto too_big = [&]() {
    for (int j = 0; j < a.n_jobs; ++j)
      if ((int64_t)S[j] * a.T * a.R * 4 >= kMaxBufferBytes) return true;
    return false;
  };
  while (total() > a.partial_cap || too_big()) {
    int jm = 0;
    for (int j = 1; j < a.n_jobs; ++j)
      if (S[j] > S[jm]) jm = j;
    if (S[jm] == 1) return false;
    S[jm] = (S[jm] + 1) / 2;
  }
  int64_t poff = 0;
  int sb = 0, eb = 0;
  for (int j = 0; j < a.n_jobs; ++j) {
    Job& jb = a.jobs[j];
    jb.Kc = cdiv(cdiv(jb.in, S[j]), gran) * gran;
    jb.S = cdiv(jb.in, jb.Kc);
    jb.poff = poff;
    poff += (int64_t)jb.S * a.T * a.R;
    // expand: work items of one block-chunk (kChunkCols per wave along the
    // columns); the launch splits them evenly over one round of blocks
    jb.cpb = (a.quad ? kQuadCols : kChunkCols) * CW;
    jb.n_col = cdiv(jb.out, jb.cpb);
    jb.shrink_base = a.shrink_base[j] = sb;
    jb.expand_base = a.expand_base[j] = eb;
    sb += shrink_tiles(a) * jb.S * a.nq;
    eb += a.n_tiles * jb.n_col;
  }
  for (int j = a.n_jobs; j < kMaxJobs; ++j) a.shrink_base[j] = a.expand_base[j] = INT32_MAX;
  a.shrink_blocks = sb;
  a.expand_items = eb;
  return true;
}

}  // namespace salt
