// Launch records and index arithmetic of the apply kernels, shared by the HIP
// kernels and by host code (the runtime that fills the records, and a plain
// C++ build of this header that walks every block of a launch and checks each
// address against its buffer).  No HIP types: it compiles with g++ as well.
//
// Every global address an apply kernel forms is `base + offset`, with the
// offset computed here from indices that are first clamped into the range of
// their buffer (token < T, slot < n_slots, rank < rank of the slot, column <
// out, k < in, sorted position < T).  A value read from device memory (a token
// record, a tile header) can therefore never move an access outside the
// allocation it belongs to, whatever it holds.
#pragma once

#include <stddef.h>
#include <stdint.h>

// SALT_HOST_ONLY: a plain C++ build (no HIP headers) for host-side checks.
#if defined(SALT_HOST_ONLY)
#define SALT_HD inline
struct int4 {
  int x, y, z, w;
};
#else
#include <hip/hip_runtime.h>
#define SALT_HD __host__ __device__ __forceinline__
#endif

namespace salt {

// ---- fixed shapes -----------------------------------------------------------
constexpr int kWaves = 4;            // waves of an apply block for tiles of up to 32 tokens
constexpr int kStepK = 64;           // k elements one wave takes per shrink step
constexpr int kChunkCols = 64;       // output columns one wave takes per expand chunk
constexpr int kQuadStep = 128;       // the same in the quad layout (lane layouts, below)
constexpr int kQuadCols = 128;
constexpr int kMaxJobs = 16;         // tables one apply launch serves
constexpr int kRankChunk = 16;       // residual ranks one shrink block accumulates
constexpr int kMaxRc = 128;          // largest centroid rank
constexpr int kMaxRu = 72;           // largest residual rank (long-tail concatenated adapters)
constexpr int kMaxC = 64;            // largest centroid library
constexpr int kMaxTokens = 65536;    // largest batch of one plan
constexpr int kSortChunk = 4096;     // keys one plan block sorts in LDS
constexpr int64_t kMaxBufferBytes = (int64_t)1 << 31;   // bound of every buffer an apply kernel addresses with 32-bit offsets

SALT_HD int imin(int a, int b) { return a < b ? a : b; }
SALT_HD int imax(int a, int b) { return a > b ? a : b; }
SALT_HD int iclamp(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
SALT_HD int cdiv(int a, int b) { return (a + b - 1) / b; }

// Waves of an apply block for tiles of M tokens: four for up to 32 tokens,
// eight for 64 (two per 16-token block: two K halves in the shrink, two column
// phases in the expand), one per 16-token block beyond.
SALT_HD constexpr int waves_of(int M) { return M > 64 ? M / 16 : (M == 64 ? 2 * kWaves : kWaves); }

// Row stride of the split-K partials: r_c + r_u rounded up to whole float4s.
SALT_HD int padded_rank(int r_c, int r_u) {
  const int r = r_c + r_u;
  return r < 4 ? 4 : (r + 3) / 4 * 4;
}

// ---- records ------------------------------------------------------------------
// A tile is a run of at most M sorted tokens of one centroid group: header
// (first sorted position i0, token count n, centroid c or -1, largest residual
// rank of its centroid group).  A token
// record at sorted position p is (token t, slot u or -1, residual rank r,
// gamma bits).

// One table served by an apply launch.
struct Job {
  const void* x;           // [T][in], caller-owned
  void* y;                 // [T][out], caller-owned
  const void* at_c;        // [C][r_c][in]   centroid A, transposed
  const void* bt_c;        // [C][out][r_c]  centroid B, transposed
  int64_t prefix;          // sum of (in + out) over the context's earlier tables
  int64_t poff;            // first float of this job's partials
  int32_t in, out;
  int32_t S;               // K ranges of the shrink
  int32_t Kc;              // length of one K range (a multiple of kStepK)
  int32_t cpb;             // output columns of one expand block-chunk (kChunkCols x the waves along the columns)
  int32_t n_col;           // expand block-chunks per tile: cdiv(out, cpb)
  int32_t shrink_base;     // first shrink block of this job
  int32_t expand_base;     // first expand work item of this job
};

struct ApplyLaunch {
  // A block's first reads stand in lines of their own (64 bytes).
  // The first shrink block and expand work item of each job (INT32_MAX past the last
  // job), a line each.  A shrink block finds its job with one scalar load instead of
  // one per job in turn (a decode layer of four tokens: 6.2 -> 5.3 us); the expand
  // walks its line, since comparing with all of it costs its column loop the scalar
  // registers (Zipf T = 512: + 1 us).
  int32_t shrink_base[kMaxJobs];
  // what every block reads of the batch, two lines
  const int4* tiles;       // [n_tiles]
  const int4* stiles;      // [n_stiles] the shrink's tiles
  const int4* srt;         // [T] token records in sorted order
  const char* pool;        // residual slot pool
  float* partials;         // split-K partial sums
  const char* zeros;       // zero page: >= max(in, out) * esize bytes of zeros (read in place of missing residual rows)
  int64_t slot_stride;     // bytes between slots
  int32_t T;
  int32_t n_jobs;
  int32_t n_tiles;
  int32_t n_stiles;
  int32_t MS;              // tokens per shrink tile: 16 with `wide`, else min(M, 64)
  int32_t M;               // tokens per tile (16, 32, 64 or 128)
  int32_t C, r_c;
  int32_t n_slots;
  int32_t r_u;             // largest residual rank of the batch (<= kMaxRu)
  int32_t nq;              // residual rank chunks: ceil(r_u / kRankChunk), >= 1
  int32_t R;               // partial row stride, padded_rank(r_c, r_u)
  int32_t expand_items;    // expand work items: sum over jobs of n_tiles x n_col
  int32_t shrink_blocks;
  // what only the host reads
  int32_t wide;            // residual ranks above 2: the shrink is k_shrink_wide's (wide_shrink)
  int32_t quad;            // the expand's lane layout is the quad one
  int32_t uneven;          // some tiles hold ranks of several chunks, others of fewer
  int32_t n_pairs;         // (shrink tile, residual rank chunk) pairs that hold a rank, or 0: n_stiles * nq
  int32_t expand_base[kMaxJobs];
  Job jobs[kMaxJobs];
  int64_t partial_cap;     // floats of `partials`
  int32_t esize;           // bytes per element (2: bf16, 4: fp32)
  int32_t n_cu;            // compute units of the device (sizes the expand grid)
};
static_assert(offsetof(ApplyLaunch, tiles) == 64 && offsetof(ApplyLaunch, n_tiles) == 128 &&
              offsetof(ApplyLaunch, expand_base) == 192 && offsetof(ApplyLaunch, jobs) == 256);

struct TileHdr {
  int i0, n, c;
  int r;                   // bound of the residual ranks of the tile's tokens
};
struct TokRec {
  int t, u, r;
  uint32_t gamma_bits;
  bool tok;                // a real token of the tile
  bool res;                // has a residual term (slot >= 0, rank > 0)
};

// A tile header with every field clamped: 0 <= i0 < T, 0 <= n <= min(M, T -
// i0), -1 <= c < C, 0 <= r <= r_u (M: the tile size of the list it comes from).
SALT_HD TileHdr clamp_tile(const ApplyLaunch& a, int4 h, int M) {
  TileHdr r;
  r.i0 = iclamp(h.x, 0, imax(a.T - 1, 0));
  r.n = iclamp(h.y, 0, imin(M, a.T - r.i0));
  r.c = (a.r_c > 0) ? iclamp(h.z, -1, a.C - 1) : -1;
  r.r = iclamp(h.w, 0, a.r_u);
  return r;
}

// Token k of a tile (k >= n reads the tile's first token and is not a real one).
SALT_HD int tile_pos(const TileHdr& h, int k) { return h.i0 + (k < h.n ? k : 0); }

SALT_HD TokRec clamp_tok(const ApplyLaunch& a, int4 rec, bool real) {
  TokRec r;
  r.t = iclamp(rec.x, 0, a.T - 1);
  r.u = iclamp(rec.y, -1, a.n_slots - 1);
  r.r = (r.u >= 0) ? iclamp(rec.z, 0, a.r_u) : 0;
  r.gamma_bits = (uint32_t)rec.w;
  r.tok = real;
  r.res = real && r.u >= 0 && r.r > 0;
  return r;
}

// ---- block decomposition ----------------------------------------------------------
SALT_HD int job_of(const int32_t (&base)[kMaxJobs], int b) {
  int n = 0;               // (whole-number steps on the scalar unit: base[i] <= b adds one)
#if defined(__clang__)
#pragma unroll
#endif
  for (int i = 1; i < kMaxJobs; ++i) n += (int)((uint32_t)(base[i] - 1 - b) >> 31);
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+s"(n));       // (one product with the record's size, not one per step)
#endif
  return n;
}
SALT_HD int job_of_shrink(const ApplyLaunch& a, int b) { return job_of(a.shrink_base, b); }
SALT_HD int job_of_expand(const ApplyLaunch& a, int b) {
  int j = 0;
  while (j + 1 < a.n_jobs && b >= a.expand_base[j + 1]) ++j;
  return j;
}

// Shrink item i of job j: shrink tile tau, K range s, residual rank chunk q
// (items of a job: (q, s, tau) with tau fastest).  one: there is one rank chunk
// only, and neither of the divisions by S is needed.
struct ShrinkCoord {
  int tau, s, q;
};
SALT_HD int shrink_tiles(const ApplyLaunch& a) { return a.n_stiles; }
SALT_HD ShrinkCoord shrink_coord(const ApplyLaunch& a, const Job& jb, int item, bool one = false) {
  const int local = item - jb.shrink_base, nt = imax(shrink_tiles(a), 1);
  ShrinkCoord c;
  c.tau = local % nt;
  const int rest = local / nt;
  if (one) {
    c.s = iclamp(rest, 0, jb.S - 1);
    c.q = 0;
    return c;
  }
  c.s = rest % jb.S;
  c.q = iclamp(rest / jb.S, 0, a.nq - 1);
  return c;
}
SALT_HD TileHdr shrink_tile(const ApplyLaunch& a, int tau) {
  return clamp_tile(a, a.stiles[iclamp(tau, 0, a.n_stiles - 1)], a.MS);
}
SALT_HD TileHdr expand_tile(const ApplyLaunch& a, int tau) {
  return clamp_tile(a, a.tiles[iclamp(tau, 0, a.n_tiles - 1)], a.M);
}

// Expand work items: (job, tile, block-chunk), job-major, then tile, block-chunk
// fastest; block-chunk bc of a job covers columns [bc cpb, min(out, (bc + 1)
// cpb)).  A launch of G blocks gives block b the contiguous items [b N / G,
// (b + 1) N / G), N = expand_items, so every block carries the same number of
// block-chunks (to within one) and walks them tile by tile, reading a tile's v
// once per visit.
SALT_HD int expand_begin(const ApplyLaunch& a, int b, int G) {
  return (int)((int64_t)iclamp(b, 0, G) * a.expand_items / imax(G, 1));
}
// Block-chunks [j0, j1) of tile tau of job `job`: the run of items that starts at
// item pos and ends at the tile's last block-chunk or at item end, whichever
// comes first (pos < end).
struct ExpandSeg {
  int job, tau, j0, j1;
};
SALT_HD ExpandSeg expand_seg(const ApplyLaunch& a, int pos, int end) {
  ExpandSeg sg;
  sg.job = job_of_expand(a, pos);
  const Job& jb = a.jobs[sg.job];
  const int local = imax(0, pos - jb.expand_base), nc = imax(jb.n_col, 1);
  sg.tau = iclamp(local / nc, 0, a.n_tiles - 1);
  sg.j0 = local - (local / nc) * nc;
  sg.j1 = imin(nc, sg.j0 + imax(1, end - pos));
  return sg;
}

// ---- element offsets (in elements of the context dtype unless stated) --------------
// x[t][k .. k+7]: k clamped to a whole 8-element vector inside the row.
SALT_HD int64_t x_off(const ApplyLaunch& a, const Job& jb, int t, int k) {
  return (int64_t)iclamp(t, 0, a.T - 1) * jb.in + iclamp(k, 0, jb.in - 8);
}
// A_c^T[c][j][k .. k+7]
SALT_HD int64_t atc_off(const ApplyLaunch& a, const Job& jb, int c, int j, int k) {
  return ((int64_t)iclamp(c, 0, a.C - 1) * a.r_c + iclamp(j, 0, a.r_c - 1)) * jb.in + iclamp(k, 0, jb.in - 8);
}
// B_c^T[c][o][j .. j+7] (j a multiple of 8 below r_c)
SALT_HD int64_t btc_off(const ApplyLaunch& a, const Job& jb, int c, int o, int j) {
  return ((int64_t)iclamp(c, 0, a.C - 1) * jb.out + iclamp(o, 0, jb.out - 1)) * a.r_c + iclamp(j, 0, a.r_c - 8);
}
// y[t][o .. o+7]
SALT_HD int64_t y_off(const ApplyLaunch& a, const Job& jb, int t, int o) {
  return (int64_t)iclamp(t, 0, a.T - 1) * jb.out + iclamp(o, 0, jb.out - 8);
}
// Byte offset in the slot pool of A_u^T[rho][k .. k+7] of slot u holding rank r:
// the slot's blob holds, table after table, At_u [r][in] then B_u [r][out].
SALT_HD int64_t atu_byte(const ApplyLaunch& a, const Job& jb, int u, int r, int rho, int k) {
  const int rr = iclamp(r, 1, a.r_u);
  const int64_t e = (int64_t)rr * jb.prefix + (int64_t)iclamp(rho, 0, rr - 1) * jb.in + iclamp(k, 0, jb.in - 8);
  return (int64_t)iclamp(u, 0, a.n_slots - 1) * a.slot_stride + e * a.esize;
}
// Byte offset in the slot pool of B_u[rho][o .. o+7] of slot u holding rank r.
SALT_HD int64_t bu_byte(const ApplyLaunch& a, const Job& jb, int u, int r, int rho, int o) {
  const int rr = iclamp(r, 1, a.r_u);
  const int64_t e = (int64_t)rr * jb.prefix + (int64_t)rr * jb.in + (int64_t)iclamp(rho, 0, rr - 1) * jb.out +
                    iclamp(o, 0, jb.out - 8);
  return (int64_t)iclamp(u, 0, a.n_slots - 1) * a.slot_stride + e * a.esize;
}
// Partial sum of K range s, sorted position p, column col (floats), inside the
// job's own region [poff, poff + S * T * R).
SALT_HD int64_t part_off(const ApplyLaunch& a, const Job& jb, int s, int p, int col) {
  return jb.poff + ((int64_t)iclamp(s, 0, jb.S - 1) * a.T + iclamp(p, 0, a.T - 1)) * a.R + iclamp(col, 0, a.R - 1);
}

// ---- loop ranges ---------------------------------------------------------------
// K range s of a job: [k_lo, k_hi).  Its kStepK-wide steps are shared by the
// kw waves along K, wave kq taking steps kq, kq + kw, ...
SALT_HD int k_lo(const Job& jb, int s) { return imin(jb.in, s * jb.Kc); }
SALT_HD int k_hi(const Job& jb, int s) { return imin(jb.in, (s + 1) * jb.Kc); }
SALT_HD int k_steps(const Job& jb, int s) { return cdiv(k_hi(jb, s) - k_lo(jb, s), kStepK); }

// Elements between the two 8-element vectors a lane holds of a 64-wide shrink
// step or expand chunk: lane group g holds g 8 + 0..7 and kPiece + g 8 + 0..7,
// so that the four groups' vector h covers 32 contiguous elements.
constexpr int kPiece = 32;

// Output column of expand A-operand row i (lane & 15) in column block b4 of a
// 64-column chunk starting at col0: arranged so that MFMA output lane (token,
// g), which receives rows 4 g + e of tile b4, holds columns col0 + 8 g + kPiece h
// + 4 (b4 & 1) + e with h = b4 >> 1, i.e. the vectors col0 + 8 g + kPiece h + 0..7.
SALT_HD int expand_col(int col0, int i, int b4) {
  return col0 + kPiece * (b4 >> 1) + 8 * (i >> 2) + 4 * (b4 & 1) + (i & 3);
}

// ---- lane layouts ----------------------------------------------------------------
// Row layout: a lane holds a token row (lane & 15), as the matrix instructions hold
// their operands, and of a 64-wide step or chunk the two vectors above.
// Quad layout: a wave works on 16 token rows x 128 consecutive elements, 16 vectors
// of eight per row, and loads them so that the four lanes of a quad take four
// consecutive vectors of one row: lane l = 16 g + 4 q + b reads in load j (0..3)
// row 4 q + j, vector 4 g + b.  The memory pipeline takes a wave's 16-byte lanes
// quad by quad, one 64-byte piece each; in the row layout every lane is a piece
// of its own (prefill T = 8192, rank 1, the expand: 236 -> 212 us).
// A transpose of 4 registers x 4 lanes inside each quad turns loads j into the
// operand form: lane l, register s holds row l & 15, vector 4 g + s, that is
// elements 32 g + 8 s + 0..7.
SALT_HD int quad_row(int lane, int j) { return 4 * ((lane >> 2) & 3) + j; }
SALT_HD int quad_elem(int lane) { return 32 * (lane >> 4) + 8 * (lane & 3); }
// Column of row i of 16-column tile t (0..7) of a 128-column chunk in the quad
// layout: the product's lane (token, g), which receives rows 4 g + e, e = 0..3,
// of every tile, holds of tiles 2 s and 2 s + 1 the columns 32 g + 8 s + 0..7.
SALT_HD int quad_col(int i, int t) { return 32 * (i >> 2) + 4 * t + (i & 3); }

// Whether the expand of ranks up to 2 runs in the quad layout: 128-token tiles of
// ranks up to 1 (for ranks above 2 see quad_rows).  Smaller
// tiles keep the row layout, whose shorter chunks, two sets of operands and
// cheaper set-up serve short groups better (Llama-3.1-8B decode T = 256: 34.5 us
// against 36 us, Zipf T = 512: 35 against 39, 64-token tiles of rank 2: 41 against
// 49), and so do 128-token tiles of rank 2, for whose second row the quad layout
// has no registers left (prefill T = 8192, r_c = 64: 266 us against 291 us), or of
// centroid ranks above 64, whose eight fragments leave one block of it to a compute
// unit (Llama-3.2-3B layer, T = 8192, rank 1: r_c = 72 396 us against 442 in the
// quad layout, 128 437 against 488; T = 4096: 237 / 255, 267 / 292).
SALT_HD constexpr bool quad_rank1(int M, int r_c, int r_u) { return M == 128 && r_c <= 64 && r_u <= 1; }

}  // namespace salt
