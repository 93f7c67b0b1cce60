// Similarity codebook replacement (Sec. "Similarity Based Token Replacement", Alg. 1): what its
// kernels share.  ut = tensor * units + unit indexes one independent (batch, kv-head, K|V)
// problem of n tokens.  The kernels, in the order spindle_compress_shallow enqueues them:
//   shallow_prep    what must start from a known value; magnitudes (Eq. 8) in double precision, of
//                   fp32 inputs unit vectors rounded to fp16, and a 64-byte sketch of every token whose
//                   products bound the cosines from above
//   shallow_pivots, shallow_order, shallow_window
//                   the tokens of a problem sorted so that similar ones stand together
//   shallow_scan    which pairs of 32-token tiles can hold a pair above theta at all: balls around the
//                   tiles' sketches first, then sketch products, in six-bit floats
//   shallow_refine  where the sketches exclude little, the same from the rows
//   shallow_rows    for those tiles the cosines themselves (Eq. 4, 9), decided exactly; degrees
//                   (Eq. 10) and neighbour lists
//   merge_onehop, merge_twohop, merge_update
//                   the first rounds of the greedy highest-degree codebook construction
//                   (Eq. 11-13) in its exact parallel form, one launch per phase
//   shallow_merge   the remaining rounds (all of them for short problems) and the codebook order of
//                   the picked tokens, one workgroup per problem
//   shallow_emit    references in codebook order and the codebook vectors
//   shallow_assign  tokens whose entry fell beyond the codebook cap go to the nearest
//                   stored entry
//
// shallow_prep.hip holds shallow_prep, shallow_tiles.hip the kernels from the order of the tokens to
// their lists, shallow_merge.hip the greedy
// merge, shallow_codebook.hip the codebook order, the outputs and the cap; shallow.hip the
// workspace layout and the entry points.
#pragma once

#include <math.h>
#include <string.h>

#include "common.h"

namespace spindle {

// Unit vectors are stored in fp16 scaled by 2^10, so that components down to 6e-8 of the
// norm stay normal numbers.  |fp16 MFMA cosine - exact cosine| then stays below kGuard:
// each component of both vectors carries a relative rounding error of at most 2^-11
// (sum over the dot product <= 2^-10 = 9.77e-4 by Cauchy-Schwarz), the fp32 normalisation
// adds < 1e-6 and the fp32 accumulation of 128 exact products < 1e-5.
constexpr float kUnitScale = 1024.f;
constexpr float kGuard = 1.05e-3f;

constexpr int kStageCols = 64;
constexpr int kLdsRow = 272;      // fp16 row of 128 + 16 B pad (shallow_prep)
// What the sums of 128 exact products in fp32, truncated or not, and the two factors may be off from a cosine is less than
// 2e-5; a result within this of theta is decided in double precision.
constexpr float kRowsGuard = 7e-5f;
constexpr int kStageBytes = kStageCols * 256;   // staged tokens: unpadded rows, 16-byte pieces swizzled

// Sketch of a token: 64 bytes, integers scaled by kSketchScale.  60 coordinates of the unit vector
// after a Walsh-Hadamard rotation, and the norm of the other 68 spread evenly over the last byte of
// each 16-byte piece, so that the product of two sketches is at least the cosine, up to rounding
// (the coordinates left out contribute at most the product of their norms).
constexpr float kSketchScale = 300.f;
constexpr int kSketchBytes = 64;
constexpr int kTile = 32;                        // tokens per tile of the sorted order
constexpr int kTileBytes = kTile * kSketchBytes;   // sketches of a tile as bytes
// What shallow_scan multiplies are the sketches in six-bit floats (two exponent and three mantissa bits, up to 7.5),
// kSixScale of the integers to the unit: twice the rate of bytes on the matrix cores.  They are off by 0.025 of a unit
// vector where the bytes are by 0.008; a clustered layer has as many tile pairs marked all the same (2.3 % of them).
// Products are multiples of 2^-6 below 2^12, so their sums are exact.
constexpr float kSixScale = 16.f;
constexpr int kSixBytes = kTile * 48;            // of a tile: 16 bytes of every lane's 24, then 8 of every lane
constexpr int kScanPanel = 16;                   // row tiles of a block of shallow_scan
constexpr int kScanStage = 8;                    // column tiles it stages at a time
constexpr int kScanRun = 16;                     // stages of a block at most
constexpr uint32_t kSketchUnknown = 1u << 20;    // error of a token whose sketch says nothing
// Tokens are sorted by bucket, two per pivot (at most kPivots, one per 16 tokens): what is near it, and what isn't but has
// it nearest.
constexpr int kPivots = 1024, kBuckets = 2 * kPivots;
constexpr int kOrderTokens = 512;                // tokens per block of shallow_pivots and shallow_order, or twice as many
constexpr int kWindow = 1024;                    // places of a block of shallow_window
constexpr int kBallTiles = 64;                   // tiles whose balls stand together: one each, and 32 seconds
constexpr int kBalls = 3 * kTile;
// Problems of 2048 tokens and more are sorted and scanned, shorter ones only where there are many: what the launches
// take, about 45 us, has to come back from shallow_rows, which then needn't take every tile.  Clusters and
// isolated tokens, without and with: 16 problems of 1280 124, 142 and 107, 151 us, of 1536 135, 152 and 111, 152; 64 of
// 1024 119, 136 and 120, 150, of 1280 203, 231 and 143, 185; 256 of 1024 294, 332 and 225, 296.
inline int scan_pays(int UT, int n) {
  const long T = (n + 31) / 32;
  return n >= 2048 || (n >= 1024 && UT * T * (T - 24) >= 18000);
}
// Tile pairs of all problems from which the scan pays for asking the balls around the tiles first, which takes shallow_window
// and shallow_scan some 10 us.  What they exclude depends on the rows (most in clusters, least where
// many are isolated) and grows with the length, so the line is where calls on the whole cost the same.  fp16, without balls and with, us: 16 problems
// of 8192 tokens (1.05 million) in clusters 158, 165, a third isolated 186, 195; 2 of 28000 (1.53) 160, 160 and 254, 257, drifting 273, 277; 16 of
// 11000 (1.9) 190, 191 and 240, 245, drifting 252, 257; 4 of 23000 (2.1) 174, 169, half isolated 261, 265; 2 of 32768 (2.1) 176, 170, a fifth
// 223, 217, half 300, 302, kept rows of repeated heads 230, 221; 128 of 4096 (2.1) 301, 299, a third isolated 413, 426, drifting 372, 374.
inline int balls_pay(int UT, int n) {
  const long T = (n + 31) / 32;
  return UT * T * T >= 2000000;
}
// Below kBallMinTheta balls exclude too little: products of unrelated tokens end at about 0.65 for a tile, and the radius
// and the errors add 0.2.  Calls, fp16, without and with, us, by theta: 64 problems of 8192 tokens in clusters 0.88 356, 319, 0.83 386, 365, 0.8
// 487, 489, 0.77 697, 765, half isolated 0.9 578, 569, 0.86 783, 899, 0.83 934, 949, 0.8 997, 1054, 0.74 1067, 1231; 16 of 32768, a
// third isolated, 0.9 826, 705, 0.86 1202, 1137, 0.8 2118, 2096, 0.74 2545, 2644, drifting 0.9 659, 649, 0.86 1038, 1100, 0.8 2539, 2595; 64 of
// 8051 in 13 clusters 0.85 on V and 0.9 on K, without on V and with, 714, 581.  Between 0.8 and 0.87 it depends on the rows.
constexpr float kBallMinTheta = 0.8f;
// Below kSketchMinTheta the sketches are not asked: a sketch product of unrelated tokens is about 0.53 with a
// spread of 0.06, so the largest of a pair of tiles is above 0.7 nearly always.  Below kVectorMinTheta the full
// vectors are not asked either: at 0.3 a third of the pairs of tiles of unrelated tokens hold a cosine above it, three
// quarters for four row tiles together, and what is left out of shallow_rows is what finding it takes.
constexpr float kSketchMinTheta = 0.7f, kVectorMinTheta = 0.3f;
enum { kByNone, kByVector, kBySketch };
// Column tiles a scan block may mark before the full vectors decide instead, counted once for the four row tiles
// that shallow_rows takes together: all pairs in shallow_refine cost a fifth of what shallow_rows takes
// for all of them (16 problems of 32768 tokens: 1.95 and 8 to 10 ms).
constexpr float kRefineShare = 0.22f;

constexpr int kCounters = 32;     // ints per ut
// (slots 6..15 hold the phase timings of shallow_merge)
enum { C_PICKS = 4, C_ROUNDS = 5 };

struct ShallowParams {
  const char *X[2];        // input tensors [U][n][128] in `dtype` (index = tensor slot)
  float theta[2];
  int dtype, U, UT, n;
  KvLayout lay;            // rows of the input tensors
  int cap;
  // workspace
  _Float16 *Xh;            // [UT][n][128] fp32 inputs: unit vectors
  _Float16 *Xe;            // [UT][n][128] unit vectors of the stored entries, where tokens were cut; the room of Xl
  double *m64;             // [UT][n]
  int *slot, *alive, *cand, *dying, *rank, *rank_vert;   // [UT][n] (cand: candidate bits in the grid rounds)
  // Lists, keys and everything after them count tokens by position: place in the sorted order.
  uint16_t *perm, *iperm;  // [UT][n] token at a position, position of a token
  float *invp;             // [UT][n] factor of a row in the cosine (see shallow_rows), by position
  uint8_t *sk0;            // [UT][n][64] sketches by token
  float2 *inv_err;         // [UT][n] by token (scan): the factor, and the distance of the sketch from what it stands for (< 0: says nothing)
  uint16_t *bucket;        // [UT][n] bucket of a token
  uint32_t *mean;          // [UT][2] first eight coordinates of the pivots' mean
  uint32_t *total;         // [UT][kBuckets] tokens per bucket
  uint16_t *before;        // [UT][order blocks][kBuckets] place within a bucket of a block's first token of it
  uint8_t *sk;             // [UT][Tp][kSixBytes] sketches by position, in six-bit floats
  uint32_t *etile;         // [UT][Tp] what a tile's sketches may be off by in a product, sketch units squared
  int balls, asks[2];      // 1: the scan asks the balls around tiles first, in any of the tensors, in each
  float *tnorm;            // [UT][Tp] longest six-bit sketch of a tile, in six-bit units (as the radii)
  // Balls around the six-bit sketches of a tile, or of its two parts: centres as 3 tiles of 32 per kBallTiles, and per centre
  // what the products of its tile may be off by, in six-bit units squared (no tile: a large negative number), and its radius.
  uint8_t *skc;            // [UT][Tp / 64][3][kSixBytes]
  float2 *ball;            // [UT][Tp / 64][kBalls]
  uint8_t *second;         // [UT][Tp / 64][kTile] tile of the 64 that a second ball belongs to
  uint32_t *tpairs;        // [UT][T][TW] bit t of row r: tiles r and t may hold a pair above theta
  int T, Tp, TW;           // tiles, rounded up to whole panels; words per row of tpairs
  int scan;                // 1: tokens are sorted and tpairs says which tiles count; 0: all tiles, positions = tokens
  int stages_per_item, njg;   // column stages of a block of the scan, runs of them in a problem
  uint32_t *todo;          // [scan_blocks] 1: left to shallow_refine
  int by[2];               // which tile pairs count: kBySketch, kByVector or, all of them, kByNone
  int scan_thr[2];         // theta in sketch units squared
  _Float16 *Xl;            // [UT][n][128] fp32 inputs: what fp16 rounding took off the unit vectors, x 2^11
  // Neighbours of a position, 16 positions at a time: words (half tile << 16 | one bit per position of
  // it), only those with a bit set; or, where a tile's rows would need more than list_row words each on
  // average, the bits of all half tiles in order (list_row words hold them).
  uint2 *rows;             // [UT][n] first word and number of words of a row; dense rows: kDenseRow | half tiles
  uint32_t *lists;         // [UT][n][list_row]
  int list_row;            // words per row on average
  int n32;                 // n rounded up to whole tiles: pitch of key and m1 (a dense row has a word for both half tiles of the last)
  uint32_t *key, *m1;      // [UT][n32] (remaining degree << 16) | (0xFFFF - token), 0 once removed; largest in the neighbourhood
  uint32_t *live[3];       // [UT][T] bit per position: still there at the start of round 0, 1, 2
  uint32_t *picked;        // [UT][T] bit per position: became a codebook entry
  uint32_t *pick_key;      // [UT][n] key of a picked position at pick time; slot = position of a token's entry
  int *counters;           // [UT][kCounters]
  unsigned *pairs_exact;   // [UT][T][rows_waves] pairs decided in double precision, by wave
  uint32_t *ovf;           // [UT][n] tokens whose codebook entry was cut, per problem
  unsigned *ovf_cnt;       // [UT] their number
  uint2 *ccand;            // [UT][n][2][kCandCap] lists of shallow_assign: (entry index, approximate cosine bits)
  // outputs (index = tensor slot)
  char *C[2];
  int32_t *n_codes[2], *n_found[2], *ref[2];
  float *mag[2];
  int32_t *deg_out[2];     // optional initial degrees
};

// Blocks are dealt round-robin to the 8 XCDs; this numbering gives each XCD a run of consecutive
// items (a problem's blocks share its L2).  The launch has a multiple of 8 blocks.
__device__ __forceinline__ int xcd_item() { return (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3); }
inline unsigned xcd_grid(size_t items) { return (unsigned)align_up(items, 8); }

__device__ __forceinline__ const char *x_row(const ShallowParams &p, int ut, int a) {
  const int t = ut / p.U, u = ut % p.U;
  return p.X[t] + kv_unit_offset(p.lay, u) + (size_t)a * (size_t)p.lay.st;
}

// Waves of shallow_rows that share a row tile: four (one row tile per block) while four row tiles per block would leave
// compute units without a block.  fp16 and fp32 heads of 512 tokens, 256 row tiles in all 12 and 15 us (four per block 21
// and 27), 512 row tiles 21 and 30 (21 and 28), 1024 38 and 47 (22 and 28); of 1000 tokens, 512 row tiles 31 and 38 (35 and
// 52), 1024 60 and 72 (36 and 47).
inline int rows_waves(int UT, int T) { return (long)UT * T < 1024 ? 4 : 1; }

constexpr uint32_t kDenseRow = 1u << 31;

// Eq. 4 evaluated the way the adjacency decision is defined: double precision,
// dimension-order dot product, 0 when either vector is zero.
template <int DT, int kBatch>
__device__ inline double cos64(const ShallowParams &p, int ut, int a, int b) {
  const double den = p.m64[(size_t)ut * p.n + a] * p.m64[(size_t)ut * p.n + b];
  if (!(den > 0.0)) return 0.0;
  return dot64<DT, kBatch>(x_row(p, ut, a), x_row(p, ut, b)) / den;
}

// Blocks of shallow_scan, a multiple of 8.
inline int scan_blocks(const ShallowParams &p) { return 8 * (p.Tp / kScanPanel) * ((p.UT * p.njg + 7) / 8); }

// Entries per cut token and lane group that shallow_assign hands to the exact comparison.
constexpr int kCandCap = 8;

// ---------------------------------------------------------------- launches, one per source file
// Each enqueues its kernels on `st` in order and returns SPINDLE_OK or the failed HIP call.
spindle_status launch_prep(const ShallowParams &p, size_t nzero, size_t cpieces, hipStream_t st);   // words to clear, 16-byte pieces of a tensor's codebooks
spindle_status launch_tiles(const ShallowParams &p, hipStream_t st);      // order, scan and lists
spindle_status launch_adjacency(const ShallowParams &p, uint32_t *const out[2], hipStream_t st);   // exports G
spindle_status launch_unit_like(const ShallowParams &p, hipStream_t st);   // operands of the next into Xe
spindle_status launch_bare_similarity(const ShallowParams &p, hipStream_t st, int mode);   // measurement aid
spindle_status launch_merge(const ShallowParams &p, hipStream_t st);
spindle_status launch_codebook(const ShallowParams &p, hipStream_t st);

}  // namespace spindle
