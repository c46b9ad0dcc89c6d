// Host-side shape bookkeeping, the workspace layout, error and timing helpers shared by the FastH kernels' launchers.
// Included by fasth.hip, the library's single translation unit.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "fasth.h"
#include "fasth_device.h"

namespace fasth {

// ------------------------------------------------------------------------------------------
// Host-side shape bookkeeping
// ------------------------------------------------------------------------------------------

constexpr int kMaxBlock = 128;     // largest k: a k x k factor must fit in LDS with scratch
constexpr int kMaxD = 16384;       // general chain kernel: 1024 threads x 4 chunks of 4 elements
constexpr int kGramChunk = 128;    // columns of V per LDS tile in the Gram kernel
constexpr int kMaxGramSplit = 16;  // partial Gram matrices per block
constexpr int kComputeUnits = 256; // of the MI355X: launches of more workgroups than this run in rounds or share units
constexpr int kDvTile = 64;        // columns of dV per workgroup
constexpr int kDvMChunk = 32;      // mini-batch columns per LDS tile in the dV kernel

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static int padded_block(int k) {
  int kp = 16;
  while (kp < k) kp *= 2;
  return kp;
}

struct TrioPlan { int xt, ct, parts; };  // chain_trio_kernel: template arguments and workgroups per tile (0: not used)

struct Layout {
  // What the kernels see: vectors padded to dp elements (a multiple of 4), np >= n rows in nb = np / ki blocks of ki rows.
  // A row of V that does not exist is a zero row whose diagonal entry of the block's triangular matrix is one: its
  // coefficients are zero and nothing downstream changes.
  int dp, np, ki;
  bool copy_v;       // the kernels read a padded copy of V (off_V) that the factor kernels write
  int kp, nb, gram_split, dv_split;
  bool dv_trio;      // dv_trio_kernel forms dV
  int kf, kpf, nbf;  // rows of a factor as stored (several of the caller's blocks when a team kernel merges them), padded; their number
  int team_wide;     // parts per column if chain_team_wide_kernel serves the shape (factors stored in its order), else 0
  int npair;         // pairs of blocks whose rows' product V_a V_b^T is formed beside the factors (chain_team_wide_kernel), else 0
  TrioPlan trio;     // .parts > 0 if chain_trio_kernel serves the shape
  size_t off_frag;   // the rows of V as that kernel's operands
  size_t off_V, off_T, off_S, off_Spart, off_ready, off_xch, off_saveA, off_saveCa, off_saveG, off_saveCg, off_dVpart, off_Zpart, total;
  size_t xch_words;  // 32-bit words of the hand-off area between workgroups that share a column (0: none)
};

// Columns of 1025 to 2048 elements are shared by two workgroups (chain_pair_kernel's SPLIT form) while both have a
// compute unit of their own. Per column the workspace then holds 2 x 2 x 16 hand-off words of 16 bytes and a tag
// counter (padded to 256 bytes).
constexpr unsigned kSplitPairWords = (2 * 2 * 16 * 16 + 256) / 4;
constexpr int kSplitPairMaxCols = kComputeUnits / 2;
static bool split_pair_serves(int d, int m, int k) {
  return d > 1024 && d <= 2048 && d % 4 == 0 && (k == 32 || k == 64 || k == 128) && m <= kSplitPairMaxCols;
}
constexpr int kDefaultWaitLimit = 1 << 20;  // polls of a bounded wait between workgroups (a fraction of a second)

// chain_team_kernel: a team of two to eight workgroups per column, 512 elements each, steps of 64 rows. Parts per
// column for a shape it serves, else 0: 512 < d <= 4096 in whole 16-byte chunks, blocks of 32 (an even number of
// them: two are merged into a factor of 64 rows), 64 or 128 rows, and a compute unit for every workgroup of the
// launch, so that no part waits for one that has not started.
constexpr int kTeamRows = 64;        // rows of V per step
constexpr int kTeamSlice = 512;      // elements of the column per workgroup
constexpr int kTeamHeadBytes = 256;  // per column: [0] tag counter, [32 + 8 j] part j's XCC_ID word
constexpr unsigned team_words_per_column(int np) { return (unsigned)(kTeamHeadBytes + np * 2 * np * kTeamRows * 8) / 4u; }
#ifndef FASTH_TEAM_MIN_D
#define FASTH_TEAM_MIN_D (kTeamSlice + 1)
#endif
// A team's workgroups need a compute unit each, all at once: a part that waited for a unit would keep its partners
// polling until a whole chain elsewhere has ended. The launch places the parts of columns c, c + 8, ... on one XCD
// (32 of the 256 units), so what must fit is np workgroups for every eight columns begun.
static bool team_fits(int m, int np) { return 8 * np * ((m + 7) / 8) <= kComputeUnits; }
// chain_team_wide_kernel: the same with 256 elements of the column per workgroup and steps of 128 rows, for columns
// of FASTH_TEAM_WIDE_MIN_D to 2048 elements while every workgroup has a compute unit of its own: half as many
// sequential steps as with 64 rows. Such a step joins two blocks of 64 rows (the caller's, halves of the caller's
// blocks of 128, or merged pairs of the caller's blocks of 32) through their 64 x 64 factors and the product
// V_a V_b^T of their rows, which the factor kernel forms beside the factors. Its hand-off words are 16 bytes
// {sum, tag, sum, tag}. The matrices of such a shape are stored in the order in which the kernel's threads read them.
constexpr int kWideRows = 128;
constexpr int kWideSlice = 256;
constexpr unsigned team_wide_words_per_column(int np) { return (unsigned)(kTeamHeadBytes + np * 2 * np * (kWideRows / 2) * 16) / 4u; }
#ifndef FASTH_TEAM_WIDE_MIN_D
#define FASTH_TEAM_WIDE_MIN_D 513
#endif
static int team_wide_parts(int d, int n, int m, int k) {
  if (d < FASTH_TEAM_WIDE_MIN_D || d > 8 * kWideSlice || d % 4 != 0 || n % kWideRows != 0) return 0;
  if (!(k == 32 || k == 64 || k == 128)) return 0;
  const int np = (d + kWideSlice - 1) / kWideSlice;
  return team_fits(m, np) ? np : 0;
}
static int team_parts(int d, int n, int m, int k) {
  if (team_wide_parts(d, n, m, k)) return 0;
  if (d < FASTH_TEAM_MIN_D || d > 8 * kTeamSlice || d % 4 != 0) return 0;
  if (!(k == 64 || k == 128 || (k == 32 && n % 64 == 0))) return 0;
  const int np = (d + kTeamSlice - 1) / kTeamSlice;
  return team_fits(m, np) ? np : 0;
}

// chain_team_tile_kernel: tiles of 16 columns on the matrix cores, each shared by a team of ceil(d / 256) workgroups
// (2 to 4; ceil(d / 512) for d > 1024), steps of 64 rows (32 for d > 1024): for mini-batches of FASTH_TEAM_TILE_MIN_COLS columns and more (d > 512; ..._SHORT for
// shorter columns), as long as every
// workgroup has a compute unit on its team's XCD. Parts per tile for a shape it serves, else 0. Per tile the
// workspace holds a 256-byte head and, per receiving part, step parity and sending part, 512 hand-off words of 16 bytes.
#ifndef FASTH_TEAM_TILE_MIN_COLS
#define FASTH_TEAM_TILE_MIN_COLS 449        // d > 512: from here on it beats the per-column kernels' rounds (and chain_quad_kernel)
#endif
#ifndef FASTH_TEAM_TILE_MIN_COLS_LONG
#define FASTH_TEAM_TILE_MIN_COLS_LONG 640   // d > 1024 (parts of 512 elements, steps of 32 rows)
#endif
#ifndef FASTH_TEAM_TILE_MIN_COLS_SHORT
#define FASTH_TEAM_TILE_MIN_COLS_SHORT 897  // d <= 512 (two parts)
#endif
// Mini-batches for which calls may overlap on the GPU although their tiles are shared by workgroups: beyond 1024 columns of more than
// 512 elements, where kernels without hand-overs served before. Teams form in the order in which workgroups start there, and calls
// that may overlap on one workspace take no teams.
static bool shared_tiles_overlap(int d, int m) { return d > 512 && m > 1024; }
constexpr unsigned team_tile_words(int np) { return (unsigned)(kTeamHeadBytes + np * 2 * np * 512 * 16) / 4u; }
static int team_tile_parts(int d, int n, int m, int k) {
  if (m < (d > 1024 ? FASTH_TEAM_TILE_MIN_COLS_LONG : d > 512 ? FASTH_TEAM_TILE_MIN_COLS : FASTH_TEAM_TILE_MIN_COLS_SHORT) ||
      d <= 256 || d > 2048 || d % 4 != 0) return 0;
  // parts of 256 elements take 64 rows per step (blocks of 32 two at a time), parts of 512 (d > 1024) take 32
  if (!(k == 64 || k == 128 || (k == 32 && (d > 1024 || n % 64 == 0)))) return 0;
  if (team_wide_parts(d, n, m, k) || team_parts(d, n, m, k)) return 0;
  if ((size_t)d * m * sizeof(float) >= 0x80000000u || (size_t)n * d * sizeof(float) >= 0x80000000u) return 0;  // 32-bit byte offsets
  const int np = d > 1024 ? (d + 511) / 512 : (d + 255) / 256;
  return np >= 2 && team_fits((m + 15) / 16, np) ? np : 0;
}

// chain_trio_kernel: tiles of 16 ct columns on the bf16 matrix cores at fp32 precision, each shared by `parts` workgroups
// of 128 xt elements, for more than 1024 columns, or 2048 where chain_team_tile_kernel with its shorter parts serves and is
// as fast (us, nothing saved: d = 1024, m = 1024: 74 against 76; forward + backward: d = 512, m = 2000: 152 against 157). Every workgroup of a team needs a compute unit on the
// team's XCD. Short parts and narrow tiles have the least to do per step (us per forward + backward, k = 32, {xt, ct}):
// d = 512, m = 4096: {4, 1} 179, {4, 2} 205; d = 1024, m = 2048: {4, 1} 324, {4, 2} 376; but 16 columns of 1024 elements keep the
// matrix cores waiting for V: d = 1024, m = 4096: {4, 2} 647, {8, 1} 699, {8, 2} 833; d = 2048, m = 2048: {4, 2} 1242,
// {8, 1} 1272, {8, 2} 1506.
// Before (chain_tile_kernel, dv_kernel), us per forward + backward: d = 256, m = 4096: 118 -> 101; d = 512, m = 4096: 311 -> 184;
// d = 1024, m = 1100: 481 -> 271, 2048: 574 -> 317, 4096: 751 -> 538; d = 2048, m = 1100: 1782 -> 935, 4096: 2651 -> 1995.
// Few steps do not pay for the operands of V, and rounding n up to whole steps weighs more: us per forward + backward without and
// with, d = 256, m = 1500: n = 96: 63, 69; n = 128: 71, 68; d = 640, m = 3000: n = 96: 80, 98; n = 128: 98, 105; n = 192: 136, 132;
// d = 1024, m = 3000: n = 96: 91, 102; n = 112: 108, 103; d = 1280, m = 1500: n = 80: 89, 89; n = 112: 109, 90; with 1024 elements per
// workgroup ({8, 2}): d = 1536, m = 4096: n = 128: 180, 222; n = 192: 242, 254; n = 256: 303, 280; d = 2048: n = 128: 215, 242.
// Up to 1280 columns of 513 to 768 elements chain_team_tile_kernel's three shorter parts serve: d = 640, m = 1100, n = 512: 138 against 159.
constexpr int kTrioMaxD = 2048;
constexpr unsigned trio_words(int np, int ct) { return (unsigned)(kTeamHeadBytes + np * 2 * np * 512 * 16 * ct) / 4u; }
static TrioPlan trio_plan(int d, int n, int m) {
  const TrioPlan none{0, 0, 0};
  if (m <= (d > 256 && d <= 512 ? 2048 : d > 512 && d <= 768 ? 1280 : 1024) || d > kTrioMaxD) return none;
  if (n <= (d <= 512 ? (m > 2048 ? 96 : 112) : d <= 768 && m > 2048 ? 160 : d <= 1024 ? 96 : 64)) return none;
  const int narrow = (m + 15) / 16, wide = (m + 31) / 32, np4 = (d + 511) / 512, np8 = (d + 1023) / 1024;
  if (d <= 512) return TrioPlan{d <= 256 ? 2 : 4, narrow <= kComputeUnits ? 1 : 2, 1};
  if (team_fits(narrow, np4)) return TrioPlan{4, 1, np4};
  if (team_fits(wide, np4)) return TrioPlan{4, 2, np4};
  if (d <= 1024) return TrioPlan{8, 2, 1};
  return n > 192 && team_fits(wide, np8) ? TrioPlan{8, 2, np8} : none;
}
// The same operands without teams, for calls that may overlap on one workspace: 1024 elements in one workgroup (at most 4096
// columns: a team served them), beyond that chain_tile_kernel. us per fasth_apply, nothing saved, chain_tile_kernel, this and teams:
// d = n = 1024: m = 1100: 174, 130, 94; m = 2048: 175, 128, 97; m = 4096: 178, 139, 120; d = n = 1536, m = 2048: 364, -, 177
// (256 elements per wave need more registers than there are).
static TrioPlan trio_solo_plan(int d, int n, int m) {
  const TrioPlan plan = trio_plan(d, n, m);
  if (plan.parts <= 1) return plan;
  return d <= 1024 ? TrioPlan{8, 1, 1} : TrioPlan{0, 0, 0};
}

// dv_trio_kernel: blocks of 64 rows, from 449 columns on and once the products are worth its longer start (us per forward +
// backward with it and without: d = n = 512, m = 512: 100, 88; d = n = 512, m = 800: 141, 135; d = n = 1024, m = 420: 193, 189;
// m = 600: 206, 207; m = 800: 220, 244; m = 1024: 239, 272; d = n = 2048, m = 700: 680, 912).
static bool dv_trio_serves(int d, int n, int m, int k) {
  return m >= 449 && (double)n * d * m >= 4e8 && k == 64 && d % 2 == 0 &&
         (size_t)m * n * sizeof(float) < 0x80000000u && (size_t)m * d * sizeof(float) < 0x80000000u && (size_t)n * d * sizeof(float) < 0x80000000u;
}
constexpr int kDvTrioTile = 256;  // elements per workgroup
// Parts of the mini-batch: what a part adds (its partial sums written and read again, the start of its workgroups)
// against fuller rounds of workgroups.
static int dv_trio_split(int d, int n, int m) {
  const int wgs = (d + kDvTrioTile - 1) / kDvTrioTile * (n / 64), chunks = (m + 31) / 32;
  int best = 1;
  double best_us = 1e30;
  for (int s = 1; s <= 16 && s <= (chunks + 1) / 2; ++s) {
    const double rounds = (wgs * s + kComputeUnits - 1) / kComputeUnits;
    const double us = rounds * (3.0 + 1.6 * ((chunks + s - 1) / s)) + (s > 1 ? 4.0 + 8e-6 / 4.0 * s * (double)n * d : 0.0);
    if (us < best_us) { best_us = us; best = s; }
  }
  return best;
}

// The dV kernel has one workgroup per (64-column tile of dV, block). When that is too few to fill the chip and the
// mini-batch is wide (a short, narrow V against many columns: a 1 x 1 convolution with few channels), the
// mini-batch is split over up to 32 workgroups whose partial sums meet in a buffer of the workspace.
static int dv_minibatch_split(int d, int n, int m, int k) {
  const int wgs = ((d + kDvTile - 1) / kDvTile) * (n / k);
  if (wgs >= 128 || m < 256) return 1;
  // a split needs every block's matrix Z formed beforehand from the coefficient matrices, which the kernel that does
  // it addresses with 32-bit byte offsets
  if ((size_t)m * n * sizeof(float) >= 0x80000000u) return 1;
  int split = 256 / wgs;
  if (split > m / 128) split = m / 128;
  if (split > 32) split = 32;
  return split < 1 ? 1 : split;
}

// Blocks of up to 32 rows are factored by one workgroup each; blocks of 64 rows only while d is short, because one
// workgroup per block then streams 64 d floats alone (measured: d = 256 18.0 -> 13.6 us, d = 1024 19.5 -> 21.5 us,
// d = 2048 23 -> 34 us against a Gram product split over d).
#ifndef FASTH_FUSED64_MAX_D
#define FASTH_FUSED64_MAX_D 512
#endif
static bool factor_is_fused(int kp, int d) { return kp <= 32 || (kp == 64 && d <= FASTH_FUSED64_MAX_D); }

#ifndef FASTH_GRAM_SPLIT_128
#define FASTH_GRAM_SPLIT_128 8
#endif
// The result does not depend on how consecutive reflections are grouped into blocks (Eq. 2 holds for any grouping), so
// the library takes the grouping that costs least, whatever the caller's block size. The last block is filled up with zero
// rows, and vectors whose length is not a multiple of 4 with zeros, in a copy of V that the factor kernels write as they fetch
// the rows. Without it such shapes ran on the general kernels (short steps, rows that are not 16-byte aligned, no matrix cores).
// Forward + backward before and after, us: d = n = 784, k = 28, m = 32: 90.7 -> 71.6, m = 200: 103.9 -> 93.7;
// d = n = 1000, k = 50, m = 32: 156 -> 82, m = 600: 569 -> 225, m = 2000: 1534 -> 542; d = n = 1023, k = 33, m = 32: 232 -> 81;
// d = 511, n = 500, k = 25, m = 64: 76.5 -> 49.2; d = n = 2047, k = 23, m = 32: 570 -> 179; d = n = 1024, k = 16, m = 32: 121 -> 75.
// Blocks of 32 rows have the cheapest factors and the smallest product E V_i; the chain kernels take 32, 64 or 128 rows per step
// whatever the block. Blocks of 64 save half as many inputs, which pays once the two chains' saved inputs are well beyond
// the 256 MB of the memory-side cache, and are what dv_trio_kernel takes. us per forward + backward with blocks of 32, 64 and 128
// rows: d = n = 128, m = 100: 25, 37, 67; d = n = 512, m = 64: 46, 59, -; m = 300: 72, 88, -; d = n = 1024, m = 32: 72, 73, 86; m = 200:
// 122, 132, 174; d = n = 2048, m = 64: 184, 185, 208; m = 440 (231 MB of saved inputs per chain): 809, 779, -; d = n = 2560, m = 200
// (164 MB): 705, 727, -; d = n = 3072, m = 130 (153 MB): 861, 877, -; m = 200 (236 MB): 1064, 923, -.
// A caller's larger blocks (k > 32) need half the memory for the saved inputs; they become blocks of 64 for vectors of more than 1536
// elements from 64 columns on, where that costs nothing on the average. us with blocks of 32 and 64, repeated / inputs and workspace
// new to the caches in each pass: d = n = 2048, m = 64: 184, 185 / 189.5, 190 (three sets in turn, which fit the cache with blocks of
// 64 only: 189.6, 185.7); d = 2048, n = 1024, m = 64: 106, 105 / 110, 109; d = n = 2048, m = 200: 393, 400 / 446, 409; d = n = 3072, m = 100: 842,
// 854 / 844, 875; d = 4096, n = 1024, m = 200: 408, 407 / 455, 413; but with fewer columns: d = n = 2048, m = 32: 157, 161 / 163, 167; d = n =
// 3072, m = 32: 281, 291 / 287, 297; d = n = 4096, m = 8: 392, 417 / 404, 430; and shorter vectors: d = n = 1600, m = 64: 145, 147 / 149, 151.
// From 897 columns on, where the chains run on the matrix cores and hardly wait, half the saved inputs pay from 25 MB per chain on: blocks
// of 32 and 64, d = 1024, m = 1000: n = 192 (25 MB): 94, 92; n = 256: 114, 107; d = 512, m = 1500: n = 384 (37 MB): 126, 122; n = 512:
// 156, 140; d = 2048, m = 1000: n = 128 (33 MB): 142, 132; but m = 800: d = 512, n = 768: 173, 187; d = 640, n = 576: 135, 142.
// Never where rounding n up to 64 adds a step of 32 that matters: d = 2048, m = 4096, n = 32: 114, 140; d = 3072, m = 800, n = 160: 281, 309;
// n = 288: 416, 437; it matters least on the matrix cores: d = 2048, m = 1000, n = 288: 200, 173; m = 4096, n = 160: 311, 286
// (d = 640, m = 2100, n = 160: 112, 129).
constexpr double kManySavedBytes = 2e8, kManySavedBytesTiles = 2.5e7;
static int padded_rows(int n, int multiple) { return (n + multiple - 1) / multiple * multiple; }
static bool fills_64(int d, int n, int m) {
  return n > 320 || padded_rows(n, 64) == padded_rows(n, 32) || (d <= 2048 && (m > 2048 && d > 1024 ? n > 128 : m > 896 ? n > 192 : m > 768 && n > 256));
}
static int inner_block(int d, int n, int m, int k) {
  const double saved = 4.0 * ((n + 31) / 32) * m * d;
  return fills_64(d, n, m) && ((k > 32 && d > 1536 && m >= 64) || saved >= (m > 896 ? kManySavedBytesTiles : kManySavedBytes)) ? 64 : 32;
}
// A caller's larger blocks bound the memory for the saved inputs (n / k of them per chain): smaller ones than the caller's are taken
// only while the workspace grows by no more than this.
constexpr double kExtraSavedBytes = 1073741824.0;
static int bounded_block(int d, int n, int m, int k, int block) {
  auto saved = [&](int rows) { return 8.0 * ((n + rows - 1) / rows) * m * d; };
  while (block >= 32 && block < 128 && block < k && saved(block) - saved(k) > kExtraSavedBytes) block *= 2;
  return block;
}
// Blocks are a grid dimension of the factor and dV launches (n / 64 of them and n / 128 pairs at most): beyond this many reflections
// blocks of 128 rows and nothing shared.
constexpr int kMaxBlocks = 65535, kManyReflections = 64 * (kMaxBlocks / 2);

// Few reflections in small blocks (the caller's k < 32): blocks of 16 rows, whose factors cost least, and steps of 16 rows on the kernels
// for one column per workgroup and on chain_tile_kernel, without hand-overs and with the least padding. How many are few depends on
// what serves otherwise. us per forward + backward with blocks of 16 and with the best other choice, d: m: (n: blocks of 16, other):
// 256: 128: (112: 24, 26), (160: 27.5, 27.7); 300: (160: 38, 39), (192: 41, 41); 1000: (112: 49.5, 50), (128: 51, 50); 1500: (112: 65, 69)
// 512: 128: (128: 29, 30), (160: 31, 31); 600: (112: 56, 59), (128: 61, 58); 1500: (64: 59, 83), (128: 77, 86), (160: 89, 84)
// 1024: 32: (128: 29, 31), (192: 35, 37), (224: 38, 37); 300: (128: 51, 58), (320: 79, 82); 600: (80: 62, 67), (112: 69, 67);
//       1000: (48: 69, 70), (64: 76, 71); 1500: (48: 73, 81), (64: 84, 81)
// 1280: 64: (160: 38, 43), (192: 44, 43); 100: (192: 48, 51); 1100: (64: 88, 103)
// 2048: 8: (96: 33, 34), (112: 38, 34); 32: (96: 34, 36), (128: 38, 35); 300: (224: 119, 122), (256: 132, 132); 1000: (32: 115, 131), (48: 129, 132), (64: 145, 131)
// 4096: 32: (16: 32, 35), (24: 41, 38); 128: (256: 128, 131); 300: (192: 201, 203); 600: (128: 237, 239); 1500: (48: 361, 419), (64: 409, 382)
// Short columns and few of them: a launch each whatever the blocks, and fewer steps with 32 rows (d = 64, m = 32, n = 64: 21.5, 20).
constexpr int kFewRows = 16;
static bool few_reflections(int d, int n, int m) {
  if (d <= 256 && m <= 128) return false;
  if (d <= 256 && m <= 2048) return n <= (m <= 512 ? 160 : 112);
  if (d <= 512) return m > 2048 ? n <= 48 || (n > 64 && n <= 80) : n <= (m <= 256 || m > 896 ? 128 : 112);
  if (m > 2048) return n <= 16 || (n > 32 && n <= 48 && d <= 1536);  // 48: a third of the second 32 would be padding
  if (m > 1024 && d > 2048) return n <= 16 || (n > 32 && n <= 48);
  if (m > 1024) return n <= (m > 1280 || d > 1536 ? 48 : d <= 768 ? 80 : d <= 1024 ? 48 : 64);
  if (d <= 1024) return n <= (m <= 256 ? 192 : m <= 480 ? 576 : m <= 768 ? 96 : d <= 896 ? 80 : 48);
  if (d <= 2048) return n <= (m <= 64 ? (d <= 1536 ? 160 : 96) : m <= 128 ? (d <= 1536 ? 192 : 128) : m < 640 ? 256 : 48);
  if (team_fits(m, (d + kTeamSlice - 1) / kTeamSlice)) return n <= (d <= 3072 ? 32 : 16);
  return n <= (m <= 256 ? 256 : m <= 512 ? 192 : 112);
}
// Blocks of 8 rows (the caller's k <= 8) where a sixth or more of the blocks of 16 would be padding, and where steps of 8 rows keep twice as
// many workgroups on a compute unit: us with blocks of 8 and of 16: d = 1024, m = 800: n = 8: 49, 54; n = 24: 56, 61; d = 2048, m = 32:
// n = 24: 23, 26; m = 449: n = 8: 50, 59; n = 64: 71, 77; n = 128: 98, 98; d = 1280, m = 300: n = 64: 49, 54; n = 160: 71, 75;
// d = 64, m = 1100: n = 64: 35, 46 (tiles); n = 128: 44, 60; d = 256, m = 1100: n = 96: 55, 57.
static bool fewest_rows(int d, int n, int m) {
  if ((n - 1) % 16 < 8) {
    if (d > 2048) return n <= (m > 1024 ? 8 : team_fits(m, (d + kTeamSlice - 1) / kTeamSlice) ? 24 : m <= 300 ? 72 : 40);
    if (n <= 40) return m <= 1024 || (d <= 256 && m <= 1280);
  }
  if (d > 1024 && d <= 2048 && m > 256 && m <= 1024) return n <= (m > 480 ? 48 : d <= 1280 ? 360 : d <= 1536 ? 160 : 120);
  return d <= 256 && m > 1024 && (d <= 128 ? m <= 1536 && n <= 256 : m <= 1280 && n <= 128);
}
// Vectors of more than 2048 elements take steps of 8 rows, so blocks of 24 save padding: us with blocks of 24 and of 16 or 32: d = 3072,
// m = 300: n = 24: 80, 86; n = 72: 102, 116; n = 360: 259, 271; but their factors cost more than those of 16: m = 32, n = 20: 40, 33.
static int least_padding(int d, int n, int rows) {
  return d > 2048 && 25 * padded_rows(n, 24) <= 24 * padded_rows(n, rows) ? 24 : rows;
}

// Rows as the kernels see them, blocks of k. The kernels in which workgroups share columns need whole steps of 64 or 128 rows, and
// padding n up to them pays where they gain more than the padding costs. us per forward + backward without and with:
// columns of up to 1024 elements: d = 1024, m = 32: n = 160: 33, 37; n = 288: 42, 44; n = 448: 61, 50 (128); longer columns always;
// tiles of 16 columns: d = 512, m = 1000: n = 160: 75, 85; n = 224: 87, 92; m = 1500: n = 224: 107, 100; d = 1024, m = 449: n = 288: 71, 73;
// m = 600: n = 160: 84, 79; m = 800: n = 96: 76, 73; d = 640, m = 800: n = 96: 62, 65; beyond 1024 elements they take
// steps of 32, two at least: d = 2048, m = 1000: n = 32: 170, 132.
// Steps of 128 rows take less than twice as long as steps of 64 (2.65 against 1.95 us at d = 1024) but their launch more: d = 2048,
// m = 32: n = 192: 40 with steps of 64, 45 padded to 256; n = 320: 50, 55; n = 576: 76, 72.
static int steps_rows(int d, int n, int m, int k) {
  const int own = padded_rows(n, k), r64 = padded_rows(n, k < 64 ? 64 : k), r128 = padded_rows(n, kWideRows);
  if (team_tile_parts(d, r64, m, k)) return (d > 1024 && n > 32) || n <= (d > 1024 ? 0 : d <= 512 ? (m <= 1024 ? 256 : 192) : m < 512 ? 320 : d <= 896 ? 96 : 64) ? own : r64;
  if (d <= 1024 && (m <= 64 ? n <= 192 || (n > 256 && n <= 288) : n <= 320)) return own;
  if (n > 448 && team_wide_parts(d, r128, m, k)) return r128;
  return team_parts(d, r64, m, k) || team_wide_parts(d, r64, m, k) ? r64 : own;
}

// kLayoutPlain: the caller's own blocks, nothing shared and nothing padded: vectors too long for the register-resident kernels, and what
// fasth_forward_static refuses by. kLayoutShared: without the operands of V for chain_trio_kernel.
constexpr int kMaxPaddedD = 4096;
enum LayoutLevel { kLayoutPlain, kLayoutShared, kLayoutTrio };
static Layout make_layout(int d, int n, int m, int k, LayoutLevel level = kLayoutTrio) {
  const bool shared = level >= kLayoutShared;
  Layout L;
  L.dp = d; L.np = n; L.ki = k;
  const int d4 = (d + 3) & ~3;
  const bool fewest = k <= 8 && fewest_rows(d4, n, m);
  const bool many = n > kManyReflections && d <= kMaxPaddedD;
  L.trio = level == kLayoutTrio && !fewest && !many ? trio_plan(d4, n, m) : TrioPlan{0, 0, 0};
  if (L.trio.parts) {
    L.dp = d4;
    L.ki = bounded_block(d4, n, m, k, 64);
    L.np = padded_rows(n, L.ki);
  } else if (shared && many) {
    L.dp = d4;
    L.ki = kMaxBlock;
    L.np = padded_rows(n, kMaxBlock);
  } else if (shared && d <= kMaxPaddedD) {
    L.dp = d4;
    L.ki = fewest ? 8 : k < 32 && few_reflections(d4, n, m) ? kFewRows : inner_block(d4, n, m, k);
    // dv_trio_kernel takes 64 rows; blocks of 32 would save twice as many inputs, and the chain kernels for so many columns
    // take 64 rows per step whatever the block
    if (L.ki > kFewRows && fills_64(d4, n, m) && dv_trio_serves(d4, n, m, 64)) L.ki = 64;
    L.ki = bounded_block(d4, n, m, k, L.ki);
    L.np = L.ki <= kFewRows ? padded_rows(n, L.ki) : steps_rows(d4, n, m, L.ki);
    // (no kernel with shared columns: those have taken whole steps)
    if ((L.ki == 32 || (L.ki == kFewRows && m > 256)) && !team_parts(d4, L.np, m, L.ki) && least_padding(d4, n, L.ki) == 24) {
      L.ki = 24;
      L.np = padded_rows(n, 24);
    }
  }
  L.copy_v = L.dp != d || L.np != n;
  d = L.dp; n = L.np; k = L.ki;
  L.kp = padded_block(k);
  L.nb = n / k;
  const bool others = shared && !L.trio.parts && !many;
  const int team = others ? team_parts(d, n, m, k) : 0, wide = others ? team_wide_parts(d, n, m, k) : 0;
  const int ttile = others ? team_tile_parts(d, n, m, k) : 0;
  // The kernels in which workgroups share columns take 64 rows (32: the shared tiles at d > 1024) of factor per step
  // whatever the caller's block size: two blocks of 32 merged by Lemma 1, or the diagonal blocks of a larger block's
  // factor, which are the factors of its row groups; so only those are built.
  L.kf = wide || team || L.trio.parts ? 64 : ttile ? (d <= 1024 ? 64 : 32) : k;
  L.team_wide = wide;
  L.npair = wide ? n / kWideRows : 0;
  L.kpf = padded_block(L.kf);
  L.nbf = n / L.kf;
  int split = (d + kGramChunk - 1) / kGramChunk;
  L.gram_split = split > kMaxGramSplit ? kMaxGramSplit : split;
  // factors of 128 rows: the workgroup that adds the partial matrices fetches four of them per trip to memory
  if (L.kpf == 128 && L.gram_split > FASTH_GRAM_SPLIT_128) L.gram_split = FASTH_GRAM_SPLIT_128;
  size_t off = 256;  // header, reserved
  auto take = [&](size_t floats) {
    size_t o = off;
    off = align_up(off + floats * sizeof(float), 256);
    return o;
  };
  L.off_V = take(L.copy_v ? (size_t)n * d : 0);
  L.off_frag = take(L.trio.parts ? (size_t)(n / 64) * ((d + 31) / 32) * (24 * 1024 / 4) : 0);
  L.off_T = take(2 * (size_t)L.nbf * L.kpf * L.kpf);  // the factors and, behind them, their transposes
  // partial Gram matrices, later the dV kernel's per-block matrices Z (nb kp^2 floats), and,
  // where the Gram product is split over workgroups, an 8-byte "ready" word per partial matrix
  L.off_Spart = take(std::max((size_t)(L.nbf + L.npair) * L.gram_split * L.kpf * L.kpf, (size_t)L.nb * L.kp * L.kp));
  L.off_ready = take(factor_is_fused(L.kpf, d) ? 0 : (size_t)(L.nbf + L.npair) * L.gram_split * 2);
  L.off_S = take(2 * (size_t)L.npair * L.kpf * L.kpf);  // per pair V_a V_b^T and its transpose
  L.xch_words = wide ? (size_t)m * team_wide_words_per_column(wide)
              : team ? (size_t)m * team_words_per_column(team)
              : ttile ? (size_t)((m + 15) / 16) * team_tile_words(ttile)
              : L.trio.parts > 1 ? (size_t)((m + 16 * L.trio.ct - 1) / (16 * L.trio.ct)) * trio_words(L.trio.parts, L.trio.ct)
              : others && split_pair_serves(d, m, k) ? (size_t)m * kSplitPairWords : 0;
  L.off_xch = take(L.xch_words);
  L.off_saveA = take((size_t)L.nb * m * d);
  L.off_saveCa = take((size_t)m * n);
  L.off_saveG = take((size_t)L.nb * m * d);
  L.off_saveCg = take((size_t)m * n);
  L.dv_trio = shared && dv_trio_serves(d, n, m, k);
  L.dv_split = L.dv_trio ? dv_trio_split(d, n, m) : dv_minibatch_split(d, n, m, k);
  L.off_dVpart = take(L.dv_split > 1 ? (size_t)L.dv_split * n * d : 0);
  L.off_Zpart = take(L.dv_trio && L.dv_split > 1 ? (size_t)L.dv_split * n * k : 0);
  L.total = off;
  return L;
}

static int check_shape(const fasth_shape* s) {
  if (!s) return FASTH_EINVAL;
  if (s->d < 1 || s->n < 1 || s->m < 1 || s->k < 1) return FASTH_EINVAL;
  if (s->n % s->k != 0) return FASTH_EINVAL;
  if (s->transpose != 0 && s->transpose != 1) return FASTH_EINVAL;
  if (s->k > kMaxBlock || s->d > kMaxD || s->m > 65535) return FASTH_EUNSUPPORTED;
  if (s->n / s->k > kMaxBlocks) return FASTH_EUNSUPPORTED;
  return FASTH_OK;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Text of the last HIP error a call of this thread ran into, for fasth_strerror(FASTH_EHIP).
static thread_local char g_hip_error_text[192] = "";
static int note_hip_error(hipError_t e, const char* what) {
  snprintf(g_hip_error_text, sizeof(g_hip_error_text), "HIP runtime call or kernel launch failed: %s (%s)",
           hipGetErrorString(e), what);
  return FASTH_EHIP;
}

#define FASTH_HIP(call)                                    \
  do {                                                     \
    hipError_t e_ = (call);                                \
    if (e_ != hipSuccess) return note_hip_error(e_, #call); \
  } while (0)

// Optional per-kernel timing for benchmarks: a pair of HIP events around every launch.
// "kernel<a, b, c>": the instantiation a launcher picked, as a profiler prints it.
static std::string variant_name(const char* base, std::initializer_list<int> args) {
  std::string s(base);
  s += "<";
  bool first = true;
  for (int a : args) {
    if (!first) s += ", ";
    s += std::to_string(a);
    first = false;
  }
  return s + ">";
}

namespace prof {
struct Rec { int id; hipEvent_t beg, end; };
constexpr size_t kMaxRecords = 1u << 16;  // launches recorded between two collects; later ones go untimed
static bool enabled = false;
static std::vector<Rec> recs;
static std::vector<hipEvent_t> pool;
static const char* variant[FASTH_KERNEL_COUNT] = {};  // instantiation last launched per slot while enabled
static hipEvent_t get_event() {
  if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}
struct Scope {
  Rec r{-1, nullptr, nullptr};
  hipStream_t st;
  Scope(int id, hipStream_t s, const char* name = nullptr) : st(s) {
    if (!enabled) return;
    if (name && id >= 0 && id < FASTH_KERNEL_COUNT) variant[id] = name;
    if (recs.size() >= kMaxRecords) return;
    r.id = id; r.beg = get_event(); r.end = get_event();
    if (r.beg) (void)hipEventRecord(r.beg, st);
  }
  ~Scope() {
    if (r.id < 0) return;
    if (r.end) (void)hipEventRecord(r.end, st);
    recs.push_back(r);
  }
};
}  // namespace prof

// Kernels that ask for more than 64 KiB of dynamic LDS must be allowed to, once per kernel and device; the size
// granted so far is remembered per kernel (a small table under a mutex) so that the timed path makes no such call.
struct LdsGrant { const void* kernel; int device; size_t bytes; };
static std::vector<LdsGrant> g_lds_grants;
static std::mutex g_lds_mutex;

template <typename K>
static int allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return FASTH_OK;
  const void* fn = reinterpret_cast<const void*>(kernel);
  int dev = 0;
  FASTH_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(g_lds_mutex);
  for (LdsGrant& g : g_lds_grants) {
    if (g.kernel == fn && g.device == dev) {
      if (g.bytes >= bytes) return FASTH_OK;
      FASTH_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
      g.bytes = bytes;
      return FASTH_OK;
    }
  }
  FASTH_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  g_lds_grants.push_back(LdsGrant{fn, dev, bytes});
  return FASTH_OK;
}

}  // namespace fasth
