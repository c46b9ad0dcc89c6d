// Dense fp32 matrix products on the bf16 matrix cores (three-piece operands, fasth_device.h): gemm_kernel, and pack_kernel, which
// lays a matrix out as its operands.
// Included by fasth_dense.h.
#pragma once
#include <hip/hip_runtime.h>

#include "fasth_chain.h"
#include "fasth_common.h"
#include "fasth_factor.h"

namespace fasth {

// ------------------------------------------------------------------------------------------
// Operands. A matrix whose rows are an operand's rows (of A) or columns (of B) and whose columns are the inner index k is stored as tiles of 16 rows
// x 32 k: three pieces of 1 KiB, slot 16 kq + row of a piece holding k = 8 kq .. 8 kq + 7 of that row, which is what lane 16 kq + row of
// v_mfma_f32_16x16x32_bf16 reads. Tiles of a row of tiles follow one another; rows and k are padded with zeros to multiples of 64,
// so that no product has an edge. 6 bytes per element. The odd tiles of k are stored with the opposite sign: where an addend is much smaller than
// another, v_mfma_f32_16x16x32_bf16 cuts it off downwards, whatever its sign (mean error -6e-9 of the sum's size per instruction, rms 3.7e-8, with an
// accumulator 2^-8 of the products). Added over all tiles of k that leaves errors of one direction, which a product with rows of one sign adds up; so half of
// a sum is formed as -(-a) b. Where both operands are stored this way the signs cancel.
// ------------------------------------------------------------------------------------------
constexpr int kTileBytes = 3 * 1024;
static __host__ __device__ __forceinline__ int pad64(int x) { return (x + 63) & ~63; }
static __host__ __device__ __forceinline__ size_t packed_bytes(int rows, int k) { return (size_t)pad64(rows) * pad64(k) * 6; }

// Eight consecutive k of a row: slot kq of (row, k / 32).
__device__ __forceinline__ void store_unit(char* pack, int kt, int row, int k8, const float (&v)[8]) {
  const unsigned sign = (unsigned)(k8 & 4) << 29;
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(__float_as_uint(v[e]) ^ sign);
  const Trio t = split8(x);
  u32x4* dst = reinterpret_cast<u32x4*>(pack + ((size_t)(row >> 4) * kt + (k8 >> 2)) * kTileBytes) + (k8 & 3) * 16 + (row & 15);
#pragma unroll
  for (int pc = 0; pc < 3; ++pc) dst[pc * 64] = __builtin_bit_cast(u32x4, t.p[pc]);
}

// A matrix of rows x cols as operands, from LDS or memory: `along`, its rows stay rows (k = column); `across`, its columns become rows (k = row).
struct PackJob {
  const float* src;   // [rows][cols]
  char* along;        // or null
  char* across;       // or null
  int rows, cols;
  int blocks;         // 64 x 64 blocks, padding included (0: no job); rows beyond `rows` are zero
};
constexpr int kPackJobs = 4;
struct PackArgs {
  PackJob job[kPackJobs];  // blockIdx.y
};

// One 64 x 64 block per workgroup of 256 threads, through LDS: reads 4 bytes per element and writes 6 per kind.
typedef float PackTile[64][65];
__device__ __forceinline__ void pack_block(const PackJob& p, int block, PackTile& tile) {
  const int bc = pad64(p.cols) / 64, r0 = block / bc * 64, c0 = block % bc * 64;
  const int tid = threadIdx.x, c = tid & 63;
  const BufferDesc desc = make_buffer(p.src + (size_t)r0 * p.cols, (size_t)max(0, min(64, p.rows - r0)) * p.cols * sizeof(float));
  float x[16];
#pragma unroll
  for (int it = 0; it < 16; ++it)
    x[it] = buffer_load<1>(desc, c0 + c < p.cols ? (unsigned)((it * 4 + (tid >> 6)) * p.cols + c0 + c) * 4u : kOob, 0).e[0];
#pragma unroll
  for (int it = 0; it < 16; ++it) tile[it * 4 + (tid >> 6)][c] = x[it];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2; ++it) {  // a wave writes a piece of a tile: rows fastest
    const int u = tid + it * 256, row = (u >> 7) * 16 + (u & 15), k8 = (u >> 4) & 7;
    float v[8];
    if (p.along) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = tile[row][8 * k8 + e];
      store_unit(p.along, pad64(p.cols) / 32, r0 + row, c0 / 8 + k8, v);
    }
    if (p.across) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = tile[8 * k8 + e][row];
      store_unit(p.across, p.blocks / bc * 2, c0 + row, r0 / 8 + k8, v);
    }
  }
}

__global__ void __launch_bounds__(256) pack_kernel(PackArgs args) {
  __shared__ PackTile tile;
  const PackJob& p = args.job[blockIdx.y];
  if ((int)blockIdx.x < p.blocks) pack_block(p, (int)blockIdx.x, tile);
}

// ------------------------------------------------------------------------------------------
// Products
// ------------------------------------------------------------------------------------------
struct GemmTerm {
  const char* A;     // operands; lda tiles of k per row of tiles
  const char* B;     // operands, or fp32 [k][cols] (the kernels' BF)
  int lda, ldb;      // tiles of k per row of tiles (fp32 B: its row length)
  int K;             // inner indices (fp32 B: its rows)
  bool upper;        // A is upper triangular: a tile of rows from r0 on needs k from r0 on
};
enum { kUpper = 1, kStrict = 2, kAccumulate = 4 };
// out = alpha sum + beta add, + 1 on the diagonal with diag = 1. Every output is optional.
struct GemmProblem {
  GemmTerm term;
  int tiles, rows, cols;
  int ldo;              // row length of the fp32 outputs and of `add`
  int flags;            // kUpper: tiles on and above the diagonal only; kStrict: zero on and below the diagonal;
                        // kAccumulate: out is added to
  float alpha, beta, diag;
  const float* add;     // [rows][ldo]
  float* out;           // [rows][ldo]
  float* scaled;        // [scaled_rows][ldo]: diag_factor(scale_mode, scale[r]) out
  const float* scale;
  int scale_mode, scaled_rows;
  char* along;          // out as operands, see PackJob
  char* across;
  int along_kt, across_kt;  // tiles of k per row of tiles
  int split;            // > 0: the inner index in this many parts, out has [split][rows][ldo]
  int xcd_rows;         // > 0: each XCD takes a block of tiles, the grid of tiles cut into xcd_rows x (8 / xcd_rows)
};
constexpr int kGemmProblems = 8;
struct GemmArgs {
  GemmProblem p[kGemmProblems];  // blockIdx.y
};

// A finished tile in LDS ([BM][BN + 4], all NT threads, after a barrier) to wherever it goes.
template <int BM, int BN, int NT>
__device__ __forceinline__ void gemm_epilogue(const GemmProblem& p, float* tile, int r0, int c0, int part) {
  constexpr int LD = BN + 4;
  const int tid = threadIdx.x;
  const bool diagonal = r0 == c0;
  float* out = p.out ? p.out + (size_t)part * p.rows * p.ldo : nullptr;
  constexpr int PER = BM * BN / NT, CHUNK = PER < 8 ? PER : 8;
#pragma unroll 1
  for (int first = 0; first < PER; first += CHUNK) {
    float add[CHUNK];  // what is added comes in one trip to memory
    if (p.add) {
#pragma unroll
      for (int it = 0; it < CHUNK; ++it) {
        const int u = tid + (first + it) * NT, r = u / BN, c = u % BN;
        add[it] = r0 + r < p.rows && c0 + c < p.cols ? p.add[(size_t)(r0 + r) * p.ldo + c0 + c] : 0.f;
      }
    }
#pragma unroll
    for (int it = 0; it < CHUNK; ++it) {
      const int u = tid + (first + it) * NT, r = u / BN, c = u % BN;
      float v = p.alpha * tile[r * LD + c];
      if (p.add) v += p.beta * add[it];
      if (diagonal && r == c) v += p.diag;
      const bool inside = r0 + r < p.rows && c0 + c < p.cols;
      if (!inside || ((p.flags & kStrict) && r0 + r >= c0 + c)) v = 0.f;
      if (inside && out) {
        float* dst = out + (size_t)(r0 + r) * p.ldo + c0 + c;
        *dst = (p.flags & kAccumulate) ? *dst + v : v;
      }
      tile[r * LD + c] = v;
    }
  }
  if (p.scaled) {
#pragma unroll 1
    for (int it = 0; it < PER; ++it) {
      const int u = tid + it * NT, r = u / BN, c = u % BN;
      if (r0 + r < p.scaled_rows && c0 + c < p.cols) p.scaled[(size_t)(r0 + r) * p.ldo + c0 + c] = diag_factor(p.scale_mode, p.scale[r0 + r]) * tile[r * LD + c];
    }
  }
  if (!p.along && !p.across) return;
  __syncthreads();
  if (p.along) {
#pragma unroll 1
    for (int it = 0; it < (PER + 7) / 8; ++it) {
      const int u = tid + it * NT, row = u / (2 * BN) * 16 + (u & 15), k8 = (u >> 4) % (BN / 8);
      if ((PER >= 8 || u < BM * BN / 8) && r0 + row < pad64(p.rows) && c0 + 8 * k8 < pad64(p.cols)) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = tile[row * LD + 8 * k8 + e];
        store_unit(p.along, p.along_kt, r0 + row, c0 / 8 + k8, v);
      }
    }
  }
  if (p.across) {
#pragma unroll 1
    for (int it = 0; it < (PER + 7) / 8; ++it) {
      const int u = tid + it * NT, row = u / (2 * BM) * 16 + (u & 15), k8 = (u >> 4) % (BM / 8);
      if ((PER >= 8 || u < BM * BN / 8) && c0 + row < pad64(p.cols) && r0 + 8 * k8 < pad64(p.rows)) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = tile[(8 * k8 + e) * LD + row];
        store_unit(p.across, p.across_kt, c0 + row, r0 / 8 + k8, v);
      }
    }
  }
}

// Tile coordinates of a workgroup. Workgroups b, b + 8, ... run on one XCD (grids are multiples of 8 wide): they take consecutive
// tiles, which share operands. False: no tile.
template <int BM, int BN>
__device__ __forceinline__ bool gemm_tile(const GemmProblem& p, int& r0, int& c0, int& part) {
  int t = (int)blockIdx.x;
  const int per = p.tiles / 8, more = p.tiles % 8, x = t & 7;
  const int index = t >> 3;
  if (index >= per + (x < more ? 1 : 0)) return false;
  t = x * per + min(x, more) + index;
  part = 0;
  if (p.split > 0) {
    const int each = p.tiles / p.split;
    part = t / each;
    t %= each;
  }
  int ti, tj;
  if (p.flags & kUpper) {  // tile columns of 1, 2, ... tiles (square outputs, square tiles)
    tj = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((tj + 1) * (tj + 2) / 2 <= t) ++tj;
    while (tj * (tj + 1) / 2 > t) --tj;
    ti = t - tj * (tj + 1) / 2;
  } else {
    // an XCD keeps few row panels, or few column panels, whichever there are more of
    const int rt = (pad64(p.rows) + BM - 1) / BM, ct = (pad64(p.cols) + BN - 1) / BN;
    if (p.xcd_rows > 0) {
      const int br = rt / p.xcd_rows, bc = ct * p.xcd_rows / 8;
      ti = x % p.xcd_rows * br + index % br;
      tj = x / p.xcd_rows * bc + index / br;
    } else if (rt > ct) { ti = t / ct; tj = t % ct; }
    else { ti = t % rt; tj = t / rt; }
  }
  r0 = ti * BM;
  c0 = tj * BN;
  return true;
}

// First and last tile of k.
__device__ __forceinline__ void gemm_range(const GemmTerm& g, int r0, int split, int part, int& beg, int& end) {
  beg = g.upper ? r0 / 32 : 0;
  end = pad64(g.K) / 32;
  if (split > 0) {
    const int each = ((end - beg) / 2 + split - 1) / split * 2;
    beg += part * each;
    end = min(end, beg + each);
  }
}

// A wave forms 16 RT x 16 CT outputs and fetches its operands straight into registers, a tile of k ahead; WM x WN waves make up a
// workgroup's tile and KS such groups share the inner index. No LDS and no barrier before the sums meet: waves that share an operand find it in
// the compute unit's cache. BF: B is fp32 [k][cols], split in registers: 1, a load per column; 2, where its rows are made of groups of four, a
// load per lane takes the columns of all column tiles, so that lane i's are CT i, CT i + 1, ... of the wave's.
// 1024 x 4096 x 1024: 54 us packed; BF 58 .. 60 us (62 with loads of one column each), 143 TF/s of fp32 products, which are six bf16 products each
// (the matrix cores' limit: 335, 25 us). Bound by what the waves issue, vector and matrix instructions after one another: of 108 thousand cycles in which a
// compute unit is busy a SIMD spends 49 on matrix instructions and 50 on others (packed: 83, 49 and 17; counters). Without the split 47 us, without the loads 45, with
// every load from the same addresses 57, so neither memory nor the L2s; some 8 are launch, first fetch and the way out. 1024 x 1024 x 1024: 17 us; 1024 x 256 x 1024: 7.2;
// the smallest: 4.9, launch and code fetch. The same products with both operands staged in LDS took 57 us at 1024 x 4096 x 1024 (packed) and 67 us
// (split on the way); a barrier per tile of k, for waves that share an operand to fetch it together: 63.
template <int RT, int CT, int WM, int WN, int KS, int BF>
__global__ void __launch_bounds__(64 * WM * WN * KS) gemm_kernel(GemmArgs args) {
  constexpr int BM = 16 * RT * WM, BN = 16 * CT * WN, LD = BN + 4;
  extern __shared__ __align__(16) float tile[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, i = lane & 15;
  const int ks = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
  const GemmProblem& p = args.p[blockIdx.y];
  int r0, c0, part;
  if (!gemm_tile<BM, BN>(p, r0, c0, part)) return;

  // A tile of k is summed by itself, the small products first and the leading one last, and added to what is there: one rounding of full size
  // per 32 terms, and another in the sum.
  f32x4 sum[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) sum[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const unsigned lane_off = (unsigned)lane * 16u;
  auto multiply_row = [&](int r, const Trio& a, const Trio (&b)[CT]) {
    f32x4 part[CT];
#pragma unroll
    for (int u = 0; u < 6; ++u) {
      constexpr int kLeft[6] = {2, 0, 1, 0, 1, 0}, kRight[6] = {0, 2, 1, 1, 0, 0};
#pragma unroll
      for (int c = 0; c < CT; ++c)
        part[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[kLeft[u]], b[c].p[kRight[u]], u == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : part[c], 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < CT; ++c) sum[r][c] += part[c];
    __builtin_amdgcn_sched_barrier(0);  // (else the sums of all rows wait for the last product, in registers that are not there)
  };
  // the wave's first tiles (panels that lie beyond the last are the last one: what they give is not stored)
  const int ra = r0 / 16 + wm * RT, cb = c0 / 16 + wn * CT, last_r = pad64(p.rows) / 16 - 1, last_c = pad64(p.cols) / 16 - 1;
  const GemmTerm g = p.term;
  int beg, end;
  gemm_range(g, r0, p.split, part, beg, end);
  int k = beg + ks;
  if (k < end) {
    const char* A[RT];
    const char* B[CT];
    unsigned uoff[BF == 1 ? CT : 1];
#pragma unroll
    for (int r = 0; r < RT; ++r) A[r] = g.A + ((size_t)min(ra + r, last_r) * g.lda + k) * kTileBytes;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      if constexpr (BF == 1) uoff[c] = ((unsigned)(8 * q) * (unsigned)g.ldb + (unsigned)min((cb + c) * 16 + i, p.cols - 1)) * 4u;
      else if constexpr (BF == 2) uoff[0] = ((unsigned)(8 * q) * (unsigned)g.ldb + (unsigned)min(cb * 16 + CT * i, p.cols - CT)) * 4u;
      else B[c] = g.B + ((size_t)min(cb + c, last_c) * g.ldb + k) * kTileBytes;
    }
    // An operand of the next tile of k is fetched as soon as its registers have been read: one tile of k ahead. Beyond its last tile
    // a wave fetches that one again, so that every wait leaves as many fetches in flight.
    Trio ta[RT], tb[CT];
    float v[BF ? CT : 1][8];
    auto fetch_a = [&](int r) {
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) ta[r].p[pc] = *reinterpret_cast<const bf16x8*>(A[r] + pc * 1024 + lane_off);
    };
    auto fetch_b = [&]() {
      if constexpr (BF) {
        // rows of B that do not exist lie beyond the buffer and read as zero
        const BufferDesc desc = make_buffer(reinterpret_cast<const float*>(g.B) + (size_t)k * 32 * g.ldb, (size_t)max(g.K - 32 * k, 0) * g.ldb * sizeof(float));
#pragma unroll
        for (int c = 0; c < (BF == 2 ? 1 : CT); ++c) {
          unsigned off = uoff[c];
          asm("" : "+v"(off));  // (the eight offsets formed here again: kept over the loop, they would take registers)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const auto got = buffer_load<(BF == 2 ? CT : 1)>(desc, off, 0);
#pragma unroll
            for (int x = 0; x < (BF == 2 ? CT : 1); ++x) v[c + x][e] = got.e[x];
            off += (unsigned)g.ldb * 4u;
          }
        }
      } else {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
          for (int pc = 0; pc < 3; ++pc) tb[c].p[pc] = *reinterpret_cast<const bf16x8*>(B[c] + pc * 1024 + lane_off);
      }
    };
    fetch_b();
#pragma unroll
    for (int r = 0; r < RT; ++r) fetch_a(r);
    for (int left = (end - k + KS - 1) / KS; left > 0; --left) {
      if (k + KS < end) {
        k += KS;
#pragma unroll
        for (int r = 0; r < RT; ++r) A[r] += KS * kTileBytes;
        if constexpr (!BF) {
#pragma unroll
          for (int c = 0; c < CT; ++c) B[c] += KS * kTileBytes;
        }
      }
      Trio b[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        if constexpr (BF) b[c] = split8(v[c]);
        else b[c] = tb[c];
      }
      fetch_b();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        multiply_row(r, ta[r], b);
        fetch_a(r);
      }
    }
  }
  if constexpr (BF) {  // A's odd tiles of k have the other sign; a wave's are all odd or all even
    static_assert(KS % 2 == 0, "groups of waves take every KS-th tile of k");
    if ((beg + ks) & 1) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) sum[r][c] = -sum[r][c];
    }
  }
  // The groups' sums meet in LDS, 16 bytes per lane and tile, and all threads add them (in fp64: KS - 1 roundings of full size less); then the tile goes into rows.
  constexpr int NT = 64 * WM * WN * KS, UNITS = BM * BN / 4, PER = (UNITS + NT - 1) / NT;
  f32x4* parts = reinterpret_cast<f32x4*>(tile);  // [group][row tile][column tile][lane]
  auto to_rows = [&](int unit, f32x4 v) {
    const int l = unit & 63, t = unit >> 6, row = t / (BN / 16) * 16 + 4 * (l >> 4), ct = t % (BN / 16);
    const int col = BF == 2 ? ct / CT * (16 * CT) + CT * (l & 15) + ct % CT : ct * 16 + (l & 15);
#pragma unroll
    for (int j = 0; j < 4; ++j) tile[(row + j) * LD + col] = v[j];
  };
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) parts[ks * UNITS + ((wm * RT + r) * (BN / 16) + wn * CT + c) * 64 + lane] = sum[r][c];
  __syncthreads();
  f32x4 v[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int unit = tid + it * NT;
    if (UNITS % NT == 0 || unit < UNITS) {
      double x[4] = {0., 0., 0., 0.};
#pragma unroll
      for (int g = 0; g < KS; ++g) {
        const f32x4 part = parts[g * UNITS + unit];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] += (double)part[j];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) v[it][j] = (float)x[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int unit = tid + it * NT;
    if (UNITS % NT == 0 || unit < UNITS) to_rows(unit, v[it]);
  }
  __syncthreads();
  gemm_epilogue<BM, BN, 64 * WM * WN * KS>(p, tile, r0, c0, part);
}
template <int BM, int BN, int KS>
constexpr size_t gemm_lds() { return sizeof(float) * std::max((size_t)KS * BM * BN, (size_t)BM * (BN + 4)); }

// How the XCDs share the tiles: the cut whose blocks need the fewest bytes of both operands, as each XCD fetches them into its own
// L2; 0 (consecutive tiles) where no cut gives equal blocks.
static int xcd_cut(int rt, int ct, double a_bytes, double b_bytes) {
  int best = 0;
  double least = 0.;
  for (int r = 1; r <= 8; r *= 2) {
    if (rt % r || ct % (8 / r)) continue;
    const double bytes = rt / r * a_bytes + ct / (8 / r) * b_bytes;
    if (best == 0 || bytes < least) { best = r; least = bytes; }
  }
  return best;
}

}  // namespace fasth
