// The product of all reflections as one matrix, for wide mini-batches.
// Included by fasth.hip after the chain and dV kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "fasth_common.h"
#include "fasth_gemm.h"

namespace fasth {

// ------------------------------------------------------------------------------------------
// All n reflections are one WY block (Lemma 1 with k = n): with S = V V^T and T = (diag(S) / 2 + striu(S))^-1,
//   H = I - V^T T V = I - V^T Y,   Y = T V,     H^T = I - V^T T^T V.
// T is formed for groups of 256 reflections only. With P = H_(g+1) ... H_G the product of the groups applied before group g, the rows
// of Y that belong to it are Y_g = T_g V_g P, and P - V_g^T Y_g is the product with it: from P = I to P = H. (All of T, by doubling
// blocks, is as much work, and H is less exact.) Errors of A, dV and dX against fp64, n = d = 1024 and in brackets the chain of blocks of 64: normal V
// 2.1e-7, 3.2e-7, 2.0e-7 (4.5e-7, 4.8e-7, 4.1e-7). Rows far from orthogonal, A and dV: positive 2.7e-7, 1.1e-6 (1.4e-6, 1.8e-6); one direction
// plus 0.3 times normal 2.9e-7, 1.4e-6 (3.4e-6, 6.3e-6); four directions plus 0.01 times normal 5.4e-7, 7.8e-6 (2.8e-6, 2.9e-5). At d = 512, where the chain has
// blocks of 32: 1.9e-7, 2.9e-7 (5.1e-7, 7.4e-7); 2.3e-7, 6.1e-7 (9.4e-7, 1.3e-6); 3.3e-7, 9.2e-7 (2.0e-6, 4.1e-6); 6.8e-7, 5.1e-6 (1.1e-6, 8.6e-6). That takes S and the
// inverse in fp64 up to T: with S from three-piece products and fp32 factors of 64 rows the last were 2.3e-6, 2.3e-5.
// The chain of blocks costs 12 d n m operations per gradient step, one block after the other. As matrices a step costs 6 d^2 m and a
// part that does not depend on m:
//   forward   A = H X
//   backward  dX = H^T G,   Q = dX X^T,   K = (Q - Q^T) / 2,   W = Y K,   dV = 2 (W - striu(W Y^T) V)
// The gradient with respect to H is D = G X^T, and dL = <D, dH> = <H^T D, H^T dH> = <Q, H^T dH>. H stays orthogonal, so H^T dH is
// skew-symmetric and only the skew part K of Q counts: D may be replaced by H K. Differentiating H = I - V^T T V gives
//   dV = -(Y D^T + Y' D) + E V,   Y' = T^T V,   E = U + U^T + diag(Z),   Z = Y' D Y^T,   U = striu(Z),
// and V H = -T^-T Y, i.e. Y = -Y' H and Y' = -Y H^T, turns it for D = H K into Z = -W Y^T with W = Y K (skew, as K is), Y' D = -W and
// Y D^T = -W H^T = -W + W V^T T^T V = -W - Z V, so that dV = 2 W + (E + Z) V = 2 W + 2 U V.
// For A = H^T X with G = dL/dA the gradient with respect to H is D = X G^T and Q = H^T D = A G^T; the rest is the same, from the same Y. So one
// preparation serves products in both directions, saved or not.
// All products are three-piece bf16 products (fasth_gemm.h): fp32 in, fp32 out, fp32 accumulators.
// ------------------------------------------------------------------------------------------

constexpr int kGroup = 256;  // reflections that share a T

// S: the groups' V_g V_g^T, its tiles of 16 x 16 on and above the diagonal, with fp64 matrix instructions from the fp32 rows as they are. With rows far from
// orthogonal the rounding of S decides the error of H (T amplifies it). One tile per workgroup, its waves share the elements of the rows. Bound by the matrix
// instructions, 109 cycles each: d = n = 1024: 544 workgroups, up to three per compute unit, 14.3 us (with fp32 instructions and a sum in fp64 every 16
// elements some 8, but T is then off by 9e-8 of its size where the rows are normal and by 8e-7 where they are near one direction; here by 1e-14 and 1e-11).
// What else the step needs of V and X as operands is packed in the same launch, by workgroups behind these.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kGroupTiles = (kGroup / 16) * (kGroup / 16 + 1) / 2;
struct GramArgs {
  const float* V;  // [n][d]
  double* S;       // [np][256]
  int n, d, tiles; // tiles: kGroupTiles per group (0: no product)
};
struct GramPair {
  GramArgs a[2];   // blockIdx.y
  int width;       // workgroups with a larger blockIdx.x pack
};
template <int VEC>  // floats per load: 4 where d is a multiple of it, else 1
__global__ void __launch_bounds__(256) gram_kernel(GramPair pair, PackArgs pack) {
  typedef double Part[4][16][17];
  __shared__ __align__(16) char lds[std::max(sizeof(Part), sizeof(PackTile))];
  if ((int)blockIdx.x >= pair.width) {
    const PackJob& job = pack.job[blockIdx.y];
    const int block = (int)blockIdx.x - pair.width;
    if (block < job.blocks) pack_block(job, block, *reinterpret_cast<PackTile*>(lds));
    return;
  }
  if (blockIdx.y >= 2) return;
  Part& part = *reinterpret_cast<Part*>(lds);
  const GramArgs& p = pair.a[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, i = lane & 15;
  const int per = p.tiles / 8, index = (int)blockIdx.x >> 3;  // workgroups of one XCD take consecutive tiles, which share rows
  if (index >= per) return;
  const int tile = ((int)blockIdx.x & 7) * per + index, g = tile / kGroupTiles, t = tile % kGroupTiles;
  int tj = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);  // tile columns of 1, 2, ... tiles
  while ((tj + 1) * (tj + 2) / 2 <= t) ++tj;
  while (tj * (tj + 1) / 2 > t) --tj;
  const int ti = t - tj * (tj + 1) / 2, rows = min(kGroup, p.n - g * kGroup);
  if (16 * tj >= pad64(rows)) return;
  const BufferDesc desc = make_buffer(p.V + (size_t)g * kGroup * p.d, (size_t)rows * p.d * sizeof(float));  // rows that do not exist read as zero
  // lane (q, i): of each 16 elements the four from 4 q on of rows i (the sum may run in any order); 64 elements are a step, a step ahead is fetched
  const unsigned left = (unsigned)(16 * ti + i) * (unsigned)p.d, right = (unsigned)(16 * tj + i) * (unsigned)p.d;
  BufVec<4> a[2][4], b[2][4];
  auto fetch = [&](int s, int k0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int k = k0 + 16 * c + 4 * q;
#pragma unroll
      for (int e = 0; e < 4; e += VEC) {
        const bool in = k + e < p.d;
        const BufVec<VEC> x = buffer_load<VEC>(desc, in ? (left + k + e) * 4u : kOob, 0), y = buffer_load<VEC>(desc, in ? (right + k + e) * 4u : kOob, 0);
#pragma unroll
        for (int u = 0; u < VEC; ++u) { a[s][c].e[e + u] = x.e[u]; b[s][c].e[e + u] = y.e[u]; }
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // (else the loads wait until they are needed)
  };
  f64x4 acc[2] = {};
  auto multiply = [&](int s) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[s][c].e[e], (double)b[s][c].e[e], acc[e & 1], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  int k = 64 * wave;
  fetch(0, k);
  for (; k < p.d; k += 512) {
    fetch(1, k + 256);
    multiply(0);
    fetch(0, k + 512);
    multiply(1);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[wave][q + 4 * e][i] = acc[0][e] + acc[1][e];
  __syncthreads();
  const int r = tid >> 4, c = tid & 15;
  p.S[(size_t)(g * kGroup + 16 * ti + r) * kGroup + 16 * tj + c] = (part[0][r][c] + part[1][r][c]) + (part[2][r][c] + part[3][r][c]);
}

// The factors of 64 rows, (diag(S_bb) / 2 + striu(S_bb))^-1 = M^-1; a row that does not exist has a one on the diagonal. The inverse in fp32, F, and one step
// of refinement in fp64, F + F (I - M F). Bound by the steps of the inversion and the two products, one after the other: 7.2 us for any number of blocks up to one
// per compute unit (4.8 without the refinement).
struct FactorArgs64 {
  const double* S;  // [np][256]
  double* factor;   // [np / 64][64][64]
  int n, np;
};
struct FactorPair64 {
  FactorArgs64 a[2];  // blockIdx.y
};
__global__ void __launch_bounds__(512) block_factor_kernel(FactorPair64 pair) {
  constexpr int LD = 68, LDD = 66;
  __shared__ __align__(16) float F[64 * LD + invert_scratch_floats(64)];
  __shared__ double M[64 * LDD];
  const FactorArgs64& p = pair.a[blockIdx.y];
  const int r0 = (int)blockIdx.x * 64, tid = threadIdx.x;
  if (r0 >= p.np) return;  // whole workgroup
  float* Xs = F + 64 * LD;
  double s[8];
#pragma unroll
  for (int it = 0; it < 8; ++it) s[it] = p.S[(size_t)(r0 + (tid >> 6) + 8 * it) * kGroup + r0 % kGroup + (tid & 63)];
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int r = (tid >> 6) + 8 * it, c = tid & 63;
    const double v = r0 + r >= p.n || r0 + c >= p.n ? (r == c ? 1. : 0.) : r < c ? s[it] : r == c ? 0.5 * s[it] : 0.;
    M[r * LDD + c] = v;
    F[r * LD + c] = (float)v;
    diag_scratch_store(Xs, 64, r, c, (float)v);
  }
  __syncthreads();
  invert_upper_lds<true>(F, Xs, 64, LD);
  // tiles of 16 x 16 on and above the diagonal, the longest sums first: a wave's one, and a second for two waves
  const int lane = tid & 63, wave = tid >> 6, q = lane >> 4, i = lane & 15;
  const int tiles = wave < 6 ? 1 : 2;
  auto row_of = [&](int u) { return u > 0 ? wave - 4 : (0x10210100 >> (4 * wave)) & 15; };
  auto column_of = [&](int u) { return u > 0 ? wave - 4 : (0x10321323 >> (4 * wave)) & 15; };
  f64x4 acc[2] = {};
#pragma unroll
  for (int u = 0; u < 2; ++u) {  // I - M F
    if (u >= tiles) break;
    const int ti = row_of(u), tj = column_of(u);
    for (int k0 = ti; k0 <= tj; ++k0) {  // lane (q, i) takes inner indices 16 k0 + 4 q ...: every read is issued before the first product
      double m[4], f[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        m[e] = M[(16 * ti + i) * LDD + 16 * k0 + 4 * q + e];
        f[e] = -(double)F[(16 * k0 + 4 * q + e) * LD + 16 * tj + i];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(m[e], f[e], acc[u], 0, 0, 0);
    }
    if (ti == tj)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[u][e] += q + 4 * e == i ? 1. : 0.;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (u < tiles)
#pragma unroll
      for (int e = 0; e < 4; ++e) M[(16 * row_of(u) + q + 4 * e) * LDD + 16 * column_of(u) + i] = acc[u][e];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    if (u >= tiles) break;
    const int ti = row_of(u), tj = column_of(u);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[u][e] = F[(16 * ti + q + 4 * e) * LD + 16 * tj + i];
    for (int k0 = ti; k0 <= tj; ++k0) {
      double f[4], m[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f[e] = (double)F[(16 * ti + i) * LD + 16 * k0 + 4 * q + e];
        m[e] = M[(16 * k0 + 4 * q + e) * LDD + 16 * tj + i];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[e], m[e], acc[u], 0, 0, 0);
    }
    // (the tiles below the diagonal are nowhere read)
#pragma unroll
    for (int e = 0; e < 4; ++e) p.factor[(size_t)(r0 + 16 * ti + q + 4 * e) * 64 + 16 * tj + i] = acc[u][e];
  }
}

// T of 256 rows from the factors of its blocks of 64 rows, as operands: block back substitution on 16 columns per workgroup,
//   X_c = T_cc E,   X_b = -T_bb (sum over b < j <= c of S_bj X_j),
// with fp64 matrix instructions (in fp32, 6 us less, its sums cost as much accuracy as all the other products of H together); wave w takes rows
// 16 w ... of every block. What a wave reads of S and T for a block is fetched under the products of the block before. The blocks below the
// diagonal are written as zeros. Bound by the chain of six products of the last block column.
struct InverseArgs {
  const double* S;       // [np][256]: a group's rows against its rows, the blocks of 64 x 64 on and above the diagonal
  const double* factor;  // [np / 64][64][64], tiles on and above the diagonal
  char* T;               // the groups' T as operands, rows stay rows (np x 256)
  int np;
};
struct InversePair {
  InverseArgs a[2];     // blockIdx.y
};

template <int C>
__device__ __forceinline__ void inverse_panel(const InverseArgs& p, int b0, int sub, double (*X)[64][17], double (*R)[17]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, i = lane & 15;
  f64x4 s[2][4 * (C > 0 ? C : 1)], t[2][4];  // lane (q, i): four consecutive inner indices 16 g + 4 q of row i, g = 0 .. 3
  auto fetch = [&](int b, f64x4 (&to_s)[4 * (C > 0 ? C : 1)], f64x4 (&to_t)[4]) {
    const size_t row = (size_t)(b0 + b) * 64 + 16 * wave + i;
#pragma unroll
    for (int j = C; j > b; --j)
#pragma unroll
      for (int g = 0; g < 4; ++g) to_s[4 * (C - j) + g] = *reinterpret_cast<const f64x4*>(p.S + row * kGroup + j * 64 + 16 * g + 4 * q);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      to_t[g] = g >= wave ? *reinterpret_cast<const f64x4*>(p.factor + row * 64 + 16 * g + 4 * q) : f64x4{0., 0., 0., 0.};
  };
  if constexpr (C > 0) fetch(C - 1, s[0], t[0]);
  {
    const int r = tid >> 2, c = (tid & 3) * 4;
    const f64x4 x = r / 16 <= sub ? *reinterpret_cast<const f64x4*>(p.factor + ((size_t)(b0 + C) * 64 + r) * 64 + 16 * sub + c) : f64x4{0., 0., 0., 0.};
#pragma unroll
    for (int e = 0; e < 4; ++e) X[C][r][c + e] = x[e];
  }
  __syncthreads();
  auto product = [&](const f64x4* a, const double (*B)[17], f64x4 (&acc)[4]) {  // 64 inner indices, four chains of instructions
    double b[16];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) b[4 * g + e] = B[16 * g + 4 * q + e][i];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int g = 0; g < 4; ++g) acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g][e], b[4 * g + e], acc[g], 0, 0, 0);
  };
#pragma unroll
  for (int b = C - 1; b >= 0; --b) {
    const int at = (C - 1 - b) & 1;
    if (b > 0) fetch(b - 1, s[at ^ 1], t[at ^ 1]);
    f64x4 acc[4] = {};
#pragma unroll
    for (int j = C; j > b; --j) product(s[at] + 4 * (C - j), X[j], acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) R[16 * wave + q + 4 * e][i] = (acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e]);
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = f64x4{0., 0., 0., 0.};
    product(t[at], R, acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) X[b][16 * wave + q + 4 * e][i] = -((acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e]));
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) block_inverse_kernel(InversePair pair) {
  __shared__ double X[4][64][17];
  __shared__ double R[64][17];
  const InverseArgs& p = pair.a[blockIdx.y];
  const int b0 = (int)blockIdx.x / 16 * 4, c = (int)blockIdx.x % 16 / 4, sub = (int)blockIdx.x % 4;
  const int blocks = min(4, p.np / 64 - b0);
  if (c >= blocks) return;
  switch (c) {
    case 0: inverse_panel<0>(p, b0, sub, X, R); break;
    case 1: inverse_panel<1>(p, b0, sub, X, R); break;
    case 2: inverse_panel<2>(p, b0, sub, X, R); break;
    default: inverse_panel<3>(p, b0, sub, X, R); break;
  }
  constexpr int kt = kGroup / 32;
  const int col0 = c * 64 + 16 * sub;  // in the group
  const double* flat = &X[0][0][0];
  for (int u = threadIdx.x; u < blocks * 128; u += 256) {  // eight columns of a row: the low bits of the row fastest
    const int row = u / 32 * 16 + (u & 15), k8 = u >> 4 & 1;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = row / 64 <= c ? (float)flat[row * 17 + 8 * k8 + e] : 0.f;
    store_unit(p.T, kt, b0 * 64 + row, col0 / 8 + k8, v);
  }
}

// K = (Q - Q^T) / 2, Q the sum of `parts` matrices of d x d: d = 1024, one part: 12 MB in 5 us, mostly launch and one trip to memory.
struct SkewArgs {
  const float* Q;
  float* K;
  int d, parts;
};
struct SkewPair {
  SkewArgs a[2];  // blockIdx.z
};
__global__ void __launch_bounds__(256) skew_kernel(SkewPair pair) {
  __shared__ float tile[32][33];
  const SkewArgs& p = pair.a[blockIdx.z];
  const int r0 = (int)blockIdx.y * 32, c0 = (int)blockIdx.x * 32, x = threadIdx.x & 31, y = threadIdx.x >> 5, d = p.d;
  if (r0 >= d || c0 >= d) return;  // whole workgroup
  // (entries that do not exist: the first one instead; the fetches of up to eight parts are in flight together)
  float own[4], other[4];
  unsigned at[4], to[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = r0 + y + 8 * it, c = c0 + x, rt = c0 + y + 8 * it, ct = r0 + x;
    at[it] = r < d && c < d ? (unsigned)(r * d + c) : 0u;
    to[it] = rt < d && ct < d ? (unsigned)(rt * d + ct) : 0u;
    own[it] = other[it] = 0.f;
  }
#pragma unroll 8
  for (int s = 0; s < p.parts; ++s) {
    const float* Q = p.Q + (size_t)s * d * d;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      own[it] += Q[at[it]];
      other[it] += Q[to[it]];
    }
  }
#pragma unroll
  for (int it = 0; it < 4; ++it) tile[y + 8 * it][x] = other[it];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = r0 + y + 8 * it, c = c0 + x;
    if (r < d && c < d) p.K[(size_t)r * d + c] = 0.5f * (own[it] - tile[x][y + 8 * it]);
  }
}

// ------------------------------------------------------------------------------------------
// Workspace
// ------------------------------------------------------------------------------------------
struct DenseLayout {
  size_t Vt;              // V^T as operands
  size_t S, factor;       // the groups' Gram matrices, the factors of 64 rows (fp64)
  size_t T;               // the groups' T as operands
  size_t TV;              // T_g V_g as operands
  size_t P;               // the product of the groups so far
  size_t Y, Ya;           // Y fp32 and as operands
  size_t H, Ht;           // H and H^T as operands
  // saved by the forward pass / used by the backward pass
  size_t left, right;     // operands of Q = left right^T: dX and X or, of a product H^T X, A and G
  size_t Q, K, W, Wa, U;
  int q_split;
  size_t total;
};

// Parts of the mini-batch for Q = dX X^T: enough workgroups for the GPU, 256 columns each at least.
static int dense_q_split(int d, int m) {
  const int t = pad64(d) / 64, tiles = t * t;
  int split = tiles >= 192 ? 1 : (256 + tiles - 1) / tiles;
  return std::max(1, std::min(split, m / 256));
}

static DenseLayout make_dense_layout(int d, int n, int m) {
  DenseLayout L{};
  size_t off = 256;  // header, reserved
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  const size_t np = pad64(n);
  L.Vt = take(packed_bytes(d, n));
  L.S = take(np * kGroup * 8);
  L.factor = take(np * 64 * 8);
  L.T = take(np * kGroup * 6);
  L.TV = take(packed_bytes(n, d));
  L.P = take((size_t)d * d * 4);
  L.Y = take((size_t)n * d * 4);
  L.Ya = take(packed_bytes(n, d));
  L.H = take(packed_bytes(d, d));
  L.Ht = take(packed_bytes(d, d));
  L.q_split = dense_q_split(d, m);
  L.left = take(packed_bytes(d, m));
  L.right = take(packed_bytes(d, m));
  L.Q = take((size_t)L.q_split * d * d * 4);
  L.K = take((size_t)d * d * 4);
  L.W = take((size_t)n * d * 4);
  L.Wa = take(packed_bytes(n, d));
  L.U = take(packed_bytes(n, n));
  L.total = off;
  return L;
}

// ------------------------------------------------------------------------------------------
// Launches
// ------------------------------------------------------------------------------------------
struct GemmList {
  GemmArgs args;
  int count = 0;
  GemmProblem& add() { return args.p[count++] = GemmProblem{}; }
};

template <int RT, int CT, int WM, int WN, int KS, int BF>
static int launch_gemm_as(GemmList& list, hipStream_t stream) {
  constexpr int BM = 16 * RT * WM, BN = 16 * CT * WN;
  int width = 0;
  for (int i = 0; i < list.count; ++i) {
    GemmProblem& p = list.args.p[i];
    const int rt = (pad64(p.rows) + BM - 1) / BM, ct = (pad64(p.cols) + BN - 1) / BN;
    p.tiles = p.flags & kUpper ? rt * (rt + 1) / 2 : rt * ct * std::max(p.split, 1);
    // (rows of a triangular operand take different times: every XCD takes all of them)
    if (!(p.flags & kUpper) && p.split <= 1)
      p.xcd_rows = p.term.upper ? (ct % 8 == 0 ? 1 : 0) : xcd_cut(rt, ct, 6. * BM, (BF ? 4. : 6.) * BN);
    width = std::max(width, (p.tiles + 7) / 8 * 8);
  }
  constexpr size_t lds = gemm_lds<BM, BN, KS>();
  auto kernel = gemm_kernel<RT, CT, WM, WN, KS, BF>;
  const int rc = allow_lds(kernel, lds);
  if (rc != FASTH_OK) return rc;
  hipLaunchKernelGGL(kernel, dim3(width, list.count), dim3(64 * WM * WN * KS), lds, stream, list.args);
  FASTH_HIP(hipGetLastError());
  list.count = 0;
  return FASTH_OK;
}

// Which tiles: the largest that give every compute unit a workgroup; a launch of short rounds of small tiles is over sooner than
// one of few large ones. us, k = 1024, packed operands, {128 x 128, 64 x 64, 32 x 32}: 1024 x 4096: 54, 71, -; 1024 x 1024: 35, 18.7, 38;
// 1024 x 256: -, 15.5, 7.9; 1024 x 100: -, -, 7.0; k = 512: 512 x 512: -, 10.3, 6.5.
template <int BF>
static int launch_gemm_tiles(GemmList& list, int slot, hipStream_t stream, int min_tile, int max_tile) {
  long t128 = 0, t32 = 0;
  for (int i = 0; i < list.count; ++i) {
    const GemmProblem& p = list.args.p[i];
    const long half = p.flags & kUpper ? 2 : 1, split = std::max(p.split, 1);
    t128 += (long)((p.rows + 127) / 128) * ((p.cols + 127) / 128) * split / half;
    t32 += (long)(pad64(p.rows) / 32) * (pad64(p.cols) / 32) * split / half;
  }
  int tile = t128 >= 192 ? 128 : t32 > 512 ? 64 : 32;
  tile = std::min(std::max(tile, min_tile), max_tile);
  static const std::string names[3] = {variant_name("gemm_kernel", {4, 4, 2, 2, 2, BF}), variant_name("gemm_kernel", {4, 4, 1, 1, 8, BF}),
                                       variant_name("gemm_kernel", {2, 2, 1, 1, 8, BF})};
  prof::Scope ps_(slot, stream, names[tile == 128 ? 0 : tile == 64 ? 1 : 2].c_str());
  if (tile == 128) return launch_gemm_as<4, 4, 2, 2, 2, BF>(list, stream);
  if (tile == 64) return launch_gemm_as<4, 4, 1, 1, 8, BF>(list, stream);
  return launch_gemm_as<2, 2, 1, 1, 8, BF>(list, stream);
}

// BF: B is fp32 [k][cols]; where its rows are made of 16-byte groups a lane loads neighbouring columns at once. us per forward + backward, a load per
// column and this: d = n = 1024, m = 4096: 334, 330; m = 1400: 259, 252; d = 512, m = 2048: 114, 113; d = 1536, m = 2048: 665, 658.
template <bool BF>
static int launch_gemm(GemmList& list, int slot, hipStream_t stream, int min_tile = 32, int max_tile = 128) {
  if (list.count == 0) return FASTH_OK;
  if constexpr (BF) {
    bool wide = true;
    for (int i = 0; i < list.count; ++i) {
      const GemmProblem& p = list.args.p[i];
      wide = wide && p.cols % 4 == 0 && p.term.ldb % 4 == 0 && reinterpret_cast<uintptr_t>(p.term.B) % 16 == 0;
    }
    if (wide) return launch_gemm_tiles<2>(list, slot, stream, min_tile, max_tile);
  }
  return launch_gemm_tiles<BF ? 1 : 0>(list, slot, stream, min_tile, max_tile);
}

static int launch_pack(PackArgs& args, int count, int slot, hipStream_t stream) {
  int width = 0;
  for (int i = 0; i < count; ++i) width = std::max(width, args.job[i].blocks);
  if (width == 0) return FASTH_OK;
  prof::Scope ps_(slot, stream, "pack_kernel");
  hipLaunchKernelGGL(pack_kernel, dim3(width, count), dim3(256), 0, stream, args);
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

// One product on its slice of a workspace.
struct Dense {
  int d = 0, n = 0, m = 0;
  const Dense* owner = nullptr;  // whose workspace has T, Y and H, if not this one's
  DenseLayout L;
  char* ws = nullptr;
  const Dense& factors() const { return owner ? *owner : *this; }
  char* at(size_t off) const { return ws + off; }
  float* f(size_t off) const { return reinterpret_cast<float*>(ws + off); }
  double* f64(size_t off) const { return reinterpret_cast<double*>(ws + off); }
  int kt(int x) const { return pad64(x) / 32; }
  PackJob pack_v(const float* V) const { return PackJob{V, nullptr, at(L.Vt), n, d, pad64(n) / 64 * (pad64(d) / 64)}; }
  // X of a product H X, or G of a product H^T X ([rows][m], rows beyond are zero), for dV
  PackJob pack_right(const float* X, int rows) const { return PackJob{X, at(L.right), nullptr, rows, m, pad64(d) / 64 * (pad64(m) / 64)}; }
  char* left() const { return at(L.left); }
  // H or H^T, and Y, as operands
  char* matrix(bool transpose) const { const Dense& F = factors(); return F.at(transpose ? F.L.Ht : F.L.H); }
  char* y() const { const Dense& F = factors(); return F.at(F.L.Ya); }
};

static int group_rows(const Dense& P, int g) { return std::min(kGroup, P.n - g * kGroup); }
// (row, k) of operands with kt tiles of k
static char* operand_cell(char* base, int kt, int row, int k) { return base + ((size_t)(row / 16) * kt + k / 32) * kTileBytes; }

static int dense_pack(const PackJob& job, int slot, hipStream_t stream) {
  PackArgs args{};
  args.job[0] = job;
  return launch_pack(args, 1, slot, stream);
}

// The groups' T of up to two products; `jobs`: what else is to be packed in the first launch.
static int dense_factors(const Dense* const* D, const float* const* V, int count, const PackJob* jobs, int njobs, hipStream_t stream) {
  const int slot = FASTH_KERNEL_FACTOR;
  PackArgs pk{};
  int pack = 0;  // blocks of the largest job
  for (int i = 0; i < count + njobs; ++i) {
    pk.job[i] = i < count ? D[i]->pack_v(V[i]) : jobs[i - count];
    pack = std::max(pack, pk.job[i].blocks);
  }
  InversePair inv{};
  FactorPair64 fac{};
  GramPair gram{};
  int width = 0;
  bool vec4 = true;
  for (int i = 0; i < count; ++i) {
    const Dense& P = *D[i];
    const int groups = (P.n + kGroup - 1) / kGroup;
    gram.a[i] = GramArgs{V[i], P.f64(P.L.S), P.n, P.d, groups * kGroupTiles};
    fac.a[i] = FactorArgs64{P.f64(P.L.S), P.f64(P.L.factor), P.n, pad64(P.n)};
    inv.a[i] = InverseArgs{P.f64(P.L.S), P.f64(P.L.factor), P.at(P.L.T), pad64(P.n)};
    width = std::max(width, groups);
    vec4 = vec4 && P.d % 4 == 0;
  }
  gram.width = width * kGroupTiles;
  {
    static_assert(kGroupTiles % 8 == 0, "every XCD takes as many tiles");
    prof::Scope ps_(slot, stream, vec4 ? "gram_kernel<4>" : "gram_kernel<1>");
    hipLaunchKernelGGL(vec4 ? gram_kernel<4> : gram_kernel<1>, dim3(gram.width + pack, count + njobs), dim3(256), 0, stream, gram, pk);
    FASTH_HIP(hipGetLastError());
  }
  {
    prof::Scope ps_(slot, stream, "block_factor_kernel");
    hipLaunchKernelGGL(block_factor_kernel, dim3(width * (kGroup / 64), count), dim3(512), 0, stream, fac);
    FASTH_HIP(hipGetLastError());
  }
  prof::Scope ps_(slot, stream, "block_inverse_kernel");
  hipLaunchKernelGGL(block_inverse_kernel, dim3(width * 16, count), dim3(256), 0, stream, inv);
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

// Y, H and H^T of up to two products.
static int dense_matrices(const Dense* const* D, const float* const* V, int count, hipStream_t stream) {
  const int slot = FASTH_KERNEL_FACTOR;
  int rc, steps = 0, groups[2] = {0, 0};
  for (int i = 0; i < count; ++i) {
    groups[i] = (D[i]->n + kGroup - 1) / kGroup;
    steps = std::max(steps, groups[i]);
  }
  auto group_at = [&](int i, int step) { return groups[i] - 1 - step; };
  auto y_of = [](GemmProblem& p, const Dense& P, int g) {
    p.rows = group_rows(P, g); p.cols = p.ldo = P.d; p.alpha = 1.f;
    p.out = P.f(P.L.Y) + (size_t)g * kGroup * P.d;
    p.along = operand_cell(P.y(), P.kt(P.d), g * kGroup, 0); p.along_kt = P.kt(P.d);
  };
  // T_g V_g: Y_g of the group that is applied first, operands for the others'
  GemmList tv;
  for (int i = 0; i < count; ++i) {
    const Dense& P = *D[i];
    for (int step = 0; step < groups[i]; ++step) {
      const int g = group_at(i, step);
      if (tv.count == kGemmProblems && (rc = launch_gemm<true>(tv, slot, stream)) != FASTH_OK) return rc;
      GemmProblem& p = tv.add();
      y_of(p, P, g);
      p.term = GemmTerm{operand_cell(P.at(P.L.T), kGroup / 32, g * kGroup, 0), reinterpret_cast<const char*>(V[i] + (size_t)g * kGroup * P.d),
                        kGroup / 32, P.d, group_rows(P, g), true};
      if (step > 0) {
        p.out = nullptr;
        p.along = operand_cell(P.at(P.L.TV), P.kt(P.d), g * kGroup, 0);
      }
    }
  }
  if ((rc = launch_gemm<true>(tv, slot, stream)) != FASTH_OK) return rc;
  // P <- P - V_g^T Y_g, Y_g = (T_g V_g) P
  for (int step = 0; step < steps; ++step) {
    GemmList y, h;
    for (int i = 0; i < count; ++i) {
      if (step >= groups[i]) continue;
      const Dense& P = *D[i];
      const int g = group_at(i, step);
      if (step > 0) {
        GemmProblem& p = y.add();
        y_of(p, P, g);
        p.term = GemmTerm{operand_cell(P.at(P.L.TV), P.kt(P.d), g * kGroup, 0), P.at(P.L.P), P.kt(P.d), P.d, P.d, false};
      }
      const bool last = step + 1 == groups[i];
      GemmProblem& p = h.add();
      p.term = GemmTerm{operand_cell(P.at(P.L.Vt), P.kt(P.n), 0, g * kGroup), reinterpret_cast<const char*>(P.f(P.L.Y) + (size_t)g * kGroup * P.d), P.kt(P.n), P.d, group_rows(P, g), false};
      p.rows = p.cols = p.ldo = P.d; p.alpha = -1.f;
      if (step == 0) p.diag = 1.f;
      else { p.add = P.f(P.L.P); p.beta = 1.f; }
      if (!last) {
        p.out = P.f(P.L.P);
      } else {
        p.along = P.matrix(false); p.along_kt = P.kt(P.d);
        p.across = P.matrix(true); p.across_kt = P.kt(P.d);
      }
    }
    if ((rc = launch_gemm<true>(y, slot, stream)) != FASTH_OK || (rc = launch_gemm<true>(h, slot, stream)) != FASTH_OK) return rc;
  }
  return FASTH_OK;
}

// out = H in, or H^T in; `in` has in_rows rows, the others are zero. Optionally the scaled rows for the next product
// and the result as operands.
static int dense_apply(const Dense& P, bool transpose, const float* in, int in_rows, float* out, const float* scale, int scale_mode, int scaled_rows,
                       float* scaled, char* along, hipStream_t stream) {
  GemmList list;
  GemmProblem& g = list.add();
  g.term = GemmTerm{P.matrix(transpose), reinterpret_cast<const char*>(in), P.kt(P.d), P.m, in_rows, false};
  g.rows = P.d; g.cols = g.ldo = P.m; g.alpha = 1.f;
  g.out = out;
  g.scaled = scaled; g.scale = scale; g.scale_mode = scale_mode; g.scaled_rows = scaled_rows;
  g.along = along; g.along_kt = P.kt(P.m);
  return launch_gemm<true>(list, FASTH_KERNEL_CHAIN, stream);
}

// dV of up to two products from their `left` and `right` operands (dense_apply, pack_right).
static int dense_dv(const Dense* const* D, const float* const* V, float* const* dV, int count, bool accumulate, hipStream_t stream) {
  const int slot = FASTH_KERNEL_DV;
  GemmList q, w, z, v;
  SkewPair sk{};
  int dmax = 0;
  for (int i = 0; i < count; ++i) {
    const Dense& P = *D[i];
    GemmProblem& a = q.add();
    a.term = GemmTerm{P.left(), P.at(P.L.right), P.kt(P.m), P.kt(P.m), P.m, false};
    a.rows = a.cols = a.ldo = P.d; a.alpha = 1.f; a.out = P.f(P.L.Q); a.split = P.L.q_split;
    sk.a[i] = SkewArgs{P.f(P.L.Q), P.f(P.L.K), P.d, P.L.q_split};
    dmax = std::max(dmax, P.d);
    GemmProblem& b = w.add();
    b.term = GemmTerm{P.y(), P.at(P.L.K), P.kt(P.d), P.d, P.d, false};
    b.rows = P.n; b.cols = b.ldo = P.d; b.alpha = 1.f; b.out = P.f(P.L.W);
    b.along = P.at(P.L.Wa); b.along_kt = P.kt(P.d);
    GemmProblem& c = z.add();
    // striu(W Y^T)
    c.term = GemmTerm{P.at(P.L.Wa), P.y(), P.kt(P.d), P.kt(P.d), P.d, false};
    c.rows = c.cols = c.ldo = P.n; c.alpha = 1.f; c.flags = kUpper | kStrict;
    c.along = P.at(P.L.U); c.along_kt = P.kt(P.n);
    GemmProblem& e = v.add();
    e.term = GemmTerm{P.at(P.L.U), reinterpret_cast<const char*>(V[i]), P.kt(P.n), P.d, P.n, true};
    e.rows = P.n; e.cols = e.ldo = P.d; e.alpha = -2.f; e.beta = 2.f; e.add = P.f(P.L.W); e.out = dV[i];
    e.flags = accumulate ? kAccumulate : 0;
  }
  int rc = launch_gemm<false>(q, slot, stream);
  if (rc != FASTH_OK) return rc;
  {
    prof::Scope ps_(slot, stream, "skew_kernel");
    const int t = (dmax + 31) / 32;
    hipLaunchKernelGGL(skew_kernel, dim3(t, t, count), dim3(256), 0, stream, sk);
    FASTH_HIP(hipGetLastError());
  }
  if ((rc = launch_gemm<true>(w, slot, stream)) != FASTH_OK) return rc;
  // the tiles of U beyond its diagonal tiles are not written: both products in tiles of one size
  const int tile = (long)(pad64(D[0]->n) / 32) * (pad64(D[0]->d) / 32) * count <= 512 ? 32 : 64;
  if ((rc = launch_gemm<false>(z, slot, stream, tile, tile)) != FASTH_OK) return rc;
  return launch_gemm<true>(v, slot, stream, tile, tile);
}

// 32-bit byte offsets into the fp32 operands; reflections far beyond the vector length would share a T of more rounding
static bool dense_fits(int d, int n, int m) {
  return d <= 4096 && 2 * n <= 3 * d && (size_t)d * m * sizeof(float) < 0x80000000u;
}
// Whether a product runs on the whole matrix. Its part of a gradient step that depends on m is 6 d^2 m operations instead of 12 d n m, the rest is as much as a
// mini-batch of some 1.2 d columns and falls on whoever forms H: fasth_forward and fasth_prepare, also where no gradients or few applies follow. So the lines lie
// where a gradient step is faster and a forward call alone, or fasth_prepare with two unsaved applies, is not slower (by more than the 5 % that runs on different machines
// differ); fasth_prepare with a single unsaved apply loses up to 1.3 times below some 8000 columns. Beside the lines the chain's times jump: its workgroups take another round
// beyond 2048 and 4096 columns (d <= 1024) or some 2600 and 4096 (d > 1024), and beyond d = 2048 no kernel shares columns. Lengths that are no multiple of four load an operand
// one column at a time (launch_gemm). us, chain of blocks and whole matrix; gradient step; forward alone; prepare and one unsaved apply:
//   d = n =  512, m =  1000: 128, 107;  56,  64;  53,  63     m =  5960: 232, 175;  88,  89;  74,  86      m =  7450: 283, 174;  98,  88;  81,  84
//   d = 448, n = 336, m =  7947: 218, 180;  79,  85;  67,  81   m =  9934: 340, 238; 124, 110; 102, 105
//   d = 512, n = 256, m = 23841: 484, 368; 157, 152; 126, 133   m = 29802: 616, 462; 212, 186; 156, 162
//   d = n =  640, m =  1953: 197, 183;  87,  99;  98,  96     m =  2441: 248, 186; 110, 100; 100,  97
//   n = 0.625 d,  m =  4882: 315, 206; 129,  96; 111,  94     m =  7629: 408, 288; 141, 129; 115, 126
//   n = 0.5 d,    m =  7812: 321, 280; 112, 127;  97, 123     m =  9765: 502, 299; 199, 132; 169, 125
//   d = n =  768, m =  2000: 233, 218; 100, 114; 112, 111     m =  2500: 295, 225; 128, 115; 115, 113
//   n = 0.75 d,   m =  3333: 259, 249; 106, 126;  96, 124     m =  4166: 380, 252; 155, 125; 129, 122
//   d = n =  833, m =  3906: 435, 323; 156, 176; 137, 172     m =  4882: 623, 407; 221, 214; 168, 211      m =  6103: 712, 421; 259, 216; 170, 212
//   d = n =  896, m =  2500: 356, 281; 147, 154; 132, 151     m =  3906: 460, 301; 166, 157; 143, 153
//   n = 0.75 d,   m =  3333: 329, 276; 127, 139; 113, 136     m =  4166: 500, 280; 190, 137; 148, 134
//   n = 0.5 d,    m =  6400: 402, 340; 140, 154; 113, 149     m =  8000: 482, 362; 170, 158; 122, 151      m = 10000: 736, 482; 292, 206; 215, 196
//   d = n = 1024, m =  1024: 231, 228; 100, 135;  90, 133     m =  2000: 328, 274; 136, 154; 149, 152      m =  2500: 427, 308; 168, 169; 151, 166
//   n = 0.75 d,   m =  3333: 385, 292; 141, 146; 126, 144     m =  4166: 567, 392; 211, 193; 158, 188
//   n = 0.5 d,    m =  6400: 490, 373; 166, 169; 123, 163     m = 10000: 880, 549; 343, 232; 240, 220
//   d = n = 1088, m =  2500: 531, 445; 199, 251; 280, 248     m =  3125: 782, 457; 312, 252; 284, 248
//   d = 1280, n = 960, m = 3333: 753, 571; 295, 296; 256, 291   m = 4166: 1245, 593; 532, 297; 476, 291
//   d = n = 1536, m =  2500: 906, 717; 332, 398; 402, 389     m =  3125: 1267, 852; 505, 460; 397, 449
//   d = n = 2048, m =  2000: 1242, 1031; 494, 562; 641, 549     m = 2500: 1654, 1189; 689, 629; 633, 621
//   n = 0.625 d,  m =  4000: 1333, 1024; 514, 500; 453, 484     m = 5000: 2221, 1230; 908, 590; 776, 561
//   d = n = 2052, m =  1280: 2663, 1374; 1215, 816; 1157, 810   d = 2560, n = 1280, m = 4096: 5325, 1566; 2462, 765; 2371, 750
//   d = n = 3072, m =  1280: 4394, 2668; 1959, 1547; 1833, 1535;  d = n = 4096: 9588, 5199; 4464, 2897; 3063, 2882
// Products of a layer of two: their launches serve both, so some lines lie at fewer columns. us per layer W X, gradient step and forward alone:
//   d = n =  512, m =   500: 142, 139;  61,  77     m =   625: 196, 152;  87,  82;    d = 512, n = 384, m = 7761: 517, 353; 144, 146
//   d = n =  640, m =  1907: 378, 312; 156, 155     m =  2384: 470, 311; 199, 152;    d = n =  768, m = 1953: 485, 398; 182, 201    m = 2441: 608, 414; 238, 204
//   d = n = 1024, m =  1953: 730, 531; 258, 272     m =  2441: 914, 618; 348, 306;    n = 0.75 d,   m = 3255: 805, 573; 291, 268
//   d = n = 1536, m =  1562: 1506, 1233; 620, 652   m =  1953: 1620, 1272; 655, 663;  d = 1280, n = 960, m = 2083: 976, 765; 380, 386; m = 2604: 1436, 782; 594, 382
//   d = n = 2048, m =  1562: 2322, 1844; 1020, 977;   d = n = 2560, m = 512: 3055, 3112; 1367, 1866; m = 800: 5498, 3299; 2573, 1945;   d = n = 4096, m = 800: 14780, 9834; 7123, 5428
// (symmetric forms, one set of factors, gain more: d = n = 768, m = 1953: 478, 388; 181, 155).
static bool dense_pays(int d, int n, int m, bool layer) {
  if (d < 448 || 2 * n < d) return false;
  n = std::min(n, d);  // (more reflections cost both sides more)
  const bool odd = d % 4 != 0;
  // columns (per_n n / d - per_d) >= full
  const auto at_least = [&](long long columns, int per_n, int per_d, long long full) { return columns * ((long long)per_n * n - (long long)per_d * d) >= full * d; };
  if (d <= 1024) {
    const long long columns = odd ? m * 5ll / 8 : m, least = d <= 512 ? 7168 : 4097;
    if (columns >= least && at_least(columns, 8, 3, (d <= 512 ? 4 : 3) * least)) return true;
    if (d > 512 && columns >= 2 * least) return true;
    // nearly as many reflections as elements
    if (odd || (d <= 512 && !layer)) return false;
    if (d <= 512) return at_least(m, 16, 15, 640);
    return at_least(m, 8, 7, d <= 768 || layer ? 2049 : 2560ll * 1024 * 1024 / (d * d));
  }
  if (d <= 2048) return at_least(layer ? (odd ? m : m * 3ll / 2) : odd ? m * 4ll / 5 : m, 1, 0, 2700);
  const long long columns = layer ? m * 3ll / 2 : m;
  return at_least(odd ? columns * 4 / 5 : columns, 1, -1, 2560);
}
static bool dense_serves(int d, int n, int m) { return dense_fits(d, n, m) && dense_pays(d, n, m, false); }
static bool dense_serves_layer(int d, int n, int m) { return dense_fits(d, n, m) && dense_pays(d, n, m, true); }

}  // namespace fasth
