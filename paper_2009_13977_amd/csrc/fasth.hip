// FastH for CDNA4 (gfx950): kernels and the C ABI declared in include/fasth.h.
//
// Notation follows the paper (arXiv 2009.13977): d = vector length, n = number of reflections,
// m = mini-batch columns, k = block size (Section 3.3), nb = n / k blocks P_i (Eq. 2).
//
// Block form used here. For the k rows V_i of one block, with S = V_i V_i^T,
//   P_i = H_{(i-1)k+1} ... H_{ik} = I - V_i^T T_i V_i,   T_i = (diag(S)/2 + striu(S))^-1.
// This is the WY form of Lemma 1 (Y = V_i^T, W = V_i^T T_i / 2) kept as the k x k factor T_i, so
// Step 1 of Algorithm 1 is one Gram product per block (matrix cores) plus a k x k triangular
// inverse, and P_i^T = I - V_i^T T_i^T V_i needs no second factor.
//
// Kernels
//   factor_fused_kernel  Algorithm 1 Step 1, one workgroup per block (block sizes up to 32; 64 for short vectors)
//   team_factor_kernel   Algorithm 1 Step 1 with a block's Gram product split over workgroups (MFMA); also the products
//                        V_a V_b^T of consecutive blocks' rows for the chain kernel that joins two blocks per step
//   chain_*_kernel       Algorithm 1 Step 2 / Algorithm 2 Step 1: the sequential block chain: per column of X
//                        (pair, pipe, general), a team of workgroups per column (team, team_wide), or 4 / 16 / 32 columns
//                        per workgroup or team on the matrix cores (quad, tile, team_tile, trio)
//   trio_rows_kernel     the rows of V as operands of chain_trio_kernel, part of Step 1
//   dv_*                 Algorithm 2 Step 2 as dense products per block (MFMA)
//   gemm_kernel, pack_kernel, gram_kernel, block_factor_kernel, block_inverse_kernel, skew_kernel
//                        wide mini-batches: H as one matrix, and Algorithms 1 and 2 as products with it (MFMA)
//   seq_*                the one-reflection-at-a-time comparison
//   dsigma_kernel        the diagonal step of the SVD layer
// The kernels live in fasth_factor.h, fasth_chain.h (+ fasth_chain_team.h, fasth_chain_pair.h, fasth_chain_quad.h,
// fasth_chain_tile.h, fasth_chain_trio.h, fasth_chain_teamtile.h), fasth_dv.h, fasth_dense.h (+ fasth_gemm.h) and fasth_sequential.h (helpers in fasth_common.h and
// fasth_device.h); this file holds the host drivers and the C entry points.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <mutex>
#include <type_traits>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "fasth.h"
#include "fasth_device.h"
#include "fasth_common.h"
#include "fasth_factor.h"
#include "fasth_chain.h"
#include "fasth_dv.h"
#include "fasth_dense.h"
#include "fasth_sequential.h"
#include "fasth_peaks.h"

namespace fasth {


// ------------------------------------------------------------------------------------------
// Host drivers
// ------------------------------------------------------------------------------------------

// Polls after which a kernel's wait for another workgroup gives up (fasth_set_wait_limit).
static std::atomic<int> g_wait_limit{kDefaultWaitLimit};
static int wait_limit() { return g_wait_limit.load(std::memory_order_relaxed); }

struct Product {  // one Householder product bound to its slice of a workspace
  int d, n, m, k;
  Layout L;
  char* ws;
  // Calls on this workspace never overlap on the GPU: they save into it, or the header says so for the shape. Cleared by
  // fasth_apply without saving, whose calls may overlap except for the header's list of shapes.
  bool exclusive = true;
  bool dense = false;  // the whole matrix instead of the chain of blocks: the workspace is D's
  Dense D;
  // the rows the kernels read: the caller's, or the padded copy the factor kernels leave in the workspace
  const float* rows(const float* V) const { return L.copy_v ? reinterpret_cast<const float*>(ws + L.off_V) : V; }
  float* copy() const { return L.copy_v ? reinterpret_cast<float*>(ws + L.off_V) : nullptr; }
  char* frag() const { return L.trio.parts ? ws + L.off_frag : nullptr; }
  float* T() const { return reinterpret_cast<float*>(ws + L.off_T); }
  float* Spart() const { return reinterpret_cast<float*>(ws + L.off_Spart); }
  unsigned* xch() const { return L.xch_words ? reinterpret_cast<unsigned*>(ws + L.off_xch) : nullptr; }
  float* saveA() const { return reinterpret_cast<float*>(ws + L.off_saveA); }
  float* saveCa() const { return reinterpret_cast<float*>(ws + L.off_saveCa); }
  float* saveG() const { return reinterpret_cast<float*>(ws + L.off_saveG); }
  float* saveCg() const { return reinterpret_cast<float*>(ws + L.off_saveCg); }
};

static Product bind(int d, int n, int m, int k, void* ws, bool dense = false, LayoutLevel level = kLayoutTrio) {
  Product P;
  P.d = d; P.n = n; P.m = m; P.k = k;
  P.ws = static_cast<char*>(ws);
  P.dense = dense;
  if (!dense) {
    P.L = make_layout(d, n, m, k, level);
    return P;
  }
  P.D.d = d; P.D.n = n; P.D.m = m; P.D.ws = P.ws;
  P.D.L = make_dense_layout(d, n, m);
  return P;
}
static size_t workspace_of(const Product& P) { return P.dense ? P.D.L.total : P.L.total; }
static size_t workspace_of(int d, int n, int m, int k, bool dense) { return workspace_of(bind(d, n, m, k, nullptr, dense)); }

static int launch_factor_fused(const FactorPair& fp, int count, int kp, bool vec4, hipStream_t stream) {
  static const std::string names[6] = {variant_name("factor_fused_kernel", {1, 4}), variant_name("factor_fused_kernel", {2, 4}),
                                       variant_name("factor_fused_kernel", {4, 4}), variant_name("factor_fused_kernel", {1, 1}),
                                       variant_name("factor_fused_kernel", {2, 1}), variant_name("factor_fused_kernel", {4, 1})};
  prof::Scope ps_(FASTH_KERNEL_FACTOR, stream, names[(vec4 ? 0 : 3) + (kp == 16 ? 0 : kp == 32 ? 1 : 2)].c_str());
  const dim3 grid(count == 2 && fp.nb[1] > fp.nb[0] ? fp.nb[1] : fp.nb[0], count), block(512);
  if (vec4) {
    if (kp == 16) hipLaunchKernelGGL((factor_fused_kernel<1, 4>), grid, block, 0, stream, fp);
    else if (kp == 32) hipLaunchKernelGGL((factor_fused_kernel<2, 4>), grid, block, 0, stream, fp);
    else hipLaunchKernelGGL((factor_fused_kernel<4, 4>), grid, block, 0, stream, fp);
  } else {
    if (kp == 16) hipLaunchKernelGGL((factor_fused_kernel<1, 1>), grid, block, 0, stream, fp);
    else if (kp == 32) hipLaunchKernelGGL((factor_fused_kernel<2, 1>), grid, block, 0, stream, fp);
    else hipLaunchKernelGGL((factor_fused_kernel<4, 1>), grid, block, 0, stream, fp);
  }
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

static void set_factor_slot(FactorPair& fp, int slot, const Product& P, const float* V) {
  fp.V[slot] = V; fp.T[slot] = P.T(); fp.d[slot] = P.d; fp.k[slot] = P.L.kf; fp.nb[slot] = P.L.nbf;
  fp.n[slot] = P.n; fp.dp[slot] = P.L.dp; fp.copy[slot] = P.copy();
  fp.xch[slot] = P.xch(); fp.xch_words[slot] = (unsigned)P.L.xch_words;
}

static std::atomic<unsigned long long> g_launch_id{0x9e3779b97f4a7c15ull};  // a new value per launch, never 0

static TeamFactorArgs team_factor_args(const Product& P, const float* V) {
  TeamFactorArgs a;
  a.V = V; a.Spart = P.Spart(); a.T = P.T();
  a.ready = reinterpret_cast<unsigned long long*>(P.ws + P.L.off_ready);
  a.launch_id = g_launch_id.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
  if (a.launch_id == 0) a.launch_id = 1;
  a.d = P.d; a.n = P.n; a.dp = P.L.dp; a.copy = P.copy();
  a.k = P.L.kf; a.kp = P.L.kpf; a.split = P.L.gram_split; a.wait_limit = wait_limit();
  a.xch = P.xch(); a.xch_words = (unsigned)P.L.xch_words;
  a.S = reinterpret_cast<float*>(P.ws + P.L.off_S); a.nblocks = P.L.nbf; a.npair = P.L.npair;
  return a;
}

// Blocks of 64 or 128 rows (the caller's, or pairs of blocks of 32 merged for the team chain kernel): the Gram
// product split over d, the block's first workgroup inverts. `count` products of the same shape in one launch.
static int launch_team_factor(const TeamFactorPair& pair, int count, int nbf, hipStream_t stream) {
  const TeamFactorArgs& a = pair.a[0];
  // (a pair's workgroups stage the rows of two blocks)
  const size_t lds = std::max(sizeof(float) * (size_t)(a.npair > 0 ? 2 : 1) * a.kp * (kGramChunk + 4), t_build_lds(a.kp));
  const bool vec4 = a.d % 4 == 0;
  int rc = FASTH_OK;
  if (a.kp == 64) rc = vec4 ? allow_lds(team_factor_kernel<4, 64>, lds) : allow_lds(team_factor_kernel<1, 64>, lds);
  else rc = vec4 ? allow_lds(team_factor_kernel<4, 128>, lds) : allow_lds(team_factor_kernel<1, 128>, lds);
  if (rc != FASTH_OK) return rc;
  static const std::string names[4] = {variant_name("team_factor_kernel", {4, 64}), variant_name("team_factor_kernel", {1, 64}),
                                       variant_name("team_factor_kernel", {4, 128}), variant_name("team_factor_kernel", {1, 128})};
  prof::Scope ps_(FASTH_KERNEL_TEAM_FACTOR, stream, names[(a.kp == 64 ? 0 : 2) + (vec4 ? 0 : 1)].c_str());
  const dim3 grid(a.split, nbf + a.npair, count), block(8 * a.kp);
  if (a.kp == 64) {
    if (vec4) hipLaunchKernelGGL((team_factor_kernel<4, 64>), grid, block, lds, stream, pair);
    else hipLaunchKernelGGL((team_factor_kernel<1, 64>), grid, block, lds, stream, pair);
  } else {
    if (vec4) hipLaunchKernelGGL((team_factor_kernel<4, 128>), grid, block, lds, stream, pair);
    else hipLaunchKernelGGL((team_factor_kernel<1, 128>), grid, block, lds, stream, pair);
  }
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

// The rows of V as chain_trio_kernel's operands, for up to two products in one launch.
static int launch_trio_rows(const Product& P0, const float* V0, const Product* P1, const float* V1, hipStream_t stream) {
  TrioRowsPair pair;
  auto bind_rows = [](const Product& P, const float* V) {
    return TrioRowsArgs{V, P.frag(), P.d, P.n, P.L.trio.parts ? (P.L.dp + 31) / 32 : 0, P.L.trio.parts ? P.L.np / 64 : 0};
  };
  pair.a[0] = bind_rows(P0, V0);
  pair.a[1] = P1 ? bind_rows(*P1, V1) : TrioRowsArgs{};
  const int xb = std::max(pair.a[0].xblocks, pair.a[1].xblocks), steps = std::max(pair.a[0].steps, pair.a[1].steps);
  if (xb == 0) return FASTH_OK;
  prof::Scope ps_(FASTH_KERNEL_TRIO_ROWS, stream, "trio_rows_kernel");
  hipLaunchKernelGGL(trio_rows_kernel, dim3(xb, steps, P1 ? 2 : 1), dim3(256), 0, stream, pair);
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

static int build_factors_only(const Product& P, const float* V, hipStream_t stream) {
  const int kp = P.L.kpf;
  if (factor_is_fused(kp, P.d)) {
    FactorPair fp;
    set_factor_slot(fp, 0, P, V);
    set_factor_slot(fp, 1, P, V);  // unused
    return launch_factor_fused(fp, 1, kp, P.d % 4 == 0, stream);
  }
  TeamFactorPair pair;
  pair.a[0] = team_factor_args(P, V);
  pair.a[1] = pair.a[0];  // unused
  return launch_team_factor(pair, 1, P.L.nbf, stream);
}

static int build_factors(const Product& P, const float* V, hipStream_t stream) {
  const int rc = launch_trio_rows(P, V, nullptr, nullptr, stream);
  return rc != FASTH_OK ? rc : build_factors_only(P, V, stream);
}

// Factors of two products (independent of each other) in one launch when both take the fused
// kernel with the same template arguments; otherwise one after the other.
static int build_factors_pair(const Product& P0, const float* V0, const Product& P1, const float* V1,
                              hipStream_t stream) {
  const int rows_rc = launch_trio_rows(P0, V0, &P1, V1, stream);
  if (rows_rc != FASTH_OK) return rows_rc;
  if (factor_is_fused(P0.L.kpf, P0.d) && factor_is_fused(P1.L.kpf, P1.d) && P0.L.kpf == P1.L.kpf &&
      (P0.d % 4 == 0) == (P1.d % 4 == 0)) {
    FactorPair fp;
    set_factor_slot(fp, 0, P0, V0);
    set_factor_slot(fp, 1, P1, V1);
    return launch_factor_fused(fp, 2, P0.L.kpf, P0.d % 4 == 0, stream);
  }
  if (!factor_is_fused(P0.L.kpf, P0.d) && P0.d == P1.d && P0.n == P1.n && P0.L.kf == P1.L.kf &&
      P0.L.gram_split == P1.L.gram_split && P0.L.npair == P1.L.npair) {
    TeamFactorPair pair;
    pair.a[0] = team_factor_args(P0, V0);
    pair.a[1] = team_factor_args(P1, V1);
    return launch_team_factor(pair, 2, P0.L.nbf, stream);
  }
  const int rc = build_factors_only(P0, V0, stream);
  return rc != FASTH_OK ? rc : build_factors_only(P1, V1, stream);
}

// A = H in (transpose = 0) or H^T in (transpose = 1); activation = true saves into the activation
// slots of the workspace, false into the gradient slots.
static int run_chain(const Product& P, const float* V, const float* in, float* out, int transpose, bool activation,
                     const float* in_scale, int in_scale_mode, hipStream_t stream, bool save = true,
                     const Product* factors = nullptr, int in_rows = -1, const float* ds_z1 = nullptr,
                     float* ds_out = nullptr, int ds_rows = 0) {
  // `factors`: the product of the same shape whose workspace holds the block factors (and the hand-off area that
  // was cleared when they were built), if not P's own
  const Product& F = factors ? *factors : P;
  ChainArgs a;
  a.V = F.rows(V); a.T = F.T(); a.in = in; a.out = out;
  // calls that may overlap on one workspace cannot hand sums over through it
  const bool no_teams = !P.exclusive && shared_tiles_overlap(P.L.dp, P.m);
  a.xch = no_teams ? nullptr : F.xch();
  a.wait_limit = wait_limit(); a.parts = 0;
  a.S = reinterpret_cast<const float*>(F.ws + F.L.off_S);
  a.Tt = a.T + (size_t)F.L.nbf * F.L.kpf * F.L.kpf;
  a.save_in = !save ? nullptr : activation ? P.saveA() : P.saveG();
  a.save_c = !save ? nullptr : activation ? P.saveCa() : P.saveCg();
  a.frag = F.frag();
  a.in_scale = in_scale; a.in_scale_mode = in_scale_mode;
  a.in_rows = in_rows < 0 ? P.d : in_rows;
  a.out_rows = P.d;
  a.d = P.L.dp; a.n = P.L.np; a.m = P.m;
  // the factors' own blocks for the kernels that stand in where nothing is saved
  a.k = no_teams || (P.L.trio.parts && !save) ? P.L.kf : P.L.ki;
  a.kp = padded_block(a.k); a.nb = P.L.np / a.k;
  a.transpose = transpose;
  a.sub = 1;
  a.ds_z1 = ds_z1; a.ds_out = ds_out; a.ds_rows = ds_rows;
  return launch_chain(a, stream);
}

static DvArgs dv_args(const Product& P, const float* V, float* dV, int transpose, bool accumulate,
                      const Product* factors = nullptr) {
  DvArgs a;
  a.accumulate = accumulate ? 1 : 0;
  a.V = (factors ? *factors : P).rows(V); a.saveA = P.saveA(); a.saveCa = P.saveCa(); a.saveG = P.saveG(); a.saveCg = P.saveCg(); a.dV = dV;
  // the partial Gram matrices are dead once the factors exist; Z needs nb kp^2 of their floats
  a.Z = P.L.dv_trio && P.L.dv_split > 1 ? reinterpret_cast<float*>(P.ws + P.L.off_Zpart) : P.Spart();
  a.msplit = P.L.dv_split;
  a.cols_per_part = ((P.m + a.msplit - 1) / a.msplit + kDvMChunk - 1) / kDvMChunk * kDvMChunk;
  a.msplit = (P.m + a.cols_per_part - 1) / a.cols_per_part;  // no empty part
  a.dVpart = reinterpret_cast<float*>(P.ws + P.L.off_dVpart);
  a.d = P.L.dp; a.n = P.L.np; a.m = P.m; a.k = P.L.ki; a.kp = P.L.kp; a.transpose = transpose;
  a.out_d = P.d; a.out_n = P.n;
  return a;
}

static int launch_dv_trio(const DvPair& pair, int count, hipStream_t stream) {
  int xt = 0, nb = 0;
  for (int c = 0; c < count; ++c) {
    xt = std::max(xt, (pair.a[c].out_d + kDvTrioTile - 1) / kDvTrioTile);
    nb = std::max(nb, (pair.a[c].out_n + kDvTrioRows - 1) / kDvTrioRows);
  }
  prof::Scope ps_(FASTH_KERNEL_DV, stream, "dv_trio_kernel");
  hipLaunchKernelGGL(dv_trio_kernel, dim3(xt, nb, count * pair.a[0].msplit), dim3(512), 0, stream, pair);
  FASTH_HIP(hipGetLastError());
  if (pair.a[0].msplit == 1) return FASTH_OK;
  static_assert(kDvTrioTile == 4 * kDvTile, "workgroups of dv_finish_kernel");
  hipLaunchKernelGGL(dv_finish_kernel, dim3(4 * xt, nb, count), dim3(256), 0, stream, pair);
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

static int launch_dv(const DvPair& pair, int count, int kp, bool vec4, hipStream_t stream) {
  const size_t lds = dv_lds(kp);
  auto blocks_of = [](const DvArgs& a) { return (a.out_n + a.k - 1) / a.k; };  // blocks of padding only have no gradient
  int xt = (pair.a[0].d + kDvTile - 1) / kDvTile, nb = blocks_of(pair.a[0]);
  if (count == 2) {
    xt = std::max(xt, (pair.a[1].d + kDvTile - 1) / kDvTile);
    nb = std::max(nb, blocks_of(pair.a[1]));
  }
  const DvArgs& a0 = pair.a[0];
  const int msplit = a0.msplit;  // the same for both products of a launch (run_dv_pair checks)
  const dim3 grid(xt, nb, count * msplit);
  // Many columns and blocks of 64 rows or more: Z of every block once, by a launch of its own (measured at
  // d = n = 1024, m = 4096: dV 374 -> 326 us at k = 64, 853 -> 545 us at k = 128, but 294 -> 309 us at k = 32, where
  // the rebuild is a fifth of the work). Same condition for both products of a pair: run_dv_pair joins only products
  // that share m and the library's k. A split mini-batch needs it too: no workgroup sees all columns.
  auto z_addressable = [](const DvArgs& a) { return (size_t)a.m * a.n * sizeof(float) < kOob && a.Z != nullptr; };
  const bool z_fits = z_addressable(a0) && (count == 1 || z_addressable(pair.a[1]));
  if (msplit > 1 && !z_fits) return FASTH_EINVAL;  // dv_minibatch_split never chooses a split for such a shape
  const bool prez = z_fits && (msplit > 1 || (a0.k >= 64 && (size_t)a0.m * a0.k >= 32768));
  static const std::string names[16] = {
      variant_name("dv_kernel", {1, 1, 0}), variant_name("dv_kernel", {1, 1, 1}), variant_name("dv_kernel", {1, 4, 0}), variant_name("dv_kernel", {1, 4, 1}),
      variant_name("dv_kernel", {2, 1, 0}), variant_name("dv_kernel", {2, 1, 1}), variant_name("dv_kernel", {2, 4, 0}), variant_name("dv_kernel", {2, 4, 1}),
      variant_name("dv_kernel", {4, 1, 0}), variant_name("dv_kernel", {4, 1, 1}), variant_name("dv_kernel", {4, 4, 0}), variant_name("dv_kernel", {4, 4, 1}),
      variant_name("dv_kernel", {8, 1, 0}), variant_name("dv_kernel", {8, 1, 1}), variant_name("dv_kernel", {8, 4, 0}), variant_name("dv_kernel", {8, 4, 1})};
  prof::Scope ps_(FASTH_KERNEL_DV, stream,
                  names[(kp == 16 ? 0 : kp == 32 ? 4 : kp == 64 ? 8 : 12) + (vec4 ? 2 : 0) + (prez ? 1 : 0)].c_str());
  if (prez) {
    const int kt = kp / 16;
    hipLaunchKernelGGL(dv_z_kernel, dim3(kt * kt, nb, count), dim3(256), 0, stream, pair);
    FASTH_HIP(hipGetLastError());
  }
#define FASTH_LAUNCH_DV_(KT, VV, PZ)                                                      \
  do {                                                                                    \
    int rc_ = allow_lds(dv_kernel<KT, VV, PZ>, lds);                                      \
    if (rc_ != FASTH_OK) return rc_;                                                      \
    hipLaunchKernelGGL((dv_kernel<KT, VV, PZ>), grid, dim3(256), lds, stream, pair);      \
  } while (0)
#define FASTH_LAUNCH_DV(KT)                                                               \
  do {                                                                                    \
    if (vec4 && prez) FASTH_LAUNCH_DV_(KT, 4, true);                                      \
    else if (vec4) FASTH_LAUNCH_DV_(KT, 4, false);                                        \
    else if (prez) FASTH_LAUNCH_DV_(KT, 1, true);                                         \
    else FASTH_LAUNCH_DV_(KT, 1, false);                                                  \
  } while (0)
  switch (kp) {
    case 16: FASTH_LAUNCH_DV(1); break;
    case 32: FASTH_LAUNCH_DV(2); break;
    case 64: FASTH_LAUNCH_DV(4); break;
    default: FASTH_LAUNCH_DV(8); break;
  }
#undef FASTH_LAUNCH_DV
#undef FASTH_LAUNCH_DV_
  FASTH_HIP(hipGetLastError());
  if (msplit > 1) {
    size_t nd = (size_t)a0.out_n * a0.out_d;
    if (count == 2) nd = std::max(nd, (size_t)pair.a[1].out_n * pair.a[1].out_d);
    hipLaunchKernelGGL(dv_sum_kernel, dim3((unsigned)((nd + 255) / 256), count), dim3(256), 0, stream, pair);
    FASTH_HIP(hipGetLastError());
  }
  return FASTH_OK;
}

static int run_dv(const Product& P, const float* V, float* dV, int transpose, hipStream_t stream,
                  bool accumulate = false, const Product* factors = nullptr) {
  DvPair pair;
  pair.a[0] = pair.a[1] = dv_args(P, V, dV, transpose, accumulate, factors);
  if (P.L.dv_trio) return launch_dv_trio(pair, 1, stream);
  return launch_dv(pair, 1, P.L.kp, P.L.dp % 4 == 0, stream);
}

// dV of two products with different outputs in one launch when both take the same template
// arguments and the same rows per block (a product of vectors beyond kMaxPaddedD elements keeps the caller's block size,
// its partner does not); otherwise one after the other.
static int run_dv_pair(const Product& P0, const float* V0, float* dV0, int transpose0, const Product& P1,
                       const float* V1, float* dV1, int transpose1, hipStream_t stream) {
  if (P0.L.ki == P1.L.ki && P0.L.kp == P1.L.kp && (P0.L.dp % 4 == 0) == (P1.L.dp % 4 == 0) && P0.L.dv_split == P1.L.dv_split && P0.L.dv_trio == P1.L.dv_trio) {
    DvPair pair;
    pair.a[0] = dv_args(P0, V0, dV0, transpose0, false);
    pair.a[1] = dv_args(P1, V1, dV1, transpose1, false);
    if (P0.L.dv_trio) return launch_dv_trio(pair, 2, stream);
    return launch_dv(pair, 2, P0.L.kp, P0.L.dp % 4 == 0, stream);
  }
  const int rc = run_dv(P0, V0, dV0, transpose0, stream);
  return rc != FASTH_OK ? rc : run_dv(P1, V1, dV1, transpose1, stream);
}

static int seq_threads(int d) {
  int threads = 256;
  if (d > 256 * 8) threads = 512;
  if (d > 512 * 8) threads = 1024;
  return threads;
}

struct SvdLayout {
  bool dense;
  size_t off_U, off_V, off_Z1, off_dZ2, off_scaled, total;
};

static SvdLayout make_svd_layout(int d, int n, int m, int k) {
  SvdLayout S;
  S.dense = dense_serves_layer(d, n, m);
  const size_t one = workspace_of(d, n, m, k, S.dense);
  const size_t dm = align_up((size_t)d * m * sizeof(float), 256);
  S.off_U = 0;
  S.off_V = align_up(one, 256);
  S.off_Z1 = S.off_V + align_up(one, 256);
  S.off_dZ2 = S.off_Z1 + dm;
  S.off_scaled = S.off_dZ2 + dm;  // the second product's inputs, scaled
  S.total = S.off_scaled + (S.dense ? dm : 0);
  return S;
}

// The layers on whole matrices: in the notation below, `first` is the factor applied transposed. Z1 = F^T X, Y = S (s Z1).
static int dense_layer_forward(const Dense& F, const float* Vf, const Dense& S, const float* Vs, const float* X, float* Z1, float* scaled,
                               const float* sigma, int mode, int rank, float* Y, hipStream_t st) {
  const Dense* D[2] = {&F, &S};
  const float* V[2] = {Vf, Vs};
  const int count = S.owner == &F ? 1 : 2;  // one set of factors?
  int rc = dense_factors(D, V, count, nullptr, 0, st);
  if (rc != FASTH_OK || (rc = dense_matrices(D, V, count, st)) != FASTH_OK) return rc;
  if ((rc = dense_apply(F, true, X, F.d, Z1, sigma, mode, rank, scaled, F.left(), st)) != FASTH_OK) return rc;
  if ((rc = dense_pack(S.pack_right(scaled, rank), FASTH_KERNEL_CHAIN, st)) != FASTH_OK) return rc;
  return dense_apply(S, false, scaled, rank, Y, nullptr, 0, 0, nullptr, nullptr, st);
}

static int dense_layer_backward(const Dense& F, const float* Vf, const Dense& S, const float* Vs, const float* G, const float* Z1, float* dZ2,
                                float* scaled, const float* sigma, int mode, int rank, float* dVf, float* dsigma, float* dVs, float* dX, hipStream_t st) {
  int rc = dense_apply(S, true, G, S.d, dZ2, sigma, mode, rank, scaled, S.left(), st);
  if (rc != FASTH_OK) return rc;
  if ((rc = dense_pack(F.pack_right(scaled, rank), FASTH_KERNEL_CHAIN, st)) != FASTH_OK) return rc;
  if ((rc = dense_apply(F, false, scaled, rank, dX, nullptr, 0, 0, nullptr, nullptr, st)) != FASTH_OK) return rc;
  {
    prof::Scope ps_(FASTH_KERNEL_DSIGMA, st, "dsigma_kernel");
    hipLaunchKernelGGL(dsigma_kernel, dim3((rank + 3) / 4), dim3(256), 0, st, (const float*)dZ2, Z1, sigma, dsigma, rank, S.m, mode);
    FASTH_HIP(hipGetLastError());
  }
  const Dense* D[2] = {&S, &F};
  if (S.owner != &F) {
    const float* V[2] = {Vs, Vf};
    float* dV[2] = {dVs, dVf};
    return dense_dv(D, V, dV, 2, false, st);
  }
  for (int i = 0; i < 2; ++i)  // both products' gradients are those of the same vectors: the second is added
    if ((rc = dense_dv(D + i, &Vf, &dVf, 1, i == 1, st)) != FASTH_OK) return rc;
  return FASTH_OK;
}

static int check_svd_shape(const fasth_svd_shape* s, fasth_shape* out) {
  if (!s) return FASTH_EINVAL;
  out->d = s->d; out->n = s->n; out->m = s->m; out->k = s->k; out->transpose = 0;
  return check_shape(out);
}

// Forward of the layer: first factor transposed, diagonal scale fused into the second chain's load.
static int svd_forward(const fasth_svd_shape* shape, const float* first, const float* sigma, const float* second,
                       const float* X, float* Y, void* workspace, size_t workspace_bytes, void* stream, int scale_mode) {
  fasth_shape fs;
  int rc = check_svd_shape(shape, &fs);
  if (rc != FASTH_OK) return rc;
  if (!first || !sigma || !second || !X || !Y || !workspace) return FASTH_EINVAL;
  if (!aligned16(first) || !aligned16(sigma) || !aligned16(second) || !aligned16(X) || !aligned16(Y) ||
      !aligned16(workspace))
    return FASTH_EALIGN;
  const SvdLayout S = make_svd_layout(fs.d, fs.n, fs.m, fs.k);
  if (workspace_bytes < S.total) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  // "first" is the factor applied transposed (V for W, U for W^-1); it owns slot off_V.
  Product Pf = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_V, S.dense);
  Product Ps = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_U, S.dense);
  float* Z1 = reinterpret_cast<float*>(ws + S.off_Z1);
  if (S.dense)
    return dense_layer_forward(Pf.D, first, Ps.D, second, X, Z1, reinterpret_cast<float*>(ws + S.off_scaled), sigma, scale_mode, fs.d, Y, st);
  if ((rc = build_factors_pair(Pf, first, Ps, second, st)) != FASTH_OK) return rc;
  if ((rc = run_chain(Pf, first, X, Z1, 1, true, nullptr, 0, st)) != FASTH_OK) return rc;
  return run_chain(Ps, second, Z1, Y, 0, true, sigma, scale_mode, st);
}

static int svd_backward(const fasth_svd_shape* shape, const float* first, const float* sigma, const float* second,
                        const float* G, float* dfirst, float* dsigma, float* dsecond, float* dX, void* workspace,
                        size_t workspace_bytes, void* stream, int scale_mode) {
  fasth_shape fs;
  int rc = check_svd_shape(shape, &fs);
  if (rc != FASTH_OK) return rc;
  if (!first || !sigma || !second || !G || !dfirst || !dsigma || !dsecond || !dX || !workspace) return FASTH_EINVAL;
  if (!aligned16(first) || !aligned16(sigma) || !aligned16(second) || !aligned16(G) || !aligned16(dfirst) ||
      !aligned16(dsigma) || !aligned16(dsecond) || !aligned16(dX) || !aligned16(workspace))
    return FASTH_EALIGN;
  const SvdLayout S = make_svd_layout(fs.d, fs.n, fs.m, fs.k);
  if (workspace_bytes < S.total) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  Product Pf = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_V, S.dense);
  Product Ps = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_U, S.dense);
  const float* Z1 = reinterpret_cast<const float*>(ws + S.off_Z1);
  float* dZ2 = reinterpret_cast<float*>(ws + S.off_dZ2);
  if (S.dense)
    return dense_layer_backward(Pf.D, first, Ps.D, second, G, Z1, dZ2, reinterpret_cast<float*>(ws + S.off_scaled), sigma, scale_mode, fs.d,
                                dfirst, dsigma, dsecond, dX, st);
  // through the second (plain) factor
  if ((rc = run_chain(Ps, second, G, dZ2, 1, false, nullptr, 0, st)) != FASTH_OK) return rc;
  // through the first (transposed) factor; dZ1 = s * dZ2 is fused into the chain's load, and the gradient of
  // sigma, which needs the same dZ2, rides along in the same launch
  if ((rc = run_chain(Pf, first, dZ2, dX, 0, false, sigma, scale_mode, st, true, nullptr, -1, Z1, dsigma, fs.d)) !=
      FASTH_OK)
    return rc;
  // both factors' vector gradients in one launch: each reads only its own saved slots
  return run_dv_pair(Ps, second, dsecond, 0, Pf, first, dfirst, 1, st);
}

static int sym_scale_mode(int function) {
  switch (function) {
    case FASTH_DIAG_IDENTITY: return 1;
    case FASTH_DIAG_EXP: return 3;
    case FASTH_DIAG_CAYLEY: return 4;
    default: return -1;
  }
}

// Rectangular layer (Section 3.3 "Rectangular Matrices"): U is rows x rows, V is cols x cols and
// Sigma is rows x cols with min(rows, cols) diagonal entries.
struct RectLayout {
  bool dense;
  size_t off_U, off_V, off_Z1, off_dZ2, off_scaled, total;
};

static int check_rect_shape(const fasth_rect_shape* s, fasth_shape* u, fasth_shape* v) {
  if (!s) return FASTH_EINVAL;
  u->d = s->rows; u->n = s->n_u; u->m = s->m; u->k = s->k; u->transpose = 0;
  v->d = s->cols; v->n = s->n_v; v->m = s->m; v->k = s->k; v->transpose = 0;
  const int rc = check_shape(u);
  return rc != FASTH_OK ? rc : check_shape(v);
}

static RectLayout make_rect_layout(const fasth_shape& u, const fasth_shape& v) {
  RectLayout S;
  S.dense = dense_serves_layer(u.d, u.n, u.m) && dense_serves_layer(v.d, v.n, v.m);
  S.off_U = 0;
  S.off_V = align_up(workspace_of(u.d, u.n, u.m, u.k, S.dense), 256);
  S.off_Z1 = S.off_V + align_up(workspace_of(v.d, v.n, v.m, v.k, S.dense), 256);
  S.off_dZ2 = S.off_Z1 + align_up((size_t)v.d * v.m * sizeof(float), 256);
  S.off_scaled = S.off_dZ2 + align_up((size_t)u.d * u.m * sizeof(float), 256);
  S.total = S.off_scaled + (S.dense ? align_up((size_t)std::min(u.d, v.d) * u.m * sizeof(float), 256) : 0);
  return S;
}

}  // namespace fasth

// ------------------------------------------------------------------------------------------
// Scratch memory of fasth_forward_static: one array per GPU, part of the loaded code object, so the call
// needs no allocation. In host code the array's name is only a handle; its device address is looked up once
// per device and kept.
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[FASTH_STATIC_SCRATCH_BYTES];

namespace fasth {
constexpr int kMaxDevices = 64;
static void* scratch_addr[kMaxDevices] = {};
static std::mutex scratch_mutex;

static int static_scratch(void** out) {
  int dev = -1;
  FASTH_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return FASTH_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_addr[dev]) {
    void* p = nullptr;
    FASTH_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return FASTH_EHIP;
    scratch_addr[dev] = p;
  }
  *out = scratch_addr[dev];
  return FASTH_OK;
}
}  // namespace fasth

// ------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------

using namespace fasth;

extern "C" {

const char* fasth_strerror(int code) {
  switch (code) {
    case FASTH_OK: return "success";
    case FASTH_EINVAL: return "invalid argument (null pointer, non-positive size, or k does not divide n)";
    case FASTH_EWORKSPACE: return "workspace too small";
    case FASTH_EALIGN: return "pointer is not 16-byte aligned";
    case FASTH_EHIP: return g_hip_error_text[0] ? g_hip_error_text : "HIP runtime call or kernel launch failed";
    case FASTH_EUNSUPPORTED: return "shape outside the supported range";
    case FASTH_ETIMEOUT: return "a kernel's wait for another workgroup gave up: results since the last check are invalid";
    default: return "unknown error code";
  }
}

int fasth_set_wait_limit(int polls) {
  g_wait_limit.store(polls < 0 ? kDefaultWaitLimit : polls, std::memory_order_relaxed);
  return FASTH_OK;
}

int fasth_wait_status(void* stream) {
  FASTH_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
  unsigned word = 0;
  FASTH_HIP(hipMemcpyFromSymbol(&word, HIP_SYMBOL(g_wait_gave_up), sizeof(word)));
  if (!word) return FASTH_OK;
  const unsigned zero = 0;
  FASTH_HIP(hipMemcpyToSymbol(HIP_SYMBOL(g_wait_gave_up), &zero, sizeof(zero)));
  return FASTH_ETIMEOUT;
}

const char* fasth_kernel_name(int id) {
  switch (id) {
    case FASTH_KERNEL_TEAM_FACTOR: return "team_factor_kernel";
    case FASTH_KERNEL_TRIO_ROWS: return "trio_rows_kernel";
    case FASTH_KERNEL_CHAIN: return "chain_kernel";
    case FASTH_KERNEL_DV: return "dv_kernel";
    case FASTH_KERNEL_SEQ_FORWARD: return "seq_forward_kernel";
    case FASTH_KERNEL_SEQ_BACKWARD: return "seq_backward_kernel";
    case FASTH_KERNEL_SEQ_REDUCE: return "seq_reduce_kernel";
    case FASTH_KERNEL_DSIGMA: return "dsigma_kernel";
    case FASTH_KERNEL_FACTOR: return "factor_fused_kernel";
    default: return "unknown";
  }
}

const char* fasth_profile_variant(int id) {
  if (id < 0 || id >= FASTH_KERNEL_COUNT || !prof::variant[id]) return "";
  return prof::variant[id];
}

int fasth_profile_enable(int on) {
  prof::enabled = on != 0;
  if (on)
    for (int i = 0; i < FASTH_KERNEL_COUNT; ++i) prof::variant[i] = nullptr;
  return FASTH_OK;
}

int fasth_profile_collect(float* ms, int* launches) {
  if (!ms || !launches) return FASTH_EINVAL;
  for (int i = 0; i < FASTH_KERNEL_COUNT; ++i) { ms[i] = 0.f; launches[i] = 0; }
  int rc = FASTH_OK;
  for (const prof::Rec& r : prof::recs) {
    float t = 0.f;
    if (r.beg && r.end && hipEventSynchronize(r.end) == hipSuccess &&
        hipEventElapsedTime(&t, r.beg, r.end) == hipSuccess && r.id >= 0 && r.id < FASTH_KERNEL_COUNT) {
      ms[r.id] += t;
      launches[r.id] += 1;
    } else {
      rc = FASTH_EHIP;
    }
    if (r.beg) prof::pool.push_back(r.beg);
    if (r.end) prof::pool.push_back(r.end);
  }
  prof::recs.clear();
  return rc;
}

int fasth_measure_peaks(void* buffer, size_t buffer_bytes, int repetitions, float* fp32_mfma_tflops,
                        float* hbm_read_gbs, float* hbm_copy_gbs, void* stream) {
  if (!buffer || !fp32_mfma_tflops || !hbm_read_gbs || !hbm_copy_gbs || repetitions < 1) return FASTH_EINVAL;
  if (!aligned16(buffer)) return FASTH_EALIGN;
  if (buffer_bytes < (size_t)(8u << 20)) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  FASTH_HIP(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return FASTH_EHIP; }
  float* fbuf = static_cast<float*>(buffer);
  const int wgs = 4 * kComputeUnits, iters = 4096;
  const size_t pieces = buffer_bytes / 16, half = pieces / 2;
  int rc = FASTH_OK;
  float best[3] = {0.f, 0.f, 0.f};
  for (int which = 0; which < 3 && rc == FASTH_OK; ++which) {
    for (int rep = 0; rep <= repetitions && rc == FASTH_OK; ++rep) {  // the first pass is not timed
      if (hipEventRecord(e0, st) != hipSuccess) { rc = FASTH_EHIP; break; }
      if (which == 0) hipLaunchKernelGGL(peak_mfma_kernel, dim3(wgs), dim3(256), 0, st, fbuf, iters);
      else if (which == 1) hipLaunchKernelGGL(peak_read_kernel, dim3(8 * kComputeUnits), dim3(256), 0, st, static_cast<const float4*>(buffer) + 4096, pieces - 4096, fbuf);
      else hipLaunchKernelGGL(peak_copy_kernel, dim3(8 * kComputeUnits), dim3(256), 0, st, static_cast<const float4*>(buffer), static_cast<float4*>(buffer) + half, half);
      float ms = 0.f;
      if (hipGetLastError() != hipSuccess || hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
          hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { rc = FASTH_EHIP; break; }
      if (rep == 0 || ms <= 0.f) continue;
      float rate;
      if (which == 0) rate = (float)((double)wgs * 4 * iters * kPeakMfmaPerIter * 2048.0 / (ms * 1e-3) / 1e12);
      else if (which == 1) rate = (float)((double)(pieces - 4096) * 16.0 / (ms * 1e-3) / 1e9);
      else rate = (float)((double)half * 32.0 / (ms * 1e-3) / 1e9);  // bytes read + bytes written
      if (rate > best[which]) best[which] = rate;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != FASTH_OK) return rc;
  *fp32_mfma_tflops = best[0]; *hbm_read_gbs = best[1]; *hbm_copy_gbs = best[2];
  return FASTH_OK;
}

size_t fasth_workspace_bytes(const fasth_shape* shape) {
  if (check_shape(shape) != FASTH_OK) return 0;
  return workspace_of(shape->d, shape->n, shape->m, shape->k, dense_serves(shape->d, shape->n, shape->m));
}

int fasth_forward(const fasth_shape* shape, const float* V, const float* X, float* A, void* workspace,
                  size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !X || !A || !workspace) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(X) || !aligned16(A) || !aligned16(workspace)) return FASTH_EALIGN;
  const Product P = bind(shape->d, shape->n, shape->m, shape->k, workspace, dense_serves(shape->d, shape->n, shape->m));
  if (workspace_bytes < workspace_of(P)) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (P.dense) {
    const bool t = shape->transpose != 0;
    const Dense* list[1] = {&P.D};
    const PackJob jobs[1] = {P.D.pack_right(X, P.d)};
    if ((rc = dense_factors(list, &V, 1, jobs, t ? 0 : 1, st)) != FASTH_OK || (rc = dense_matrices(list, &V, 1, st)) != FASTH_OK) return rc;
    return dense_apply(P.D, t, X, P.d, A, nullptr, 0, 0, nullptr, t ? P.D.left() : nullptr, st);
  }
  if ((rc = build_factors(P, V, st)) != FASTH_OK) return rc;
  return run_chain(P, V, X, A, shape->transpose, true, nullptr, 0, st);
}

int fasth_forward_static(const fasth_shape* shape, const float* V, const float* X, float* A, void* stream) {
  int rc = check_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !X || !A) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(X) || !aligned16(A)) return FASTH_EALIGN;
  // Only the regions Step 1 writes and Step 2 reads: nothing is saved for a backward pass. Where the operands of V for wide
  // mini-batches do not fit, the layout without them. Where that does not fit either (a large V that is copied or whose shared-column
  // kernels need much), the reflections go in segments, one after the other on the same array and in place: H X = H_1 ... H_s (H_{s+1}
  // ... H_n X). us, the rows as the caller has them and segments: d = 1000, n = 6000, m = 32, k = 50: 515, 192; d = 1023, n = 7000,
  // m = 32, k = 28: 519, 234; d = 1000, n = 6000, m = 600, k = 24: 1540, 463; d = 2048, n = 6400, m = 32, k = 32: 494, 258. The caller's
  // own blocks decide what is refused, and serve vectors that no layout pads.
  const int d = shape->d, n = shape->n, m = shape->m, k = shape->k;
  auto fits = [&](int rows, LayoutLevel l) { return make_layout(d, rows, m, k, l).off_saveA <= FASTH_STATIC_SCRATCH_BYTES; };
  LayoutLevel level = kLayoutTrio;
  int rows = n;  // of a segment; the last one has what is left
  if (!fits(n, level)) {
    level = kLayoutShared;
    if (!fits(n, level)) {
      if (!fits(n, kLayoutPlain)) return FASTH_EUNSUPPORTED;
      if (d > kMaxPaddedD) level = kLayoutPlain;
      else
        for (int parts = 2; rows > kWideRows && !(fits(rows, level) && fits(n - (n - 1) / rows * rows, level)); ++parts)
          rows = padded_rows((n + parts - 1) / parts, kWideRows);
    }
  }
  void* ws = nullptr;
  if ((rc = static_scratch(&ws)) != FASTH_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int segments = (n + rows - 1) / rows;
  for (int i = 0; i < segments; ++i) {
    const int first = (shape->transpose ? i : segments - 1 - i) * rows;
    const Product P = bind(d, std::min(rows, n - first), m, k, ws, false, level);
    const float* Vs = V + (size_t)first * d;
    if ((rc = build_factors(P, Vs, st)) != FASTH_OK) return rc;
    if ((rc = run_chain(P, Vs, i == 0 ? X : A, A, shape->transpose, true, nullptr, 0, st, false)) != FASTH_OK) return rc;
  }
  return FASTH_OK;
}

int fasth_prepare(const fasth_shape* shape, const float* V, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !workspace) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(workspace)) return FASTH_EALIGN;
  const Product P = bind(shape->d, shape->n, shape->m, shape->k, workspace, dense_serves(shape->d, shape->n, shape->m));
  if (workspace_bytes < workspace_of(P)) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (P.dense) {
    const Dense* D[1] = {&P.D};
    if ((rc = dense_factors(D, &V, 1, nullptr, 0, st)) != FASTH_OK) return rc;
    return dense_matrices(D, &V, 1, st);
  }
  return build_factors(P, V, st);
}

int fasth_apply(const fasth_shape* shape, const float* V, const float* X, float* A, void* workspace,
                size_t workspace_bytes, int save_for_backward, void* stream) {
  int rc = check_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !X || !A || !workspace) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(X) || !aligned16(A) || !aligned16(workspace)) return FASTH_EALIGN;
  Product P = bind(shape->d, shape->n, shape->m, shape->k, workspace, dense_serves(shape->d, shape->n, shape->m));
  if (workspace_bytes < workspace_of(P)) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (P.dense) {
    const bool t = shape->transpose != 0, save = save_for_backward != 0;
    if (save && !t && (rc = dense_pack(P.D.pack_right(X, P.d), FASTH_KERNEL_CHAIN, st)) != FASTH_OK) return rc;
    return dense_apply(P.D, t, X, P.d, A, nullptr, 0, 0, nullptr, save && t ? P.D.left() : nullptr, st);
  }
  P.exclusive = save_for_backward != 0;
  return run_chain(P, V, X, A, shape->transpose, true, nullptr, 0, st, save_for_backward != 0);
}

int fasth_backward(const fasth_shape* shape, const float* V, const float* G, float* dV, float* dX, void* workspace,
                   size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !G || !dV || !dX || !workspace) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(G) || !aligned16(dV) || !aligned16(dX) || !aligned16(workspace)) return FASTH_EALIGN;
  const Product P = bind(shape->d, shape->n, shape->m, shape->k, workspace, dense_serves(shape->d, shape->n, shape->m));
  if (workspace_bytes < workspace_of(P)) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (P.dense) {
    const bool t = shape->transpose != 0;
    const Dense* list[1] = {&P.D};
    if (t && (rc = dense_pack(P.D.pack_right(G, P.d), FASTH_KERNEL_CHAIN, st)) != FASTH_OK) return rc;
    if ((rc = dense_apply(P.D, !t, G, P.d, dX, nullptr, 0, 0, nullptr, t ? nullptr : P.D.left(), st)) != FASTH_OK) return rc;
    return dense_dv(list, &V, &dV, 1, false, st);
  }
  if ((rc = run_chain(P, V, G, dX, !shape->transpose, false, nullptr, 0, st)) != FASTH_OK) return rc;
  return run_dv(P, V, dV, shape->transpose, st);
}

int fasth_tune_block_size(const fasth_shape* shape, const int* candidates, int ncandidates, int repetitions,
                          const float* V, const float* X, const float* G, float* A, float* dV, float* dX,
                          void* workspace, size_t workspace_bytes, int* best_k, float* best_ms, void* stream) {
  if (!shape || !best_k) return FASTH_EINVAL;
  if (shape->d < 1 || shape->n < 1 || shape->m < 1 || repetitions < 1) return FASTH_EINVAL;
  if ((candidates && ncandidates < 1) || (shape->transpose != 0 && shape->transpose != 1)) return FASTH_EINVAL;
  if (!V || !X || !G || !A || !dV || !dX || !workspace) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(X) || !aligned16(G) || !aligned16(A) || !aligned16(dV) || !aligned16(dX) ||
      !aligned16(workspace))
    return FASTH_EALIGN;
  std::vector<int> ks;
  if (candidates) {
    ks.assign(candidates, candidates + ncandidates);
  } else {
    for (int k = 2; k <= kMaxBlock && k <= shape->n; ++k)
      if (shape->n % k == 0) ks.push_back(k);
    if (ks.empty()) ks.push_back(1);
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  FASTH_HIP(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return FASTH_EHIP; }
  int rc = FASTH_OK, found = 0;
  float best = 0.f;
  std::vector<Layout> tried;
  for (int k : ks) {
    fasth_shape s = *shape;
    s.k = k;
    if (check_shape(&s) != FASTH_OK || fasth_workspace_bytes(&s) > workspace_bytes) continue;  // not a usable candidate
    // the library's blocks decide what runs: a candidate that leads to the same ones has been tried (its first stands for all)
    if (dense_serves(s.d, s.n, s.m) && found) break;  // no blocks
    const Layout L = make_layout(s.d, s.n, s.m, k);
    if (std::any_of(tried.begin(), tried.end(), [&](const Layout& t) { return t.ki == L.ki && t.np == L.np && t.trio.parts == L.trio.parts; }))
      continue;
    tried.push_back(L);
    // one untimed pass, then `repetitions` timed ones
    for (int pass = 0; pass < 2 && rc == FASTH_OK; ++pass) {
      const int reps = pass == 0 ? 1 : repetitions;
      if (pass == 1 && hipEventRecord(e0, st) != hipSuccess) { rc = FASTH_EHIP; break; }
      for (int r = 0; r < reps && rc == FASTH_OK; ++r) {
        rc = fasth_forward(&s, V, X, A, workspace, workspace_bytes, stream);
        if (rc == FASTH_OK) rc = fasth_backward(&s, V, G, dV, dX, workspace, workspace_bytes, stream);
      }
      if (pass == 1 && rc == FASTH_OK) {
        float ms = 0.f;
        if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
          rc = FASTH_EHIP;
          break;
        }
        ms /= repetitions;
        if (!found || ms < best) { best = ms; *best_k = k; found = 1; }
      }
    }
    if (rc != FASTH_OK) break;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != FASTH_OK) return rc;
  if (!found) return FASTH_EUNSUPPORTED;
  if (best_ms) *best_ms = best;
  return FASTH_OK;
}

size_t fasth_sequential_workspace_bytes(const fasth_shape* shape) {
  if (!shape || shape->d < 1 || shape->n < 1 || shape->m < 1) return 0;
  if (shape->d > kMaxD || shape->m > 65535) return 0;
  return (size_t)shape->m * shape->n * shape->d * sizeof(float);
}

static int check_seq_shape(const fasth_shape* s) {
  if (!s) return FASTH_EINVAL;
  if (s->d < 1 || s->n < 1 || s->m < 1) return FASTH_EINVAL;
  if (s->transpose != 0 && s->transpose != 1) return FASTH_EINVAL;
  if (s->d > kMaxD || s->m > 65535) return FASTH_EUNSUPPORTED;
  return FASTH_OK;
}

#define FASTH_SEQ_DISPATCH(KERNEL, per, grid, block, stream, ...)                         \
  do {                                                                                    \
    if ((per) <= 1) hipLaunchKernelGGL(KERNEL<1>, grid, block, 0, stream, __VA_ARGS__);      \
    else if ((per) <= 2) hipLaunchKernelGGL(KERNEL<2>, grid, block, 0, stream, __VA_ARGS__); \
    else if ((per) <= 4) hipLaunchKernelGGL(KERNEL<4>, grid, block, 0, stream, __VA_ARGS__); \
    else if ((per) <= 8) hipLaunchKernelGGL(KERNEL<8>, grid, block, 0, stream, __VA_ARGS__); \
    else hipLaunchKernelGGL(KERNEL<16>, grid, block, 0, stream, __VA_ARGS__);                \
  } while (0)

int fasth_sequential_forward(const fasth_shape* shape, const float* V, const float* X, float* A, void* stream) {
  int rc = check_seq_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !X || !A) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(X) || !aligned16(A)) return FASTH_EALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int threads = seq_threads(shape->d), per = (shape->d + threads - 1) / threads;
  {
    prof::Scope ps_(FASTH_KERNEL_SEQ_FORWARD, st, "seq_forward_kernel");
    FASTH_SEQ_DISPATCH(seq_forward_kernel, per, dim3(shape->m), dim3(threads), st, V, X, A, shape->d, shape->n,
                       shape->m, shape->transpose);
  }
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

int fasth_sequential_backward(const fasth_shape* shape, const float* V, const float* A, const float* G, float* dV,
                              float* dX, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_seq_shape(shape);
  if (rc != FASTH_OK) return rc;
  if (!V || !A || !G || !dV || !dX || !workspace) return FASTH_EINVAL;
  if (!aligned16(V) || !aligned16(A) || !aligned16(G) || !aligned16(dV) || !aligned16(dX) || !aligned16(workspace))
    return FASTH_EALIGN;
  if (workspace_bytes < fasth_sequential_workspace_bytes(shape)) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int d = shape->d, n = shape->n, m = shape->m;
  float* dVpart = static_cast<float*>(workspace);
  const int threads = seq_threads(d), per = (d + threads - 1) / threads;
  {
    prof::Scope ps_(FASTH_KERNEL_SEQ_BACKWARD, st, "seq_backward_kernel");
    FASTH_SEQ_DISPATCH(seq_backward_kernel, per, dim3(m), dim3(threads), st, V, A, G, dVpart, dX, d, n, m,
                       shape->transpose);
  }
  FASTH_HIP(hipGetLastError());
  const size_t nd = (size_t)n * d;
  {
    prof::Scope ps_(FASTH_KERNEL_SEQ_REDUCE, st, "seq_reduce_kernel");
    hipLaunchKernelGGL(seq_reduce_kernel, dim3((unsigned)((nd + 255) / 256)), dim3(256), 0, st, (const float*)dVpart,
                       dV, nd, m);
  }
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

size_t svd_layer_workspace_bytes(const fasth_svd_shape* shape) {
  fasth_shape fs;
  if (check_svd_shape(shape, &fs) != FASTH_OK) return 0;
  return make_svd_layout(fs.d, fs.n, fs.m, fs.k).total;
}

int svd_sym_apply(const fasth_svd_shape* shape, int function, const float* Uv, const float* sigma, const float* X,
                  float* Y, void* workspace, size_t workspace_bytes, void* stream) {
  fasth_shape fs;
  int rc = check_svd_shape(shape, &fs);
  if (rc != FASTH_OK) return rc;
  const int mode = sym_scale_mode(function);
  if (mode < 0 || !Uv || !sigma || !X || !Y || !workspace) return FASTH_EINVAL;
  if (!aligned16(Uv) || !aligned16(sigma) || !aligned16(X) || !aligned16(Y) || !aligned16(workspace)) return FASTH_EALIGN;
  const SvdLayout S = make_svd_layout(fs.d, fs.n, fs.m, fs.k);
  if (workspace_bytes < S.total) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  Product Pin = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_V, S.dense);   // U^T X; owns the factors
  Product Pout = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_U, S.dense);  // U (s * Z1); saves only
  float* Z1 = reinterpret_cast<float*>(ws + S.off_Z1);
  if (S.dense) {
    Pout.D.owner = &Pin.D;
    return dense_layer_forward(Pin.D, Uv, Pout.D, Uv, X, Z1, reinterpret_cast<float*>(ws + S.off_scaled), sigma, mode, fs.d, Y, st);
  }
  if ((rc = build_factors(Pin, Uv, st)) != FASTH_OK) return rc;
  if ((rc = run_chain(Pin, Uv, X, Z1, 1, true, nullptr, 0, st)) != FASTH_OK) return rc;
  return run_chain(Pout, Uv, Z1, Y, 0, true, sigma, mode, st, true, &Pin);
}

int svd_sym_apply_backward(const fasth_svd_shape* shape, int function, const float* Uv, const float* sigma,
                           const float* G, float* dUv, float* dsigma, float* dX, void* workspace,
                           size_t workspace_bytes, void* stream) {
  fasth_shape fs;
  int rc = check_svd_shape(shape, &fs);
  if (rc != FASTH_OK) return rc;
  const int mode = sym_scale_mode(function);
  if (mode < 0 || !Uv || !sigma || !G || !dUv || !dsigma || !dX || !workspace) return FASTH_EINVAL;
  if (!aligned16(Uv) || !aligned16(sigma) || !aligned16(G) || !aligned16(dUv) || !aligned16(dsigma) ||
      !aligned16(dX) || !aligned16(workspace))
    return FASTH_EALIGN;
  const SvdLayout S = make_svd_layout(fs.d, fs.n, fs.m, fs.k);
  if (workspace_bytes < S.total) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  Product Pin = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_V, S.dense);
  Product Pout = bind(fs.d, fs.n, fs.m, fs.k, ws + S.off_U, S.dense);
  const float* Z1 = reinterpret_cast<const float*>(ws + S.off_Z1);
  float* dZ2 = reinterpret_cast<float*>(ws + S.off_dZ2);
  if (S.dense) {
    Pout.D.owner = &Pin.D;
    return dense_layer_backward(Pin.D, Uv, Pout.D, Uv, G, Z1, dZ2, reinterpret_cast<float*>(ws + S.off_scaled), sigma, mode, fs.d, dUv, dsigma,
                                dUv, dX, st);
  }
  if ((rc = run_chain(Pout, Uv, G, dZ2, 1, false, nullptr, 0, st, true, &Pin)) != FASTH_OK) return rc;
  if ((rc = run_dv(Pout, Uv, dUv, 0, st, false, &Pin)) != FASTH_OK) return rc;
  if ((rc = run_chain(Pin, Uv, dZ2, dX, 0, false, sigma, mode, st, true, nullptr, -1, Z1, dsigma, fs.d)) != FASTH_OK)
    return rc;
  return run_dv(Pin, Uv, dUv, 1, st, true);
}

int svd_layer_log_abs_det(int d, const float* sigma, float* log_abs_det, float* dsigma, void* stream) {
  if (d < 1 || !sigma || !log_abs_det) return FASTH_EINVAL;
  if (!aligned16(sigma) || (dsigma && !aligned16(dsigma))) return FASTH_EALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(logabsdet_kernel, dim3(1), dim3(256), 0, st, sigma, log_abs_det, dsigma, d);
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

int svd_layer_apply(const fasth_svd_shape* shape, const float* Uv, const float* sigma, const float* Vv, const float* X,
                    float* Y, void* workspace, size_t workspace_bytes, void* stream) {
  return svd_forward(shape, Vv, sigma, Uv, X, Y, workspace, workspace_bytes, stream, 1);
}

int svd_layer_inverse_apply(const fasth_svd_shape* shape, const float* Uv, const float* sigma, const float* Vv,
                            const float* X, float* Y, void* workspace, size_t workspace_bytes, void* stream) {
  return svd_forward(shape, Uv, sigma, Vv, X, Y, workspace, workspace_bytes, stream, 2);
}

int svd_layer_apply_backward(const fasth_svd_shape* shape, const float* Uv, const float* sigma, const float* Vv,
                             const float* G, float* dUv, float* dsigma, float* dVv, float* dX, void* workspace,
                             size_t workspace_bytes, void* stream) {
  return svd_backward(shape, Vv, sigma, Uv, G, dVv, dsigma, dUv, dX, workspace, workspace_bytes, stream, 1);
}

int svd_layer_inverse_apply_backward(const fasth_svd_shape* shape, const float* Uv, const float* sigma,
                                     const float* Vv, const float* G, float* dUv, float* dsigma, float* dVv,
                                     float* dX, void* workspace, size_t workspace_bytes, void* stream) {
  return svd_backward(shape, Uv, sigma, Vv, G, dUv, dsigma, dVv, dX, workspace, workspace_bytes, stream, 2);
}

size_t svd_rect_workspace_bytes(const fasth_rect_shape* shape) {
  fasth_shape fu, fv;
  if (check_rect_shape(shape, &fu, &fv) != FASTH_OK) return 0;
  return make_rect_layout(fu, fv).total;
}

int svd_rect_apply(const fasth_rect_shape* shape, const float* Uv, const float* sigma, const float* Vv, const float* X,
                   float* Y, void* workspace, size_t workspace_bytes, void* stream) {
  fasth_shape fu, fv;
  int rc = check_rect_shape(shape, &fu, &fv);
  if (rc != FASTH_OK) return rc;
  if (!Uv || !sigma || !Vv || !X || !Y || !workspace) return FASTH_EINVAL;
  if (!aligned16(Uv) || !aligned16(sigma) || !aligned16(Vv) || !aligned16(X) || !aligned16(Y) || !aligned16(workspace))
    return FASTH_EALIGN;
  const RectLayout S = make_rect_layout(fu, fv);
  if (workspace_bytes < S.total) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  Product Pu = bind(fu.d, fu.n, fu.m, fu.k, ws + S.off_U, S.dense);
  Product Pv = bind(fv.d, fv.n, fv.m, fv.k, ws + S.off_V, S.dense);
  float* Z1 = reinterpret_cast<float*>(ws + S.off_Z1);
  const int r = fu.d < fv.d ? fu.d : fv.d;
  if (S.dense) return dense_layer_forward(Pv.D, Vv, Pu.D, Uv, X, Z1, reinterpret_cast<float*>(ws + S.off_scaled), sigma, 1, r, Y, st);
  if ((rc = build_factors_pair(Pv, Vv, Pu, Uv, st)) != FASTH_OK) return rc;
  if ((rc = run_chain(Pv, Vv, X, Z1, 1, true, nullptr, 0, st)) != FASTH_OK) return rc;
  // Sigma Z1: the first r rows of Z1 scaled by sigma, rows r..rows-1 zero; fused into the chain's load
  return run_chain(Pu, Uv, Z1, Y, 0, true, sigma, 1, st, true, nullptr, r);
}

int svd_rect_apply_backward(const fasth_rect_shape* shape, const float* Uv, const float* sigma, const float* Vv,
                            const float* G, float* dUv, float* dsigma, float* dVv, float* dX, void* workspace,
                            size_t workspace_bytes, void* stream) {
  fasth_shape fu, fv;
  int rc = check_rect_shape(shape, &fu, &fv);
  if (rc != FASTH_OK) return rc;
  if (!Uv || !sigma || !Vv || !G || !dUv || !dsigma || !dVv || !dX || !workspace) return FASTH_EINVAL;
  if (!aligned16(Uv) || !aligned16(sigma) || !aligned16(Vv) || !aligned16(G) || !aligned16(dUv) ||
      !aligned16(dsigma) || !aligned16(dVv) || !aligned16(dX) || !aligned16(workspace))
    return FASTH_EALIGN;
  const RectLayout S = make_rect_layout(fu, fv);
  if (workspace_bytes < S.total) return FASTH_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  Product Pu = bind(fu.d, fu.n, fu.m, fu.k, ws + S.off_U, S.dense);
  Product Pv = bind(fv.d, fv.n, fv.m, fv.k, ws + S.off_V, S.dense);
  const float* Z1 = reinterpret_cast<const float*>(ws + S.off_Z1);
  float* dZ2 = reinterpret_cast<float*>(ws + S.off_dZ2);
  const int r = fu.d < fv.d ? fu.d : fv.d;
  if (S.dense)
    return dense_layer_backward(Pv.D, Vv, Pu.D, Uv, G, Z1, dZ2, reinterpret_cast<float*>(ws + S.off_scaled), sigma, 1, r, dVv, dsigma, dUv, dX, st);
  if ((rc = run_chain(Pu, Uv, G, dZ2, 1, false, nullptr, 0, st)) != FASTH_OK) return rc;
  // Sigma^T dZ2: first r rows scaled, rows r..cols-1 zero
  if ((rc = run_chain(Pv, Vv, dZ2, dX, 0, false, sigma, 1, st, true, nullptr, r, Z1, dsigma, r)) != FASTH_OK) return rc;
  return run_dv_pair(Pu, Uv, dUv, 0, Pv, Vv, dVv, 1, st);
}

}  // extern "C"
