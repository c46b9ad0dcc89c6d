// Every layout against what the kernels that will read it expect, over all forms a call can take: run on the host only.
#include <hip/hip_runtime.h>

#include <cstdio>

#include "fasth_common.h"
#include "fasth_factor.h"
#include "fasth_chain.h"
#include "fasth_dense.h"

using namespace fasth;

static long failures = 0, layouts = 0;

static void check(int d, int n, int m, int k, LayoutLevel level) {
  const bool own = d > kMaxPaddedD || level == kLayoutPlain;  // the caller's blocks: k divides n
  if (own && n % k) return;
  ++layouts;
  const Layout L = make_layout(d, n, m, k, level);
  auto expect = [&](bool ok, const char* what) {
    if (ok || ++failures > 20) return;
    printf("%s: d=%d n=%d m=%d k=%d level=%d: blocks of %d, %d rows, factors of %d\n", what, d, n, m, k, (int)level, L.ki, L.np, L.kf);
  };
  expect(L.np >= n && L.np % L.ki == 0 && L.np % L.kf == 0 && L.np - n < 128 && L.nb == L.np / L.ki, "whole blocks and factors");
  expect(L.dp >= d && L.dp - d < 4 && L.copy_v == (L.dp != d || L.np != n), "padding and the copy of V");
  expect(L.off_ready - L.off_Spart >= (size_t)L.nb * L.kp * L.kp * sizeof(float), "room for Z");
  expect(L.nb <= kMaxBlocks && (own || L.nbf + L.npair <= kMaxBlocks), "grid dimensions");
  if (own) return;
  for (int call = 0; call < 3; ++call) {  // saving; without, alone on its workspace; without, overlapping
    const bool save = call == 0, no_teams = call == 2 && shared_tiles_overlap(L.dp, m);
    ChainArgs a{};
    a.xch = no_teams || !L.xch_words ? nullptr : reinterpret_cast<unsigned*>(16);
    a.frag = L.trio.parts ? reinterpret_cast<const char*>(16) : nullptr;
    a.d = L.dp; a.n = L.np; a.m = m;
    a.k = no_teams || (L.trio.parts && !save) ? L.kf : L.ki;
    a.kp = padded_block(a.k); a.nb = L.np / a.k;
    int rows = a.k;  // of a stored factor, as the kernel that is launched reads it
    bool wide = false;
    if (chain_uses_trio(a)) rows = 64;
    else if (chain_uses_team_tile(a)) rows = L.dp > 1024 ? 32 : 64;
    else if (chain_uses_tile(a) || chain_uses_quad(a)) rows = a.k;
    else if (chain_uses_team_wide(a)) { rows = 64; wide = true; }
    else if (chain_uses_team(a)) rows = 64;
    else if (!chain_uses_split_pair(a))
      expect(a.k == 32 || a.k == 64 || a.k == 128 || (a.d <= 2048 ? a.k == 16 || a.k == 8 : a.k % 8 == 0), "blocks of chain_pipe_kernel");
    expect(rows == L.kf, save ? "factors (saving)" : "factors (not saving)");
    expect(wide == (L.team_wide != 0), "order of the factors");
    expect(!a.xch || no_teams || L.xch_words > 0, "hand-off area");
  }
}

// The whole matrix: every area holds what its kernels write and read, padding included, and ends before the next; the kernels' 32-bit
// offsets and launch sizes.
static void check_dense(int d, int n, int m) {
  if (!dense_serves(d, n, m) && !dense_serves_layer(d, n, m)) return;
  ++layouts;
  const DenseLayout L = make_dense_layout(d, n, m);
  const size_t dp = (d + 63) / 64 * 64, np = (n + 63) / 64 * 64, mp = (m + 63) / 64 * 64, nd = (size_t)n * d, dd = (size_t)d * d;
  const struct { size_t at, bytes; } areas[] = {
      {L.Vt, dp * np * 6}, {L.S, np * 256 * 8}, {L.factor, np * 64 * 8}, {L.T, np * 256 * 6}, {L.TV, np * dp * 6}, {L.P, dd * 4}, {L.Y, nd * 4}, {L.Ya, np * dp * 6},
      {L.H, dp * dp * 6}, {L.Ht, dp * dp * 6}, {L.left, dp * mp * 6}, {L.right, dp * mp * 6}, {L.Q, (size_t)L.q_split * dd * 4}, {L.K, dd * 4}, {L.W, nd * 4},
      {L.Wa, np * dp * 6}, {L.U, np * np * 6}};
  bool ok = L.q_split >= 1 && L.q_split <= std::max(1, m / 256);
  for (const auto& a : areas) {
    ok = ok && a.at % 256 == 0 && a.at + a.bytes <= L.total;
    for (const auto& b : areas) ok = ok && (&a == &b || a.at + a.bytes <= b.at || b.at + b.bytes <= a.at);
  }
  const size_t limit = 1ull << 31;  // bytes of a buffer, and offsets into it
  ok = ok && dd * 4 < limit && nd * 4 < limit && (size_t)d * m * 4 < limit && (size_t)kGroup * d * 4 < limit;
  ok = ok && (long)((n + kGroup - 1) / kGroup) * kGroupTiles + (long)(dp / 64) * std::max(np / 64, mp / 64) < (1l << 31);
  if (ok || ++failures > 20) return;
  printf("whole matrix: d=%d n=%d m=%d: total %zu\n", d, n, m, L.total);
}

int main() {
  for (int d = 400; d <= 4096; d = d < 700 ? d + 7 : d * 9 / 8 + 1)
    for (int n = d / 3; n <= 3 * d / 2 + 3; n = n * 8 / 7 + 1)
      for (int m = 300; m <= 65535; m = m < 3000 ? m * 9 / 8 : m * 2 - 1) check_dense(d, n, m);
  for (int d : {448, 512, 640, 768, 1024, 2048, 4096})
    for (int n : {d / 2, d, 3 * d / 2})
      for (int m : {1024, 65535}) check_dense(d, n, m);
  for (int d : {1, 63, 64, 130, 256, 257, 512, 513, 640, 768, 769, 897, 1024, 1025, 1280, 1281, 1536, 1537, 2047, 2048, 2049, 3072, 3073, 4096, 4097, 16384})
    for (int n = 1; n < 9000000; n = n < 700 ? n + 1 + n / 25 : n * 3 + 1)
      for (int m = 1; m <= 65535; m = m < 70 ? m * 3 + 1 : m < 5000 ? m * 6 / 5 : m * 3)
        for (int k : {1, 8, 9, 16, 31, 32, 33, 64, 100, 128})
          for (LayoutLevel level : {kLayoutTrio, kLayoutShared, kLayoutPlain})
            if (n / k <= kMaxBlocks) check(d, n, m, k, level);
  printf("%ld layouts, %ld failures\n", layouts, failures);
  return failures != 0;
}
