// Algorithm 1 Step 2 and Algorithm 2 Step 1 for mini-batches of more than a thousand columns on the bf16 matrix cores
// at fp32 precision (chain_trio_kernel), and the kernel that lays the rows of V out for it (trio_rows_kernel).
// Included by fasth_chain.h after ChainArgs, diag_factor and dsigma_row.
#pragma once
#include <hip/hip_runtime.h>

#include "fasth_common.h"

namespace fasth {

// ------------------------------------------------------------------------------------------
// The fp32 matrix instructions of this GPU run at 157 TFLOP/s, the bf16 ones at 2.5 PFLOP/s with fp32 accumulation. An
// fp32 number is the sum of three bf16 numbers (device helper split8), and a product of two such sums without its three
// smallest terms is six bf16 products: 2.4 times the fp32 rate measured (2.0 PFLOP/s / 6 against 146 TFLOP/s).
// The leading products h h accumulate by themselves, the five others, together about 2^-7 of them at most, in a second accumulator,
// and the two are added once at the end: a sum then has one rounding of full size per 32 terms where the fp32
// instruction has one per 4, and its error is SMALLER (2-norm against fp64, normal operands: 64 terms 5.5e-8 against
// 8.4e-8, 256 terms 9.1e-8 against 1.5e-7, 1024 terms 1.9e-7 against 2.9e-7; all six in one accumulator: 4.9e-7).
// Results below 2^-126 behave alike: these instructions keep denormal operands (same errors with operands of 1e-33).
//
// Layout. A workgroup of 8 waves holds CT tiles of 16 columns; wave w of part j of NP holds XW = 16 XT consecutive rows of
// the columns from x_w = (8 j + w) XW on, in the accumulators of the second product, for the whole chain: register jj of
// lane (q, i) of accumulator t = 2 b + h is A(x_w + 32 b + 8 q + 4 h + jj, column i). A contraction may take its terms in any
// order, and this one makes the eight registers (h, jj) of a lane the eight consecutive inner indices that it supplies as
// the B operand of v_mfma_f32_16x16x32_bf16, so A is split in registers and never moves between lanes.
// The rows of V come as matrix-instruction operands of 1 KiB (64 lanes x 16 bytes, three pieces each), straight from the
// workspace into registers: trio_rows_kernel writes, per 64 rows and 32 elements, the 12 operands of the first product
// (4 row tiles) and the 12 of the second (2 element tiles x 2 halves of the rows). No wave needs another wave's
// elements, so V never passes through LDS.
// A step takes 64 rows, whose 64 x 64 factor the factor kernels build: B = V_rows A (64 x 16 CT) is summed over the waves in
// LDS and, with NP > 1, over the parts through the workspace (all to all, words {sum, tag, sum, tag}, tagged and bounded
// as in chain_team_tile_kernel); a wave forms one 16 x 16 tile of C = op(T) B with fp32 instructions, splits it and
// leaves it in LDS as operands of A -= V_rows^T C. Three barriers per step. The operands of the second product are
// fetched while the sums are handed over, those of the next step's first product during the second product.
// What bounds it: d = n = 1024, m = 4096 ({4, 2}, two parts), a step of 6.2 us: 2.9 us first product and the wait for the slower
// wave, 1.1 us hand-over, 0.9 us C, 1.3 us second product; the products take 1.3 us each at the matrix cores' rate: the 24 KiB
// per wave and product come into a compute unit at about 36 bytes per clock. (Touching the next steps' cache lines ahead
// made it slower, 122 -> 139 us per chain, as the hand-over's loads then wait for those; the first product's operands of the next
// step fetched before the hand-over: 76 -> 88 us at m = 1024, {2, 1}.) Per chain, nothing saved: 178 -> 122 us (chain_tile_kernel),
// m = 2048: 174 -> 101, m = 8192: 305 -> 198; d = 256, m = 4096: 31 -> 16; d = 512, m = 4096: 71 -> 45; d = 2048, m = 4096: 603 -> 395.
// ------------------------------------------------------------------------------------------
constexpr int kTrioOperand = 1024;                      // bytes of one operand
constexpr int kTrioCell = 24 * kTrioOperand;            // bytes per 64 rows x 32 elements

struct TrioRowsArgs {
  const float* V;   // [n][d], the caller's
  char* frag;       // [rows / 64][xblocks][24][1024]
  int d, n, xblocks, steps;
};
struct TrioRowsPair {
  TrioRowsArgs a[2];
};

// One workgroup per cell: its 64 x 32 elements through LDS, then each wave forms two of the eight operand triples.
// Rows and elements that do not exist are zero. Reads 4 and writes 12 bytes per element.
__global__ void __launch_bounds__(256) trio_rows_kernel(TrioRowsPair pair) {
  __shared__ float tile[64][33];
  const TrioRowsArgs& p = pair.a[blockIdx.z];
  const int st = blockIdx.y, xb = blockIdx.x;
  if (st >= p.steps || xb >= p.xblocks) return;  // whole workgroup
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, i = lane & 15;
  const BufferDesc vdesc = make_buffer(p.V + (size_t)st * 64 * p.d, (size_t)max(0, min(64, p.n - st * 64)) * p.d * sizeof(float));
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int r = (tid >> 5) + 8 * it, x = xb * 32 + (tid & 31);
    tile[r][tid & 31] = buffer_load<1>(vdesc, x < p.d ? (unsigned)(r * p.d + x) * 4u : kOob, 0).e[0];
  }
  __syncthreads();
  char* cell = p.frag + ((size_t)st * p.xblocks + xb) * kTrioCell;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int f = 2 * wave + u;  // 0 .. 3: row tile f of the first product; 4 .. 7: element tile h, half kb of the second
    float v[8];
    if (f < 4) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = tile[16 * f + i][8 * q + e];
    } else {
      const int h = (f - 4) >> 1, kb = f & 1, x = 8 * (i >> 2) + 4 * h + (i & 3);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = tile[32 * kb + 8 * q + e][x];
    }
    Trio t = split8(v);
    u32x4* dst = reinterpret_cast<u32x4*>(cell + (size_t)f * 3 * kTrioOperand) + lane;
#pragma unroll
    for (int pc = 0; pc < 3; ++pc) dst[pc * 64] = __builtin_bit_cast(u32x4, t.p[pc]);
  }
}

constexpr size_t trio_lds(int ct) { return (size_t)(9 * 1024 * sizeof(float) + 6 * kTrioOperand) * ct; }

// XT: accumulator tiles of 16 elements per wave and column tile (2, 4, 8); CT: column tiles of 16 (1, 2); TEAM: more than one part
template <int XT, int CT, bool TEAM>
__global__ void __launch_bounds__(512) chain_trio_kernel(ChainArgs p) {
  extern __shared__ __align__(16) float smem[];
  constexpr int XW = 16 * XT, NB = XT / 2, COLS = 16 * CT, MAXP = kTrioMaxD / (128 * XT);
  const int NP = TEAM ? p.parts : 1;
  f32x4* Bp = reinterpret_cast<f32x4*>(smem);             // the waves' shares of B: [8][tile CT rt + ct][lane]
  f32x4* Btot = Bp + 8 * 256 * CT;                        // B summed, [tile][lane]
  char* Cs = reinterpret_cast<char*>(Btot + 256 * CT);        // C as operands: [ct][kb][piece][1024 bytes]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, i = lane & 15;
  const int m = p.m, d = p.d, n = p.n;
  const int tiles = (m + COLS - 1) / COLS;
  const int chain_wgs = TEAM ? 8 * NP * ((tiles + 7) / 8) : tiles;
  if ((int)blockIdx.x >= chain_wgs) {  // the side product, on compute units the chain leaves idle
    const int row = ((int)blockIdx.x - chain_wgs) * 8 + wave;
    if (row < p.ds_rows) dsigma_row(p.in, p.ds_z1, p.in_scale, p.ds_out, row, m, p.in_scale_mode);
    return;
  }
  int part = 0, tile = (int)blockIdx.x;
  if constexpr (TEAM) {
    const int drawn = draw_team_ticket(p.xch, trio_words(NP, CT), chain_wgs);
    part = drawn % NP;
    tile = drawn / NP * 8 + (int)(blockIdx.x & 7u);
    if ((unsigned)tile >= (unsigned)tiles) return;
  }
  const int col0 = tile * COLS + i;  // column tile ct: col0 + 16 ct
  const int x_w = (part * 8 + wave) * XW;  // this wave's first element
  auto x_of = [&](int t, int jj) { return x_w + 32 * (t >> 1) + 8 * q + 4 * (t & 1) + jj; };

  // this wave's operands of V: a step's cells are consecutive, this wave's NB cells among them; cells beyond the last
  // element read as zero
  const int xblocks = (d + 31) / 32;
  const size_t step_bytes = (size_t)xblocks * kTrioCell;
  const unsigned lane_off = (unsigned)lane * 16u;
  const int first_cell = x_w / 32;
  auto step_desc = [&](int st) { return make_buffer(reinterpret_cast<const float*>(p.frag + (size_t)st * step_bytes), step_bytes); };
  auto load_triple = [&](BufferDesc desc, int b, int f, Trio& t) {
    const unsigned cell = first_cell + b < xblocks ? (unsigned)(first_cell + b) * (unsigned)kTrioCell : kOob;
#pragma unroll
    for (int pc = 0; pc < 3; ++pc)
      t.p[pc] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(desc, lane_off + cell, (unsigned)(f * 3 + pc) * kTrioOperand, 0));
  };
  // operand g of the second product: rows half g / XT, element tile g % XT
  auto load_second = [&](BufferDesc desc, int g, Trio& t) { load_triple(desc, (g % XT) >> 1, 4 + 2 * (g & 1) + g / XT, t); };

  const int ns = n / 64;
  auto step_of = [&](int s) { return p.transpose ? s : ns - 1 - s; };
  Trio f1[4];
  {
    const BufferDesc d0 = step_desc(step_of(0));
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) load_triple(d0, 0, rt, f1[rt]);
  }

  // the input tile: rows beyond those that exist and columns beyond m read as zero
  f32x4 A[XT][CT];
  {
    const BufferDesc xdesc = make_buffer(p.in, (size_t)p.in_rows * m * sizeof(float));
#pragma unroll
    for (int t = 0; t < XT; ++t) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int x = x_of(t, jj), col = col0 + 16 * ct;
          const unsigned off = col < m && x < p.in_rows ? ((unsigned)x * (unsigned)m + (unsigned)col) * 4u : kOob;
          A[t][ct][jj] = buffer_load<1>(xdesc, off, 0).e[0];
        }
      }
    }
    if (p.in_scale_mode) {
      // all fetches first, then the mode as a compile-time constant: rows that do not exist hold zero in A already;
      // their sigma is replaced by 1 so that the factor stays finite
      const BufferDesc sdesc = make_buffer(p.in_scale, (size_t)p.in_rows * sizeof(float));
      f32x4 sg[XT];
#pragma unroll
      for (int t = 0; t < XT; ++t) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) sg[t][jj] = buffer_load<1>(sdesc, (unsigned)x_of(t, jj) * 4u, 0).e[0];
      }
      auto scale_rows = [&](auto mode) {
#pragma unroll
        for (int t = 0; t < XT; ++t) {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const float f = diag_factor(decltype(mode)::value, x_of(t, jj) < p.in_rows ? sg[t][jj] : 1.f);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) A[t][ct][jj] *= f;
          }
        }
      };
      switch (p.in_scale_mode) {
        case 1: scale_rows(std::integral_constant<int, 1>()); break;
        case 2: scale_rows(std::integral_constant<int, 2>()); break;
        case 3: scale_rows(std::integral_constant<int, 3>()); break;
        default: scale_rows(std::integral_constant<int, 4>()); break;
      }
    }
  }

  BufferDesc hdesc = make_buffer(nullptr, 0);
  unsigned tag0 = 0u;
  bool gave_up = false, same_xcd = false;
  if constexpr (TEAM) {
    hdesc = make_buffer(reinterpret_cast<const float*>(p.xch + (size_t)tile * trio_words(NP, CT)), trio_words(NP, CT) * 4u);
    tag0 = __builtin_amdgcn_raw_buffer_load_b32(hdesc, 0u, 0, 16);
    const unsigned my_xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u;
    const unsigned hs_tag = tag0 + 1u;
    if (tid == 0) {
      const u32x2 w = {my_xcc, hs_tag};
      __builtin_amdgcn_raw_buffer_store_b64(w, hdesc, 32u + (unsigned)part * 8u, 0, 16);
    }
    unsigned peer_xcc = my_xcc;
    const unsigned hs_from = 32u + (unsigned)(lane < NP ? lane : part) * 8u;
    const long long start_limit = kStartPolls * p.wait_limit;
    long long polls = 0;
    for (;;) {
      const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(hdesc, hs_from, 0, 16);
      peer_xcc = w.x;
      if (__all(w.y == hs_tag)) break;
      if (polls++ >= start_limit) { gave_up = true; break; }
      asm volatile("" ::: "memory");
    }
    same_xcd = !gave_up && __all(peer_xcc == my_xcc);
  }

  // A lane's registers (h, jj) of a cell are eight consecutive elements of its column
  auto save_input = [&](int block) {
    const BufferDesc adesc = make_buffer(p.save_in + (size_t)block * m * d, (size_t)m * d * sizeof(float));
#pragma unroll
    for (int t = 0; t < XT; ++t) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int x = x_of(t, 0), col = col0 + 16 * ct;
        BufVec<4> v;
        v.e[0] = A[t][ct][0]; v.e[1] = A[t][ct][1]; v.e[2] = A[t][ct][2]; v.e[3] = A[t][ct][3];
        buffer_store<4>(adesc, col < m && x < d ? ((unsigned)col * (unsigned)d + (unsigned)x) * 4u : kOob, 0, v);
      }
    }
  };

  const int crt = wave & 3, cct = wave >> 2;  // this wave's tile of C (CT = 1: the first four waves)
  const int sub = p.sub;                      // steps per block
  for (int s = 0; s < ns; ++s) {
    const int st = step_of(s), stn = step_of(s + 1 < ns ? s + 1 : s);
    const BufferDesc cur = step_desc(st), nxt = step_desc(stn);
    // this wave's share of B = V_rows A
    {
      f32x4 hi[4][CT], lo[4][CT];
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) hi[rt][ct] = lo[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        Trio a[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          float v[8];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) { v[jj] = A[2 * b][ct][jj]; v[4 + jj] = A[2 * b + 1][ct][jj]; }
          a[ct] = split8(v);
        }
        const Trio* right[4] = {a, a, a, a};
        f32x4* lead[4] = {hi[0], hi[1], hi[2], hi[3]};
        trio_mma<4, CT>(f1, right, lead, lo);
        if (b + 1 < NB) {
#pragma unroll
          for (int rt = 0; rt < 4; ++rt) load_triple(cur, b + 1, rt, f1[rt]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) Bp[wave * 256 * CT + (CT * rt + ct) * 64 + lane] = hi[rt][ct] + lo[rt][ct];
      }
    }
    // row 16 crt + i of op(T), entries 16 g + 4 q .. + 3
    float4 tr[4];
    {
      const float* Ts = (p.transpose ? p.Tt : p.T) + (size_t)st * 4096 + (16 * crt + i) * 64 + 4 * q;
#pragma unroll
      for (int g = 0; g < 4; ++g) tr[g] = *reinterpret_cast<const float4*>(Ts + 16 * g);
    }
    // the first operands of the second product arrive while the sums are formed and handed over
    Trio f2[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) load_second(cur, g, f2[g]);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    {
      // thread t adds 2 CT entries of the eight waves' shares, sends the sums to the other parts and receives theirs
      struct Own { float2 e[CT]; };
      const Own* share = reinterpret_cast<const Own*>(Bp) + tid;
      Own own = share[0];
#pragma unroll
      for (int w = 1; w < 8; ++w) {
        const Own o = share[w * 512];
#pragma unroll
        for (int h = 0; h < CT; ++h) { own.e[h].x += o.e[h].x; own.e[h].y += o.e[h].y; }
      }
      if constexpr (TEAM) {
        const unsigned tag = tag0 + 1u + (unsigned)s, par = (unsigned)s & 1u;
        auto slot = [&](int to, int from, int h) {
          return (unsigned)kTeamHeadBytes + (((((unsigned)to * 2u + par) * (unsigned)NP + (unsigned)from) * CT + h) * 512u + (unsigned)tid) * 16u;
        };
#pragma unroll
        for (int j = 0; j < MAXP; ++j) {
          if (j < NP && j != part) {
#pragma unroll
            for (int h = 0; h < CT; ++h) {
              const u32x4 out = {__float_as_uint(own.e[h].x), tag, __float_as_uint(own.e[h].y), tag};
              if (same_xcd) __builtin_amdgcn_raw_buffer_store_b128(out, hdesc, slot(j, part, h), 0, 0);
              else __builtin_amdgcn_raw_buffer_store_b128(out, hdesc, slot(j, part, h), 0, 16);
            }
          }
        }
        Own got[MAXP];  // part j's sums (zero once a wait has given up)
#pragma unroll
        for (int j = 0; j < MAXP; ++j) {
#pragma unroll
          for (int h = 0; h < CT; ++h) got[j].e[h] = make_float2(0.f, 0.f);
        }
        if (!gave_up) {
          int polls = 0;
          for (;;) {
            bool all_in = true;
#pragma unroll
            for (int j = 0; j < MAXP; ++j) {
              if (j < NP && j != part) {
#pragma unroll
                for (int h = 0; h < CT; ++h) {
                  const u32x4 w = same_xcd ? __builtin_amdgcn_raw_buffer_load_b128(hdesc, slot(part, j, h), 0, 2)
                                           : __builtin_amdgcn_raw_buffer_load_b128(hdesc, slot(part, j, h), 0, 16);
                  const unsigned t0 = w.y, t1 = w.w;
                  got[j].e[h] = make_float2(__uint_as_float(w.x), __uint_as_float(w.z));
                  all_in = all_in && t0 == tag && t1 == tag;
                }
              }
            }
            if (__all(all_in)) break;
            if (polls++ >= p.wait_limit) { gave_up = true; break; }
            asm volatile("" ::: "memory");
          }
        }
        // the parts' sums in the order of the parts: every part gets the same bits
        Own total;
#pragma unroll
        for (int h = 0; h < CT; ++h) total.e[h] = make_float2(0.f, 0.f);
#pragma unroll
        for (int j = 0; j < MAXP; ++j) {
          if (j < NP) {
#pragma unroll
            for (int h = 0; h < CT; ++h) {
              total.e[h].x += j == part ? own.e[h].x : got[j].e[h].x;
              total.e[h].y += j == part ? own.e[h].y : got[j].e[h].y;
            }
          }
        }
        own = total;
      }
      reinterpret_cast<Own*>(Btot)[tid] = own;
    }
    lds_barrier();
    if (CT == 2 || wave < 4) {
      // tile (crt, cct) of C = op(T) B: instruction (g, jj) takes inner index 16 g + 4 q + jj of lane (q, i)
      f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 b = Btot[(CT * g + cct) * 64 + lane];
        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(tr[g].x, b[0], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(tr[g].y, b[1], c1, 0, 0, 0);
        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(tr[g].z, b[2], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(tr[g].w, b[3], c1, 0, 0, 0);
      }
      const f32x4 c = c0 + c1;
      // lane (q, i) has rows 16 crt + 4 q + jj of column i: half of the eight inner indices that lane
      // 16 (2 (crt % 2) + q / 2) + i supplies to the second product's half kb = crt / 2
      unsigned w0[3], w1[3];
      split2(-c[0], -c[1], w0[0], w0[1], w0[2]);
      split2(-c[2], -c[3], w1[0], w1[1], w1[2]);
      char* dst = Cs + (cct * 2 + (crt >> 1)) * 3 * kTrioOperand + ((2 * (crt & 1) + (q >> 1)) * 16 + i) * 16 + 8 * (q & 1);
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) *reinterpret_cast<u32x2*>(dst + pc * kTrioOperand) = u32x2{w0[pc], w1[pc]};
      const int ccol = col0 + 16 * cct;
      if (p.save_c && part == 0 && ccol < m)
        *reinterpret_cast<float4*>(p.save_c + (size_t)ccol * n + (size_t)st * 64 + 16 * crt + 4 * q) = make_float4(c[0], c[1], c[2], c[3]);
    }
    // the block's input is saved here and not at the step's start: the waits of the hand-over would wait for these stores
    if (p.save_in && st % sub == (p.transpose ? 0 : sub - 1)) save_input(st / sub);
    lds_barrier();
    // A -= V_rows^T C, four operands at a time, the first half of the rows before the other
    {
      Trio c[2][CT];
      auto load_c = [&](int kb) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
          for (int pc = 0; pc < 3; ++pc)
            c[kb][ct].p[pc] = *reinterpret_cast<const bf16x8*>(Cs + ((ct * 2 + kb) * 3 + pc) * kTrioOperand + lane * 16);
        }
      };
      if constexpr (XT == 2) {
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) load_triple(nxt, 0, rt, f1[rt]);
      }
#pragma unroll
      for (int g = 0; g < 2 * XT; g += 4) {
        if (g % XT == 0) load_c(g / XT);
        if (XT == 2) load_c(1);
        f32x4 lo[4][CT];
        const Trio* right[4];
        f32x4* lead[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          right[r] = c[(g + r) / XT];
          lead[r] = A[(g + r) % XT];
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) lo[r][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        trio_mma<4, CT>(f2, right, lead, lo);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (g + 4 < 2 * XT) load_second(cur, g + 4 + r, f2[r]);
          else if (XT > 2) load_triple(nxt, 0, r, f1[r]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) A[(g + r) % XT][ct] += lo[r][ct];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if constexpr (TEAM) {
    // the next launch on this workspace counts on from here
    if (part == 0 && tid == 0) __builtin_amdgcn_raw_buffer_store_b32(tag0 + (unsigned)ns, hdesc, 0u, 0, 16);
    if (gave_up && lane == 0) __hip_atomic_store(&g_wait_gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const BufferDesc odesc = make_buffer(p.out, (size_t)p.out_rows * m * sizeof(float));
#pragma unroll
  for (int t = 0; t < XT; ++t) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int x = x_of(t, jj), col = col0 + 16 * ct;
        BufVec<1> v;
        v.e[0] = A[t][ct][jj];
        buffer_store<1>(odesc, col < m && x < p.out_rows ? ((unsigned)x * (unsigned)m + (unsigned)col) * 4u : kOob, 0, v);
      }
    }
  }
}

// No hand-off area: the call may overlap with others on its workspace.
static TrioPlan chain_trio_plan(const ChainArgs& a) {
  if (!a.frag) return TrioPlan{0, 0, 0};
  return a.xch ? trio_plan(a.d, a.n, a.m) : trio_solo_plan(a.d, a.n, a.m);
}
static bool chain_uses_trio(const ChainArgs& a) { return chain_trio_plan(a).parts > 0; }

static int launch_chain_trio(const ChainArgs& args, hipStream_t stream) {
  ChainArgs a = args;
  const TrioPlan plan = chain_trio_plan(a);
  if (plan.parts == 0 || a.k % 64 != 0 || a.n % 64 != 0 || (plan.parts > 1 && !a.xch)) return FASTH_EINVAL;
  a.parts = plan.parts;
  a.sub = a.k / 64;
  const int side = a.ds_out ? (a.ds_rows + 7) / 8 : 0;
  const int tiles = (a.m + 16 * plan.ct - 1) / (16 * plan.ct);
  const dim3 grid((plan.parts > 1 ? 8 * plan.parts * ((tiles + 7) / 8) : tiles) + side), block(512);
#define FASTH_LAUNCH_TRIO(XT_, CT_, TEAM_)                                                            \
  do {                                                                                                 \
    int rc_ = allow_lds(chain_trio_kernel<XT_, CT_, TEAM_>, trio_lds(CT_));                            \
    if (rc_ != FASTH_OK) return rc_;                                                                   \
    static const std::string name_ = variant_name("chain_trio_kernel", {XT_, CT_, TEAM_});             \
    prof::Scope ps_(FASTH_KERNEL_CHAIN, stream, name_.c_str());                                        \
    hipLaunchKernelGGL((chain_trio_kernel<XT_, CT_, TEAM_>), grid, block, trio_lds(CT_), stream, a);   \
  } while (0)
  const bool team = plan.parts > 1;
  if (plan.xt == 2 && plan.ct == 1) FASTH_LAUNCH_TRIO(2, 1, false);
  else if (plan.xt == 2) FASTH_LAUNCH_TRIO(2, 2, false);
  else if (plan.xt == 4 && plan.ct == 1 && !team) FASTH_LAUNCH_TRIO(4, 1, false);
  else if (plan.xt == 4 && plan.ct == 1) FASTH_LAUNCH_TRIO(4, 1, true);
  else if (plan.xt == 4 && !team) FASTH_LAUNCH_TRIO(4, 2, false);
  else if (plan.xt == 4) FASTH_LAUNCH_TRIO(4, 2, true);
  else if (plan.ct == 1) FASTH_LAUNCH_TRIO(8, 1, false);
  else if (!team) FASTH_LAUNCH_TRIO(8, 2, false);
  else FASTH_LAUNCH_TRIO(8, 2, true);
#undef FASTH_LAUNCH_TRIO
  FASTH_HIP(hipGetLastError());
  return FASTH_OK;
}

}  // namespace fasth
