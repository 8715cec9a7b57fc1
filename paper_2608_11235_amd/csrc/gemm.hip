// bf16 MFMA GEMM for gfx950: C[M, N] = A[M, K] . W[N, K]^T with fp32 accumulation.
//
// A workgroup of WAVES_M x WAVES_N wavefronts owns a BM x BN tile; each wavefront owns
// TM x TN blocks of 16 x 16 computed with v_mfma_f32_16x16x32_bf16.  The 16 x 16 shape is
// chosen over 32 x 32 x 16 for power: large products run into the card's power limit, and a
// register-only loop on random data sustains 1.99 PFLOP/s with it against 1.79.
//
// Operands come in K panels of 32, so that every 1 KB load reads 1 KB of contiguous memory:
//   A  [K / 32][M][32]: 16 rows of one panel are 1 KB
//   W  (W_BLOCKS) 64 x 32 blocks, row-major inside, block (n / 64, k / 32) at
//      ((n / 64) * K / 32 + k / 32) * 4 KB, N % 64 == 0; or (W_LM_HEAD) the LM head's
//      layout (lm_head.hip), 1 KB blocks of 16 rows x 32 k in the MFMA operand's lane order,
//      zero rows up to N's next multiple of 32.  These blocks go to LDS and come back as they
//      are: a load that gathers their 16-byte chunks into 64-byte rows touches four times the
//      cache lines and runs at 38 GB/s a CU out of L2, a linear one at 131.
// What bounds the loop is the rate of cache lines that a CU's loads touch: with row-major
// operands (64 bytes of each of 16 rows, twice the lines) the same loop runs 18 % slower at
// 4096 x 37888 x 3584, and 25 % slower at 256 x 128 tiles.
//
// Pipeline: a ring of ST stages of one 32-wide K slice in LDS, filled by buffer loads that
// write LDS directly (no staging registers, no LDS store instructions).  Section kt waits for
// this wavefront's loads of slice kt + 1, passes one barrier, and then issues the MFMAs of
// slice kt (fragments already in registers) with everything else spread between them: the
// fragment reads of slice kt + 1 and the loads of slice kt + ST - 1, one per few MFMAs (loads
// issued in a burst fill the address unit's queue and stall the MFMAs behind them).  An A
// fragment is overwritten by the next slice's as soon as its row of MFMAs is issued; only the
// B fragments have two register sets.  The loads of section kt go to the stage of slice
// kt - 1, whose fragments every wavefront had in registers before this barrier, so the
// barrier drains nothing but the loads it needs.
// The 16-byte chunks of a 64-byte LDS row are XOR-permuted (on the global side of the load,
// which can gather; the LDS side is linear): a 16-byte LDS read serves 16 lanes a cycle,
// lanes {0-3, 12-15, 20-27} together, and the permutation puts their chunks on 16 distinct
// 16-byte slots of the 256-byte bank window (counted conflicts: 0).
//
// Measured (back-to-back launches, weights from HBM, same box, against the register-staged
// 32 x 32 x 16 loop with row-major A that this one replaced): gate/up + SwiGLU at
// 4096 x 37888 x 3584 955 -> 789 us (1.41 PFLOP/s), 1280 x 24576 x 4096 229 -> 184 us
// (1.40 PFLOP/s), 512 x 24576 x 4096 92.4 -> 83 us (1.24 PFLOP/s).
//
// Split-K (for outputs with too few tiles to fill the chip): split s of a tile
// accumulates K-slices [s*nk, (s+1)*nk) and stores its fp32 partial tile (EPI_PART_F32);
// a row-wise kernel downstream adds the partials in split order, so results do not depend
// on scheduling, and applies what the output needs next (residual add + RMSNorm, or bias +
// RoPE + head layout for q/k/v).  Every tile config sums K in the same order, so the split
// count alone decides an output's bits.
//
// The MFMA takes W as its first operand, so a lane holds one row of C and 4 consecutive
// columns: epilogues store 8 or 16 bytes per lane straight from the accumulators, RoPE pairs
// and gate/up pairs meet in one lane, and a row's statistics need two lane exchanges.
// Epilogues:  EPI_BF16    C = bf16((acc + bias[n]) * scale), row-major
//             EPI_ADD_F32 C(fp32) += acc            (residual stream update)
//             EPI_PART_F32  split s stores acc to its own fp32 slab of C
//             EPI_SWIGLU  weights interleave gate/up rows in groups of 16:
//                         C = bf16(silu(g) * u), stored as K panels [ffn / 32][M][32].
//             EPI_QKV_ROPE  bias, rotate-half RoPE on q and k, head-major q/k and
//                         transposed v written straight from the accumulators.
//             EPI_TOP1    no C: per row and wavefront column range, (max, first arg max,
//                         sum of exp) of the bf16 logits EPI_BF16 would store (Eq. 1).
// Requirements: K % (64 * splits) == 0; M, N arbitrary (tails clamped on load, masked
// on store).
#include <hip/hip_ext.h>
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"

namespace cora {

constexpr int BK = 32;
constexpr int GROUP_M = 8;  // M tiles walked before the next N tile (see tile_of)

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// 16 bytes per lane from buffer offset voff + soff straight into LDS: lane l's bytes land at
// lds_off + 16 l.  Inline asm, because the compiler would wait for every such load before
// the next LDS read; it has no register output.
__device__ __forceinline__ void load_lds(uint32_t lds_off, int voff, u32x4_t rs, int soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_off),
               "v"(voff), "s"(rs), "s"(soff)
               : "memory", "m0");
}

__device__ __forceinline__ u32x4_t buffer_rsrc(const void* p, int64_t bytes) {
  const uint64_t a = (uint64_t)p;
  return u32x4_t{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu,
                 (uint32_t)(bytes > 0xffffffffLL ? 0xffffffffLL : bytes), 0x00020000u};
}

// Tile of logical index t: N tiles in order, all M tiles (at most GROUP_M at a time) of one
// before the next.  xcd_remap hands each XCD a contiguous run of that order, so the tiles an
// XCD runs at once cover about as many M as N tiles and share both operands in its L2
// (at 16 M tiles, 4096 x 37888 x 3584: 970 -> 949 us).
__device__ __forceinline__ void tile_of(int t, int num_m, int n_tiles, int& tm, int& tn) {
  if (num_m <= GROUP_M) {
    tm = t % num_m;
    tn = t / num_m;
    return;
  }
  const int per = GROUP_M * (n_tiles / num_m), grp = t / per, first = grp * GROUP_M;
  const int gm = min(GROUP_M, num_m - first), r = t - grp * per;
  tm = first + r % gm;
  tn = r / gm;
}

template <int WAVES_M, int WAVES_N, int TM, int TN, int ST, int OCC, int EPI>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, OCC) void k_gemm(GemmArgs g) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WR = TM * 16, WC = TN * 16;  // wavefront tile
  constexpr int BM = WAVES_M * WR, BN = WAVES_N * WC;
  constexpr int GA = BM / 16, GB = BN / 16;  // 1 KB loads (16 rows of 64 bytes) per slice
  // loads per wavefront and slice; where they do not divide evenly some load twice the same
  // 1 KB to the same place, so that every wavefront counts alike
  constexpr int LA = (GA + NW - 1) / NW, LB = (GB + NW - 1) / NW, LPW = LA + LB;
  constexpr int ROWB = BK * 2, STAGE = (BM + BN) * ROWB;
  static_assert(ST % 2 == 1 && ST >= 3 && ST <= 9, "the tail pairs sections: an odd number of stages");
  static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "SwiGLU epilogue pairs 16-column blocks");
  // dynamic: a static array of more than half the CU's LDS would tell the compiler that one
  // wavefront per SIMD is all there is, and it then spreads accumulators over AGPRs and moves
  // them back and forth in the loop (128 x 192 as 4 wavefronts: 63 us, without moves 53 us)
  extern __shared__ __attribute__((aligned(1024))) uint16_t lds[];
  constexpr size_t LDS_BYTES = (size_t)ST * STAGE;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  // logical order: split-major, then tile_of.  An XCD's workgroups share one K range (its L2
  // holds only that range of A).
  const int li = xcd_remap(blockIdx.x, gridDim.x);
  const int n_tiles = gridDim.x / g.splits;
  const int split = li / n_tiles;
  int tile_m, tile_n;
  tile_of(li - split * n_tiles, (g.M + BM - 1) / BM, n_tiles, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nk = g.K / BK / g.splits;  // even: K % (64 * splits) == 0
  const int kt0 = split * nk;

  // W is addressed from this tile's first row group (64-bit base, 32-bit offsets inside);
  // rows past M or N are clamped to the last one, so no load leaves the operands
  const bool lm = g.w_layout == W_LM_HEAD;
  const int n_rows = lm ? (g.N + 31) / 32 * 32 : g.N;
  const int64_t w_base = (int64_t)(n0 >> 6) * 64 * g.K * 2;
  const u32x4_t a_rs = buffer_rsrc(g.A, (int64_t)g.M * g.K * 2);
  const u32x4_t b_rs = buffer_rsrc(reinterpret_cast<const char*>(g.W) + w_base, (int64_t)n_rows * g.K * 2 - w_base);
  const int lr = lane >> 2, ls = lane & 3;  // this lane's row and 16-byte slot of a load
  auto swz = [](int r) {                    // 0, 2, 3, 1 for r / 4 = 0 .. 3
    const int k = (r >> 2) & 3;
    return (k >> 1) | (((k ^ (k >> 1)) & 1) << 1);
  };
  int voa[LA], vob[LB];
#pragma unroll
  for (int t = 0; t < LA; ++t) {
    const int r = (t * NW + wave) % GA * 16 + lr;
    voa[t] = min(m0 + r, g.M - 1) * 64 + (ls ^ swz(lr)) * 16;
  }
#pragma unroll
  for (int t = 0; t < LB; ++t) {
    const int nb = n0 + (t * NW + wave) % GB * 16;  // n_rows is a multiple of 16
    const int n = min(nb + (lm ? 0 : lr), n_rows - (lm ? 16 : 1)) - (n0 & ~63), c = ls ^ swz(lr);
    vob[t] = lm ? (n >> 5) * 64 * g.K + ((n >> 4) & 1) * 2048 + lane * 16
                : (n >> 6) * 128 * g.K + (n & 63) * 64 + c * 16;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  // load t of this wavefront's share of slice kt, into the stage at byte offset st
  auto issue = [&](int kt, uint32_t st, int t) {
    const int k = kt0 + kt;
    if (t < LA)
      load_lds(lds0 + st + (GA % NW ? (t * NW + wave) % GA : t * NW + wave) * 1024, voa[t < LA ? t : 0], a_rs,
               k * g.M * 64);
    else
      load_lds(lds0 + st + BM * ROWB + (GB % NW ? ((t - LA) * NW + wave) % GB : (t - LA) * NW + wave) * 1024,
               vob[t >= LA ? t - LA : 0], b_rs, lm ? (k >> 1) * 4096 + (k & 1) * 1024 : k * 4096);
  };

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // fragments: lane holds row (lane % 16), k chunk (lane / 16) * 8
  const int fr = lane & 15, fc = lane >> 4;
  const int slot = (fc ^ swz(fr)) * 16;
  const int ka = (wm * WR + fr) * ROWB + slot, kb = BM * ROWB + wn * WC * ROWB + (lm ? lane * 16 : fr * ROWB + slot);
  const char* lp = reinterpret_cast<const char*>(lds);
  auto frag = [&](int off) { return as_bf16x8(*reinterpret_cast<const u32x4_t*>(lp + off)); };
  constexpr int NM = TM * TN;
  bf16x8_t fa[TM], fb0[TN], fb1[TN];
  auto section = [&](auto load_c, auto read_c, int st_next, int kt_load, uint32_t st_load,
                     const bf16x8_t(&fb)[TN], bf16x8_t(&nb)[TN]) {
    constexpr bool LOAD = decltype(load_c)::value, READ = decltype(read_c)::value;
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      const int i = q / TN, j = q % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
      if constexpr (READ) {
        if (i == 0) nb[j] = frag(st_next + kb + j * 16 * ROWB);
        if (j == TN - 1) fa[i] = frag(st_next + ka + i * 16 * ROWB);
      }
      if constexpr (LOAD) {
#pragma unroll
        for (int t = 0; t < LPW; ++t)
          if (t * NM / LPW + (NM > LPW ? 1 : 0) == q) issue(kt_load, st_load, t);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // prologue: slices 0 .. ST - 2 in flight (past the last one: it again, never read)
#pragma unroll
  for (int u = 0; u < ST - 1; ++u)
#pragma unroll
    for (int t = 0; t < LPW; ++t) issue(u < nk ? u : nk - 1, u * STAGE, t);
  wait_vm<(ST - 2) * LPW>();
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TN; ++j) fb0[j] = frag(kb + j * 16 * ROWB);
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[i] = frag(ka + i * 16 * ROWB);
  __builtin_amdgcn_sched_barrier(0);
  int rd = 0, wr = (ST - 1) * STAGE;  // stage of slice kt, and of slices kt - 1 and kt + ST - 1
  // section KT; NEWER: slices after KT + 1 whose loads may still be in flight at the barrier
#define SECTION(LOAD, READ, NEWER, KT, FB, NB)                                              \
  do {                                                                                      \
    const int nx = rd + STAGE == ST * STAGE ? 0 : rd + STAGE;                               \
    if constexpr (READ) {                                                                   \
      wait_vm<((NEWER) > 0 ? (NEWER) : 0) * LPW>();                                         \
      asm volatile("s_barrier" ::: "memory");                                               \
    }                                                                                       \
    section(std::bool_constant<(LOAD)>{}, std::bool_constant<(READ)>{}, nx, (KT) + ST - 1, (uint32_t)wr, FB, NB); \
    wr = rd;                                                                                \
    rd = nx;                                                                                \
  } while (0)
  // nk and ST - 1 are even, so the sections that load come in pairs too
  for (int kt = 0; kt + ST - 1 < nk; kt += 2) {
    SECTION(true, true, ST - 3, kt, fb0, fb1);
    SECTION(true, true, ST - 3, kt + 1, fb1, fb0);
  }
  // the last ST - 1 slices (or all nk of them): nothing left to load
#define TAIL(P)                                     \
  if constexpr (2 * (P) <= ST - 1) {                \
    if (nk >= 2 * (P)) {                            \
      SECTION(false, true, 2 * (P)-2, 0, fb0, fb1); \
      SECTION(false, (P) > 1, 2 * (P)-3, 0, fb1, fb0); \
    }                                               \
  }
  TAIL(4) TAIL(3) TAIL(2) TAIL(1)
#undef TAIL
#undef SECTION
  wait_vm<0>();

  // epilogue: acc[i][j][e] is C[row, col] with
  //   row = m0 + wm WR + 16 i + lane % 16,  col = n0 + wn WC + 16 j + 4 (lane / 16) + e
  const int row0 = m0 + wm * WR + fr, col0 = n0 + wn * WC + 4 * fc;
  if constexpr (EPI == EPI_SWIGLU) {
    // lanes of 16 rows x 16 outputs write 32 bytes of each of 16 consecutive 64-byte rows
    uint16_t* C = reinterpret_cast<uint16_t*>(g.C);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = row0 + i * 16;
      if (row >= g.M) continue;
#pragma unroll
      for (int t = 0; t < TN / 2; ++t) {
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gt = acc[i][2 * t][e], up = acc[i][2 * t + 1][e];
          const float sg = gt / (1.0f + __expf(-gt));
          o[e] = sg * up;
        }
        const int col = (n0 + wn * WC) / 2 + t * 16 + 4 * fc;
        if (col < g.N / 2)
          *reinterpret_cast<u32x2_t*>(C + ((int64_t)(col >> 5) * g.M + row) * 32 + (col & 31)) =
              u32x2_t{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
      }
    }
  } else if constexpr (EPI == EPI_QKV_ROPE) {
    // q/k columns are pair-interleaved within a head, so the rotate-half partner of an even
    // column is the next one, in the same lane.  A 16-column block lies in one head of one
    // section (q, k or v): section widths are multiples of 64.  v leaves transposed: the
    // block passes through this wavefront's part of LDS (free once every wavefront is past
    // its last slice) and is written as runs of 8 positions.
    // The cos/sin loads of a block row are issued before the stores of the one before it: a
    // load queued behind a store waits for that store too (loaded per block column, the
    // epilogue was 20 to 30 us of 4096 x 4608 x 3584 and of 1280 x 12288 x 4096).
    const QkvOut& o = g.qkv;
    const int hd = o.head_dim, hsh = 31 - __builtin_clz(hd);  // 64 or 128
    const int hq = o.n_heads * hd, hqk = hq + o.n_kv_heads * hd;
    constexpr int SPV = WR + 16;  // staged pitch, bf16: a shift of up to 7, and up to 7 between two sequences
    static_assert(LDS_BYTES >= (size_t)NW * 16 * SPV * 2, "stage");
    const int c_wave = n0 + wn * WC;  // wave-uniform, like everything derived from it
    if (g.bias) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (c_wave + j * 16 >= g.N) continue;
        const f32x4_t bias = *reinterpret_cast<const f32x4_t*>(g.bias + c_wave + j * 16 + 4 * fc);
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i][j] += bias;
      }
    }
    if (c_wave < hqk) {
      // batch row and position of this lane's rows: divided out once, not per block column
      int rp[TM];
      int64_t oq[TM], ok[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int m = min(row0 + i * 16, g.M - 1), rb = m / o.L;
        rp[i] = m - rb * o.L;
        oq[i] = ((int64_t)rb * o.n_heads * o.Ls + rp[i]) * hd + 4 * fc;
        ok[i] = ((int64_t)rb * o.n_kv_heads * o.Ls + rp[i]) * hd + 4 * fc;
      }
      f32x4_t tab[2][TN];  // (cos, sin) of this lane's two pairs
      auto load_tab = [&](int i, f32x4_t(&t)[TN]) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
          t[j] = *reinterpret_cast<const f32x4_t*>(o.cs_t + rp[i] * hd + ((c_wave + j * 16) & (hd - 1)) + 4 * fc);
      };
      load_tab(0, tab[0]);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM) load_tab(i + 1, tab[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        const bool in = row0 + i * 16 < g.M;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int c0 = c_wave + j * 16;
          if (c0 >= hqk || !in) continue;
          const int cc0 = c0 < hq ? c0 : c0 - hq;
          uint16_t* base = (c0 < hq ? o.q : o.k) + (int64_t)(cc0 >> hsh) * o.Ls * hd + (cc0 & (hd - 1));
          const f32x4_t x = acc[i][j], t = tab[i & 1][j];
          *reinterpret_cast<u32x2_t*>(base + (c0 < hq ? oq[i] : ok[i])) =
              u32x2_t{pack_bf16x2(x[0] * t[0] - x[1] * t[1], x[1] * t[0] + x[0] * t[1]),
                      pack_bf16x2(x[2] * t[2] - x[3] * t[3], x[3] * t[2] + x[2] * t[3])};
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    if (c_wave + WC > hqk) {
      // A block of 16 dimensions passes through this wavefront's part of LDS and leaves as runs
      // of 8 positions that start at multiples of 8, whatever position the wavefront's first row
      // has: row r is staged at index s1 + r, those of the next sequence from s2 on, both
      // multiples of 8 away from their position.  (Runs of 8 rows instead, which an odd length
      // leaves unaligned, went element by element: three
      // sequences of 333, 999 x 4608 x 3584, 56.8 us against 51.3.)
      uint16_t* scr = lds + wave * 16 * SPV;
      const int mw = m0 + wm * WR, b0 = mw / o.L, p0 = mw - b0 * o.L;
      const int len = min(WR, g.M - mw), len1 = min(len, o.L - p0), len2 = len - len1;
      const int s1 = p0 & 7, s2 = (s1 + len1 + 7) & ~7;
      const int n1 = s2 >> 3, nr = n1 + ((len2 + 7) >> 3);  // runs of the first sequence, of both
      const bool two = len2 <= o.L;  // else a third sequence begins here: rows staged as they come
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int c0 = c_wave + j * 16;
        if (c0 < hqk || c0 >= g.N || len <= 0) continue;
        const int head = (c0 - hqk) >> hsh, d0 = (c0 - hqk) & (hd - 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int r = i * 16 + fr, at = two ? (r < len1 ? s1 + r : s2 + r - len1) : r;
#pragma unroll
          for (int e = 0; e < 4; ++e) scr[(4 * fc + e) * SPV + at] = (uint16_t)f32_to_bf16_bits(acc[i][j][e]);
        }
        wave_lds_sync();
        const uint16_t* src = scr + (lane >> 2) * SPV;
        const int64_t dim = (int64_t)head * hd + d0 + (lane >> 2), seq = (int64_t)o.n_kv_heads * hd;
        if (two) {
          for (int run = lane & 3; run < nr; run += 4) {
            const bool first = run < n1;
            const int pp = first ? (p0 & ~7) + 8 * run : 8 * (run - n1);
            const int lo = first ? p0 : 0, hi = first ? p0 + len1 : len2;
            uint16_t* dst = o.vt + ((b0 + (first ? 0 : 1)) * seq + dim) * o.Ls + pp;
            if (pp >= lo && pp + 8 <= hi) {
              *reinterpret_cast<u32x4_t*>(dst) = *reinterpret_cast<const u32x4_t*>(src + 8 * run);
            } else {
              for (int t = max(lo - pp, 0); t < 8 && pp + t < hi; ++t) dst[t] = src[8 * run + t];
            }
          }
        } else {
          for (int r = lane & 3; r < len; r += 4) {
            const int m = mw + r, bb = m / o.L;
            o.vt[(bb * seq + dim) * o.Ls + m - bb * o.L] = src[r];
          }
        }
        wave_lds_sync();  // the next block is staged in the same place
      }
    }
  } else if constexpr (EPI == EPI_TOP1) {
    // Row statistics of Eq. (1) over this wavefront's TN x 16 columns, of the rounded logits
    // EPI_BF16 would write: a lane reduces its TN x 4 columns, then the 4 lanes of a row
    // agree on the max (lowest column among equals) and add their sums.
    const int part = tile_n * WAVES_N + wn;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float v[TN * 4];
      float m = -INFINITY;
      int arg = INT_MAX;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = col0 + j * 16 + e;
          float x = bf16_bits_to_f32(f32_to_bf16_bits(acc[i][j][e] * g.scale));
          if (c >= g.N || c == g.mask_id) x = -INFINITY;
          v[4 * j + e] = x;
          if (x > m) { m = x; arg = c; }
        }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float om = __shfl_xor(m, o, 64);
        const int oa = __shfl_xor(arg, o, 64);
        arg = om > m ? oa : (m > om ? arg : min(arg, oa));
        m = fmaxf(m, om);
      }
      float s = 0.f;
      if (m != -INFINITY) {
        const ExpBelow ex(m);
#pragma unroll
        for (int k = 0; k < TN * 4; ++k) s += ex(v[k]);
        s = ex.sum(s);
      }
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      const int row = row0 + i * 16;
      if (fc == 0 && row < g.M) {
        const int64_t o = (int64_t)row * g.n_parts + part;
        g.part_m[o] = m;
        g.part_s[o] = s;
        g.part_arg[o] = arg;
      }
    }
  } else if constexpr (EPI == EPI_ADD_F32 || EPI == EPI_PART_F32) {
    // N % 4 == 0 (checked at launch): a lane's 4 columns are in or out together
    float* C = reinterpret_cast<float*>(g.C) +
               (EPI == EPI_PART_F32 ? (int64_t)split * g.M * g.ldc : (int64_t)0);
    if constexpr (EPI == EPI_ADD_F32) {
      // the next block row's loads go out before this one's stores (see EPI_QKV_ROPE)
      f32x4_t h[2][TN];
      auto load_h = [&](int i, f32x4_t(&v)[TN]) {
        if (row0 + i * 16 >= g.M) return;
#pragma unroll
        for (int j = 0; j < TN; ++j)
          if (col0 + j * 16 < g.N) v[j] = *reinterpret_cast<const f32x4_t*>(C + (int64_t)(row0 + i * 16) * g.ldc + col0 + j * 16);
      };
      load_h(0, h[0]);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM) load_h(i + 1, h[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (row0 + i * 16 < g.M) {
          float* dst = C + (int64_t)(row0 + i * 16) * g.ldc + col0;
#pragma unroll
          for (int j = 0; j < TN; ++j)
            if (col0 + j * 16 < g.N) *reinterpret_cast<f32x4_t*>(dst + j * 16) = h[i & 1][j] + acc[i][j];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = row0 + i * 16;
        if (row >= g.M) continue;
        float* dst = C + (int64_t)row * g.ldc + col0;
#pragma unroll
        for (int j = 0; j < TN; ++j)
          if (col0 + j * 16 < g.N) *reinterpret_cast<f32x4_t*>(dst + j * 16) = acc[i][j];
      }
    }
  } else {
    uint16_t* C = reinterpret_cast<uint16_t*>(g.C);
    const bool vec = (g.ldc & 3) == 0 && ((uintptr_t)C & 7) == 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = row0 + i * 16;
      if (row >= g.M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = col0 + j * 16;
        uint16_t* dst = C + (int64_t)row * g.ldc + col;
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x[e] = (acc[i][j][e] + (g.bias && col + e < g.N ? g.bias[col + e] : 0.f)) * g.scale;
        if (vec && col + 3 < g.N) {
          *reinterpret_cast<u32x2_t*>(dst) = u32x2_t{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < g.N) dst[e] = (uint16_t)f32_to_bf16_bits(x[e]);
        }
      }
    }
  }
}

// ---- tile configurations ---------------------------------------------------------------
// X(cfg, WAVES_M, WAVES_N, TM, TN, stages, minimum waves per SIMD, workgroups per CU (LDS),
//   slice_us, cu_us, tile_us): the last three are gemm_us's constants per 32-wide slice of a
//   lone tile, per slice and resident tile on a busy chip, and per tile.
// 0 to 4 and 9 serve the wide products (a larger tile moves fewer bytes per FLOP from L2 into
// LDS); 5 to 8 products whose larger tiles would leave CUs idle: few rows, or few rows and
// columns.  1, 3 and 9 hold their tile in wavefronts of 64 or 96 rows: the same tiles in
// wavefronts of 32 rows read a third more bytes from LDS per MFMA (cold weights,
// 512 x 24576 x 4096 at 256 x 192 91.6 -> 87.4 us, 512 x 12288 x 4096 at 128 x 192 57.8 ->
// 53.2 us; 999 x 4608 x 3584 at 192 x 128 38.5 us, the others 42 and more).
#define GEMM_CFGS(X)                              \
  X(0, 4, 2, 4, 8, 5, 1, 1, 0.508, 0.626, 4.05)   \
  X(1, 4, 2, 4, 6, 5, 2, 1, 0.439, 0.506, 3.42)   \
  X(2, 4, 2, 4, 4, 5, 1, 1, 0.319, 0.363, 2.56)   \
  X(3, 2, 2, 4, 6, 5, 2, 1, 0.286, 0.300, 2.55)   \
  X(4, 2, 2, 4, 4, 5, 2, 2, 0.230, 0.217, 1.32)   \
  X(5, 2, 2, 4, 2, 5, 2, 2, 0.187, 0.155, 0.41)   \
  X(6, 2, 2, 2, 4, 5, 2, 2, 0.192, 0.161, 0.40)   \
  X(7, 2, 2, 2, 2, 7, 2, 2, 0.113, 0.100, 0.52)   \
  X(8, 2, 2, 1, 2, 9, 2, 2, 0.088, 0.078, 0.68)   \
  X(9, 2, 2, 6, 4, 5, 2, 1, 0.250, 0.283, 2.39)
struct CfgShape {
  int bm, bn, waves_n, per_cu;
  double slice_us, cu_us, tile_us;
};
static CfgShape cfg_shape(int cfg) {
  switch (cfg) {
#define X(C, WM, WN, TM, TN, ST, OCC, PER_CU, SL, CU, TILE) \
  case C: return {WM * TM * 16, WN * TN * 16, WN, PER_CU, SL, CU, TILE};
    GEMM_CFGS(X)
#undef X
  }
  return {};
}

int gemm_num_cfgs() { return 10; }

// wavefront columns per tile and their width (TN x 16) of each config
int gemm_top1_parts(const GemmPlan& p, int N) {
  const CfgShape sh = cfg_shape(p.cfg);
  return (N + sh.bn - 1) / sh.bn * sh.waves_n;
}

// Estimated time of one launch in microseconds: rounds of resident tiles, each the larger of
// a tile's own latency per 32-wide slice and the chip's throughput with that many tiles
// resident (a few busy CUs run faster than all: power), plus prologue and epilogue; the time
// to stream the weights, of which a little over half overlaps with it; plus the traffic of
// split-K partials and, in the kernel downstream, of folding them (fold_us more where that
// kernel is an extra one).  The constants are fitted to a sweep of all configs and split
// counts over 47 shapes (64 to 4096 rows, 768 to 152064 columns, K 256 to 18944); the config
// it picks is on average 0.3 %, at most 7 % slower than the fastest measured one of these.
// Where 0.363 against 0.357 for the 256 x 128 tiles decides (55 of 19299 random shapes of those
// ranges, none of them fitted), its picks measured 0.3 % faster in the mean: from 6.7 % faster
// (1686 x 22016 x 2432; 2 to 4 % at K above 7000) to 10 % slower (2084 x 29056 x 1600).
static double gemm_us(int M, int N, int K, int num_cus, int cfg, int splits, double fold_us) {
  const CfgShape sh = cfg_shape(cfg);
  const double nk = (double)K / BK / splits;
  const int64_t grid = (int64_t)((M + sh.bm - 1) / sh.bm) * ((N + sh.bn - 1) / sh.bn) * splits;
  const int64_t slots = (int64_t)num_cus * sh.per_cu;
  auto round_us = [&](int64_t n) {
    const double per_cu = (double)std::min<int64_t>(sh.per_cu, (n + num_cus - 1) / num_cus);
    const double busy = std::min(1.0, (double)n / num_cus);
    return nk * std::max(sh.slice_us, per_cu * sh.cu_us * (0.54 + 0.46 * busy)) + sh.tile_us;
  };
  double us = 1.4 + (double)(grid / slots) * round_us(slots);
  if (grid % slots) us += round_us(grid % slots);
  const double stream_us = 1.4 + (double)N * K * 2 / 7.3e6;  // the weights at 7.3 TB/s
  us = std::max(us, stream_us) + 0.44 * std::min(us, stream_us);
  if (splits > 1) us += 0.37 * (double)splits * M * N * 4.0 / (1 << 20) + fold_us;
  return us;
}

GemmPlan gemm_plan_cfg(int M, int N, int K, int cfg, int splits) {
  GemmPlan p{};
  p.cfg = cfg;
  const CfgShape sh = cfg_shape(cfg);
  p.tiles = ((M + sh.bm - 1) / sh.bm) * ((N + sh.bn - 1) / sh.bn);
  p.splits = splits;
  p.ws_floats = splits > 1 ? (size_t)splits * M * N : 0;
  return p;
}

GemmPlan gemm_plan(int M, int N, int K, int num_cus) {
  return gemm_plan_split(M, N, K, num_cus, 1, 0.0);
}

GemmPlan gemm_plan_split(int M, int N, int K, int num_cus, int splits, double fold_us) {
  int best_cfg = 0, best_sp = splits > 0 ? splits : 1;
  double best_us = -1;
  for (int sp = 1; sp <= 8; sp *= 2) {
    if (splits > 0 && sp != splits) continue;
    if (sp > 1 && (K % (64 * sp) != 0 || K / sp < 256 ||
                   (size_t)sp * M * N > gemm_ws_floats_bound(num_cus)))
      continue;
    for (int c = 0; c < gemm_num_cfgs(); ++c) {
      const double us = gemm_us(M, N, K, num_cus, c, sp, fold_us);
      if (best_us < 0 || us < best_us) { best_cfg = c; best_sp = sp; best_us = us; }
    }
  }
  return gemm_plan_cfg(M, N, K, best_cfg, best_sp);
}


// With timing events, the dispatch itself stamps them with the kernel's start and end
// (hipExtLaunchKernel), so no marker packet sits between the events and the kernel.
template <int WM, int WN, int TM, int TN, int ST, int OCC, int EPI>
static hipError_t run(const GemmArgs& a, int grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  constexpr unsigned LDS = ST * (WM * TM + WN * TN) * 16 * BK * 2;  // ST stages of both operands
  static_assert(LDS <= 160 * 1024, "LDS of a CU");
  if (e0 || e1)
    hipExtLaunchKernelGGL((k_gemm<WM, WN, TM, TN, ST, OCC, EPI>), dim3(grid), dim3(WM * WN * 64), LDS, s, e0, e1, 0, a);
  else
    hipLaunchKernelGGL((k_gemm<WM, WN, TM, TN, ST, OCC, EPI>), dim3(grid), dim3(WM * WN * 64), LDS, s, a);
  return hipGetLastError();
}

template <int EPI>
static hipError_t run_cfg(int cfg, const GemmArgs& a, int grid, hipStream_t s, hipEvent_t e0,
                          hipEvent_t e1) {
  switch (cfg) {
#define X(C, WM, WN, TM, TN, ST, OCC, ...) \
  case C: return run<WM, WN, TM, TN, ST, OCC, EPI>(a, grid, s, e0, e1);
    GEMM_CFGS(X)
#undef X
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(int epi, const GemmArgs& in, const GemmPlan& p, hipStream_t s,
                       hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (in.M == 0 || in.N == 0) return hipSuccess;
  // pairs of 32-wide slices; whole 64-row weight blocks; fp32 outputs in groups of 4 columns
  if (p.splits < 1 || in.K % (64 * p.splits) != 0) return hipErrorInvalidValue;
  if (in.w_layout != W_LM_HEAD && (in.w_layout != W_BLOCKS || in.N % 64 != 0)) return hipErrorInvalidValue;
  if ((epi == EPI_ADD_F32 || epi == EPI_PART_F32) && in.N % 4 != 0) return hipErrorInvalidValue;
  if (p.splits > 1 && epi != EPI_PART_F32) return hipErrorInvalidValue;
  GemmArgs a = in;
  a.splits = p.splits;
  const int grid = p.tiles * p.splits;
  switch (epi) {
    case EPI_BF16: return run_cfg<EPI_BF16>(p.cfg, a, grid, s, ev_start, ev_stop);
    case EPI_ADD_F32: return run_cfg<EPI_ADD_F32>(p.cfg, a, grid, s, ev_start, ev_stop);
    case EPI_SWIGLU: return run_cfg<EPI_SWIGLU>(p.cfg, a, grid, s, ev_start, ev_stop);
    case EPI_QKV_ROPE: return run_cfg<EPI_QKV_ROPE>(p.cfg, a, grid, s, ev_start, ev_stop);
    case EPI_PART_F32: return run_cfg<EPI_PART_F32>(p.cfg, a, grid, s, ev_start, ev_stop);
    case EPI_TOP1:
      if (a.n_parts != gemm_top1_parts(p, a.N) || !a.part_m || !a.part_s || !a.part_arg)
        return hipErrorInvalidValue;
      return run_cfg<EPI_TOP1>(p.cfg, a, grid, s, ev_start, ev_stop);
  }
  return hipErrorInvalidValue;
}

}  // namespace cora
