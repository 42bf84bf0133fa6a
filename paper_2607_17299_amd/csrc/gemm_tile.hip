// Tiled bf16 GEMM on gfx950 MFMA for many rows: the projections of prefill
// chunks and wide verify batches, and their LM head (more than 80 rows, a large LM
// head more than 96; fewer run in gemm.hip's skinny kernels).
//
// C[m][n] = sum_k A[m][k] * W[n][k] over the packed weights of gemm.hip (1 KB
// MFMA fragments, step-major).  At these sizes the matrix cores bound it, so a
// workgroup computes a large tile (up to 256 x 256) from LDS and every operand
// byte comes straight from memory to LDS:
//   * 8 waves as WM x WN, each with (BM / WM) x (BN / WN) of the tile in
//     accumulators; v_mfma_f32_16x16x32_bf16, fp32 sums over all of the split's k;
//   * ST stages of one 64-wide k-step each.  W arrives as the 1 KB fragments it is
//     stored in; an A row of the step is one 128-byte line, its eight 16-byte
//     chunks permuted so that fragment reads fall on different banks;
//   * one barrier a step, and the loads of a stage spread over the slots between
//     (issued together they hold up the LDS reads behind them: gate/up at 2048
//     rows 327 us against 304).
// A third stage pays where it fits (128 rows by 256 columns or less): 256-row
// gate/up 72 -> 57 us.
// Measured (4096-wide decoder, weights rotated), against the skinny kernels that
// ran these rows before: qkv / o / gate+up / down at 256 rows 28 / 19 / 86 / 48 us
// -> 19 / 14 / 57 / 33; at 1152 rows 74 / 44 / 249 / 141 -> 53 / 39 / 199 / 98; at
// 2048 rows 130 / 85 / 477 / 263 -> 93 / 58 / 308 / 153 (1340 TFLOP/s); over a
// long append's passes of 2048 rows the matrix pipes are busy 62% (gate/up), 59%
// (down), 48% (o) and 42% (qkv, 192 tiles on 256 CUs) of all cycles.
#include "lds_load.h"

namespace {

constexpr int KS = 64;          // k-step
constexpr int kThreads = 512;   // 8 waves

// LPS = loads issued per slot (see below).  WNT: one m-block, so every weight
// byte is used by one workgroup and its load is non-temporal.
template <int BM, int BN, int WM, int WN, int LPS, int ST, int EPI, bool WNT>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) k_gemm_tile(GemmArgs g) {
  static_assert(WM * WN == 8 && BM % 64 == 0 && BN % 128 == 0, "8 waves, whole loads");
  constexpr int MT = BM / WM / 16, NT = BN / WN / 16;  // 16 x 16 tiles per wave
  constexpr int A_INS = BM / 64, W_INS = BN / 64;      // 1 KB loads per wave and step
  constexpr int INS = A_INS + W_INS;
  constexpr int NGB = BN / 128;                        // weight groups per tile
  constexpr int A_B = BM * 128, STAGE = (BM + BN) * 128;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[ST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, lg = lane >> 4;
  const int wi = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wi % WM, wn = wi / WM;
  const int mblocks = (g.M + BM - 1) / BM;
  const int NG = g.N / 128;                            // weight groups
  const int NB = (NG + NGB - 1) / NGB;                 // the last tile may be half empty
  // Workgroups are dealt to the 8 XCDs round-robin by linear id: the m-blocks of
  // one weight block get ids 8 apart, so all but the first find W in that XCD's
  // L2; a ragged tail of fewer than 8 n-blocks falls back to consecutive ids.
  const int full = (NB / 8) * 8 * mblocks;
  int nb, mb;
  if ((int)blockIdx.x < full) {
    const int r = blockIdx.x % (8 * mblocks);
    nb = (blockIdx.x / (8 * mblocks)) * 8 + (r & 7);
    mb = r >> 3;
  } else {
    const int r = blockIdx.x - full;
    nb = (NB / 8) * 8 + r / mblocks;
    mb = r % mblocks;
  }
  const int split = blockIdx.y;
  const int m0 = mb * BM;
  const int kb = split * g.kper;
  const int nsteps = (min(g.K, kb + g.kper) - kb) / KS;
  const int sstride = NG * (KS * 256);  // bytes per k-step of the packed weights
  const int64_t wbase = (int64_t)nb * NGB * (8 * KS * 16);
  const i32x4 wres = make_rsrc(g.Wp + wbase, ((int64_t)g.N * g.K - wbase) * 2);
  // rows at or beyond M read as zero (the LM head's gathered rows: row 0)
  const i32x4 ares = make_rsrc(g.A, EPI == EPI_ARGMAX ? 0xffffffffLL : (int64_t)g.M * g.lda * 2);

  // A: load i of wave wi brings rows (i * 8 + wi) * 8 .. + 7, lane l the 16-byte
  // slot l % 8 of row l / 8.  Slot c of row r holds chunk c ^ ((r / 2) % 8).
  // (av is the offset of load 0 of step 0; offsets are carried whole in the
  // lanes, so that the descriptor's size check covers them.)
  const int ar = wi * 8 + (lane >> 3);
  const int av = ((m0 + ar) * g.lda + kb + (((lane & 7) ^ ((ar >> 1) & 7)) * 8)) * 2;
  int avr[EPI == EPI_ARGMAX ? A_INS : 1];
  if constexpr (EPI == EPI_ARGMAX) {
#pragma unroll
    for (int i = 0; i < A_INS; ++i) {
      const int r = m0 + ar + i * 64 < g.M ? m0 + ar + i * 64 : 0;
      avr[i] = ((g.a_rows ? g.a_rows[r] : r) * g.lda + (((lane & 7) ^ ((ar >> 1) & 7)) * 8)) * 2;
    }
  }
  const int wv = (kb / KS) * sstride + wi * 1024 + lane * 16;
  // load i of k-step s into stage q
  auto load1 = [&](int q, int s, int i) __attribute__((always_inline)) {
    const uint32_t to = lds_addr(smem) + q * STAGE + wi * 1024;
    if (i < A_INS)
      load_lds16<false>(to + i * 8192, EPI == EPI_ARGMAX ? avr[EPI == EPI_ARGMAX ? i : 0] + s * KS * 2
                                                  : av + (s * KS + i * 64 * g.lda) * 2, ares);
    else load_lds16<WNT>(to + A_B + (i - A_INS) * 8192, wv + s * sstride + (i - A_INS) * 8192, wres);
  };

  // Weight tiles of this wave: NT consecutive ones; SwiGLU takes NT / 2 gate
  // tiles of a group and then the matching up tiles, 4 further.
  constexpr int NG2 = NT / 2;
  static_assert(EPI != EPI_SWIGLU || 4 % NG2 == 0, "a wave's gate tiles lie in one group");
  const int q0 = EPI == EPI_SWIGLU ? (wn * NG2 / 4) * 8 + wn * NG2 % 4 : wn * NT;
  auto wtile = [&](int n) { return EPI == EPI_SWIGLU ? (n < NG2 ? n : 4 + n - NG2) : n; };
  const int woff = q0 * 2048 + lane * 16;
  int aoff[2];
  {
    const int r = wm * (BM / WM) + ln;   // (r + 16 mt) / 2 % 8 is the same for every mt
#pragma unroll
    for (int j = 0; j < 2; ++j) aoff[j] = r * 128 + (((lg * 2 + j) ^ ((r >> 1) & 7)) * 16);
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  // own loads of the next stage arrived (`left` later ones may be in flight) and
  // own LDS reads done, then everyone's
  auto sync = [&](auto left) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(decltype(left)::value) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // A step is 2 MT slots, one A fragment (and NT MFMAs) each: slot i is row tile
  // i % MT of k-half i / MT.  A fragments are read LOOK slots ahead into a ring,
  // the weight fragments of half 1 during half 0 and those of the next step's
  // half 0 in the last LOOK slots.  Before these last slots, the next stage must
  // be complete (sync); every read of this stage is then done, and step s + ST is
  // requested into it, LPS loads a slot, on into the next step's first slots.
  constexpr int SLOTS = 2 * MT, LOOK = 3, RING = 4;
  static_assert(SLOTS % RING == 0 && SLOTS - LOOK >= MT && INS <= LPS * SLOTS, "reads and loads fit the slots");
  constexpr int HEAD = LPS * LOOK < INS ? LPS * LOOK : INS;  // loads in the last LOOK slots
  bf16x8 ra[RING], rb[2][NT];
  auto read_a = [&](const unsigned char* sA, int i) __attribute__((always_inline)) {
    ra[i % RING] = as_bf16x8(*reinterpret_cast<const uint4*>(sA + aoff[i / MT] + (i % MT) * 2048));
  };
  auto read_b = [&](const unsigned char* sW, int h, int n) __attribute__((always_inline)) {
    rb[h][n] = as_bf16x8(*reinterpret_cast<const uint4*>(sW + woff + wtile(n) * 2048 + h * 1024));
  };
  auto step = [&](int s, auto tag) __attribute__((always_inline)) {
    constexpr int C = decltype(tag)::value, N = (C + 1) % ST, Pv = (C + ST - 1) % ST;
    const unsigned char *SA = smem + C * STAGE, *SW = SA + A_B, *NA = smem + N * STAGE, *NW = NA + A_B;
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) {
      if (i == SLOTS - LOOK) {
        // stages s + 2 .. s + ST - 1 may still be in flight
        if (s + ST - 1 < nsteps) sync(std::integral_constant<int, (ST - 2) * INS>{});
        else sync(std::integral_constant<int, 0>{});
      }
      if (i < SLOTS - LOOK) read_a(SA, i + LOOK);
      else read_a(NA, i + LOOK - SLOTS);
      if (i < MT) {
#pragma unroll
        for (int n = 0; n < NT; ++n)
          if (n * MT / NT == i) read_b(SW, 1, n);
      }
      if (i >= SLOTS - LOOK) {
#pragma unroll
        for (int n = 0; n < NT; ++n)
          if (n * LOOK / NT == i - (SLOTS - LOOK)) read_b(NW, 0, n);
        if (s + ST < nsteps) {
#pragma unroll
          for (int q = 0; q < LPS; ++q)
            if ((i - (SLOTS - LOOK)) * LPS + q < INS) load1(C, s + ST, (i - (SLOTS - LOOK)) * LPS + q);
        }
      } else if (HEAD + i * LPS < INS) {
        if (s > 0 && s + ST - 1 < nsteps) {
#pragma unroll
          for (int q = 0; q < LPS; ++q)
            if (HEAD + i * LPS + q < INS) load1(Pv, s + ST - 1, HEAD + i * LPS + q);
        }
      }
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[i % MT][n] = mfma16(ra[i % RING], rb[i / MT][n], acc[i % MT][n]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int q = 0; q < ST; ++q)
    if (q < nsteps) {
#pragma unroll
      for (int i = 0; i < INS; ++i) load1(q, q, i);
    }
  if (ST - 1 < nsteps) sync(std::integral_constant<int, (ST - 1) * INS>{});
  else sync(std::integral_constant<int, 0>{});
#pragma unroll
  for (int n = 0; n < NT; ++n) read_b(smem + A_B, 0, n);
#pragma unroll
  for (int i = 0; i < LOOK; ++i) read_a(smem, i);
  __builtin_amdgcn_sched_barrier(0);
  // (the reads past the last step are of no use, and in bounds)
  for (int s = 0; s < nsteps; s += ST) {
    step(s, std::integral_constant<int, 0>{});
    if (s + 1 < nsteps) step(s + 1, std::integral_constant<int, 1>{});
    if constexpr (ST > 2)
      if (s + 2 < nsteps) step(s + 2, std::integral_constant<int, 2>{});
  }

  // lane holds C[m0 + wm BM/WM + m 16 + lg 4 + i][tile column + ln]; the second
  // half of the last tile may lie past N
  const int row0 = m0 + wm * (BM / WM) + lg * 4;
  const int grp = nb * NGB + wn * NT / 8;              // this wave's 128-column group
  static_assert(EPI == EPI_SWIGLU || NT <= 8, "a wave's columns lie in one group");
  const bool live = grp < NG;
  if constexpr (EPI == EPI_SWIGLU) {
    if (!live) return;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + m * 16 + i;
        if (row >= g.M) continue;
#pragma unroll
        for (int n = 0; n < NG2; ++n) {
          const float a = acc[m][n][i];
          g.out[(int64_t)row * g.ld_out + (nb * NGB * 4 + wn * NG2 + n) * 16 + ln] =
              f2bf(a / (1.f + expf(-a)) * acc[m][n + NG2][i]);
        }
      }
  } else if constexpr (EPI == EPI_PARTIAL) {
    if (!live) return;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + m * 16 + i;
        if (row >= g.M) continue;
        float* pr = g.P + ((int64_t)split * g.M + row) * g.N + nb * BN + wn * NT * 16 + ln;
#pragma unroll
        for (int n = 0; n < NT; ++n) pr[n * 16] = acc[m][n][i];
      }
  } else {
    // each row's best (value, lowest index) among this wave's columns, then
    // among the waves of each 128-column group
    float* sv = reinterpret_cast<float*>(smem);                    // [WN][BM]
    int* si = reinterpret_cast<int*>(smem + WN * BM * 4);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + m * 16 + i;
        const int c0 = nb * BN + wn * NT * 16 + ln;
        float v = acc[m][0][i];
        int idx = c0;
#pragma unroll
        for (int n = 1; n < NT; ++n)
          if (acc[m][n][i] > v) {
            v = acc[m][n][i];
            idx = c0 + n * 16;
          }
        if (g.logits && live && row < g.M) {
#pragma unroll
          for (int n = 0; n < NT; ++n) g.logits[(int64_t)row * g.ld_logits + c0 + n * 16] = acc[m][n][i];
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
          const float ov = __shfl_xor(v, o, 64);
          const int oi = __shfl_xor(idx, o, 64);
          if (ov > v || (ov == v && oi < idx)) {
            v = ov;
            idx = oi;
          }
        }
        if (g.nan_max) {  // the comparisons drop most NaNs
          bool has = false;
#pragma unroll
          for (int n = 0; n < NT; ++n) has |= acc[m][n][i] != acc[m][n][i];
          if ((__ballot(has) >> (lg * 16)) & 0xffff) v = __builtin_nanf("");
        }
        if (ln == 0) {
          sv[wn * BM + row - m0] = v;
          si[wn * BM + row - m0] = idx;
        }
      }
    __syncthreads();
    constexpr int WPG = WN / NGB;  // waves per group
    for (int e = tid; e < BM * NGB; e += kThreads) {
      const int r = e % BM, gi = e / BM;
      if (m0 + r >= g.M || nb * NGB + gi >= NG) continue;
      float v = sv[gi * WPG * BM + r];
      int idx = si[gi * WPG * BM + r];
      for (int w = 1; w < WPG; ++w) {
        const float ov = sv[(gi * WPG + w) * BM + r];
        const int oi = si[(gi * WPG + w) * BM + r];
        if (ov > v || (ov == v && oi < idx) || (g.nan_max && ov != ov)) {
          v = ov;
          idx = oi;
        }
      }
      g.amax_v[(int64_t)(m0 + r) * NG + nb * NGB + gi] = v;
      g.amax_i[(int64_t)(m0 + r) * NG + nb * NGB + gi] = idx;
    }
  }
}

template <int BM, int BN, int WM, int WN, int LPS, int ST, bool WNT = false>
void go(const GemmArgs& g, int epi, int splits, hipStream_t st) {
  if constexpr (BN == 128 && !WNT)
    if (g.M <= BM) return go<BM, BN, WM, WN, LPS, ST, true>(g, epi, splits, st);
  const dim3 grid(cdiv_i(g.N, BN) * cdiv_i(g.M, BM), splits);
  if constexpr (BM != 2 * BN)  // (gate/up matrices are whole 256-column tiles: 128 x 256 is never worse)
    if (epi == EPI_SWIGLU) {
      k_gemm_tile<BM, BN, WM, WN, LPS, ST, EPI_SWIGLU, WNT><<<grid, kThreads, 0, st>>>(g);
      return;
    }
  if (epi == EPI_PARTIAL)
    k_gemm_tile<BM, BN, WM, WN, LPS, ST, EPI_PARTIAL, WNT><<<grid, kThreads, 0, st>>>(g);
  else
    k_gemm_tile<BM, BN, WM, WN, LPS, ST, EPI_ARGMAX, WNT><<<grid, kThreads, 0, st>>>(g);
}

// Tile shapes and what a k-step of one tile takes with every CU busy (us).
struct TileShape {
  int bm, bn;
  float step_us;
};
constexpr TileShape kTiles[kTileShapes] = {{256, 256, 1.29f}, {192, 256, 1.06f}, {128, 256, 0.77f},
                                {256, 128, 0.77f}, {192, 128, 0.64f}, {128, 128, 0.48f}};

}  // namespace

// The tile shape and split count with the least estimated time: whole waves of
// tiles over the 256 CUs times their k-steps, plus the partial sums' way through
// memory (0.19 us a MB) and 0.3 us a split for their consumer.  Over 19 row
// counts from 96 to 2048 of the 4096-wide decoder's four projections the choices
// take 1% more in all than the best of every shape and 1, 2, 3, 4, 6 or 8 splits
// (5.1 ms together; the skinny kernels took 6.8).  256 x 128 only differs from
// 128 x 256 in what an odd number of 128-column groups wastes.
TilePlan plan_gemm_tile(int M, int N, int K, int epi, int64_t cap_elems) {
  const int steps = K / KS;
  TilePlan best{-1, 1, K};
  float best_us = 1e30f;
  for (int c = 0; c < kTileShapes; ++c) {
    const TileShape& t = kTiles[c];
    for (int s = 1; s <= (epi == EPI_PARTIAL ? std::min(8, steps) : 1); ++s) {
      const int per = cdiv_i(steps, s);
      if (cdiv_i(steps, per) != s) continue;  // fewer splits than asked: seen before
      if (epi == EPI_PARTIAL && (int64_t)s * M * N > cap_elems) break;
      const int64_t wgs = (int64_t)cdiv_i(M, t.bm) * cdiv_i(N, t.bn) * s;
      float us = (float)((wgs + 255) / 256) * (per * t.step_us + 0.33f);
      if (epi == EPI_PARTIAL) us += (float)s * M * N * 4e-6f * 0.19f + 0.3f * s;
      if (us < best_us) {
        best_us = us;
        best = {c, s, per * KS};
      }
    }
  }
  return best;
}

void launch_gemm_tile(const GemmArgs& g, int epi, int shape, int splits, hipStream_t st) {
  switch (shape) {
    case 0: go<256, 256, 2, 4, 2, 2>(g, epi, splits, st); break;
    case 1: go<192, 256, 2, 4, 2, 2>(g, epi, splits, st); break;
    case 2: go<128, 256, 2, 4, 2, 3>(g, epi, splits, st); break;
    case 3: go<256, 128, 4, 2, 2, 3>(g, epi, splits, st); break;
    case 4: go<192, 128, 2, 4, 2, 3>(g, epi, splits, st); break;
    default: go<128, 128, 2, 4, 2, 3>(g, epi, splits, st); break;
  }
}
