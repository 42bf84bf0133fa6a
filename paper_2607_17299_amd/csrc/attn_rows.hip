// Prefill attention over the paged KV cache (gfx950): row blocks of 128 rows, a
// causal run of one sequence's new tokens with G query heads per token.
//
// The matrix cores bound it (P V twice: P as bf16 hi + lo), with the softmax's
// VALU work close behind, so both have to run at once and nothing else may stand
// in the way:
//   * Wave w of 4 owns rows [32w, 32w + 32) and walks 32-key blocks (two pages)
//     that the workgroup shares.  v_mfma_f32_32x32x16_bf16: S^T = K Q^T with the
//     keys as the M side, one query row per lane, so the softmax needs one
//     exchange between the wave's halves; key m of a block is page m / 16, slot
//     8 (m/4 % 2) + 4 (m/8 % 2) + m % 4, which leaves each lane the 8 + 8
//     consecutive keys that O^T += V^T P^T wants of its row.
//   * Step i multiplies block i + 1's keys and block i - 1's values while it does
//     the softmax of block i: no MFMA of a step waits for its VALU work.
//   * Keys and values go straight from memory to LDS, as 1 KB MFMA fragments in
//     lane order (each lane names its own 16 bytes), so that fragment reads are
//     contiguous.  Four stages each, keys requested four steps and values two
//     before the step that holds them: a load has two steps to arrive.
// 2048 rows of 32 heads over 25600 keys (head_dim 128): 1403 -> 1151-1162 us (the
// kernel it replaces staged blocks through registers and took scores, softmax and
// product one after the other).  Over an append of 16 x 2048 tokens to 8192-26624 keys
// the matrix pipes are busy 60% of all cycles (41% before), 1.12 PFLOP/s executed, the
// masked keys of the last blocks and both halves of P counted (a large bf16 matrix
// product 1.3-1.57).  Fewer VALU instructions (the low parts by v_dot2c_f32_bf16: 1185
// us) or addresses (per-lane ones: 1151) change nothing.
#include "attn.h"
#include "lds_load.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

WAR_DEV f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// One unit's rows and keys, decoded from its work-order descriptor (the fields
// k_attn reads inline; prefill units are never shared-prefix units).
struct UnitRows {
  int item, b, chunk, t0, nt, seq, pos0, row0, nrows, last_pos;
  __device__ void decode(const AttnArgs& a, int it) {
    const int4 u0 = a.meta.udesc[2 * (it / a.n_kv_heads)], u1 = a.meta.udesc[2 * (it / a.n_kv_heads) + 1];
    item = u0.x;
    b = u0.y;
    chunk = u0.z;
    t0 = u0.w & 0xffff;
    nt = u0.w >> 16;
    seq = u1.y;
    pos0 = u1.z;
    row0 = u1.w;
    nrows = nt * a.G;
    last_pos = pos0 + t0 + nt - 1;
  }
  // row r -> (query row, query head) and its partial row; false if r is not live
  __device__ bool src(const AttnArgs& a, int kvh, int r, int& qrow, int& h, int64_t& prow) const {
    if (r >= nrows) return false;
    qrow = row0 + t0 + r / a.G;
    h = kvh * a.G + r % a.G;
    prow = ((int64_t)item * a.n_kv_heads + kvh) * a.prb + r;
    return true;
  }
};

// own loads but the last LEFT have arrived and own LDS reads are done, then
// everyone's
template <int LEFT>
WAR_DEV void wait_sync() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LEFT) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int HD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) k_attn_rows(AttnArgs a) {
  constexpr int KF = HD / 16;    // 1 KB fragments of a block's keys (MFMA k-steps), and of its values
  constexpr int NDT = HD / 32;   // 32-dim output tiles
  constexpr int PW = KF / 4;     // fragments a wave loads, of each
  constexpr int ST = 4;          // stages
  constexpr int SB = KF * 1024;  // bytes per stage
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * ST * SB];  // keys, then values
  const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = a.meta.n_items[1] * a.n_kv_heads;
  const int CH = a.meta.n_items[3];
  constexpr int P = 16;          // page size
  const uint32_t lds0 = lds_addr(smem);

  // A load is 1 KB of one page, the page's address in scalar registers.  Keys:
  // load q is pair q / 2 of k-steps in page q % 2, in LDS [k-step][dims 8 g .. + 7]
  // [key row]; values: load q is tile q % NDT in page q / NDT, [keys 8 g .. + 7][dim].
  uint32_t koff[PW], voff[PW];   // this lane's byte offset in the page
#pragma unroll
  for (int i = 0; i < PW; ++i) {
    const int q = w * PW + i;
    koff[i] = ((((lane >> 3) & 1) * (HD / 32) + q / 2) * 8 + (lane & 7)) * 64 + g * 32 + ((lane >> 4) & 1) * 16;
    voff[i] = (P * HD + ((q % NDT) * 32 + ln) * P + g * 8) * 2;
  }
  const int kread = (ln >> 4) * 1024 + g * 256 + (lane & 15) * 16, vread = ST * SB + lane * 16;

  const UnitQueue uq(total);
  __shared__ int s_it;
  if (tid == 0) s_it = blockIdx.x;
  __syncthreads();
  for (;;) {
    const int it = __builtin_amdgcn_readfirstlane(s_it);  // (scalar: so are the unit's addresses)
    if (it >= total) break;
    const int kvh = it % a.n_kv_heads;
    UnitRows u;
    u.decode(a, it);
    const int S = u.last_pos + 1;
    const int qpos0 = u.pos0 + u.t0;  // the first row's position
    const int kbeg = u.chunk * CH, kend = min(S, kbeg + CH);
    const int nb = kend > kbeg ? (kend - kbeg + 31) / 32 : 0;
    // blocks before nfull lie at or below every row's position
    const int nfull = qpos0 - 31 - kbeg < 0 ? 0 : min(nb, (qpos0 - 31 - kbeg) / 32 + 1);
    const int64_t pstride = (int64_t)a.kv.n_kv_heads * 2 * P * HD;
    const bf16_t* kvb = a.kv.kv + a.kv.page_elems(a.layer, 0, kvh, 0);

    // Page ids: lane l of pv holds page 64 n + l of the chunk (the sequence's
    // last page beyond its end), pn those of the next n.
    const int32_t* trow = a.table + (int64_t)u.seq * a.max_pages + kbeg / P;
    const int plast = (S - 1) / P - kbeg / P;
    auto page_vec = [&](int n) { return trow[min(n * 64 + lane, plast)]; };
    int pv = page_vec(0), pn = page_vec(1), pgrp = 0;
    // pages of block b (b grows by at most one from call to call)
    auto pages = [&](int b, int& p0, int& p1) __attribute__((always_inline)) {
      if ((b >> 5) != pgrp) {
        pgrp = b >> 5;
        pv = pn;
        pn = page_vec(pgrp + 1);
      }
      p0 = __builtin_amdgcn_readlane(pv, (2 * b) & 63);
      p1 = __builtin_amdgcn_readlane(pv, (2 * b + 1) & 63);
    };
    auto load_k = [&](int stage, int p0, int p1) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const int q = w * PW + i;
        load_lds16(lds0 + stage * SB + q * 1024, kvb + (int64_t)(q % 2 ? p1 : p0) * pstride, koff[i]);
      }
    };
    auto load_v = [&](int stage, int p0, int p1) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const int q = w * PW + i;
        load_lds16(lds0 + (ST + stage) * SB + q * 1024, kvb + (int64_t)(q / NDT ? p1 : p0) * pstride, voff[i]);
      }
    };

    // queries (B operand of S^T) and position of this lane's row
    const int r = w * 32 + ln;
    int qrow, h;
    int64_t prow;
    const bool live = u.src(a, kvh, r, qrow, h, prow);
    const int rpos = live ? qpos0 + r / a.G : u.last_pos;
    bf16x8 qf[KF];
#pragma unroll
    for (int f = 0; f < KF; ++f)
      qf[f] = as_bf16x8(live ? *reinterpret_cast<const uint4*>(a.q + (int64_t)qrow * a.q_stride + h * HD + f * 16 + g * 8)
                             : make_uint4(0, 0, 0, 0));

    float m_run = -INFINITY, l_run = 0.f;
    f32x16 o_acc[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o_acc[dt][e] = 0.f;

    struct Pw {
      uint4 hi[2], lo[2];  // weights of the block's two pages
    };
    auto kfrag = [&](int stage, int f) __attribute__((always_inline)) {
      return as_bf16x8(*reinterpret_cast<const uint4*>(smem + stage * SB + (f >> 1) * 2048 + (f & 1) * 512 + kread));
    };
    auto vfrag = [&](int stage, int f) __attribute__((always_inline)) {
      return as_bf16x8(*reinterpret_cast<const uint4*>(smem + stage * SB + f * 1024 + vread));
    };
    f32x16 zero;
#pragma unroll
    for (int e = 0; e < 16; ++e) zero[e] = 0.f;
    auto scores = [&](int stage, f32x16& s) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
      for (int f = 0; f < KF; ++f) s = mfma32(kfrag(stage, f), qf[f], s);
    };

    // Step i: keys and values of blocks i + 4 and i + 2 are requested, S(i + 1)
    // and the product of block i - 1's weights and values are taken, and the
    // softmax of block i makes its weights.  Past the end the requests repeat the
    // last block and S(i + 1) is of no use; block -1 has zero weights and zeros.
    auto step = [&](int i, f32x16& s, f32x16& snext, const Pw& pin, Pw& pout, int k0, int k1, int v0,
                    int v1) __attribute__((always_inline)) {
      load_k(i & 3, k0, k1);
      load_v((i + 2) & 3, v0, v1);
      if (i >= nfull) {  // keys above some row's position or past the sequence end
        const int kb = kbeg + 32 * i;
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (kb + 16 * (e >> 3) + 8 * g + (e & 7) > rpos) s[e] = -INFINITY;
      }
      __builtin_amdgcn_sched_barrier(0);
      // 3 KF slots of one MFMA each: k-step f of S(i + 1), then the two products
      // (hi, lo) of value fragment f, whose operands are read LOOK triples
      // ahead; the softmax of block i is dealt over the slots.
      // Lane holds S^T[key kb + 16 (e / 8) + 8 g + e % 8][row].
      constexpr int LOOK = 2, RING = 3;
      bf16x8 rk[RING], rv[RING];
      auto read = [&](int f) __attribute__((always_inline)) {
        rk[f % RING] = kfrag((i + 1) & 3, f);
        rv[f % RING] = vfrag((i + 3) & 3, f);
      };
#pragma unroll
      for (int f = 0; f < LOOK; ++f) read(f);
      float lm = 0.f, m_new = 0.f, m_use = 0.f, sum = 0.f, p0 = 0.f, p1 = 0.f;
      uint32_t hi[8], lo[8];
      constexpr int SLOTS = 3 * KF, HEAD = 3 * KF / 8;  // the row maximum takes the first HEAD slots
      auto softmax = [&](int t) __attribute__((always_inline)) {  // task t of 16: half of the work of a pair of keys
        const int e = t / 2 * 2;
        if (t % 2 == 0) {
          float s0 = s[e], s1 = s[e + 1];
          asm volatile("" : "+v"(s0), "+v"(s1));  // (the empty asm keep the work in its slot)
          p0 = __builtin_amdgcn_exp2f(fmaf(s0, a.scale_log2, -m_use));
          p1 = __builtin_amdgcn_exp2f(fmaf(s1, a.scale_log2, -m_use));
          hi[e / 2] = pack2(p0, p1);
          asm volatile("" : "+v"(hi[e / 2]), "+v"(p0), "+v"(p1));
        } else {
          sum += p0 + p1;
          lo[e / 2] = pack2(p0 - lo_f(hi[e / 2]), p1 - hi_f(hi[e / 2]));
          asm volatile("" : "+v"(lo[e / 2]), "+v"(sum));
        }
      };
#pragma unroll
      for (int z = 0; z < SLOTS; ++z) {
        const int f = z / 3;
        if (z % 3 == 0) {
          if (f + LOOK < KF) read(f + LOOK);
          snext = mfma32(rk[f % RING], qf[f], f == 0 ? zero : snext);
        } else {
          o_acc[f % NDT] = mfma32(rv[f % RING], as_bf16x8(z % 3 == 1 ? pin.hi[f / NDT] : pin.lo[f / NDT]), o_acc[f % NDT]);
        }
        if (z == 0) {
          lm = fmaxf(s[0], s[1]);
#pragma unroll
          for (int e = 2; e < 16; e += 2) lm = fmaxf(fmaxf(s[e], s[e + 1]), lm);
          lm *= a.scale_log2;
        }
        if (z == HEAD - 1) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(lm), __float_as_uint(lm), false, false);
          const float mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
          m_new = mx > m_run + 8.f ? mx : m_run;  // lazy rescaling, decided per row as in k_attn
          m_use = m_new == -INFINITY ? 0.f : m_new;
        }
#pragma unroll
        for (int t = 0; t < 16; ++t)
          if (z >= HEAD && t * (SLOTS - HEAD) / 16 == z - HEAD) softmax(t);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int pg = 0; pg < 2; ++pg) {
        pout.hi[pg] = make_uint4(hi[pg * 4], hi[pg * 4 + 1], hi[pg * 4 + 2], hi[pg * 4 + 3]);
        pout.lo[pg] = make_uint4(lo[pg * 4], lo[pg * 4 + 1], lo[pg * 4 + 2], lo[pg * 4 + 3]);
      }
      if (__any(m_new != m_run)) {
        const float alpha = m_new == m_run ? 1.f : exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o_acc[dt] *= alpha;
        m_run = m_new;
      }
      l_run += sum;
      wait_sync<4 * PW>();  // K(i + 2) and V(i) are here; steps i - 1 and i may be in flight
    };

    if (nb > 0) {
      const int lb = nb - 1;
      int k0, k1, v0[2], v1[2];  // v: pages of the blocks whose values are requested next
      pages(0, k0, k1);
      load_k(0, k0, k1);
      const int f0 = k0, f1 = k1;
      pages(min(1, lb), k0, k1);
      load_k(1, k0, k1);
      const int g0 = k0, g1 = k1;
      pages(min(2, lb), v0[0], v1[0]);
      load_k(2, v0[0], v1[0]);
      load_v(0, f0, f1);
      pages(min(3, lb), v0[1], v1[1]);
      load_k(3, v0[1], v1[1]);
      load_v(1, g0, g1);
      // block -1's values
      for (int e = tid; e < SB / 16; e += 256)
        *reinterpret_cast<uint4*>(smem + (ST + 3) * SB + e * 16) = make_uint4(0, 0, 0, 0);
      f32x16 sa, sb;
      Pw pa, pb;
#pragma unroll
      for (int pg = 0; pg < 2; ++pg) pa.hi[pg] = pa.lo[pg] = make_uint4(0, 0, 0, 0);
      wait_sync<5 * PW>();
      scores(0, sa);
      wait_sync<4 * PW>();
      for (int i = 0;;) {
        pages(min(i + 4, lb), k0, k1);
        step(i, sa, sb, pa, pb, k0, k1, v0[0], v1[0]);
        v0[0] = k0;
        v1[0] = k1;
        if (++i == nb) {
          pa = pb;
          break;
        }
        pages(min(i + 4, lb), k0, k1);
        step(i, sb, sa, pb, pa, k0, k1, v0[1], v1[1]);
        v0[1] = k0;
        v1[1] = k1;
        if (++i == nb) break;
      }
      // the last block's product; slots past the sequence end may hold anything
      const int kb = kbeg + 32 * lb;
#pragma unroll
      for (int pg = 0; pg < 2; ++pg)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          uint4 v = __builtin_bit_cast(uint4, vfrag(lb & 3, pg * NDT + dt));
          if (kb + 32 > S) v = keep_first(v, min(max(S - (kb + 16 * pg + 8 * g), 0), 8));
          o_acc[dt] = mfma32(as_bf16x8(v), as_bf16x8(pa.hi[pg]), o_acc[dt]);
          o_acc[dt] = mfma32(as_bf16x8(v), as_bf16x8(pa.lo[pg]), o_acc[dt]);
        }
    }

    int next_it = 0;
    if (tid == 0) next_it = uq.next(a.unit_ctr);
    // this wave's rows: partial O, running max and sum
    const float l = l_run + __shfl_xor(l_run, 32, 64);
    if (live) {
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(&a.po[prow * HD + dt * 32 + q * 8 + g * 4]) =
              make_float4(o_acc[dt][q * 4], o_acc[dt][q * 4 + 1], o_acc[dt][q * 4 + 2], o_acc[dt][q * 4 + 3]);
      if (g == 0) {
        a.pm[prow] = m_run;
        a.pl[prow] = l;
      }
    }
    if (tid == 0) s_it = next_it;
    wait_sync<0>();
  }
}

}  // namespace

void launch_attn_rows(const AttnArgs& a, int head_dim, int grid, hipStream_t st) {
  if (head_dim == 128) k_attn_rows<128><<<grid, 256, 0, st>>>(a);
  else k_attn_rows<64><<<grid, 256, 0, st>>>(a);
}
