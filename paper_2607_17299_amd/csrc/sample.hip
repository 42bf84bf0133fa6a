// Sampled verification: lossless speculative sampling with a deterministic
// drafter over top-k / temperature target distributions (gfx950).
//
// Target distribution of a row: keep the top_k largest logits (value
// descending, ties to the lowest token id), p = softmax(z_kept / T).  The
// draft d at row i is accepted iff u_i < p_i(d); at the first rejection the
// next token is drawn from p_i with d removed, and after the last draft from
// p_n; a draw with uniform v is the smallest token t (in id order) whose
// cumulative weight exceeds v times the total.  (The paper samples with
// temperature 1 and top-k 200 and requires lossless speculation; the rule is
// the standard one for a point-mass drafter.)
//
// k_sample_rows: one workgroup per row.  Each row's outcome (accepted?, token
// if rejected here, token if every draft up to here is accepted) is computed
// for every row; k_sample_accept then walks the rows of a request.
//
// The LM head leaves the largest logit of every 128-id block.  The top_k-th
// largest of these block maxima is at most the top_k-th largest logit, so every
// kept id lies in a block whose maximum reaches it and is itself at least that
// large: sample_from_blocks reads only those blocks (about top_k of the V / 128)
// and does the rest, an exact 3-pass radix select on an order-preserving integer
// image of the logits and ordered scans for tie ranks and draws, on the few
// candidates in LDS.  At top_k 200 of 151,936 ids a row has about 220
// candidates.  What bounds it is latency: a dozen block-wide scans.  80 rows of
// 151,936 ids: 454 us with sample_from_row (six passes over all logits),
// 28.5 us from the block maxima.
//
// sample_from_row walks the whole row instead: the radix select over all ids,
// then ordered passes (each wave walks its own id segment in coalesced 64-id
// chunks, with wave scans).  It takes what the blocks cannot narrow down: more
// kept ids than blocks, rows with more candidates than fit LDS (many equal
// logits), rows with a NaN (a block that holds one has a NaN maximum).
#include "kernels.h"

namespace {

constexpr int kST = 1024;   // threads per row workgroup
constexpr int kBins = 2048; // radix-select bins (11-bit digits)

constexpr int kBlk = 128;       // ids per block maximum (the LM head's column block)
constexpr int kMinBlk = 32;     // fewer blocks: the row walk is the faster
constexpr int kMaxBlk = 4096;   // block maxima a workgroup handles (4 per thread)
constexpr int kMaxCand = 4096;  // candidates held in LDS (4 per thread)

__device__ __forceinline__ uint32_t fkey(float x) {
  const uint32_t u = __float_as_uint(x + 0.f);  // -0 and +0 are the same value
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // larger float -> larger key
}

__device__ int block_excl_scan_i(int v, int* sh, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) sh[w] = x;
  __syncthreads();
  int off = 0, tot = 0;
  for (int i = 0; i < nw; ++i) {
    if (i < w) off += sh[i];
    tot += sh[i];
  }
  *total = tot;
  __syncthreads();
  return off + x - v;
}

// inclusive scan over the 64 lanes of a wave
template <class T>
__device__ __forceinline__ T wave_incl_scan(T x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Scan over the block's threads (in thread order) of one float each: thread
// t's (lower, upper) running sums.  Upper of a thread is bit for bit the lower
// of the next one, so the intervals tile [0, total) without gaps or overlaps.
__device__ float2 block_scan_f(float v, float* sh, float* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const float x = wave_incl_scan(v);
  const float below = __shfl_up(x, 1, 64);
  __syncthreads();
  if (lane == 63) sh[w] = x;
  __syncthreads();
  float off = 0.f, tot = 0.f;
  for (int i = 0; i < nw; ++i) {
    if (i == w) off = tot;
    tot += sh[i];
  }
  *total = tot;
  __syncthreads();
  return make_float2(lane ? off + below : off, off + x);
}

struct SampleShared {
  int hist[2 * kBins];
  int sh_i[kST / 64];
  float sh_f[kST / 64], sh_g[kST / 64];
  uint32_t prefix;
  int need;
  float max, wd;
  int tok[2];
  int flag;
};

// One pass of the radix select after its histogram (nb bins of `bits` at
// `shift`, two copies in hist): moves to the bin holding the need-th largest.
// Thread t looks at bins 2t and 2t + 1.
__device__ void radix_pick(SampleShared& sh, uint32_t pre, int shift, int nb) {
  const int t = threadIdx.x;
  const int* hist = sh.hist;
  const int c1 = 2 * t + 1 < nb ? hist[2 * t + 1] + hist[kBins + 2 * t + 1] : 0;
  const int c0 = 2 * t < nb ? hist[2 * t] + hist[kBins + 2 * t] : 0;
  int total;
  const int below = block_excl_scan_i(c0 + c1, sh.sh_i, &total);
  const int above = total - below - c0 - c1;  // elements in bins above 2t+1
  const int need = sh.need;
  __syncthreads();
  if (above < need && need <= above + c1) {
    sh.prefix = pre | ((uint32_t)(2 * t + 1) << shift);
    sh.need = need - above;
  } else if (above + c1 < need && need <= above + c1 + c0) {
    sh.prefix = pre | ((uint32_t)(2 * t) << shift);
    sh.need = need - above - c1;
  }
  __syncthreads();
}

// The row's outcome from the LM head's block maxima; false (by every thread)
// when they leave too many candidates or hold a NaN, and nothing is written.
__device__ bool sample_from_blocks(const SampleArgs& s, int r, int d, SampleShared& sh, uint32_t* c_key, int* c_id) {
  constexpr int NW = kST / 64;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const float* z = s.logits + (int64_t)r * s.V;
  const int nblk = s.V / kBlk;
  const float* bm = s.block_max + (int64_t)r * nblk;
  // the first two digits (22 bits) of the top_k-th largest block maximum: the
  // low edge of its bin bounds the kept logits from below
  uint32_t mk[4];
  bool has[4], nan = false;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int q = 4 * t + e;
    has[e] = q < nblk;
    const float v = has[e] ? bm[q] : 0.f;
    nan |= v != v;
    mk[e] = fkey(v);
  }
  if (t == 0) {
    sh.prefix = 0;
    sh.need = s.top_k;
    sh.flag = 0;
    sh.tok[0] = sh.tok[1] = 0x7fffffff;
  }
  __syncthreads();
  if (nan) sh.flag = 1;  // every writer stores 1
  for (int pass = 0; pass < 2; ++pass) {
    const int shift = pass == 0 ? 21 : 10;
    for (int k = t; k < 2 * kBins; k += kST) sh.hist[k] = 0;
    __syncthreads();
    const uint32_t pre = sh.prefix, hmask = pass == 0 ? 0u : 0xffe00000u;
    int* hh = sh.hist + (w & 1) * kBins;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (has[e] && (mk[e] & hmask) == pre) atomicAdd(&hh[(mk[e] >> shift) & (kBins - 1)], 1);
    __syncthreads();
    radix_pick(sh, pre, shift, kBins);
  }
  if (sh.flag) return false;
  const uint32_t low = sh.prefix;
  // the blocks that reach it, in id order (c_id holds their list)
  int nsel;
  int mine = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) mine += has[e] && mk[e] >= low;
  int at = block_excl_scan_i(mine, sh.sh_i, &nsel);
  int* sel = sh.hist;                                  // [nsel] <= kMaxBlk = 2 kBins
  static_assert(kMaxBlk <= 2 * kBins, "the block list shares the histogram");
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (has[e] && mk[e] >= low) sel[at++] = 4 * t + e;
  __syncthreads();
  // candidates per wave (wave w takes selected blocks [w0, w1)): count, then
  // write at the wave's place, in id order (lane l holds ids l and l + 64)
  const int per = (nsel + NW - 1) / NW;
  const int w0 = min(nsel, w * per), w1 = min(nsel, w0 + per);
  int cnt = 0;
  for (int q = w0; q < w1; ++q) {
    const float* zb = z + (int64_t)sel[q] * kBlk + lane;
    cnt += __popcll(__ballot(fkey(zb[0]) >= low)) + __popcll(__ballot(fkey(zb[64]) >= low));
  }
  if (lane == 0) sh.sh_i[w] = cnt;
  __syncthreads();
  int pos = 0, nc = 0;
  for (int k = 0; k < NW; ++k) {
    if (k < w) pos += sh.sh_i[k];
    nc += sh.sh_i[k];
  }
  __syncthreads();
  if (nc > kMaxCand) return false;
  for (int q = w0; q < w1; ++q) {
    const int id0 = sel[q] * kBlk + lane;
    const uint32_t k0 = fkey(z[id0]), k1 = fkey(z[id0 + 64]);
    const unsigned long long b0 = __ballot(k0 >= low), b1 = __ballot(k1 >= low);
    const unsigned long long before = (1ull << lane) - 1;
    if (k0 >= low) {
      const int o = pos + __popcll(b0 & before);
      c_key[o] = k0;
      c_id[o] = id0;
    }
    pos += __popcll(b0);
    if (k1 >= low) {
      const int o = pos + __popcll(b1 & before);
      c_key[o] = k1;
      c_id[o] = id0 + 64;
    }
    pos += __popcll(b1);
  }
  if (t == 0) {
    sh.prefix = 0;
    sh.need = s.top_k;
  }
  __syncthreads();
  // thread t owns candidates 4t .. 4t+3 (id order)
  uint32_t key[4];
  bool in[4];
  uint32_t top = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    in[e] = 4 * t + e < nc;
    key[e] = in[e] ? c_key[4 * t + e] : 0;
    top = max(top, key[e]);
  }
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
    const int nb = pass == 2 ? kBins / 2 : kBins;
    for (int k = t; k < 2 * kBins; k += kST) sh.hist[k] = 0;
    __syncthreads();
    const uint32_t pre = sh.prefix;
    const uint32_t hmask = pass == 0 ? 0u : pass == 1 ? 0xffe00000u : 0xfffffc00u;
    int* hh = sh.hist + (w & 1) * kBins;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (in[e] && (key[e] & hmask) == pre) atomicAdd(&hh[(key[e] >> shift) & (nb - 1)], 1);
    __syncthreads();
    radix_pick(sh, pre, shift, nb);
  }
  const uint32_t kth = sh.prefix;   // key of the top_k-th largest logit
  const int ties_kept = sh.need;    // how many logits equal to it are kept (lowest ids first)
  for (int o = 32; o >= 1; o >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, o, 64));
  __syncthreads();
  if (lane == 0) sh.sh_i[w] = (int)top;
  __syncthreads();
  for (int k = 0; k < NW; ++k) top = max(top, (uint32_t)sh.sh_i[k]);
  auto value = [](uint32_t k) { return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k); };
  const float zmax = value(top), invT = 1.f / s.temperature;
  int ntie = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) ntie += in[e] && key[e] == kth;
  int all_ties;
  int rank = block_excl_scan_i(ntie, sh.sh_i, &all_ties);
  float wv[4], wr[4], sum = 0.f, sumr = 0.f;
  int id[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    id[e] = in[e] ? c_id[4 * t + e] : -1;
    const bool tie = in[e] && key[e] == kth;
    rank += tie ? 1 : 0;
    const bool kept = in[e] && (key[e] > kth || (tie && rank <= ties_kept));
    wv[e] = kept ? expf((value(key[e]) - zmax) * invT) : 0.f;
    wr[e] = id[e] == d ? 0.f : wv[e];
    sum += wv[e];
    sumr += wr[e];
    if (id[e] == d && in[e]) sh.wd = wv[e];
  }
  if (t == 0) sh.flag = 0;
  float W, Wr;
  const float2 ce = block_scan_f(sum, sh.sh_f, &W);
  const float2 cr = block_scan_f(sumr, sh.sh_g, &Wr);
  // the draft's weight: 0 unless it is a candidate
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (in[e] && id[e] == d) sh.flag = 1;
  __syncthreads();
  const float wdraft = sh.flag ? sh.wd : 0.f;
  const float u = s.uniforms[(int64_t)r * 2], vv = s.uniforms[(int64_t)r * 2 + 1];
  const float tgt_end = vv * W, tgt_rej = vv * Wr;
  // the thread whose interval holds a target looks for it among its candidates
  // (the last kept one takes what rounding leaves at the interval's end)
  int last_end = -1, last_rej = -1;  // highest kept ids (fallback below)
  int hit_end = -1, hit_rej = -1;
  float pe = ce.x, pr = cr.x;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    pe += wv[e];
    pr += wr[e];
    if (wv[e] > 0.f) {
      last_end = id[e];
      if (hit_end < 0 && pe > tgt_end) hit_end = id[e];
    }
    if (wr[e] > 0.f) {
      last_rej = id[e];
      if (hit_rej < 0 && pr > tgt_rej) hit_rej = id[e];
    }
  }
  if (ce.x <= tgt_end && tgt_end < ce.y && last_end >= 0) atomicMin(&sh.tok[1], hit_end >= 0 ? hit_end : last_end);
  if (cr.x <= tgt_rej && tgt_rej < cr.y && last_rej >= 0) atomicMin(&sh.tok[0], hit_rej >= 0 ? hit_rej : last_rej);
  // a target that rounds to the total lies in no interval: the last kept token
  for (int o = 32; o >= 1; o >>= 1) {
    last_end = max(last_end, __shfl_xor(last_end, o, 64));
    last_rej = max(last_rej, __shfl_xor(last_rej, o, 64));
  }
  if (lane == 0) {
    sh.sh_i[w] = last_end;
    sh.hist[w] = last_rej;
  }
  __syncthreads();
  if (t == 0) {
    int le = -1, lr = -1;
    for (int k = 0; k < NW; ++k) {
      le = max(le, sh.sh_i[k]);
      lr = max(lr, sh.hist[k]);
    }
    int* o = s.row_out + (int64_t)r * 3;
    o[0] = d >= 0 && u * W < wdraft ? 1 : 0;
    o[1] = sh.tok[0] != 0x7fffffff ? sh.tok[0] : lr;
    o[2] = sh.tok[1] != 0x7fffffff ? sh.tok[1] : le;
  }
  return true;
}

__device__ void sample_from_row(const SampleArgs& s, int r, int d, SampleShared& sh) {
  constexpr int NW = kST / 64;
  int *hist = sh.hist, *sh_i = sh.sh_i, *s_tok = sh.tok;
  float *sh_f = sh.sh_f, *sh_g = sh.sh_g;
  const float* z = s.logits + (int64_t)r * s.V;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;

  // ---- radix select of the top_k-th largest key: digits of 11, 11 and 10
  // bits, high first (the first digit spans sign, exponent and two mantissa
  // bits, so that logits of similar size spread over many bins), into two
  // histogram copies (even and odd waves) to halve atomic contention
  if (t == 0) {
    sh.prefix = 0;
    sh.need = s.top_k;
    s_tok[0] = s_tok[1] = -1;
  }
  float mx = -INFINITY;
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
    const int nbits = pass == 2 ? 10 : 11;
    const int nb = 1 << nbits;
    for (int k = t; k < 2 * kBins; k += kST) hist[k] = 0;
    __syncthreads();
    const uint32_t pre = sh.prefix;
    const uint32_t hmask = pass == 0 ? 0u : (0xffffffffu << (shift + nbits));
    int* hh = hist + (w & 1) * kBins;
    for (int v = t; v < s.V; v += kST) {
      const float x = z[v];
      if (pass == 0) mx = fmaxf(mx, x);
      const uint32_t key = fkey(x);
      if ((key & hmask) == pre) atomicAdd(&hh[(key >> shift) & (nb - 1)], 1);
    }
    __syncthreads();
    radix_pick(sh, pre, shift, nb);
  }
  const uint32_t kth = sh.prefix;  // key of the top_k-th largest logit
  const int ties_kept = sh.need;   // how many logits equal to it are kept (lowest ids first)
  // row maximum
  for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) sh_f[w] = mx;
  __syncthreads();
  if (t == 0) {
    float m = sh_f[0];
    for (int k = 1; k < NW; ++k) m = fmaxf(m, sh_f[k]);
    sh.max = m;
  }
  __syncthreads();
  const float zmax = sh.max;
  const float invT = 1.f / s.temperature;

  // ---- ordered passes: wave w owns ids [seg0, seg1), walked in 64-id chunks
  // (lane l reads id c + l: coalesced); prefixes inside a chunk come from
  // wave scans, across chunks from a running carry, across waves from a block
  // scan of the wave totals
  const int seg = (s.V + NW - 1) / NW;
  const int seg0 = min(s.V, w * seg), seg1 = min(s.V, seg0 + seg);
  // (1) ties per wave -> the rank of each wave's first tie
  int ties = 0;
  for (int c = seg0; c < seg1; c += 64) {
    const int v = c + lane;
    ties += (v < seg1 && fkey(z[v]) == kth) ? 1 : 0;
  }
  for (int o = 32; o >= 1; o >>= 1) ties += __shfl_xor(ties, o, 64);
  if (lane == 0) sh_i[w] = ties;
  __syncthreads();
  int tie0 = 0;
  for (int k = 0; k < w; ++k) tie0 += sh_i[k];
  __syncthreads();
  // weight of id v given the rank of the ties before it
  auto weight = [&](int v, int tie_rank_incl, bool is_tie, float x) -> float {
    const uint32_t key = fkey(x);
    const bool kept = key > kth || (is_tie && tie_rank_incl <= ties_kept);
    return kept ? expf((x - zmax) * invT) : 0.f;
  };
  // (2) weights per wave (all, and without the draft)
  float wsum = 0.f, wdr = 0.f;
  {
    int carry = tie0;
    for (int c = seg0; c < seg1; c += 64) {
      const int v = c + lane;
      const float x = v < seg1 ? z[v] : -INFINITY;
      const bool tie = v < seg1 && fkey(x) == kth;
      const int rank = carry + wave_incl_scan(tie ? 1 : 0);
      carry = __shfl(rank, 63, 64);
      const float wv = v < seg1 ? weight(v, rank, tie, x) : 0.f;
      wsum += wv;
      if (v == d) wdr = wv;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    wsum += __shfl_xor(wsum, o, 64);
    wdr += __shfl_xor(wdr, o, 64);
  }
  if (lane == 0) {
    sh_f[w] = wsum;
    sh_g[w] = wdr;
  }
  __syncthreads();
  float W = 0.f, wdraft = 0.f, off_all = 0.f, off_rej = 0.f;
  for (int k = 0; k < NW; ++k) {
    if (k < w) {
      off_all += sh_f[k];
      off_rej += sh_f[k] - sh_g[k];
    }
    W += sh_f[k];
    wdraft += sh_g[k];
  }
  const float Wr = W - wdraft;
  // the acceptance test, then the token for either outcome
  const float u = s.uniforms[(int64_t)r * 2], vv = s.uniforms[(int64_t)r * 2 + 1];
  const bool accept = d >= 0 && u * W < wdraft;
  // (3) cumulative weights in id order: the draws
  const float tgt_end = vv * W, tgt_rej = vv * Wr;
  int last_end = -1, last_rej = -1;  // highest kept ids (fallback below)
  {
    int carry = tie0;
    float ce = off_all, cr = off_rej;
    for (int c = seg0; c < seg1; c += 64) {
      const int v = c + lane;
      const float x = v < seg1 ? z[v] : -INFINITY;
      const bool tie = v < seg1 && fkey(x) == kth;
      const int rank = carry + wave_incl_scan(tie ? 1 : 0);
      carry = __shfl(rank, 63, 64);
      const float wv = v < seg1 ? weight(v, rank, tie, x) : 0.f;
      const float wr = v == d ? 0.f : wv;
      const float ie = wave_incl_scan(wv), ir = wave_incl_scan(wr);
      const float cum_e = ce + ie, cum_r = cr + ir;
      if (wv > 0.f) {
        last_end = v;
        if (v != d) last_rej = v;
        if (cum_e > tgt_end && cum_e - wv <= tgt_end) s_tok[1] = v;
        if (v != d && cum_r > tgt_rej && cum_r - wr <= tgt_rej) s_tok[0] = v;
      }
      ce += __shfl(ie, 63, 64);
      cr += __shfl(ir, 63, 64);
    }
  }
  // a target at the very top of the cumulative sum can miss every crossing
  // through rounding between partial sums: take the last kept token then
  for (int o = 32; o >= 1; o >>= 1) {
    last_end = max(last_end, __shfl_xor(last_end, o, 64));
    last_rej = max(last_rej, __shfl_xor(last_rej, o, 64));
  }
  if (lane == 0) {
    sh_i[w] = last_end;
    hist[w] = last_rej;
  }
  __syncthreads();
  if (t == 0) {
    int le = -1, lr = -1;
    for (int k = 0; k < NW; ++k) {
      le = max(le, sh_i[k]);
      lr = max(lr, hist[k]);
    }
    int* o = s.row_out + (int64_t)r * 3;
    o[0] = accept ? 1 : 0;
    o[1] = s_tok[0] >= 0 ? s_tok[0] : lr;
    o[2] = s_tok[1] >= 0 ? s_tok[1] : le;
  }
}

// BLOCKS: the LM head's block maxima are there and can narrow the row down.
template <bool BLOCKS>
__global__ void __launch_bounds__(kST) k_sample_rows(SampleArgs s) {
  __shared__ SampleShared sh;
  __shared__ uint32_t c_key[BLOCKS ? kMaxCand : 1];
  __shared__ int c_id[BLOCKS ? kMaxCand : 1];
  const int r = blockIdx.x;
  const int b = r / s.kp1, i = r % s.kp1;
  const int dl = s.ntok[b] - 1;  // drafts of the request (-1: inactive step)
  if (i > dl) return;
  const int d = i < dl ? s.drafts[(int64_t)b * s.k_max + i] : -1;
  if constexpr (BLOCKS) {
    if (sample_from_blocks(s, r, d, sh, c_key, c_id)) return;
    __syncthreads();
  }
  sample_from_row(s, r, d, sh);
}

// block_max[row][block] over rows of V logits (V a multiple of kBlk): what the
// LM head's epilogue leaves, for logits that come from elsewhere.
__global__ void __launch_bounds__(64) k_block_max(const float* z, int V, float* block_max) {
  const int64_t at = (int64_t)blockIdx.y * V + (int64_t)blockIdx.x * kBlk + threadIdx.x;
  const float a = z[at], b = z[at + 64], m = wave_max(fmaxf(a, b));
  const bool nan = __any(a != a || b != b);
  if (threadIdx.x == 0) block_max[(int64_t)blockIdx.y * (V / kBlk) + blockIdx.x] = nan ? __builtin_nanf("") : m;
}

__global__ void k_sample_accept(SampleArgs s, int32_t* accept_lens, int32_t* next_tokens) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= s.B) return;
  const int dl = s.ntok[b] - 1;
  if (dl < 0) {  // no rows: the step's setup failed
    if (accept_lens) accept_lens[b] = -1;
    next_tokens[b] = -1;
    return;
  }
  int a = 0, nxt = -1;
  for (int i = 0; i <= dl; ++i) {
    const int* o = s.row_out + (int64_t)(b * s.kp1 + i) * 3;
    if (i < dl && o[0]) continue;
    a = i;
    nxt = i < dl ? o[1] : o[2];
    break;
  }
  if (accept_lens) accept_lens[b] = a;
  next_tokens[b] = nxt;
}

}  // namespace

void launch_sample(const SampleArgs& s, int32_t* accept_lens, int32_t* next_tokens, hipStream_t st) {
  // A block maximum bounds the kept logits only when there are at least top_k
  // of them; a workgroup handles kMaxBlk.  A short row is walked in less time than
  // the block path's scans take, with top_k 8: 1024 ids 16 us against 21.5, 3072 ids
  // 20 and 21.5, 4096 ids 22 and 21.5, 8192 ids 32 and 21.5.
  const int nblk = s.block_max && s.V % kBlk == 0 ? s.V / kBlk : 0;
  if (s.top_k <= nblk && nblk >= kMinBlk && nblk <= kMaxBlk)
    k_sample_rows<true><<<s.B * s.kp1, kST, 0, st>>>(s);
  else
    k_sample_rows<false><<<s.B * s.kp1, kST, 0, st>>>(s);
  k_sample_accept<<<cdiv_i(s.B, 64), 64, 0, st>>>(s, accept_lens, next_tokens);
}

void launch_block_max(const float* logits, int rows, int V, float* block_max, hipStream_t st) {
  k_block_max<<<dim3(V / kBlk, rows), 64, 0, st>>>(logits, V, block_max);
}
