// HSA Step 2 (Algorithm 1 of arXiv 2502.14051, assignments i1, g, P, s1, i2) as a workgroup-level
// routine: one workgroup of NT threads handles one (sequence, KV head).  It picks the top-k1
// channels of the group-summed |q|, streams only those rows of the channel-major page summaries
// (K_max where the group-summed q is >= 0, K_min otherwise), forms one fp32 score per page in LDS
// and keeps the top-kp pages with an exact 4-pass radix select.  Ties go to the lower index in both
// picks; the page list comes out ascending.
//
// Traffic: k1 rows of P bf16 values, read as 16-byte runs of eight pages; everything else lives in
// LDS.  Summation order is fixed, so results are bit-reproducible run to run.  The routine is
// latency-bound (a chain of a few dependent memory and LDS round trips), hence the batched loads,
// the one-barrier radix passes and the lane-shift scans.
#pragma once

#include <type_traits>

#include "common.h"

namespace rkv {

__device__ __forceinline__ uint32_t f32_order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // larger float <=> larger unsigned key
}

__device__ __forceinline__ float f32_from_order_key(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

template <int NT>
struct SelectShared {
  __align__(16) float s_abs[kHeadDim];
  float s_sum[kHeadDim];
  int s_chan[kHeadDim];
  float s_wgt[kHeadDim];
  int s_rank[kHeadDim];
  __align__(16) float partial[NT * 8];
  __align__(16) uint32_t hist[4][256];  // one histogram per radix pass
  uint32_t wsum[NT / kWave];
  uint32_t cnt0;
};

// exclusive prefix sum of one uint32 per thread over the NT-thread workgroup.  REUSE = false leaves out the
// trailing barrier, for a caller that does not touch `wsum` again before its next barrier.  The wavefronts' totals
// are summed by a scan of their own, a lane each: walking the ones in front took a sixteen-wavefront workgroup up
// to fifteen LDS reads one after the other.
template <int NT, bool REUSE = true>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* wsum) {
  constexpr int kWaves = NT / kWave;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t inc = wave_incl_scan(v);
  if (lane == kWave - 1) wsum[wave] = inc;
  __syncthreads();
  const uint32_t upto = wave_incl_scan(lane < kWaves ? wsum[lane] : 0u);
  const uint32_t base = wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto, wave - 1) : 0u;
  if (REUSE) __syncthreads();
  return base + inc - v;
}

// accumulate eight rows' worth of eight-page runs.  The rows are j0 + t * jstep, t = 0..7, with
// `jbase` the smallest j0 of the workgroup in this batch: whether batch slot t holds a row at all is
// then the same for every thread (a scalar branch), and a thread whose own row falls beyond k1 reads
// the last picked row with weight zero.  The channel / weight lookups (LDS) all come first and the
// eight 16-byte loads go out back to back, so the batch costs one LDS and one memory round trip.
// (In the general routine the page that is receiving a token in the same launch gets its score from
// the tail-page routines below instead.)
template <bool STREAM = false>
__device__ __forceinline__ void score_rows8(const SelectArgs& a, const int* s_chan, const float* s_wgt,
                                            int64_t rows, int pages_cap, int o, int j0, int jbase, int jstep,
                                            float (&acc)[8]) {
  uint4 v[8];
  float w[8];
  int ch[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int j = j0 + t * jstep;
    const int jj = j < a.k1 ? j : a.k1 - 1;
    ch[t] = s_chan[jj];
    w[t] = s_wgt[jj];
    if (j >= a.k1) w[t] = 0.f;
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    v[t] = make_uint4(0, 0, 0, 0);
    if (jbase + t * jstep < a.k1) {  // uniform over the workgroup
      const bf16_t* row = (w[t] >= 0.f ? a.kmax : a.kmin) + (rows + ch[t]) * pages_cap + o * 8;
      v[t] = ld16<STREAM>(row);
    }
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const uint32_t x[4] = {v[t].x, v[t].y, v[t].z, v[t].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] = fmaf(w[t], bf16lo_to_f32(x[i]), acc[2 * i]);
      acc[2 * i + 1] = fmaf(w[t], bf16hi_to_f32(x[i]), acc[2 * i + 1]);
    }
  }
}

// What the rows hold for a page that is receiving a token (tp.page) is stale.  Its score is computed on its own by
// the last wavefront from the page's old bounds and the new key, one or two picked channels a lane: the bound of a
// channel is the old one folded with the new key's value, or the new value alone when the token opens the page
// (whatever memory holds for that column is then not looked at).  Cheaper than patching the rows in the wavefronts
// that read the page's run (1.6 of 30.3 us a layer at 65536 tokens, 3 of 39.2 at 50000 with 120 channels).  In two
// parts, so that the lookup of the old bounds goes out before the caller's row loads and is used after them (one
// memory round trip for both).
//
// tail_page_finish leaves sums to be added up in order behind a barrier, min(R, 128) of them in sh.s_abs.  Every
// other page is summed up in R row groups, rows r, r + R, ... each in order, and then over the groups; these are
// the groups' sums, so that the score equals what a later launch makes of the stored bounds, to the bit: pages that
// tie then are ranked alike.  ONE_GROUP: R is 1.
struct TailRows {
  uint32_t old[2], key[2];    // bf16 bits: the bounds of rows `lane` and 64 + `lane`, the new key at their channels
  uint32_t old_pad, key_pad;  // of the row the padding reads: the last one, upper bound
};
template <int NT>
__device__ __forceinline__ TailRows tail_page_load(const SelectArgs& a, const SelectShared<NT>& sh, int64_t rows,
                                                   int pages_cap, const TailPatch& tp) {
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  TailRows t = {{0u, 0u}, {0u, 0u}, 0u, 0u};
  if (tp.page < 0 || wave != NT / kWave - 1) return t;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = h * kWave + lane;
    if (j < a.k1) {
      const int ch = sh.s_chan[j];
      if (tp.slot != 0) t.old[h] = (sh.s_wgt[j] >= 0.f ? a.kmax : a.kmin)[(rows + ch) * pages_cap + tp.page];
      t.key[h] = tp.knew[ch];
    }
  }
  const int ch = sh.s_chan[a.k1 - 1];
  if (tp.slot != 0) t.old_pad = a.kmax[(rows + ch) * pages_cap + tp.page];
  t.key_pad = tp.knew[ch];
  return t;
}
template <int NT, bool ONE_GROUP = false>
__device__ __forceinline__ void tail_page_finish(const SelectArgs& a, SelectShared<NT>& sh, const TailPatch& tp,
                                                 const TailRows& rows, int R) {
  constexpr int kUnroll = ONE_GROUP ? 32 : 8;  // rows of a group whose operands are read together
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (tp.page < 0 || wave != NT / kWave - 1) return;
  const auto fold = [&](uint32_t old, uint32_t key, bool upper) {
    const float f = bf16_to_f32((bf16_t)key), fo = bf16_to_f32((bf16_t)use_late(old));
    return tp.slot == 0 ? f : upper ? fmaxf(fo, f) : fminf(fo, f);
  };
  float* value = sh.s_abs;  // free since the channel pick ended
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = h * kWave + lane;
    if (j < a.k1) value[j] = fold(rows.old[h], rows.key[h], sh.s_wgt[j] >= 0.f);
  }
  // (the exchange stays within the wavefront, whose LDS accesses keep their order)
  __builtin_amdgcn_wave_barrier();
  float sum[2] = {0.f, 0.f};  // row groups `lane` and 64 + `lane`
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h * kWave >= min(R, a.k1)) break;  // (the same for every lane)
    for (int i = 0; i * R < a.k1; i += kUnroll) {
#pragma unroll
      for (int t = 0; t < kUnroll; ++t) {
        const int j = ONE_GROUP ? i + t : h * kWave + lane + (i + t) * R, jj = ONE_GROUP ? j : min(j, kHeadDim - 1);
        const float w = sh.s_wgt[jj], f = value[jj];
        sum[h] = fmaf(j < a.k1 ? w : 0.f, j < a.k1 ? f : 0.f, sum[h]);
      }
    }
  }
  // groups of unequal length are filled up with the last row's upper bound, weight zero
  if (a.k1 % R != 0) sum[0] = fmaf(0.f, fold(rows.old_pad, rows.key_pad, true), sum[0]);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int h = 0; h < 2; ++h) value[h * kWave + lane] = sum[h];
}

// lanes below this one whose bit is set
__device__ __forceinline__ int bits_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The unit's q at channel `tid` for every head of the group (threads below 128), requested but not
// used here: a caller can put its own loads behind these before anything waits, so that all of them
// share one memory round trip.  Heads beyond the group re-read head 0 (and are ignored later); the
// blocks of heads are skipped by branches that are the same for the whole workgroup.
__device__ __forceinline__ void load_q_column(const CacheView& c, const SelectArgs& a, int unit,
                                              uint32_t (&qv)[kMaxGroup]) {
  const int tid = threadIdx.x;
  const int b = unit / c.n_kv_heads, g = unit % c.n_kv_heads;
  const int G = c.group;
#pragma unroll
  for (int h = 0; h < kMaxGroup; ++h) qv[h] = 0;
  if (tid < kHeadDim) {
    const bf16_t* qp = a.q + ((int64_t)b * c.n_q_heads + (int64_t)g * G) * kHeadDim + tid;
#pragma unroll
    for (int h = 0; h < 4; ++h) qv[h] = qp[(h < G ? h : 0) * kHeadDim];
    if (G > 4) {
#pragma unroll
      for (int h = 4; h < 8; ++h) qv[h] = qp[(h < G ? h : 0) * kHeadDim];
    }
    if (G > 8) {
#pragma unroll
      for (int h = 8; h < kMaxGroup; ++h) qv[h] = qp[(h < G ? h : 0) * kHeadDim];
    }
  }
}

// Step 2, first half (needs only q): a = sum_h |q|, s = sum_h q, i1 = top-k1 channels of a, left in
// sh.s_chan / sh.s_wgt.  `qv` comes from load_q_column.  All NT threads of the workgroup take part;
// ends with a barrier.
template <int NT>
__device__ __forceinline__ void select_channels(const CacheView& c, const SelectArgs& a, int unit,
                                                SelectShared<NT>& sh, bool write_global,
                                                const uint32_t (&qv)[kMaxGroup]) {
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int G = c.group;

#pragma unroll
  for (int i = 0; i < 4 * 256 / NT; ++i) (&sh.hist[0][0])[tid + i * NT] = 0;

  // ---- a[c] = sum_h |q|, s[c] = sum_h q (fp32, head order) -----------------------------------
  if (tid < kHeadDim) {
    float sa = 0.f, ss = 0.f;
#pragma unroll
    for (int h = 0; h < kMaxGroup; ++h) {
      const float x = h < G ? bf16_to_f32((bf16_t)qv[h]) : 0.f;
      sa += fabsf(x);
      ss += x;
    }
    sh.s_abs[tid] = sa;
    sh.s_sum[tid] = ss;
  }
  __syncthreads();
  // ---- i1: rank by counting ---------------------------------------------------------------------
  // kParts neighbouring lanes rank one channel against a slice of the channels each (4 LDS values per
  // read) and add up; ranks are unique (ties go to the lower channel), so the k1 picked channels go
  // straight to slot `rank`: no compaction, and the order of the score sums stays fixed.
  constexpr int kParts = NT / kHeadDim, kSlice = kHeadDim / kParts;
  static_assert(kParts >= 2 && kParts <= 8, "the parts of a channel are added up within eight lanes");
  {
    const int ch = tid / kParts, part = tid % kParts;
    const float mine = sh.s_abs[ch];
    const float4* v4 = reinterpret_cast<const float4*>(sh.s_abs + part * kSlice);
    int rank = 0;
#pragma unroll
    for (int i = 0; i < kSlice / 4; ++i) {
      const float4 v = v4[i];
      const int o = part * kSlice + 4 * i;
      rank += (v.x > mine) || (v.x == mine && o + 0 < ch);
      rank += (v.y > mine) || (v.y == mine && o + 1 < ch);
      rank += (v.z > mine) || (v.z == mine && o + 2 < ch);
      rank += (v.w > mine) || (v.w == mine && o + 3 < ch);
    }
    // neighbouring lanes' parts add up by lane moves: pairs, quads, then the two quads
    rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xf, 0xf, false);
    if (kParts >= 4) rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xf, 0xf, false);
    if (kParts >= 8) rank += __builtin_amdgcn_update_dpp(0, rank, 0x141, 0xf, 0xf, false);
    if (part == 0) {
      sh.s_rank[ch] = rank;
      if (rank < a.k1) {
        sh.s_chan[rank] = ch;
        sh.s_wgt[rank] = sh.s_sum[ch];
      }
    }
  }
  __syncthreads();
  // the caller's copy of i1 is ascending by channel: compacted here, only when it is asked for
  if (write_global && a.out_channels) {
    bool sel = false;
    if (tid < kHeadDim) sel = sh.s_rank[tid] < a.k1;
    const unsigned long long bal = __ballot(sel);
    if (tid == 0) sh.cnt0 = (uint32_t)__popcll(bal);
    __syncthreads();
    if (sel) {
      const int pos = __popcll(bal & ((1ull << lane) - 1ull)) + (wave == 1 ? (int)sh.cnt0 : 0);
      a.out_channels[(int64_t)unit * a.k1 + pos] = tid;
    }
  }
}

// The kp-th largest of the P order keys in `keys` (LDS) by four 8-bit radix passes, as (tau, need_eq):
// the selection is every key above tau plus the first need_eq keys equal to it.  Needs kp < P and
// `hist` (LDS, 4 x 256 counters, 16-byte aligned) zeroed; every thread gets the result.
// FIRST_DONE: the caller has already counted every key's top digit into hist[0] (and synchronised).
template <int NT, bool FIRST_DONE = false>
__device__ __forceinline__ void radix_threshold(const uint32_t* keys, int P, int kp, uint32_t (*hist)[256],
                                                uint32_t& tau, uint32_t& need_eq) {
  const int tid = threadIdx.x, lane = tid % kWave;
  uint32_t prefix = 0, mask = 0, k = (uint32_t)kp;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    if (!(FIRST_DONE && pass == 0)) {
      for (int p = tid; p < P; p += NT) {
        const uint32_t key = keys[p];
        if ((key & mask) == prefix) atomicAdd(&hist[pass][(key >> shift) & 255u], 1u);
      }
      __syncthreads();
    }
    // every wavefront finds the bucket holding the k-th largest on its own (no broadcast needed):
    // lane L owns bins 4(63-L)..4(63-L)+3, so a prefix sum over lanes counts the keys in higher bins
    const int b0 = 4 * (kWave - 1 - lane);
    const uint4 h = *reinterpret_cast<const uint4*>(&hist[pass][b0]);
    const uint32_t s3 = h.w, s2 = h.z + s3, s1 = h.y + s2, s0 = h.x + s1;  // suffix sums inside the lane
    const uint32_t above = wave_incl_scan(s0) - s0;                          // keys in bins of lower lanes
    const uint32_t in[4] = {above + s0, above + s1, above + s2, above + s3};
    const uint32_t hc[4] = {h.x, h.y, h.z, h.w};
    int found = -1;
    uint32_t newk = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t exc = in[j] - hc[j];
      if (exc < k && k <= in[j]) {
        found = b0 + j;
        newk = k - exc;
      }
    }
    const unsigned long long who = __ballot(found >= 0);
    const int src = __ffsll((long long)who) - 1;
    const uint32_t bucket = (uint32_t)__builtin_amdgcn_readlane(found, src);
    k = (uint32_t)__builtin_amdgcn_readlane((int)newk, src);
    prefix |= bucket << shift;
    mask |= 0xffu << shift;
  }
  tau = prefix;
  need_eq = k;
}

// Step 2, second half for a sequence of n tokens: page scores from the picked summary rows, exact
// top-kp pages.  `keys` is LDS scratch of ceil8(pages_cap) words.  The ascending list goes to
// `list_lds` (if not null, kp entries) and, when `write_global`, to a.out_pages / a.out_pages2 (-1
// padded) and the optional score output.  Returns kp.  Ends WITHOUT a final barrier: the caller
// synchronises before reading `list_lds`.
template <int NT>
__device__ __forceinline__ int select_pages_any(const CacheView& c, const SelectArgs& a, int unit, int n,
                                                SelectShared<NT>& sh, uint32_t* keys, int32_t* list_lds,
                                                bool write_global, const TailPatch& tp) {
  const int tid = threadIdx.x;
  const int ps = c.page_size;
  int P = (n + ps - 1) / ps;
  if (P > c.pages_cap) P = c.pages_cap;
  int kp = pages_to_pick(n, ps, a.T);
  if (kp > P) kp = P;
  if (kp > a.row_len) kp = a.row_len;
  if (write_global) {
    // -1 padding of the list rows beyond kp
    if (a.out_pages)
      for (int i = kp + tid; i < a.row_len; i += NT) a.out_pages[(int64_t)unit * a.row_len + i] = -1;
    if (a.out_pages2)
      for (int i = kp + tid; i < a.row_len2; i += NT) a.out_pages2[(int64_t)unit * a.row_len2 + i] = -1;
  }
  if (P == 0) return 0;
  const int n_rec = min(a.n_recent, kp);  // no more forced pages than pages picked: the newest ones win

  // ---- s1: page scores ---------------------------------------------------------------------------
  const int n_oct = (P + 7) / 8;
  const int64_t rows = (int64_t)unit * kHeadDim;
  float* out_scores = write_global ? a.out_scores : nullptr;
  const TailRows tail = tail_page_load<NT>(a, sh, rows, c.pages_cap, tp);
  if (n_oct < NT) {
    int npow = 1;
    while (npow < n_oct) npow <<= 1;
    const int R = NT / npow;  // row groups summed separately, then in order
    const int r = tid / npow, o = tid % npow;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    if (o < n_oct)
      for (int jb = 0; jb < a.k1; jb += 8 * R)
        score_rows8(a, sh.s_chan, sh.s_wgt, rows, c.pages_cap, o, jb + r, jb, R, acc);
    tail_page_finish<NT>(a, sh, tp, tail, R);
    RKV_STAMP(2);
#pragma unroll
    for (int i = 0; i < 8; ++i) sh.partial[(r * npow + o) * 8 + i] = acc[i];
    __syncthreads();
    for (int p = tid; p < npow * 8; p += NT) {
      const bool is_tail = p == tp.page;
      const float* part = is_tail ? sh.s_abs : sh.partial + p;
      const int step = is_tail ? 1 : npow * 8, n_part = is_tail ? min(R, kHeadDim) : R;
      float s = 0.f;
      for (int rr = 0; rr < n_part; ++rr) s += part[rr * step];
      if (p < n_oct * 8) {
        if (p < P && out_scores) out_scores[(int64_t)unit * c.pages_cap + p] = s;
        if (p >= P) s = -INFINITY;
        else if (p >= P - n_rec) s = INFINITY;
        const uint32_t key = f32_order_key(s);
        keys[p] = key;
        if (p < P) atomicAdd(&sh.hist[0][key >> 24], 1u);  // the first radix pass, counted on the way
      }
    }
  } else {
    const auto keep = [&](int p, float s) {
      if (p < P && out_scores) out_scores[(int64_t)unit * c.pages_cap + p] = s;
      if (p >= P) s = -INFINITY;
      else if (p >= P - n_rec) s = INFINITY;
      const uint32_t key = f32_order_key(s);
      keys[p] = key;
      if (p < P) atomicAdd(&sh.hist[0][key >> 24], 1u);  // the first radix pass, counted on the way
    };
    for (int o = tid; o < n_oct; o += NT) {
      float acc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = 0.f;
      for (int j0 = 0; j0 < a.k1; j0 += 8)
        score_rows8(a, sh.s_chan, sh.s_wgt, rows, c.pages_cap, o, j0, j0, 1, acc);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (o * 8 + i != tp.page) keep(o * 8 + i, acc[i]);
    }
    tail_page_finish<NT, true>(a, sh, tp, tail, 1);
    if (tp.page >= 0 && tid == NT - kWave) keep(tp.page, sh.s_abs[0]);  // the thread that left it there
  }
  __syncthreads();

  // ---- i2: exact kp-th largest key by 4 x 8-bit radix passes -------------------------------------
  RKV_STAMP(3);
  uint32_t tau = 0, need_eq = (uint32_t)P;  // defaults select everything (kp == P)
  if (kp < P) radix_threshold<NT, true>(keys, P, kp, sh.hist, tau, need_eq);
  RKV_STAMP(4);

  // ---- emit ascending: every key > tau, plus the first need_eq keys == tau -----------------------
  const int ipt = (P + NT - 1) / NT;
  const int lo = min(P, tid * ipt), hi = min(P, lo + ipt);
  uint32_t cnt = 0;  // low 16 bits: keys > tau, high 16 bits: keys == tau
  for (int p = lo; p < hi; ++p) {
    const uint32_t key = keys[p];
    cnt += (key > tau) ? 1u : 0u;
    cnt += (key == tau) ? 0x10000u : 0u;
  }
  const uint32_t before = block_excl_scan<NT, false>(cnt, sh.wsum);  // the caller's barrier follows
  uint32_t gt = before & 0xffffu, eq = before >> 16;
  for (int p = lo; p < hi; ++p) {
    const uint32_t key = keys[p];
    bool take = key > tau;
    if (key == tau) {
      take = eq < need_eq;
      ++eq;
    }
    if (take) {
      const uint32_t eq_taken = (key == tau) ? eq - 1 : min(eq, need_eq);
      const uint32_t pos = gt + eq_taken;
      if ((int)pos < kp) {
        if (list_lds) list_lds[pos] = p;
        if (write_global) {
          if (a.out_pages) a.out_pages[(int64_t)unit * a.row_len + pos] = p;
          if (a.out_pages2 && (int)pos < a.row_len2) a.out_pages2[(int64_t)unit * a.row_len2 + pos] = p;
        }
      }
    }
    if (key > tau) ++gt;
  }
  return kp;
}

// Step 2, second half, for caches of at most ROUNDS * NT pages (every fused decode launch of the usual
// shapes): the same result as select_pages_any, arranged for latency.  The routine sits in front of the
// K/V stream with HBM idle, so what counts is the number of dependent steps, not the work:
//   - eight lanes of a wavefront share an eight-page run and split the picked rows between them; the row sums meet in three
//     lane-exchange steps and a permutation, so that thread t holds the scores of pages t, NT + t, ... (one per round).
//     Eight neighbouring lanes read the same row, i.e. 128 contiguous bytes: with the lanes of a run side by side a load
//     touched eight rows per eight lanes, and the rows came in at the rate the first-level cache looks up lines.  us a
//     layer, so / now: one sequence of 16000 tokens 15.7 / 15.2, of 24000 17.3 / 16.4, of 32700 (rows of whole cache lines)
//     19.7 / 17.4, of 32768 18.8 / 17.6, 7 with 1856 pages at 68 channels 28.0 / 24.9, 16 with 1488 at 81 28.5 / 27.9; with
//     one round (16 of 4122) 22.3 / 22.3;
//   - the kp-th largest score is found by counting into 256 or 512 equal-width value bins between the
//     smallest and the largest finite score (the forced recent pages, +inf, in the top bin): one
//     histogram, scanned by every wavefront for itself.  Binning is monotone, so every page above the
//     threshold's bin is in, every page below is out, and only the few pages sharing that bin are
//     ranked exactly (by order key, ties to the lower page).  Page scores of one cache differ in
//     their mantissas, not their exponents: radix digits pile them onto a few counters (hundreds of
//     LDS atomics on one address), value bins spread them;
//   - scores without a finite range, or more than 64 pages in the threshold's bin, go through the
//     radix passes of the general routine instead.
// Ends WITHOUT a final barrier, like select_pages_any.
template <int NT, int ROUNDS>
__device__ __forceinline__ int select_pages_small(const CacheView& c, const SelectArgs& a, int unit, int n,
                                                  SelectShared<NT>& sh, uint32_t* keys, int32_t* list_lds,
                                                  bool write_global, const TailPatch& tp) {
  constexpr int kRuns = NT / 8;   // eight-page runs per round
  constexpr int kRounds = ROUNDS;
  constexpr int kWaves = NT / kWave;
  constexpr int kCandMax = 64;
  const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int ps = c.page_size;
  int P = (n + ps - 1) / ps;
  if (P > c.pages_cap) P = c.pages_cap;
  int kp = pages_to_pick(n, ps, a.T);
  if (kp > P) kp = P;
  if (kp > a.row_len) kp = a.row_len;
  if (write_global) {
    if (a.out_pages)
      for (int i = kp + tid; i < a.row_len; i += NT) a.out_pages[(int64_t)unit * a.row_len + i] = -1;
    if (a.out_pages2)
      for (int i = kp + tid; i < a.row_len2; i += NT) a.out_pages2[(int64_t)unit * a.row_len2 + i] = -1;
  }
  if (P == 0) return 0;
  const int n_rec = min(a.n_recent, kp);  // no more forced pages than pages picked: the newest ones win
  const int n_oct = (P + 7) / 8;
  const int64_t rows = (int64_t)unit * kHeadDim;
  const int o = wave * 8 + lane % 8, r = lane / 8;  // this lane's run of a round, and its rows
  // the wavefront's first run of a round: a wavefront without any skips the round's arithmetic (a scalar branch)
  const int o_wave = __builtin_amdgcn_readfirstlane(tid / kWave) * (kWave / 8);
  // scratch words in sh.partial (unused by the channel pick): candidate keys, their counter, the
  // wavefronts' score ranges and emission counts
  uint32_t* scr = reinterpret_cast<uint32_t*>(sh.partial);
  uint32_t* cand = scr;                             // [kCandMax]
  uint32_t* cand_n = scr + kCandMax;                // [1]
  uint32_t* wlo = scr + kCandMax + 8;               // [kWaves]
  uint32_t* whi = wlo + kWaves;                     // [kWaves]
  uint32_t* wcnt = whi + kWaves;                    // [kRounds][kWaves]

  // The page that is receiving a token is always the sequence's last.  What the rows hold for it is stale: the last
  // wavefront, which has the fewest pages of its own, sums its score up from the page's old bounds folded with the
  // new key, or from the new key alone when the token opens the page (what memory holds for that column is then not
  // looked at), and the workgroup's last thread takes the page in its last round: still the last page in (round,
  // thread) order.  The sum is formed like every other page's, rows r, r + 8, ... by lane r and then the eight
  // lanes, so that it equals what a later launch makes of the stored bounds, to the bit: pages that tie then are
  // ranked alike.  The old bounds travel with the rows.
  const bool tail_wave = tp.page >= 0 && o_wave == (kWaves - 1) * (kWave / 8);
  const bool has_tail = tp.page >= 0 && tid == NT - 1;
  // Lane l fetches rows l and 64 + l; rows beyond k1 count as below.  (The weight is read and then dropped: read
  // under the condition, it has the compiler fetch the base pointer per lane from the kernel arguments, a round
  // trip: 0.4 us a layer.)
  const auto tail_row = [&](int j, float& w) {
    const int jj = min(j, a.k1 - 1);
    w = sh.s_wgt[jj];
    if (j >= a.k1) w = 0.f;
    return sh.s_chan[jj];
  };
  const int tail_rows = (a.k1 + 7) / 8 * 8;
  uint32_t tail_old[2] = {0u, 0u};
  if (tail_wave && tp.slot != 0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = h * kWave + lane;
      float w;
      if (j < tail_rows) {
        const int ch = tail_row(j, w);
        tail_old[h] = (w >= 0.f ? a.kmax : a.kmin)[(rows + ch) * c.pages_cap + tp.page];
      }
    }
  }
  // ---- s1: page scores.  Lane (o, r) takes the rows r, r + 8, ... of the picked
  // channels for the runs o, o + kRuns, ... (one per round); the loads of every round go out before the
  // first is used, so the rounds share one memory round trip.
  float score[kRounds];
  const auto plus_ror8 = [](float keep, float give) {  // `give` of the lane eight away in its row of sixteen
    return keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xf, 0xf, true));
  };
  {
    constexpr int kBatch = 4;  // rows of a thread whose loads are in flight together, for every round (registers)
    float acc[kRounds][8];
#pragma unroll
    for (int i = 0; i < kRounds; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;
    for (int jb = 0; jb < a.k1; jb += 8 * kBatch) {
      float w[kBatch];
      int ch[kBatch];
#pragma unroll
      for (int t = 0; t < kBatch; ++t) {
        const int j = jb + r + t * 8;
        const int jj = j < a.k1 ? j : a.k1 - 1;  // a row beyond k1: the last picked row again, weight zero
        ch[t] = sh.s_chan[jj];
        w[t] = sh.s_wgt[jj];
        if (j >= a.k1) w[t] = 0.f;
      }
      const bf16_t* row[kBatch];
#pragma unroll
      for (int t = 0; t < kBatch; ++t) row[t] = (w[t] >= 0.f ? a.kmax : a.kmin) + (rows + ch[t]) * c.pages_cap + o * 8;
      uint4 v[kRounds][kBatch];
#pragma unroll
      for (int i = 0; i < kRounds; ++i)
#pragma unroll
        for (int t = 0; t < kBatch; ++t) {
          v[i][t] = make_uint4(0, 0, 0, 0);
          // (the first two conditions are the same for the whole workgroup)
          if (i * kRuns < n_oct && jb + t * 8 < a.k1 && i * kRuns + o < n_oct) v[i][t] = ld16<false>(row[t] + i * NT);
        }
#pragma unroll
      for (int i = 0; i < kRounds; ++i) {
        if (i * kRuns + o_wave >= n_oct) continue;
#pragma unroll
        for (int t = 0; t < kBatch; ++t) {
          const uint32_t x[4] = {v[i][t].x, v[i][t].y, v[i][t].z, v[i][t].w};
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            acc[i][2 * q4] = fmaf(w[t], bf16lo_to_f32(x[q4]), acc[i][2 * q4]);
            acc[i][2 * q4 + 1] = fmaf(w[t], bf16hi_to_f32(x[q4]), acc[i][2 * q4 + 1]);
          }
        }
      }
    }
    // The eight lanes of a run add up their row groups: r and r + 4, then r and r + 2, then r and r + 1, each step leaving a
    // lane with half of its pages; lane (r, o) ends with page r of its run, and passes it to the lane whose own page it is.
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
      score[i] = 0.f;
      if (i * kRuns + o_wave < n_oct) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][e]), __float_as_uint(acc[i][e + 4]), false, false);
          x[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[e]), __float_as_uint(x[e + 2]), false, false);
          x[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
        const bool up = (lane & 8) != 0;
        score[i] = __shfl(plus_ror8(up ? x[1] : x[0], up ? x[0] : x[1]), lane % 8 * 8 + lane / 8);
      }
    }
    if (tail_wave) {
      float sum = 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h * kWave >= a.k1) break;  // (the same for the whole launch, as the next one)
        const int j = h * kWave + lane;
        float w = 0.f, f = 0.f;
        if (j < tail_rows) {
          f = bf16_to_f32(tp.knew[tail_row(j, w)]);
          if (tp.slot != 0) {
            const float fo = bf16_to_f32((bf16_t)use_late(tail_old[h]));
            f = w >= 0.f ? fmaxf(fo, f) : fminf(fo, f);
          }
        }
#pragma unroll
        for (int t0 = 0; t0 < 8; t0 += 4) {
          if (h * kWave + t0 * 8 >= a.k1) break;
          float wt[4], ft[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            wt[t] = __shfl(w, r + (t0 + t) * 8);
            ft[t] = __shfl(f, r + (t0 + t) * 8);
          }
#pragma unroll
          for (int t = 0; t < 4; ++t) sum = fmaf(wt[t], ft[t], sum);
        }
      }
      SwapPair sw = swap_rows32(__float_as_uint(sum));
      sum = __uint_as_float(sw.a) + __uint_as_float(sw.b);
      sw = swap_rows16(__float_as_uint(sum));
      sum = __uint_as_float(sw.a) + __uint_as_float(sw.b);
      sum = plus_ror8(sum, sum);
      if (has_tail) score[kRounds - 1] = sum;
    }
  }
  // the page of round i, and whether it is this thread's
  const auto page_of = [&](int i) { return has_tail && i == kRounds - 1 ? tp.page : i * NT + tid; };
  const auto owns = [&](int i) { return page_of(i) < P && (page_of(i) != tp.page || (has_tail && i == kRounds - 1)); };
  RKV_STAMP(2);

  // ---- order keys, and the range of the finite scores ---------------------------------------------
  float* out_scores = write_global ? a.out_scores : nullptr;
  uint32_t key[kRounds];
  float val[kRounds];
  bool live[kRounds];
  uint32_t klo = 0xffffffffu, khi = 0u;  // the range of the finite scores, as order keys
#pragma unroll
  for (int i = 0; i < kRounds; ++i) {
    const int p = page_of(i);
    live[i] = owns(i);
    float sc = score[i];
    if (live[i] && out_scores) out_scores[(int64_t)unit * c.pages_cap + p] = sc;
    if (live[i] && p >= P - n_rec) sc = INFINITY;
    val[i] = sc;
    key[i] = live[i] ? f32_order_key(sc) : 0u;
    if (live[i] && fabsf(sc) < INFINITY) {
      klo = min(klo, key[i]);
      khi = max(khi, key[i]);
    }
  }
  uint32_t tau = 0, need_eq = (uint32_t)P;  // defaults select everything (kp == P)
  bool by_bin = false;                     // picked by bin alone: every page of the threshold's bin is in
  int bstar = 0;
  int bin[kRounds];
#pragma unroll
  for (int i = 0; i < kRounds; ++i) bin[i] = 0;
  if (kp < P) {
    klo = wave_min_u32(klo);
    khi = wave_max_u32(khi);
    if (lane == 0) {
      wlo[wave] = klo;
      whi[wave] = khi;
    }
    if (tid == 0) *cand_n = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; w += 4) {
      const uint4 l = *reinterpret_cast<const uint4*>(wlo + w), h = *reinterpret_cast<const uint4*>(whi + w);
      klo = min(min(min(klo, l.x), min(l.y, l.z)), l.w);
      khi = max(max(max(khi, h.x), max(h.y, h.z)), h.w);
    }
    const float lo = f32_from_order_key(klo), hi = f32_from_order_key(khi);  // (no finite score: lo is a NaN)
    // bins, and bins per lane of a scanning wavefront.  Every wavefront walks its lanes' bins one after the other,
    // so fewer bins make a shorter scan and more pages per bin a longer exact rank; with at most two pages per
    // thread 256 bins measured 0.4 us ahead of 1024 at the benchmark shape, with five (one sequence of 32768
    // tokens) 512 are 0.4 us ahead of 1024.
    constexpr int NB = ROUNDS <= 2 ? 256 : 512, BPL = NB / kWave;
    // (any positive factor makes monotone bins, so the hardware's reciprocal will do)
    const float scale = (float)(NB - 2) * __builtin_amdgcn_rcpf(hi - lo);
    bool decided = (hi > lo) && (scale < 3.0e38f);  // the same for every thread
    if (decided) {
      uint32_t* hist = &sh.hist[0][0];  // 4 x 256 counters, all zero
#pragma unroll
      for (int i = 0; i < kRounds; ++i) {
        // clamped as a float, so that -inf, +inf and NaN never reach the conversion
        int b = (int)fminf(fmaxf((val[i] - lo) * scale, 0.f), (float)(NB - 2));
        if (val[i] == INFINITY) b = NB - 1;
        bin[i] = b;
        if (live[i]) atomicAdd(&hist[b], 1u);
      }
      __syncthreads();
      // every wavefront finds the bin of the kp-th largest for itself: lane L owns the BPL bins below
      // NB - L * BPL, so a prefix sum over the lanes counts the pages in higher bins
      const int btop = NB - 1 - lane * BPL;  // the lane's highest bin
      uint32_t hc[BPL], total = 0;
#pragma unroll
      for (int v = 0; v < BPL / 4; ++v) {
        const uint4 h = *reinterpret_cast<const uint4*>(&hist[btop - 4 * v - 3]);
        hc[4 * v + 0] = h.w;
        hc[4 * v + 1] = h.z;
        hc[4 * v + 2] = h.y;
        hc[4 * v + 3] = h.x;
        total += h.x + h.y + h.z + h.w;
      }
      uint32_t above = wave_incl_scan(total) - total;
      int found = -1;
      uint32_t need = 0, cnum = 0;
#pragma unroll
      for (int j = 0; j < BPL; ++j) {  // j = 0: the lane's highest bin
        if (above < (uint32_t)kp && (uint32_t)kp <= above + hc[j]) {
          found = btop - j;
          need = (uint32_t)kp - above;
          cnum = hc[j];
        }
        above += hc[j];
      }
      const int src = __ffsll((long long)__ballot(found >= 0)) - 1;
      bstar = __builtin_amdgcn_readlane(found, src);
      need = (uint32_t)__builtin_amdgcn_readlane((int)need, src);
      cnum = (uint32_t)__builtin_amdgcn_readlane((int)cnum, src);
      if (cnum == need) {
        by_bin = true;
      } else if (cnum <= (uint32_t)kCandMax) {
        // exact rank among the pages of the threshold's bin
#pragma unroll
        for (int i = 0; i < kRounds; ++i)
          if (live[i] && bin[i] == bstar) cand[atomicAdd(cand_n, 1u)] = key[i];
        __syncthreads();
        const uint32_t ki = lane < (int)cnum ? cand[lane] : 0u;
        uint32_t gt = 0, ge = 0;
        for (uint32_t j = 0; j < cnum; ++j) {
          const uint32_t kj = cand[j];
          gt += kj > ki;
          ge += kj >= ki;
        }
        const bool is_tau = lane < (int)cnum && gt < need && need <= ge;  // equal keys give the same pair
        const int who = __ffsll((long long)__ballot(is_tau)) - 1;
        tau = (uint32_t)__builtin_amdgcn_readlane((int)ki, who);
        need_eq = need - (uint32_t)__builtin_amdgcn_readlane((int)gt, who);
      } else {
        decided = false;
      }
    }
    if (!decided) {
      // the general routine's radix passes, on the keys in LDS
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kRounds; ++i)
        if (live[i]) keys[page_of(i)] = key[i];
      for (int i = tid; i < 4 * 256; i += NT) (&sh.hist[0][0])[i] = 0;
      __syncthreads();
      radix_threshold<NT, false>(keys, P, kp, sh.hist, tau, need_eq);
      bstar = -1;  // every live page is ranked by its key
    }
  }
  RKV_STAMP(3);

  // ---- emit ascending.  Page order is (round, thread) order: a prefix sum over the threads per round.
  // In: every page above the threshold (by bin, then by key), plus the first need_eq pages equal to it.
  bool above_t[kRounds], equal_t[kRounds];
  unsigned long long m_above[kRounds], m_equal[kRounds];
#pragma unroll
  for (int i = 0; i < kRounds; ++i) {
    if (kp >= P) {
      above_t[i] = false;
      equal_t[i] = live[i];  // key == tau is not needed: need_eq == P takes every live page
    } else if (by_bin) {
      above_t[i] = live[i] && bin[i] >= bstar;
      equal_t[i] = false;
    } else if (bstar >= 0) {
      above_t[i] = live[i] && (bin[i] > bstar || (bin[i] == bstar && key[i] > tau));
      equal_t[i] = live[i] && bin[i] == bstar && key[i] == tau;
    } else {
      above_t[i] = live[i] && key[i] > tau;
      equal_t[i] = live[i] && key[i] == tau;
    }
    m_above[i] = __ballot(above_t[i]);
    m_equal[i] = __ballot(equal_t[i]);
    // low 16 bits: pages above the threshold, high 16 bits: pages equal to it
    if (lane == 0) wcnt[i * kWaves + wave] = (uint32_t)__popcll(m_above[i]) + ((uint32_t)__popcll(m_equal[i]) << 16);
  }
  if (by_bin) need_eq = 0;
  __syncthreads();
  // what lies in front of each wavefront's pages of each round: one prefix sum over the counts, (round, wave) order
  // (every thread adding up the counts it has before it cost 0.2-0.3 of 19.5 us a layer with five rounds)
  static_assert(kRounds * kWaves <= kWave, "a lane per count");
  const uint32_t counts = wave_incl_scan(lane < kRounds * kWaves ? wcnt[lane] : 0u);
#pragma unroll
  for (int i = 0; i < kRounds; ++i) {
    const int at = i * kWaves + wave;
    const uint32_t before = at > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)counts, at - 1) : 0u;
    const uint32_t gt = (before & 0xffffu) + (uint32_t)bits_below(m_above[i]);
    const uint32_t eq = (before >> 16) + (uint32_t)bits_below(m_equal[i]);
    const bool take = above_t[i] || (equal_t[i] && eq < need_eq);
    if (take) {
      const uint32_t pos = gt + (equal_t[i] ? eq : min(eq, need_eq));
      const int p = page_of(i);
      if ((int)pos < kp) {
        if (list_lds) list_lds[pos] = p;
        if (write_global) {
          if (a.out_pages) a.out_pages[(int64_t)unit * a.row_len + pos] = p;
          if (a.out_pages2 && (int)pos < a.row_len2) a.out_pages2[(int64_t)unit * a.row_len2 + pos] = p;
        }
      }
    }
  }
  RKV_STAMP(4);
  return kp;
}

// Step 2, second half, with the form chosen by the cache's capacity: ROUNDS of select_rounds().  The fused kernels have
// it as a template parameter and are instantiated per form.  us a layer, forms 1 to 6 behind branches in one kernel / a kernel
// per form, the step with a token taken in: one sequence of 4096 tokens (one round) 14.2 / 13.4, of 16000 (two) 15.8 / 14.9, of
// 24000 (three) 16.9 / 16.1, of 32700 (four) 18.0 / 17.1, of 40000 (five) 19.2 / 18.2, four of 24000 18.5 / 17.5, 8 of 4122 at a
// budget of 256 13.7 / 13.0; without the token one of 24000 14.2 / 13.8.  That is where half of the output channels are a
// workgroup's share; with all of them the two are the same within 1 % (8 of 4122 16.7 / 16.6, 16 22.0 / 22.1, with all eight
// forms behind branches 64 of 4122 56.6 / 56.4, 40 of 8000 51.7 / 51.8, 13 unequal ones 20.9 / 20.7).  It is not the registers,
// which are as many in both (171; 215 with forms 7 and 8 beside the others, at the same times).
// Six to eight rounds against select_pages_any: one sequence of 42000 tokens 24.6 / 20.1, of 50000 25.4 / 21.0, of 64000
// 27.5 / 22.2, 13 of 50000 35.0 / 30.8, 40 of 25000 (256 threads) 60.0 / 55.8.  A thread's counts leave a lane each for at
// most eight rounds of eight wavefronts.
__host__ __device__ constexpr int select_rounds(int pages_cap, int nt) {
  return pages_cap <= 8 * nt ? (pages_cap + nt - 1) / nt : 0;
}

template <int NT, int ROUNDS>
__device__ __forceinline__ int select_pages(const CacheView& c, const SelectArgs& a, int unit, int n,
                                            SelectShared<NT>& sh, uint32_t* keys, int32_t* list_lds,
                                            bool write_global, const TailPatch& tp) {
  if constexpr (ROUNDS == 0) return select_pages_any<NT>(c, a, unit, n, sh, keys, list_lds, write_global, tp);
  else return select_pages_small<NT, ROUNDS>(c, a, unit, n, sh, keys, list_lds, write_global, tp);
}

// A kernel instance per form: runs fn(std::integral_constant<int, ROUNDS>) with the form of this capacity.
template <class Fn>
inline void with_select_rounds(int pages_cap, int nt, const Fn& fn) {
  switch (select_rounds(pages_cap, nt)) {
    case 1: fn(std::integral_constant<int, 1>{}); break;
    case 2: fn(std::integral_constant<int, 2>{}); break;
    case 3: fn(std::integral_constant<int, 3>{}); break;
    case 4: fn(std::integral_constant<int, 4>{}); break;
    case 5: fn(std::integral_constant<int, 5>{}); break;
    case 6: fn(std::integral_constant<int, 6>{}); break;
    case 7: fn(std::integral_constant<int, 7>{}); break;
    case 8: fn(std::integral_constant<int, 8>{}); break;
    default: fn(std::integral_constant<int, 0>{});
  }
}

// Step 2's top-k (Algorithm 1, i2) on page scores that an earlier launch left in a.in_scores: the
// pick of the large-summary path.  A thread keeps its contiguous run of a few scores in registers
// from the one batch of loads to the ordered emission, so no pass waits on LDS reads.
//
// The kp-th largest score is found by counting, not by radix digits: one pass over 1023 equal-width
// value bins between the smallest and the largest finite score (+inf, the forced recent pages, has a
// bin of its own), a scan over the bins, then an exact rank among the few scores that share the bin
// of the kp-th.  Page scores differ in their low mantissa bits rather than in their exponents, so
// value bins spread them where the leading radix digits would pile them into one or two counters.
// Binning is monotone, hence the result is exactly the radix select's, ties to the lower page
// included.  Scores without a finite range, or more than 1024 of them in that one bin, fall back to
// radix passes over the same registers.  Up to ROCKETKV_MAX_PAGES pages.
template <int NT>
struct PickShared {
  __align__(16) uint32_t hist[4][256];  // 1024 value bins, or the four radix histograms of the fallback
  uint32_t cand[1024];
  uint32_t wmin[NT / kWave], wmax[NT / kWave];
  uint32_t wsum[NT / kWave];
  int found[6];
  uint32_t cnt0;
};

// COHERENT: the scores were written earlier in the SAME launch by other workgroups (with device-scope
// write-through stores): they are read with device-scope loads, which do not trust this XCD's L2.
// kVec: float4 loads per thread, i.e. NT * kVec * 4 >= pages_cap (the wrapper below picks it).
// sh.hist must be all zero on entry (the caller clears it, and synchronises, before the call).
template <int NT, bool COHERENT, int kVec>
__device__ __forceinline__ void pick_from_scores_n(const CacheView& c, const SelectArgs& a, int unit, int n,
                                                   PickShared<NT>& sh) {
  constexpr int NB = 1024, BPT = NB / NT, CAP = 1024;
  static_assert(kVec >= 1 && NB % NT == 0, "thread count does not fit the pick");
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  // ---- this thread's run of pages, [4 * v_begin, 4 * v_begin + 4 * per), laid out on pages_cap so
  // that the loads go out before the sequence length is known ---------------------------------------
  const int per = (c.pages_cap / 4 + NT - 1) / NT;  // rows hold pages_cap (a multiple of 8) floats
  const int v_begin = tid * per;
  const float4* in4 = reinterpret_cast<const float4*>(a.in_scores + (int64_t)unit * c.pages_cap);
  float4 v[kVec];
#pragma unroll
  for (int i = 0; i < kVec; ++i) {
    v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < per && (v_begin + i) * 4 < c.pages_cap) {
      if (COHERENT) {
        const float* f = reinterpret_cast<const float*>(in4 + v_begin + i);
        v[i] = make_float4(__hip_atomic_load(f + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                           __hip_atomic_load(f + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                           __hip_atomic_load(f + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                           __hip_atomic_load(f + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      } else {
        v[i] = in4[v_begin + i];
      }
    }
  }
  const int ps = c.page_size;
  int P = (n + ps - 1) / ps;
  if (P > c.pages_cap) P = c.pages_cap;
  int kp = pages_to_pick(n, ps, a.T);
  if (kp > P) kp = P;
  if (kp > a.row_len) kp = a.row_len;
  if (a.out_pages)
    for (int i = kp + tid; i < a.row_len; i += NT) a.out_pages[(int64_t)unit * a.row_len + i] = -1;
  if (a.out_pages2)
    for (int i = kp + tid; i < a.row_len2; i += NT) a.out_pages2[(int64_t)unit * a.row_len2 + i] = -1;
  if (P == 0) return;
  const int n_rec = min(a.n_recent, kp);  // no more forced pages than pages picked: the newest ones win
  uint32_t key[kVec * 4];
  uint32_t klo = 0xffffffffu, khi = 0u;  // the range of the finite scores, as order keys
#pragma unroll
  for (int i = 0; i < kVec; ++i) {
    const float x[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int pg = (v_begin + i) * 4 + e;
      const bool live = i < per && pg < P;
      float sc = live ? x[e] : -INFINITY;
      if (live && pg >= P - n_rec) sc = INFINITY;
      key[i * 4 + e] = f32_order_key(sc);
      if (live) {
        if (fabsf(sc) < INFINITY) {
          klo = min(klo, key[i * 4 + e]);
          khi = max(khi, key[i * 4 + e]);
        }
      }
    }
  }
  // `live` again, as a test on the register index alone
  const auto is_live = [&](int r) { return r / 4 < per && (v_begin + r / 4) * 4 + (r & 3) < P; };

  uint32_t tau = 0, need_eq = (uint32_t)P;  // defaults select everything (kp == P)
  if (kp < P) {
    uint32_t* hist = &sh.hist[0][0];
    uint32_t* cand = sh.cand;
    klo = wave_min_u32(klo);
    khi = wave_max_u32(khi);
    if (lane == 0) {
      sh.wmin[wave] = klo;
      sh.wmax[wave] = khi;
    }
    if (tid == 0) sh.cnt0 = 0;
    __syncthreads();
    constexpr int kWaves = NT / kWave;
    klo = wave_min_u32(lane < kWaves ? sh.wmin[lane] : 0xffffffffu);
    khi = wave_max_u32(lane < kWaves ? sh.wmax[lane] : 0u);
    const float lo = f32_from_order_key(klo), hi = f32_from_order_key(khi);  // (no finite score: lo is a NaN)
    // (any positive factor makes monotone bins, so the hardware's reciprocal will do)
    const float scale = (float)(NB - 1) * __builtin_amdgcn_rcpf(hi - lo);
    bool decided = (hi > lo) && (scale < 3.0e38f);  // same for every thread
    if (decided) {
      const auto bin_of = [&](uint32_t k) -> int {
        const float f = f32_from_order_key(k);
        if (f == INFINITY) return NB - 1;
        const int b = (int)((f - lo) * scale);
        return min(max(b, 0), NB - 2);
      };
      int bin[kVec * 4];
#pragma unroll
      for (int r = 0; r < kVec * 4; ++r) {
        bin[r] = bin_of(key[r]);
        if (is_live(r)) atomicAdd(&hist[bin[r]], 1u);
      }
      __syncthreads();
      // thread t owns the BPT bins below NB - t*BPT: a prefix sum over threads counts the bins above
      uint32_t h[BPT], total = 0;
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        h[j] = hist[NB - 1 - tid * BPT - j];  // j = 0: the thread's highest bin
        total += h[j];
      }
      uint32_t above = block_excl_scan<NT>(total, sh.wsum);
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        if (above < (uint32_t)kp && (uint32_t)kp <= above + h[j]) {
          sh.found[0] = NB - 1 - tid * BPT - j;
          sh.found[1] = (int)((uint32_t)kp - above);
          sh.found[2] = (int)h[j];
        }
        above += h[j];
      }
      __syncthreads();
      const int bstar = sh.found[0], need = sh.found[1], cnum = sh.found[2];
      decided = cnum <= CAP;
      if (decided) {
#pragma unroll
        for (int r = 0; r < kVec * 4; ++r)
          if (is_live(r) && bin[r] == bstar) cand[atomicAdd(&sh.cnt0, 1u)] = key[r];
        __syncthreads();
        for (int i = tid; i < cnum; i += NT) {
          const uint32_t ki = cand[i];
          int gt = 0, ge = 0;
          for (int j = 0; j < cnum; ++j) {
            const uint32_t kj = cand[j];
            gt += kj > ki;
            ge += kj >= ki;
          }
          if (gt < need && need <= ge) {  // ki is the need-th largest; equal keys write the same pair
            sh.found[4] = (int)ki;
            sh.found[5] = need - gt;
          }
        }
        __syncthreads();
        tau = (uint32_t)sh.found[4];
        need_eq = (uint32_t)sh.found[5];
      }
    }
    if (!decided) {
      // four 8-bit radix passes over the keys in registers (same scan as radix_threshold)
      __syncthreads();
      for (int i = tid; i < 4 * 256; i += NT) hist[i] = 0;
      __syncthreads();
      uint32_t prefix = 0, mask = 0, k = (uint32_t)kp;
      for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
#pragma unroll
        for (int r = 0; r < kVec * 4; ++r) {
          const bool on = is_live(r) && (key[r] & mask) == prefix;
          const uint32_t digit = (key[r] >> shift) & 255u;
          if (on) atomicAdd(&sh.hist[pass][digit], 1u);
        }
        __syncthreads();
        const int b0 = 4 * (kWave - 1 - lane);
        const uint4 h = *reinterpret_cast<const uint4*>(&sh.hist[pass][b0]);
        const uint32_t s3 = h.w, s2 = h.z + s3, s1 = h.y + s2, s0 = h.x + s1;
        const uint32_t above = wave_incl_scan(s0) - s0;
        const uint32_t in[4] = {above + s0, above + s1, above + s2, above + s3};
        const uint32_t hc[4] = {h.x, h.y, h.z, h.w};
        int found = -1;
        uint32_t newk = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t exc = in[j] - hc[j];
          if (exc < k && k <= in[j]) {
            found = b0 + j;
            newk = k - exc;
          }
        }
        const unsigned long long who = __ballot(found >= 0);
        const int src = __ffsll((long long)who) - 1;
        const uint32_t bucket = (uint32_t)__builtin_amdgcn_readlane(found, src);
        k = (uint32_t)__builtin_amdgcn_readlane((int)newk, src);
        prefix |= bucket << shift;
        mask |= 0xffu << shift;
      }
      tau = prefix;
      need_eq = k;
      __syncthreads();
    }
  }

  // ---- emit ascending: every key > tau, plus the first need_eq keys == tau -----------------------
  uint32_t cnt = 0;  // low 16 bits: keys > tau, high 16 bits: keys == tau
#pragma unroll
  for (int r = 0; r < kVec * 4; ++r) {
    if (is_live(r)) {
      cnt += (key[r] > tau) ? 1u : 0u;
      cnt += (key[r] == tau) ? 0x10000u : 0u;
    }
  }
  const uint32_t before = block_excl_scan<NT>(cnt, sh.wsum);
  uint32_t gt = before & 0xffffu, eq = before >> 16;
#pragma unroll
  for (int r = 0; r < kVec * 4; ++r) {
    if (is_live(r)) {
      const int pg = (v_begin + r / 4) * 4 + (r & 3);
      bool take = key[r] > tau;
      if (key[r] == tau) {
        take = eq < need_eq;
        ++eq;
      }
      if (take) {
        const uint32_t eq_taken = (key[r] == tau) ? eq - 1 : min(eq, need_eq);
        const uint32_t pos = gt + eq_taken;
        if ((int)pos < kp) {
          if (a.out_pages) a.out_pages[(int64_t)unit * a.row_len + pos] = pg;
          if (a.out_pages2 && (int)pos < a.row_len2) a.out_pages2[(int64_t)unit * a.row_len2 + pos] = pg;
        }
      }
      if (key[r] > tau) ++gt;
    }
  }
}

// The pick with the per-thread run sized to the cache (instruction count follows the unrolled run
// length, so a short cache must not pay for the longest one).
template <int NT, bool COHERENT = false>
__device__ __forceinline__ void pick_from_scores(const CacheView& c, const SelectArgs& a, int unit, int n,
                                                 PickShared<NT>& sh) {
  constexpr int kMaxVec = ROCKETKV_MAX_PAGES / 4 / NT;
  static_assert(kMaxVec >= 1, "thread count does not fit the pick");
  const int per = (c.pages_cap / 4 + NT - 1) / NT;  // same for every thread
  if (per <= 1) pick_from_scores_n<NT, COHERENT, 1>(c, a, unit, n, sh);
  else if (per <= 2 || kMaxVec < 4) pick_from_scores_n<NT, COHERENT, (kMaxVec < 2 ? kMaxVec : 2)>(c, a, unit, n, sh);
  else if (per <= 4 || kMaxVec < 8) pick_from_scores_n<NT, COHERENT, (kMaxVec < 4 ? kMaxVec : 4)>(c, a, unit, n, sh);
  else pick_from_scores_n<NT, COHERENT, kMaxVec>(c, a, unit, n, sh);
}

// Page scores of the eight-page runs [o_begin, o_begin + n_runs) of one unit, n_runs <= NT, written as
// raw fp32 sums to `scores_row[page]` for page < P.  For summaries too large for one workgroup to
// stream at a useful rate: several workgroups take a slice each (every one repeats the cheap channel
// pick), and the top-k runs afterwards on the scores.  Needs sh.s_chan / sh.s_wgt; ends with a barrier.
template <int NT, bool COHERENT = false>
__device__ __forceinline__ void score_chunk(const CacheView& c, const SelectArgs& a, int unit, int P,
                                            SelectShared<NT>& sh, int o_begin, int n_runs,
                                            float* scores_row, const TailPatch& tp) {
  const int tid = threadIdx.x;
  const int64_t rows = (int64_t)unit * kHeadDim;
  int npow = 1;
  while (npow < n_runs) npow <<= 1;
  const int R = NT / npow;  // row groups summed separately, then in order
  const int r = tid / npow, o = tid % npow;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  // the page that is receiving a token, if it lies in this slice: scored on its own (see tail_page_load)
  const int tail_local = tp.page >= 0 ? tp.page - o_begin * 8 : -1;
  const bool owns_tail = tail_local >= 0 && tail_local < n_runs * 8;  // same for the whole workgroup
  TailPatch mine = tp;
  if (!owns_tail) mine.page = -1;
  const TailRows tail = tail_page_load<NT>(a, sh, rows, c.pages_cap, mine);
  if (o < n_runs)
    for (int jb = 0; jb < a.k1; jb += 8 * R)  // each slice of the rows has this one reader: streamed
      score_rows8<true>(a, sh.s_chan, sh.s_wgt, rows, c.pages_cap, o_begin + o, jb + r, jb, R, acc);
  tail_page_finish<NT>(a, sh, mine, tail, R);
#pragma unroll
  for (int i = 0; i < 8; ++i) sh.partial[(r * npow + o) * 8 + i] = acc[i];
  __syncthreads();
  for (int p = tid; p < n_runs * 8; p += NT) {
    const bool is_tail = owns_tail && p == tail_local;
    const float* part = is_tail ? sh.s_abs : sh.partial + p;
    const int step = is_tail ? 1 : npow * 8, n_part = is_tail ? min(R, kHeadDim) : R;
    float s = 0.f;
    for (int rr = 0; rr < n_part; ++rr) s += part[rr * step];
    const int page = o_begin * 8 + p;
    if (page < P) {
      if (COHERENT)  // read back by another workgroup of this launch: write through, device scope
        __hip_atomic_store(&scores_row[page], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        scores_row[page] = s;
    }
  }
  if (COHERENT) drain_stores();  // the scores are acknowledged before the barrier that the caller's report follows
  __syncthreads();
}

// Both halves back to back, the list to global memory.
template <int NT>
__device__ __forceinline__ void select_block(const CacheView& c, const SelectArgs& a, int unit, int n,
                                             SelectShared<NT>& sh, uint32_t* keys) {
  const TailPatch none = {-1, 0, nullptr, nullptr};
  uint32_t qv[kMaxGroup];
  load_q_column(c, a, unit, qv);
  select_channels<NT>(c, a, unit, sh, true, qv);
  // (the same for the whole launch)  One kernel for every capacity, in which the forms of three, four and six to eight rounds
  // have not been built.  What they would give, us a launch of 256 threads a unit, so / with them: one sequence of 9000 tokens
  // (three rounds) 7.8 / 6.9, of 16000 (four) 8.1 / 7.7, of 21000 (six) 13.1 / 9.1, of 32000 (eight) 14.9 / 10.7, sixteen of
  // 32000 17.7 / 14.0, 64 of 16000 15.6 / 14.9, at 216 registers instead of 142.
  switch (select_rounds(c.pages_cap, NT)) {
    case 1: select_pages<NT, 1>(c, a, unit, n, sh, keys, nullptr, true, none); break;
    case 2: select_pages<NT, 2>(c, a, unit, n, sh, keys, nullptr, true, none); break;
    case 3:
    case 4:
    case 5: select_pages<NT, 5>(c, a, unit, n, sh, keys, nullptr, true, none); break;
    default: select_pages<NT, 0>(c, a, unit, n, sh, keys, nullptr, true, none);
  }
}

}  // namespace rkv
