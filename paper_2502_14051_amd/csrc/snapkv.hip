// Stage 1 of RocketKV (Section 3.3 of arXiv 2502.14051; window / kernel sizes from Appendix A.3):
// GQA-aware SnapKV.  Per (sequence, KV head):
//   pass 1  row statistics (max, sum-exp) of the causal softmax of every (head, window row) over the
//           whole prompt, split along the key axis, then merged (by a launch or in pass 2);
//   pass 2  probabilities recomputed from the statistics and summed over heads and window rows into
//           one vote per prefix token;
//   pool    stride-1 max-pool of the votes (odd kernel, clipped at the ends), written as votes and as
//           runs of equal votes;
//   select  exact top-(N-W) of the pooled votes from the runs, ties to the lower position, emitted
//           ascending, followed by the W window positions;
//   gather  K rows and V columns of the kept tokens copied into the destination cache.
// The two score passes are the one dense contraction of the method (G*W query rows against every
// key): they run on the matrix cores with the (head, window-row) index as the MFMA column, so a lane
// owns a fixed set of softmax rows and their statistics stay in registers.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "select_core.h"
#include "vote_bins.h"

namespace rkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kLog2eS = 1.4426950408889634f;
constexpr float kNegBigS = -1.0e30f;

constexpr int kCountStride = 64;  // uint32 between the run counters of two units

struct SnapArgs {
  const bf16_t* qobs;
  int W, NC, CG, n_chunks, chunk_pages, keep, s_cap, pool_r;
  float* stats_part;  // [units][n_chunks][NC][2], where pooled, kept and runs are written later
  float* stats;       // [units][NC][2]   (max in log2 domain, 1/sum)
  float* votes;       // [units][s_cap]
  float* pooled;      // [units][s_cap]
  int32_t* kept;      // [units][keep]
  int32_t* kept_user; // optional copy for the caller, rows of kept_stride entries
  int kept_stride;
  int32_t* n_out;     // [batch]: number of tokens kept per sequence
  uint2* runs;        // [units][s_cap]: the pooled votes as runs of equal ones
  uint32_t* n_runs;   // [units], kCountStride apart
  uint32_t* hist;     // [units][kSelBins]: pooled votes per bin
  int sel_split;      // workgroups a unit's row is divided between in the select
};

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// max of three without the input canonicalisation fmaxf() brings along (three extra instructions
// per call here); the inputs are matrix-core outputs and running maxima, never signalling NaNs.  A matrix-core output
// must have been read by an instruction of the compiler's before (see the one use).
__device__ __forceinline__ float max3_raw(float x, float y, float w) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(x), "v"(y), "v"(w));
  return d;
}

// 16 bytes per lane from `src` straight to LDS: lane l's land 16 l bytes behind the wavefront's `dst`
template <int POLICY>
__device__ __forceinline__ void load_to_lds(const void* src, void* dst) {
#ifdef __HIP_DEVICE_COMPILE__  // the builtin is unknown to the host pass
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, POLICY);
#endif
}

constexpr int kSnapCols = 128;            // softmax rows (columns of the products) per wavefront, in blocks of 32
constexpr int kSnapMaxPairs = kWave;      // page pairs one wavefront walks, at most: a lane each
constexpr int kSnapSegPairs = 8;          // page pairs between two write-outs of the votes
constexpr int kSnapMaxChunkPages = 128;   // pages per workgroup
constexpr int kRowsBytes = 4 * kHeadDim * (int)sizeof(bf16_t) + 16;  // four rows in LDS, and what shifts the next four's banks
constexpr int kTileBytes = 4 * kRowsBytes, kSlotBytes = 2 * kTileBytes;
constexpr int kRingBytes = 4 * 2 * kSlotBytes;
constexpr int kMergeLoads = 16;            // chunk statistics a thread of pass 2 has in flight
constexpr int kMergeStats = 64 * 128;      // statistics of a unit that pass 2 merges itself, at most
constexpr int kMergeWorkgroups = 1024;     // in up to this many workgroups, two rounds over the chip
constexpr int kSnapStatBytes = 2 * 4 * kSnapCols * (int)sizeof(float);
constexpr int kSnapVoteBytes = 2 * kSnapSegPairs * 4 * 2 * kAttnPage * (int)sizeof(float);

// Four bytes to LDS, in assembly: in front of a store it can see the compiler waits for every load to LDS in flight,
// which it cannot tell apart from the store's target.
__device__ __forceinline__ void lds_store(float* dst, float x) {
#ifdef __HIP_DEVICE_COMPILE__
  const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)dst;
  asm volatile("ds_write_b32 %0, %1" ::"v"(at), "v"(x) : "memory");
#endif
}

// A lane's values x[0 .. 15], each to be summed over the 32 lanes of its half wavefront: lane l is left with the
// total of x[8 (l / 16 % 2) + 4 (l / 8 % 2) + 2 (l / 4 % 2) + l / 2 % 2], which the lanes below and above it in a
// pair share.  Every step halves the values a lane holds, so that 38 instructions do it; the order of the additions
// is fixed.
__device__ __forceinline__ float half_wave_sums(float (&x)[16], int lane) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {  // rows of 16 lanes: an even row keeps x[j], an odd one x[j + 8]
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[j]), __float_as_uint(x[j + 8]), false, false);
    x[j] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  const auto step = [&](auto ctrl, int bit, int n) {  // the lane `ctrl` names differs in `bit` (and covers the rest later)
    const bool up = (lane & bit) != 0;
#pragma unroll
    for (int j = 0; j < n; ++j) {
      const float keep = up ? x[j + n] : x[j], give = up ? x[j] : x[j + n];
      x[j] = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), decltype(ctrl)::value, 0xf, 0xf, true));
    }
  };
  step(std::integral_constant<int, 0x128>{}, 8, 4);  // row_ror:8
  step(std::integral_constant<int, 0x141>{}, 4, 2);  // row_half_mirror
  step(std::integral_constant<int, 0x4E>{}, 2, 1);   // quad_perm 2,3,0,1
  return x[0] + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x[0]), 0xB1, 0xf, 0xf, true));  // quad_perm 1,0,3,2
}

// MERGE (pass 2): the statistics of pass 1's chunks are merged by every workgroup for itself, not by a launch in between.
// That launch takes 4-5 us whatever there is to merge; here up to 64 KiB come from L2 beside the queries.  us a call
// with the summaries, by a launch / so: 1 x 2048 tokens 36.6 / 35.1, 1 x 8192 48.6 / 46.0, 1 x 16384 53.0 / 51.4, 1 x 32768
// 70.8 / 69.4, 4 x 16000 89.3 / 86.5, 8 x 32000 unequal 179.8 / 177.5 (1024 workgroups), 16 x 32768 541.3 / 543.6 (2048).
// The two meet between 64 and 128 KiB of statistics a unit, of which kMergeStats is the lower end.  By KiB a unit, a launch / so:
//    80  1 x 20000 with 64 query heads 75.2 / 74.4, 1 x 5000 with 8 query heads and one KV head 42.5 / 41.4
//    94  1 x 24000 with 64 77.7 / 77.2
//    98  1 x 200000 with 32 239.3 / 238.0, 1 x 50000 with 16 and four KV heads 66.3 / 65.8
//   110  1 x 28000 with 64 80.8 / 81.6
//   118  2 x 120000 with 64 364.0 / 372.3
//   126  1 x 32000 with 64 88.3 / 89.3, 1 x 8000 with 8 and one KV head 42.5 / 42.6
// NB: blocks of 32 softmax rows every wavefront works through (blocks without any hold zero queries and are
// discarded).  A wavefront takes 32 tokens, a pair of neighbouring pages, at a time, against one block after the
// other: a 32 x 32 product leaves a lane one softmax row and sixteen of the tokens.
//
// What bounds it: vector issue and HBM, nearly equally, and under sustained load the clock.  With 16 x 16 products
// a lane held four tokens of a softmax row, so that a maximum, a rescale and their exponential were paid for every
// four logits, and a product kept the vector port busy for half of its 16 cycles; with 32 x 32 ones it is sixteen
// logits, and a product covers twice the work in the same issue time.  The call with the summaries, 8 KV heads, us
// on keys that are in no cache / again and again on the same keys: 16 x 32768 tokens 582 -> 548 / 579 -> 547, 4 x
// 32768 175 -> 168 / 171 -> 162, 1 x 131072 164 -> 154 / 156 -> 152, 1 x 32768 81.5 -> 78 / 74.2 -> 74.3, 1 x 8192
// 56 -> 51 / 53.5 -> 48.8.  Under the long set-up loop of the benchmark, where the clock drops, 16 x 32768 stays at
// 580-595 a layer.  (Bare stream of 16 x 32768 keys: 161 us a pass.)
template <bool PASS2, int NB, bool MERGE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void snap_score_kernel(CacheView c, SnapArgs a) {
  typedef uint32_t ring_u32x4 __attribute__((ext_vector_type(4)));
  // Two pairs of key tiles per wavefront, then in pass 1 maxima and sums by wavefront, in pass 2 the votes of two
  // segments, [2][column groups][tokens].
  extern __shared__ __align__(16) unsigned char s_ring[];
  float* s_out = reinterpret_cast<float*>(s_ring + kRingBytes);
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // scalar: page indices stay in SGPRs
  const int hn = lane % 16, half = lane / 32;
  const int unit = blockIdx.y, chunk = blockIdx.x;
  const int b = unit / c.n_kv_heads, g = unit % c.n_kv_heads;
  const int S = c.seq_lens[b];
  if (S <= a.keep || S > c.pages_cap * kAttnPage) return;
  const int L = S - a.W;
  const int cgi = wave % a.CG, pw = wave / a.CG, npw = 4 / a.CG;
  const int p_begin = chunk * a.chunk_pages;
  const int p_limit = PASS2 ? (L + kAttnPage - 1) / kAttnPage : (S + kAttnPage - 1) / kAttnPage;
  const int p_end = min(p_begin + a.chunk_pages, p_limit);
  if (p_begin >= p_end) return;  // a chunk beyond the prompt: its statistics are never read
  const int n_pairs = (p_end - p_begin + 2 * npw - 1) / (2 * npw);  // <= kSnapMaxPairs (host)
  const auto first_page = [&](int it) { return p_begin + 2 * (it * npw + pw); };

  // Where this wavefront's pages live: lane i looks up pair i once, up front, and the loop hands the
  // pages out by readlane, so it contains no table lookups and no waits on them.  -1: absent.
  int pp0 = -1, pp1 = -1;
  if (lane < n_pairs) {
    const int p = first_page(lane);
    if (p < p_end) pp0 = (int)phys_page(c, b, p);
    if (p + 1 < p_end) pp1 = (int)phys_page(c, b, p + 1);
  }

  bf16x8 qf[NB][8];
  float M2[NB], invZ[NB];
  float m[NB], z[NB];
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) { m[cb] = kNegBigS; z[cb] = 0.f; }
  const float sc = kLog2eS * 0.08838834764831845f;
  const char* k_head = reinterpret_cast<const char*>(c.k_pool + (int64_t)g * c.stride_head);

  // Key tiles travel through two slots of LDS per wavefront, a pair of pages each, filled by loads that write LDS
  // directly (no registers are held for tiles in flight): the pair for iteration it + 2 is requested as soon
  // as iteration it has its own in registers.  An absent or out-of-range page reads tile 0 of the pool
  // and is masked below; those loads are issued all the same, which keeps the number of loads younger
  // than the pair being waited for constant.
  unsigned char* ring = s_ring + wave * 2 * kSlotBytes;
  const int row_at = hn / 4 * kRowsBytes + hn % 4 * kHeadDim * (int)sizeof(bf16_t) + half * 16;
  const auto pages_at = [&](int it, int& a0, int& a1) {  // `it` is wave-uniform
    a0 = __builtin_amdgcn_readlane(pp0, it & (kWave - 1));
    a1 = __builtin_amdgcn_readlane(pp1, it & (kWave - 1));
    if (it >= n_pairs) a0 = a1 = -1;
  };
  // Both passes load the keys with the streaming hint.  Without it in pass 2 the gather that follows finds part of
  // the keys in the last-level cache, which gives less than the hint gives the pass: pass + gather on keys not scored
  // before, 16 x 32768 tokens 239 + 100 us without, 215 + 117 with; 1 x 32768 22.5 + 11.4 and 20.1 + 12.3.  The call
  // with the summaries, without / with: 16 x 32768 570 / 548, 4 x 32768 176 / 168, 1 x 131072 160 / 154, 1 x 32768
  // 80.3 / 78, 1 x 8192 51.1 / 50.7; only one prompt of 32768 scored over and over is ahead without (73.8 / 74.3).
  constexpr int kPolicyStream = 2;  // the "nt" bit of the load's cache policy
  // Load instruction j of a tile brings in token rows 4j .. 4j+3 (1 KiB, whole cache lines); lane l lands 16 l
  // bytes behind the instruction's place in the slot, and fetches the 16-byte chunk that belongs there: chunk x of
  // row 4j + i stands at position x ^ 4i, and the instructions' places are 16 bytes more than a KiB apart, so that
  // the reads below (16 rows at one chunk position) spread over all LDS banks.
  const uint32_t dma_off = (uint32_t)((lane >> 4) * kHeadDim + ((lane & 15) ^ (lane >> 4) * 4) * 8) * sizeof(bf16_t);
  const auto fetch = [&](const char* rows, unsigned char* dst, auto policy) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      load_to_lds<decltype(policy)::value>(rows + j * 4 * kHeadDim * (int)sizeof(bf16_t) + dma_off, dst + j * kRowsBytes);
  };
  const auto issue = [&](int it) {
    int a0, a1;
    pages_at(it, a0, a1);
    unsigned char* dst = ring + (it & 1) * kSlotBytes;
    constexpr std::integral_constant<int, kPolicyStream> policy{};
    fetch(k_head + (int64_t)max(a0, 0) * c.stride_page * (int)sizeof(bf16_t), dst, policy);
    fetch(k_head + (int64_t)max(a1, 0) * c.stride_page * (int)sizeof(bf16_t), dst + kTileBytes, policy);
  };
  // Row hn of a tile, channels 16 j + 8 half .., j = 0 .. 7: chunk 2 j + half
  const auto read_row = [&](const unsigned char* tile, bf16x8 (&f)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      f[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const ring_u32x4*>(tile + row_at + ((j / 2 ^ hn % 4) * 64 + j % 2 * 32)));
  };
  bf16x8 kf[8];
  const auto read_pair = [&](int it) {  // this lane's row is token lane % 32 of the pair
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // everything but the younger pair has landed
    read_row(ring + (it & 1) * kSlotBytes + lane % 32 / 16 * kTileBytes, kf);
  };
  const auto product = [&](int cb, int j, f32x16& acc) {
    const f32x16 zero = {};
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j], qf[cb][j], j == 0 ? zero : acc, 0, 0, 0);
  };
  // The votes of a pair: staged in LDS, one copy per column group, and written out once per segment of
  // kSnapSegPairs pairs (a global store per pair would sit among the tile loads the wait above counts, and
  // make it wait for more of them than it needs).  Two buffers in turn, so one barrier per segment.
  const int seg_tokens = kSnapSegPairs * 2 * npw * kAttnPage;
  const int vote_at = pw * 2 * kAttnPage + lane / 16 % 2 * kAttnPage + lane / 8 % 2 * 8 + half * 4 + lane / 2 % 4;
  const auto vote_slot = [&](int seg, int cg) { return s_out + ((seg & 1) * a.CG + cg) * seg_tokens; };
  const auto emit_votes = [&](float (&v)[16], int it) {
    // (element i of an accumulator is token 16 (i / 8) + 8 (i / 4 % 2) + 4 half + i % 4 of the pair)
    const float total = half_wave_sums(v, lane);
    lds_store(vote_slot(it / kSnapSegPairs, cgi) + it % kSnapSegPairs * (2 * npw * kAttnPage) + vote_at, total);
  };
  const auto write_out = [&](int it) {  // after iteration `it`, in every wavefront alike
    if (!PASS2 || (it % kSnapSegPairs != kSnapSegPairs - 1 && it + 1 != n_pairs)) return;
    // (not __syncthreads(), which would wait for the tiles in flight as well)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int seg = it / kSnapSegPairs, tok = p_begin * kAttnPage + seg * seg_tokens + tid * 4;
    if (tid * 4 < seg_tokens && tok < min(p_end * kAttnPage, L)) {  // rows hold a multiple of four votes
      float4 x = *reinterpret_cast<const float4*>(vote_slot(seg, 0) + tid * 4);
      if (a.CG == 2) {
        const float4 y = *reinterpret_cast<const float4*>(vote_slot(seg, 1) + tid * 4);
        x = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
      }
      *reinterpret_cast<float4*>(a.votes + (int64_t)unit * a.s_cap + tok) = x;
    }
  };

  // Softmax update of block `cb` from its products `s`
  float v[16];  // pass 2: this pair's votes
  const auto update = [&](int cb, f32x16& s) {
    if (PASS2) {
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const float e = exp2_fast(fmaf(s[x], sc, -M2[cb]));
        v[x] = cb == 0 ? e * invZ[cb] : fmaf(e, invZ[cb], v[x]);
      }
    } else {
      // m[] is the running maximum in the log2 domain; an unchanged maximum rescales by exactly 1
      // max3_raw() is assembly, in front of which the compiler leaves no time for the products to reach their
      // registers.  It does in front of this multiplication, and the empty assembly puts the rest behind it.
      const float last = s[15] * sc;
      asm volatile("" : "+v"(s) : "v"(last));
      const float x0 = max3_raw(s[0], s[1], s[2]), x1 = max3_raw(s[3], s[4], s[5]), x2 = max3_raw(s[6], s[7], s[8]);
      const float x3 = max3_raw(s[9], s[10], s[11]), x4 = max3_raw(s[12], s[13], s[14]);
      const float top = max3_raw(max3_raw(x0, x1, x2), x3, x4);
      const float mn = max3_raw(m[cb], top * sc, last);
      float sum = 0.f;
#pragma unroll
      for (int x = 0; x < 16; x += 4) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = exp2_fast(fmaf(s[x + i], sc, -mn));
        const float four = (e[0] + e[1]) + (e[2] + e[3]);
        sum = x == 0 ? four : sum + four;
      }
      z[cb] = fmaf(z[cb], exp2_fast(m[cb] - mn), sum);
      m[cb] = mn;
    }
  };

  // The leading run of pairs that need no mask takes the hot variant: none of the wavefront's pages
  // absent, and the pair's last token inside the prefix, so that every window row sees all of it.
  int n_hot = 0;
  // (A pair at or beyond the chunk's end is not an absent one: taken for one, it sent every pair of a wavefront down
  // the masked path in the last chunk of most prompts: 25 us of pass 2 over 16 x 32768 tokens.)
  const bool gone0 = first_page(lane) < p_end && pp0 < 0, gone1 = first_page(lane) + 1 < p_end && pp1 < 0;
  if (__ballot(lane < n_pairs && (gone0 || gone1)) == 0ull) {
    // pairs whose second page p has p * 16 + 15 <= L, i.e. p <= (L - 15) / 16, and lies below p_end
    const int p_last = min(p_end - 1, (L - (kAttnPage - 1)) >= 0 ? (L - (kAttnPage - 1)) / kAttnPage : -1);
    if (p_last >= p_begin + 2 * pw + 1) n_hot = (p_last - 1 - p_begin - 2 * pw) / (2 * npw) + 1;
    n_hot = min(n_hot, n_pairs);
  }
  const auto hot_pairs = [&](int n) {
    read_pair(0);
    for (int it = 0; it < n; ++it) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        f32x16 acc;
#pragma unroll
        for (int j = 0; j < 8; ++j) product(cb, j, acc);
        if (cb == 0) {  // the keys are in registers (the products had to wait for the LDS reads): refill their slot
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          issue(it + 2);
        }
        if (cb == NB - 1) read_pair(it + 1);  // lands under the last update (behind the last pair, in vain)
        // keep the blocks in program order: products of a later block hoisted above this one's update
        // would need a second accumulator the register file has no room for
        __builtin_amdgcn_sched_barrier(0);
        update(cb, acc);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (PASS2) emit_votes(v, it);
      write_out(it);
    }
  };
  const int first_w = __builtin_amdgcn_readfirstlane(cgi * kSnapCols % a.W);
  // A pair of any kind (pages absent, or at the end of the prefix, where rows differ in what they see).
  const auto masked_pair = [&](int it) {
    int a0, a1;
    pages_at(it, a0, a1);
    const int ln = (int)use_late((uint32_t)lane);  // nothing of this is worth a register across the hot pairs
    const int tok0 = first_page(it) * kAttnPage + ln / 32 * 4;
    read_pair(it);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue(it + 2);
    int w0 = first_w;  // the place in the window of a block's first softmax row; window and blocks are multiples of 16
    const auto next16 = [&](int w) { return w + 16 == a.W ? 0 : w + 16; };
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      f32x16 acc;
#pragma unroll
      for (int j = 0; j < 8; ++j) product(cb, j, acc);
      const int w1 = next16(w0);
      int limit = L + ln % 16 + (ln & 16 ? w1 : w0);  // the last token this softmax row sees
      if (cgi * kSnapCols + cb * 32 + ln % 32 >= a.NC) limit = -1;
      w0 = next16(w1);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const bool sees = (i < 8 ? a0 : a1) >= 0 && tok0 + i / 4 * 8 + i % 4 <= limit;
        acc[i] = sees ? acc[i] : -INFINITY;
      }
      update(cb, acc);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (PASS2) emit_votes(v, it);
    write_out(it);
  };

  // The queries: fetched once per workgroup, as whole cache lines, into the second slot of every wavefront, laid
  // out like the key tiles (16 softmax rows for 16 tokens) and read from there; the first pair of key
  // tiles travels beside them into the first.  (Every wavefront fetching its fragments from memory by itself
  // took 9 us per workgroup: 128 loads of 16 half lines each through one first-level cache.)  The rows of a
  // group's heads lie one after the other, so column `col` is simply row `col`.
  static_assert(kSnapCols == 8 * 16, "eight blocks of 16 queries fill one slot of four wavefronts");
  const auto block_at = [&](int x) {  // where block x of 16 lies: tile x / 4 of the second slot of wavefront x % 4
    return s_ring + (x % 4 * 2 + 1) * kSlotBytes + x / 4 * kTileBytes;
  };
  // MERGE: this workgroup merges the chunks' statistics itself, requested ahead of the queries.  A softmax row's chunks are
  // dealt to `parts` threads, in an order that is the same in every workgroup; the partial results meet in LDS behind the
  // queries' barrier.
  const auto merge = [](float& mm, float& zz, float mo, float zo) {
    const float mn = fmaxf(mm, mo);
    zz = zz * exp2_fast(mm - mn) + zo * exp2_fast(mo - mn);
    mm = mn;
  };
  const int ncp = a.NC <= 64 ? 64 : a.NC <= 128 ? 128 : 256, parts = 256 / ncp;  // NC <= 256 (host)
  const int my_row = tid & (ncp - 1), my_part = tid / ncp;
  const int chunks = ((S + kAttnPage - 1) / kAttnPage + a.chunk_pages - 1) / a.chunk_pages;
  float2 first_stats[MERGE ? kMergeLoads : 1];
  const auto fetch_stats = [&](int ch0) {
    const float2* row = reinterpret_cast<const float2*>(a.stats_part) + (int64_t)unit * a.n_chunks * a.NC + my_row;
#pragma unroll
    for (int u = 0; u < kMergeLoads; ++u) {
      const int ch = ch0 + my_part + u * parts;
      first_stats[u] = make_float2(kNegBigS, 0.f);
      if (ch < chunks && my_row < a.NC) first_stats[u] = row[(int64_t)ch * a.NC];
    }
  };
  if (MERGE) fetch_stats(0);
  if (PASS2 && !MERGE) {  // requested ahead of the queries: one round trip for both
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      const int col = cgi * kSnapCols + cb * 32 + lane % 32;
      const float2 st2 = col < a.NC ? *reinterpret_cast<const float2*>(a.stats + ((int64_t)unit * a.NC + col) * 2)
                                    : make_float2(0.f, 0.f);
      M2[cb] = st2.x;
      invZ[cb] = st2.y;
    }
  }
  const char* q_rows =
      reinterpret_cast<const char*>(a.qobs + ((int64_t)b * c.n_q_heads + (int64_t)g * c.group) * a.W * kHeadDim);
  for (int cg = 0; cg < a.CG; ++cg) {
    if (cg > 0) __syncthreads();  // the blocks of the group before have been read
#pragma unroll
    for (int h = 0; h < (NB + 1) / 2; ++h) {
      const int x = h * 4 + wave, block = cg * (kSnapCols / 16) + x;
      if (block * 16 < a.NC)
        fetch(q_rows + (int64_t)block * 16 * kHeadDim * sizeof(bf16_t), block_at(x), std::integral_constant<int, 0>{});
    }
    if (cg == 0) {
      issue(0);
      if (MERGE) {
        float mm = kNegBigS, zz = 0.f;
        for (int ch0 = 0;;) {
#pragma unroll
          for (int u = 0; u < kMergeLoads; ++u) merge(mm, zz, first_stats[u].x, first_stats[u].y);
          ch0 += kMergeLoads * parts;
          if (ch0 >= chunks) break;
          fetch_stats(ch0);
        }
        s_out[tid] = mm;
        s_out[256 + tid] = zz;
      }
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // all but the first pair of key tiles
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if (cg == cgi) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        read_row(block_at(2 * cb + lane % 32 / 16), qf[cb]);
        if (cg * kSnapCols + cb * 32 + lane % 32 >= a.NC) {
#pragma unroll
          for (int j = 0; j < 8; ++j) qf[cb][j] = __builtin_bit_cast(bf16x8, (ring_u32x4){0u, 0u, 0u, 0u});
        }
      }
    }
  }
  if (MERGE) {
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      const int col = cgi * kSnapCols + cb * 32 + lane % 32;
      float mm = kNegBigS, zz = 0.f;
      if (col < a.NC)
        for (int p = 0; p < parts; ++p) merge(mm, zz, s_out[p * ncp + col], s_out[256 + p * ncp + col]);
      M2[cb] = col < a.NC ? mm : 0.f;
      invZ[cb] = zz > 0.f ? 1.f / zz : 0.f;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();  // the blocks have been read: their slots take key tiles now
  issue(1);
  if (n_hot > 0) hot_pairs(n_hot);
  for (int it = n_hot; it < n_pairs; ++it) masked_pair(it);
  // the last refills (unused) land before the workgroup's LDS is given back
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (PASS2) return;
  if (chunk == 0) {  // the pool, which counts into these, is at least a launch away
    if (tid == 0) a.n_runs[unit * kCountStride] = 0;
    uint4* hist = reinterpret_cast<uint4*>(a.hist + (int64_t)unit * kSelBins);
    for (int i = tid; i < kSelBins / 4; i += 256) hist[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  // ---- pass 1: merge statistics over the half wavefronts and the wavefronts, and hand the chunk's partial out
  float (*sM)[kSnapCols] = reinterpret_cast<float (*)[kSnapCols]>(s_out);
  float (*sZ)[kSnapCols] = sM + 4;
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) {
    const float mo = __shfl_xor(m[cb], 32), zo = __shfl_xor(z[cb], 32);
    const float mn = fmaxf(m[cb], mo);
    z[cb] = z[cb] * exp2_fast(m[cb] - mn) + zo * exp2_fast(mo - mn);
    if (half == 0) {
      sM[wave][cb * 32 + lane] = mn;
      sZ[wave][cb * 32 + lane] = z[cb];
    }
  }
  __syncthreads();
  for (int idx = tid; idx < a.CG * kSnapCols; idx += 256) {
    const int cg2 = idx / kSnapCols, lc = idx % kSnapCols;
    if (idx >= a.NC) continue;
    float mm = kNegBigS, zz = 0.f;
    for (int w2 = cg2; w2 < 4; w2 += a.CG) {
      const float mo = sM[w2][lc], zo = sZ[w2][lc];
      const float mn = fmaxf(mm, mo);
      zz = zz * exp2_fast(mm - mn) + zo * exp2_fast(mo - mn);
      mm = mn;
    }
    float* o = a.stats_part + (((int64_t)unit * a.n_chunks + chunk) * a.NC + idx) * 2;
    o[0] = mm;
    o[1] = zz;
  }
}

// merge the per-chunk statistics of one unit, where there are too many for pass 2 (MERGE above).  A long
// prompt has hundreds of chunks: the chunks of a softmax row are dealt to 1024 / ncp threads (ncp = the row
// count rounded up to a power of two), each merges its share with eight loads in flight, and one thread per
// row merges the partial results in a fixed order.
constexpr int kStatsT = 1024;
__global__ __launch_bounds__(kStatsT) void snap_stats_kernel(CacheView c, SnapArgs a) {
  __shared__ float pm[kStatsT], pz[kStatsT];
  const int tid = threadIdx.x;
  const int unit = blockIdx.x;
  const int b = unit / c.n_kv_heads;
  const int S = c.seq_lens[b];
  if (S <= a.keep || S > c.pages_cap * kAttnPage) return;
  const int chunks = ((S + kAttnPage - 1) / kAttnPage + a.chunk_pages - 1) / a.chunk_pages;
  int ncp = 64;
  while (ncp < a.NC) ncp <<= 1;  // NC <= 256 (host)
  const int col = tid % ncp, part = tid / ncp, parts = kStatsT / ncp;
  const auto merge = [](float& mm, float& zz, float mo, float zo) {
    const float mn = fmaxf(mm, mo);
    zz = zz * exp2_fast(mm - mn) + zo * exp2_fast(mo - mn);
    mm = mn;
  };
  float mm = kNegBigS, zz = 0.f;
  if (col < a.NC) {
    const float2* row = reinterpret_cast<const float2*>(a.stats_part) + (int64_t)unit * a.n_chunks * a.NC + col;
    for (int ch0 = part; ch0 < chunks; ch0 += parts * 8) {
      float2 o[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int ch = ch0 + u * parts;
        o[u] = ch < chunks ? row[(int64_t)ch * a.NC] : make_float2(kNegBigS, 0.f);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) merge(mm, zz, o[u].x, o[u].y);
    }
  }
  pm[tid] = mm;
  pz[tid] = zz;
  __syncthreads();
  if (tid < a.NC) {
    mm = kNegBigS;
    zz = 0.f;
    for (int p = 0; p < parts; ++p) merge(mm, zz, pm[p * ncp + tid], pz[p * ncp + tid]);
    a.stats[((int64_t)unit * a.NC + tid) * 2] = mm;
    a.stats[((int64_t)unit * a.NC + tid) * 2 + 1] = zz > 0.f ? 1.f / zz : 0.f;
  }
}

__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Stride-1 max-pool over the prefix votes, window [j-r, j+r] clipped to [0, L), and the list of runs
// the select works from.  A workgroup pools kPoolTile positions, a thread eight neighbours: their
// windows share [j0+7-r, j0+r], which is 2q+1 whole groups of eight (their maxima stand in LDS) and a
// few elements at either end; what the eight windows do not share is seven elements on each side,
// walked once.  At kernel 63 that is 21 LDS reads for eight votes (window maxima by doubling take 17
// for each).  A maximum is exact, so the order of taking it does not matter.
//
// Pooling repeats every local maximum up to 2r+1 times, so the pooled row is written once more as runs
// of equal votes, cut at multiples of eight: (ordered bits of the vote, group * 16 + length), in no
// particular order, and counted into the unit's histogram of kSelBins bins, 64 to the octave (votes are
// small probabilities under a few heavy tokens: equal-width bins would put nearly all into the lowest).
// The select starts from those: about a sixth of the votes, and its first counting pass done.  The
// counters of different units sit in lines of their own (adds to one line queue up: 128 units sharing
// four lines took 27 us here and 8 units of 131072 votes sharing one 16.5; 17.7 and 10.1 apart.
// Clearing and reading the bins is the same work for a workgroup of any size: 14.5 and 8.1 with 512
// threads instead of 256, no more with 1024.).
constexpr int kPoolT = 512;
constexpr int kPoolTile = kPoolT * 8;
__global__ __launch_bounds__(kPoolT) void snap_pool_kernel(CacheView c, SnapArgs a) {
  extern __shared__ float smem[];  // raw[], one float of padding per eight, then the groups' maxima
  __shared__ uint32_t s_wave[kPoolT / kWave], s_base;
  __shared__ uint32_t hist[kSelBins];
  const int unit = blockIdx.y;
  const int b = unit / c.n_kv_heads;
  const int S = c.seq_lens[b];
  if (S <= a.keep || S > c.pages_cap * kAttnPage) return;
  const int L = S - a.W, r = a.pool_r;
  const int j0 = blockIdx.x * kPoolTile;
  if (j0 >= L) return;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int HG = (r + 7) / 8;           // halo in groups of eight
  const int groups = kPoolT + 2 * HG;   // groups of the tile with its halo
  float* raw = smem;                    // group x, element i at x * 9 + i: no bank conflicts
  float* gmax = smem + groups * 9;
  const float* v = a.votes + (int64_t)unit * a.s_cap;
  for (int i = tid; i < kSelBins; i += kPoolT) hist[i] = 0;
  for (int x = tid; x < groups; x += kPoolT) {
    const int j = j0 + (x - HG) * 8;
    float e[8], m = -INFINITY;
    if (j >= 0 && j < L) {  // rows hold a multiple of eight floats: a group that begins below L is in bounds
      const float4 lo = *reinterpret_cast<const float4*>(v + j), hi = *reinterpret_cast<const float4*>(v + j + 4);
      e[0] = lo.x; e[1] = lo.y; e[2] = lo.z; e[3] = lo.w;
      e[4] = hi.x; e[5] = hi.y; e[6] = hi.z; e[7] = hi.w;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (j < 0 || j + i >= L) e[i] = -INFINITY;
      m = fmaxf(m, e[i]);
      raw[x * 9 + i] = e[i];
    }
    gmax[x] = m;
  }
  __syncthreads();
  const int t = tid + HG;  // this thread's group
  const auto at = [&](int x) { return raw[x + (x >> 3)]; };  // element x of the tile, the halo's first is 0
  float o[8];
  if (r >= 7) {
    const int q = (r - 7) / 8, e = r - 8 * q - 7;  // 2q+1 whole groups, e elements beyond them at either end
    float core = gmax[t];
    for (int x = 1; x <= q; ++x) core = fmaxf(core, fmaxf(gmax[t - x], gmax[t + x]));
    for (int x = 0; x < e; ++x) core = fmaxf(core, fmaxf(at(8 * (t - q) - 1 - x), at(8 * (t + q + 1) + x)));
    float left = core, right = core;
    o[7] = core;
#pragma unroll
    for (int i = 6; i >= 0; --i) {
      left = fmaxf(left, at(8 * t - r + i));
      o[i] = left;
    }
#pragma unroll
    for (int i = 1; i < 8; ++i) {
      right = fmaxf(right, at(8 * t + r + i));
      o[i] = fmaxf(o[i], right);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      o[i] = at(8 * t + i);
      for (int x = 1; x <= r; ++x) o[i] = fmaxf(o[i], fmaxf(at(8 * t + i - x), at(8 * t + i + x)));
    }
  }
  const int j = j0 + tid * 8;
  const int n = min(8, L - j);  // votes of this thread (none below 1)
  uint32_t key[8], starts = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    key[i] = order_key(o[i]);
    if (i < n && (i == 0 || key[i] != key[i - 1])) starts |= 1u << i;
  }
  if (n > 0) {
    float4* out = reinterpret_cast<float4*>(a.pooled + (int64_t)unit * a.s_cap + j);
    out[0] = make_float4(o[0], o[1], o[2], o[3]);
    out[1] = make_float4(o[4], o[5], o[6], o[7]);
  }
  const uint32_t mine = __popc(starts);
  const uint32_t inc = wave_incl_scan(mine);
  if (lane == kWave - 1) s_wave[wave] = inc;
  __syncthreads();
  uint32_t at0 = inc - mine, all = 0;
#pragma unroll
  for (int w = 0; w < kPoolT / kWave; ++w) {
    if (w < wave) at0 += s_wave[w];
    all += s_wave[w];
  }
  if (tid == 0) s_base = atomicAdd(&a.n_runs[unit * kCountStride], all);
  int len[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if ((starts >> i) & 1u) {
      const uint32_t rest = (starts >> i) >> 1;  // the next run begins at i + ffs(rest), or the votes end
      len[i] = rest ? __ffs(rest) : n - i;
      atomicAdd(&hist[vote_bin(key[i])], (uint32_t)len[i]);
    }
  }
  __syncthreads();
  uint2* runs = a.runs + (int64_t)unit * a.s_cap + s_base + at0;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if ((starts >> i) & 1u) *runs++ = make_uint2(key[i], (uint32_t)(j / 8) * 16u + (uint32_t)len[i]);
  for (int i = tid; i < kSelBins; i += kPoolT)
    if (hist[i] != 0u) atomicAdd(&a.hist[(int64_t)unit * kSelBins + i], hist[i]);
}

// Exact top-(keep-W) of the pooled votes, ties to the lower position, and the window, ascending.  A
// unit's row is cut into `sel_split` slices, one workgroup each; every workgroup finds the unit's
// threshold for itself, counts what lies above it and at it before its slice, and emits its slice in
// order.  The threshold: the pool's histogram names the bin of the wanted rank; one pass over the runs
// collects the runs in it and counts the ones above it before the slice; the few collected are ranked
// by counting.  Only if more than kSelCand runs share the bin is it divided again.
//
// One workgroup per unit over the votes themselves took 26 us for 8 units of 32768 votes and 30 for
// 128 units, bound by the vector instructions of the one compute unit (32 votes a thread through the
// counting and the emission); seven launches of radix passes took 35 us for 8 units of 131072.  Now
// 7.4 / 15 / 10.8 us.  Slices stay at 4096 positions or more, and at one round over the chip.
constexpr int kSelT = 1024;
constexpr int kSelCand = 512;
constexpr int kSelSlice = 4 * kSelT;  // positions emitted at a time
constexpr int kSelBatch = 8;          // runs a thread has in flight

struct SelShared {
  uint32_t hist[kSelBins];
  uint2 cand[kSelCand];
  uint32_t wsum[2][kSelT / kWave];
  uint32_t n_cand, bin, rank, tau, need;
};

// The wanted rank's bin by a scan from the top, four bins a thread, in h[] the highest first:
// sh.bin and, within it, sh.rank.  Ends with a barrier.
__device__ __forceinline__ void find_bin(const uint32_t (&h)[4], uint32_t k, SelShared& sh) {
  const int top = kSelBins - 1 - (int)threadIdx.x * 4;
  uint32_t above = block_excl_scan<kSelT>(h[0] + h[1] + h[2] + h[3], sh.wsum[0]);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (above < k && k <= above + h[j]) {
      sh.bin = (uint32_t)(top - j);
      sh.rank = k - above;
    }
    above += h[j];
  }
  __syncthreads();
}

__device__ __forceinline__ void snap_threshold(const uint2* runs, int n_runs, const uint32_t* ghist, uint32_t want,
                                               uint32_t group0, SelShared& sh, uint32_t& tau, uint32_t& need_eq,
                                               uint32_t& gt_before, uint32_t& eq_before) {
  static_assert(kSelBins == 4 * kSelT, "four bins a thread");
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const auto fetch = [&](uint2 (&v)[kSelBatch], int x0) {  // an absent run has length 0
#pragma unroll
    for (int u = 0; u < kSelBatch; ++u) {
      const int x = x0 + u * kSelT + tid;
      v[u] = x < n_runs ? runs[x] : make_uint2(0u, 0u);
    }
  };
  uint2 first[kSelBatch];  // on their way while the histogram is scanned
  fetch(first, 0);
  const auto each = [&](const auto& fn) {
#pragma unroll
    for (int u = 0; u < kSelBatch; ++u)
      if (first[u].y != 0u) fn(first[u].x, first[u].y);
    for (int x0 = kSelBatch * kSelT; x0 < n_runs; x0 += kSelBatch * kSelT) {
      uint2 v[kSelBatch];
      fetch(v, x0);
#pragma unroll
      for (int u = 0; u < kSelBatch; ++u)
        if (v[u].y != 0u) fn(v[u].x, v[u].y);
    }
  };
  const uint4 gh = reinterpret_cast<const uint4*>(ghist)[kSelT - 1 - tid];
  if (tid == 0) sh.n_cand = 0;
  const uint32_t h0[4] = {gh.w, gh.z, gh.y, gh.x};
  find_bin(h0, want, sh);
  uint32_t k = sh.rank;
  KeyRange in = bin_range(sh.bin);  // where the wanted key lies
  uint32_t gt = 0, eq = 0;  // this thread's share of what lies before the slice
  each([&](uint32_t key, uint32_t gl) {
    if (key < in.lo) return;
    if (key - in.lo > in.span) {
      if ((gl >> 4) < group0) gt += gl & 15u;
    } else {
      const uint32_t at = atomicAdd(&sh.n_cand, 1u);
      if (at < (uint32_t)kSelCand) sh.cand[at] = make_uint2(key, gl);
    }
  });
  __syncthreads();
  int n_cand = (int)sh.n_cand;
  const bool few = n_cand <= kSelCand;
  while (n_cand > kSelCand && in.span != 0u) {
    const int shift = part_shift(in);
    __syncthreads();  // n_cand and the bin have been read
    for (int i = tid; i < kSelBins; i += kSelT) sh.hist[i] = 0;
    if (tid == 0) sh.n_cand = 0;
    __syncthreads();
    each([&](uint32_t key, uint32_t gl) {
      if (key >= in.lo && key - in.lo <= in.span) atomicAdd(&sh.hist[(key - in.lo) >> shift], gl & 15u);
    });
    __syncthreads();
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = sh.hist[kSelBins - 1 - tid * 4 - j];
    find_bin(h, k, sh);
    k = sh.rank;
    in = part_range(in, sh.bin, shift);
    each([&](uint32_t key, uint32_t gl) {
      if (key >= in.lo && key - in.lo <= in.span) {
        const uint32_t at = atomicAdd(&sh.n_cand, 1u);
        if (at < (uint32_t)kSelCand) sh.cand[at] = make_uint2(key, gl);
      }
    });
    __syncthreads();
    n_cand = (int)sh.n_cand;
  }
  if (n_cand <= kSelCand) {
    if (tid < n_cand) {
      const uint32_t ki = sh.cand[tid].x;
      uint32_t above = 0, upto = 0;
      for (int j = 0; j < n_cand; ++j) {
        const uint2 o = sh.cand[j];
        above += o.x > ki ? o.y & 15u : 0u;
        upto += o.x >= ki ? o.y & 15u : 0u;
      }
      if (above < k && k <= upto) {  // equal keys write the same pair
        sh.tau = ki;
        sh.need = k - above;
      }
    }
    __syncthreads();
    tau = sh.tau;
    need_eq = sh.need;
  } else {  // one key left
    tau = in.lo;
    need_eq = k;
  }
  const auto before = [&](uint32_t key, uint32_t gl) {
    const uint32_t len = (gl >> 4) < group0 ? gl & 15u : 0u;
    gt += key > tau ? len : 0u;
    eq += key == tau ? len : 0u;
  };
  if (few) {  // the ones above the bin are in `gt`
    if (tid < n_cand) before(sh.cand[tid].x, sh.cand[tid].y);
  } else {
    gt = 0;
    each(before);
  }
  gt = wave_incl_scan(gt);
  eq = wave_incl_scan(eq);
  if (lane == kWave - 1) {
    sh.wsum[0][wave] = gt;
    sh.wsum[1][wave] = eq;
  }
  __syncthreads();
  constexpr int kWaves = kSelT / kWave;
  const auto total = [&](const uint32_t* w) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(lane < kWaves ? w[lane] : 0u), kWaves - 1);
  };
  gt_before = total(sh.wsum[0]);
  eq_before = total(sh.wsum[1]);
  __syncthreads();
}

__global__ __launch_bounds__(kSelT) void snap_select_kernel(CacheView c, SnapArgs a) {
  __shared__ SelShared sh;
  const int tid = threadIdx.x;
  const int unit = blockIdx.y, slice = blockIdx.x;
  const int b = unit / c.n_kv_heads, g = unit % c.n_kv_heads;
  const int S = c.seq_lens[b];
  int32_t* kept = a.kept + (int64_t)unit * a.keep;
  int32_t* kept2 = a.kept_user ? a.kept_user + (int64_t)unit * a.kept_stride : nullptr;
  const bool small = S <= a.keep;
  const bool bad = S > c.pages_cap * kAttnPage;
  if (small || bad) {
    if (slice != 0) return;
    const int cnt = bad ? 0 : S;
    for (int i = tid; i < a.keep; i += kSelT) {
      const int v = i < cnt ? i : -1;
      kept[i] = v;
      if (kept2) kept2[i] = v;
    }
    if (g == 0 && tid == 0) a.n_out[b] = cnt;
    return;
  }
  const int L = S - a.W;
  const int k_pref = a.keep - a.W;
  const int blocks = (L + kSelSlice - 1) / kSelSlice, per = (blocks + a.sel_split - 1) / a.sel_split;
  const int j_begin = slice * per * kSelSlice, j_end = min(j_begin + per * kSelSlice, L);
  if (j_begin >= L) return;
  // the slice's first votes travel while the threshold is found
  const float* row = a.pooled + (int64_t)unit * a.s_cap;
  const auto load = [&](int j) { return j < L ? *reinterpret_cast<const float4*>(row + j) : make_float4(0.f, 0.f, 0.f, 0.f); };
  float4 v = load(j_begin + tid * 4);

  uint32_t tau, need_eq, gt, eq;
  snap_threshold(a.runs + (int64_t)unit * a.s_cap, (int)a.n_runs[unit * kCountStride], a.hist + (int64_t)unit * kSelBins,
                 (uint32_t)k_pref, (uint32_t)j_begin / 8, sh, tau, need_eq, gt, eq);

  // ordered emission: kSelSlice positions at a time, four neighbours a thread
  for (int j0 = j_begin; j0 < j_end; j0 += kSelSlice) {
    const int j = j0 + tid * 4;
    const float x[4] = {v.x, v.y, v.z, v.w};
    if (j0 + kSelSlice < j_end) v = load(j + kSelSlice);
    uint32_t key[4], cnt = 0;  // low 16 bits: keys above the threshold, high 16 bits: keys at it
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      key[e] = order_key(x[e]);
      if (j + e < j_end) cnt += (key[e] > tau ? 1u : 0u) + (key[e] == tau ? 0x10000u : 0u);
    }
    const uint32_t before = block_excl_scan<kSelT>(cnt, sh.wsum[0]);
    uint32_t mgt = gt + (before & 0xffffu), meq = eq + (before >> 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (j + e >= j_end || key[e] < tau) continue;
      if (key[e] > tau || meq < need_eq) {
        const uint32_t pos = mgt + min(meq, need_eq);
        if ((int)pos < k_pref) {
          kept[pos] = j + e;
          if (kept2) kept2[pos] = j + e;
        }
      }
      if (key[e] > tau) ++mgt; else ++meq;
    }
    if (j0 + kSelSlice < j_end) {  // what this block adds to the ones after it
      if (tid == kSelT - 1) {
        sh.rank = (before & 0xffffu) + (cnt & 0xffffu);
        sh.need = (before >> 16) + (cnt >> 16);
      }
      __syncthreads();
      gt += sh.rank;
      eq += sh.need;
      __syncthreads();
    }
  }
  if (slice == 0) {
    for (int w = tid; w < a.W; w += kSelT) {
      kept[k_pref + w] = L + w;
      if (kept2) kept2[k_pref + w] = L + w;
    }
    if (g == 0 && tid == 0) a.n_out[b] = a.keep;
  }
}

// copy the kept tokens into the destination cache; one workgroup per kGatherBlocks x 16 kept tokens
// (each workgroup is a chain of dependent round trips: index, rows, stores; several blocks per
// workgroup put several times the loads in flight behind one such chain).  K rows move as 256-byte
// rows.  The V values of 16 tokens are staged in LDS as [channel][token] whatever the source layout,
// then leave as one contiguous channel-major tile (page size 16) or as token rows.
constexpr int kGatherBlocks = 4;
__global__ __launch_bounds__(256) void snap_gather_kernel(CacheView src, CacheView dst, SnapArgs a) {
  constexpr int NB = kGatherBlocks, NTOK = NB * kAttnPage;
  __shared__ int s_tok[NTOK];
  __shared__ int64_t s_src[NTOK];  // element offset of the token's source tile (page and head), or -1
  __shared__ __align__(16) bf16_t s_v[NB][kHeadDim * kAttnPage];
  const int tid = threadIdx.x;
  const int unit = blockIdx.y, blk0 = blockIdx.x * NB;
  const int b = unit / src.n_kv_heads, g = unit % src.n_kv_heads;
  const int S = src.seq_lens[b];
  const int cnt = S > src.pages_cap * kAttnPage ? 0 : min(S, a.keep);
  if (blk0 * kAttnPage >= cnt) return;
  const int64_t dhead = (int64_t)g * dst.stride_head, shead = (int64_t)g * src.stride_head;
  if (tid < NTOK) {
    const int t = blk0 * kAttnPage + tid;
    const int tok = t < cnt ? a.kept[(int64_t)unit * a.keep + t] : -1;
    const int64_t spp = tok >= 0 ? phys_page(src, b, tok / kAttnPage) : -1;
    s_tok[tid] = spp >= 0 ? tok : -1;
    s_src[tid] = spp >= 0 ? spp * src.stride_page + shead : -1;
  }
  __syncthreads();
  const int dps = dst.page_size;
  // rows: thread -> (row = tid/16 of each block, 16-byte piece = tid%16)
  const int row = tid / 16, piece = tid % 16;
  int tok[NB];
  int64_t so[NB], dof[NB];  // source tile, destination row (-1: none)
  bool in_cnt[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    tok[i] = s_tok[i * kAttnPage + row];
    so[i] = s_src[i * kAttnPage + row];
    const int dt = (blk0 + i) * kAttnPage + row;  // destination position of this thread's row
    in_cnt[i] = (blk0 + i) * kAttnPage < cnt;     // the block exists at all
    const int64_t dpp = (in_cnt[i] && dt / dps < dst.pages_cap) ? phys_page(dst, b, dt / dps) : -1;
    dof[i] = dpp >= 0 ? dpp * dst.stride_page + dhead + (dt % dps) * kHeadDim + piece * 8 : -1;
  }
  // the K rows: loaded now, stored after the V loads have gone out as well (one wait for both)
  uint4 kval[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    kval[i] = make_uint4(0, 0, 0, 0);
    if (tok[i] >= 0) kval[i] = ld16<false>(src.k_pool + so[i] + (tok[i] % kAttnPage) * kHeadDim + piece * 8);
  }
  // a channel-major destination gets whole tiles (zero rows past the end); a token-major one only
  // the rows that exist, as later pages may belong to something else
  const auto store_k = [&]() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (dof[i] >= 0 && (tok[i] >= 0 || !dst.v_token_major)) *reinterpret_cast<uint4*>(dst.k_pool + dof[i]) = kval[i];
  };
  if (src.v_token_major && dst.v_token_major) {
    uint4 val[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (tok[i] >= 0) val[i] = ld16<false>(src.v_pool + so[i] + (tok[i] % kAttnPage) * kHeadDim + piece * 8);
    store_k();
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (tok[i] >= 0 && dof[i] >= 0) *reinterpret_cast<uint4*>(dst.v_pool + dof[i]) = val[i];
    return;
  }
  // stage V as s_v[block][channel][token]
  if (src.v_token_major) {
    uint4 val[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      val[i] = make_uint4(0, 0, 0, 0);
      if (tok[i] >= 0) val[i] = ld16<false>(src.v_pool + so[i] + (tok[i] % kAttnPage) * kHeadDim + piece * 8);
    }
    store_k();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const uint32_t w[4] = {val[i].x, val[i].y, val[i].z, val[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s_v[i][(piece * 8 + 2 * e) * kAttnPage + row] = (bf16_t)(w[e] & 0xffffu);
        s_v[i][(piece * 8 + 2 * e + 1) * kAttnPage + row] = (bf16_t)(w[e] >> 16);
      }
    }
  } else {
    // thread -> (slot = tid%16, channels tid/16 + 16 j): the loads of all blocks go out before the first LDS store
    const int slot = tid % kAttnPage, ch0 = tid / kAttnPage;
    bf16_t val[NB][8];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int tk = s_tok[i * kAttnPage + slot];
      const int64_t sv = s_src[i * kAttnPage + slot];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        val[i][j] = 0;
        if (tk >= 0) val[i][j] = src.v_pool[sv + (ch0 + 16 * j) * kAttnPage + tk % kAttnPage];
      }
    }
    store_k();
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) s_v[i][(ch0 + 16 * j) * kAttnPage + slot] = val[i][j];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (!dst.v_token_major) {
      // page size 16: the staged block is the destination tile
      const int dt0 = (blk0 + i) * kAttnPage;
      const int64_t dpp = (in_cnt[i] && dt0 / kAttnPage < dst.pages_cap) ? phys_page(dst, b, dt0 / kAttnPage) : -1;
      if (dpp >= 0)
        reinterpret_cast<uint4*>(dst.v_pool + dpp * dst.stride_page + dhead)[tid] =
            reinterpret_cast<const uint4*>(s_v[i])[tid];
    } else if (tok[i] >= 0 && dof[i] >= 0) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = (uint32_t)s_v[i][(piece * 8 + 2 * e) * kAttnPage + row] |
               ((uint32_t)s_v[i][(piece * 8 + 2 * e + 1) * kAttnPage + row] << 16);
      *reinterpret_cast<uint4*>(dst.v_pool + dof[i]) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

SnapPlan plan_snapkv(const CacheView& src, int window, int keep) {
  SnapPlan p;
  const size_t units = (size_t)src.batch * src.n_kv_heads;
  const int NC = src.group * window;
  // Pages per workgroup in the score passes.  A workgroup fetches its query block before its first page, which long
  // chunks amortise; short ones keep the chip full when there are few (sequence, KV head) units.
  // Up to 32 pages: doubled while there are more than 256 workgroups, one per compute unit.  With 32 pages from the
  // start a short prompt left most of the chip idle.  us a call with the summaries, 32 pages / by this rule, 8 KV
  // heads: 1 x 2048 tokens 43.9 / 37.0, 1 x 4100 46.7 / 41.2, 1 x 8192 51.4 / 48.8, 2 x 4096 47.4 / 43.3; with 64
  // query heads 1 x 5000 56.5 / 47.4.  Why one and not two per compute unit: 1 x 12000 takes 51.5 with 188 workgroups of
  // 32 pages, 53.4 with 376 of 16; 4 heads 1 x 18000 45.1 with 141, 46.4 with 282.
  // Beyond: doubled while there are more than 512 (1 x 131072 takes 153 us a call so, 158 at a bound of
  // 1024 and 170 at 2048), up to 128 pages.  Longer ones, in one round over the chip, are faster on keys seen
  // before and slower on new ones, where the workgroups are less alike: 16 x 32768 tokens 536 us a call on the same
  // keys and 620 a layer in the benchmark's set-up loop with 512 pages, 545 and 592 with 128.
  static_assert(kSnapMaxChunkPages <= 2 * 2 * kSnapMaxPairs, "a pair per lane, also where two wavefronts share a chunk's pages");
  const auto workgroups = [&](int pages) { return units * ((src.pages_cap + pages - 1) / pages); };
  int chunk_pages = 8;  // a pair for each of four wavefronts
  while (chunk_pages < 32 && workgroups(chunk_pages) > 256) chunk_pages *= 2;
  while (chunk_pages < kSnapMaxChunkPages && workgroups(chunk_pages) > 512) chunk_pages *= 2;
  p.chunk_pages = chunk_pages;
  p.n_chunks = (src.pages_cap + chunk_pages - 1) / chunk_pages;
  const size_t s_cap = (size_t)src.pages_cap * kAttnPage;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t off = 0;
  p.stats_off = off;
  off += up(units * NC * 2 * sizeof(float));
  p.votes_off = off;
  off += up(units * s_cap * sizeof(float));
  p.pooled_off = off;
  off += up(units * s_cap * sizeof(float));
  p.kept_off = off;
  off += up(units * (size_t)keep * sizeof(int32_t));
  // the select: one round of workgroups over the chip, slices of kSelSlice positions or more
  const size_t slices = (s_cap + kSelSlice - 1) / kSelSlice;
  p.sel_split = (int)(units >= 256 ? 1 : 256 / units);
  if ((size_t)p.sel_split > slices) p.sel_split = (int)slices;
  p.runs_off = off;
  off += up(units * s_cap * sizeof(uint2));
  // The chunk statistics lie where the pool and the select write, launches after their last reader: 192 bytes a page
  // and the kept indices, which up to 192 softmax rows fit at any chunk.  More rows take up to 256 bytes a page.  What is
  // reserved then is what the rule above reaches for this capacity or any smaller one (256 workgroups of 8 or 16
  // pages, 512 of 32 or 64), and not what this capacity's chunks take: a workspace sized for the longest prompt serves
  // every shorter one.
  p.stats_part_off = p.pooled_off;
  const size_t most = std::max({std::min<size_t>(workgroups(8), 256), std::min<size_t>(workgroups(32), 512),
                                (size_t)workgroups(kSnapMaxChunkPages)});
  off = std::max(off, p.stats_part_off + up(most * NC * 2 * sizeof(float)));
  p.counts_off = off;
  off += up(units * (kCountStride + kSelBins) * sizeof(uint32_t));
  p.total_bytes = off;
  return p;
}

hipError_t launch_snapkv(const bf16_t* q_obs, const CacheView& src, int window, int pool_kernel,
                         int keep, const CacheView* dst, int32_t* kept_idx, int kept_stride,
                         int32_t* n_out, void* ws, const SnapPlan& plan, hipStream_t st) {
  const int units = src.batch * src.n_kv_heads;
  char* base = static_cast<char*>(ws);
  SnapArgs a;
  a.qobs = q_obs;
  a.W = window;
  a.NC = src.group * window;
  a.CG = a.NC > kSnapCols ? 2 : 1;
  a.n_chunks = plan.n_chunks;
  a.chunk_pages = plan.chunk_pages;
  a.keep = keep;
  a.s_cap = src.pages_cap * kAttnPage;
  a.pool_r = (pool_kernel - 1) / 2;
  a.stats_part = reinterpret_cast<float*>(base + plan.stats_part_off);
  a.stats = reinterpret_cast<float*>(base + plan.stats_off);
  a.votes = reinterpret_cast<float*>(base + plan.votes_off);
  a.pooled = reinterpret_cast<float*>(base + plan.pooled_off);
  a.kept = reinterpret_cast<int32_t*>(base + plan.kept_off);
  a.kept_user = kept_idx;
  a.kept_stride = kept_stride;
  a.n_out = n_out;
  a.runs = reinterpret_cast<uint2*>(base + plan.runs_off);
  a.n_runs = reinterpret_cast<uint32_t*>(base + plan.counts_off);
  a.hist = a.n_runs + (size_t)units * kCountStride;
  a.sel_split = plan.sel_split;

  const dim3 sgrid(plan.n_chunks, units);
  const bool wide = a.NC > kSnapCols / 2;  // some wavefront owns more than two blocks of 32 softmax rows
  if (wide)
    hipLaunchKernelGGL((snap_score_kernel<false, 4>), sgrid, dim3(256), kRingBytes + kSnapStatBytes, st, src, a);
  else
    hipLaunchKernelGGL((snap_score_kernel<false, 2>), sgrid, dim3(256), kRingBytes + kSnapStatBytes, st, src, a);
  const bool merge = plan.n_chunks * a.NC <= kMergeStats && plan.n_chunks * units <= kMergeWorkgroups;
  if (!merge) hipLaunchKernelGGL(snap_stats_kernel, dim3(units), dim3(kStatsT), 0, st, src, a);
  const auto pass2 = [&](auto kernel) { hipLaunchKernelGGL(kernel, sgrid, dim3(256), kRingBytes + kSnapVoteBytes, st, src, a); };
  if (merge) {
    if (wide) pass2(snap_score_kernel<true, 4, true>); else pass2(snap_score_kernel<true, 2, true>);
  } else {
    if (wide) pass2(snap_score_kernel<true, 4>); else pass2(snap_score_kernel<true, 2>);
  }
  const dim3 pgrid((a.s_cap + kPoolTile - 1) / kPoolTile, units);
  const size_t pool_groups = kPoolT + 2 * ((a.pool_r + 7) / 8);
  hipLaunchKernelGGL(snap_pool_kernel, pgrid, dim3(kPoolT), pool_groups * 10 * sizeof(float), st, src, a);
  hipLaunchKernelGGL(snap_select_kernel, dim3(plan.sel_split, units), dim3(kSelT), 0, st, src, a);
  if (!dst) return hipGetLastError();  // filter only: the indices are the result
  const dim3 ggrid((keep + kGatherBlocks * kAttnPage - 1) / (kGatherBlocks * kAttnPage), units);
  hipLaunchKernelGGL(snap_gather_kernel, ggrid, dim3(256), 0, st, src, *dst, a);
  return hipGetLastError();
}

}  // namespace rkv
