// How the Full-KV baseline divides the pages its sequences hold between workgroups.  Plain constexpr
// arithmetic that needs no device, so a host program can sweep it.
//
// Per KV head, a sequence of P pages gets max(1, ceil(P / c)) workgroups and divides its pages evenly
// between those; a workgroup works for one unit only and never meets another one's.  HBM bounds the
// kernel as long as every compute unit has a share of the stream to the end, so c is the smallest whose
// workgroups fit one, two or four rounds over the chip:
//   - one round has no start-up but its own, and is what most calls get;
//   - but with about as many sequences as workgroups, rounding up to whole workgroups leaves compute
//     units idle or one with a multiple of the others' pages.  Shares of half or a quarter of the size
//     even that out for the price of a start-up per round.
// us a call, 8 KV heads, one round / two / four and (in brackets) the capacity divided instead: 33 sequences of
// 8192 tokens 254 / 200 / 184 (186); 28 of unequal lengths up to 8192 73 / 59 / 65 (120); 17 of 32768
// 408 / 355 / 344 (360); 11 of 8192 64 / 66 / 72 (67); 28 of 2048 40 / 47 / 56 (51).
#pragma once
#include <stdint.h>

namespace rkv {

constexpr int kDenseMaxBatch = 128; // two sequences per lane of a wavefront

struct DenseGrid {  // per KV head
  int limit;  // workgroups launched, what any lengths can ask for
  int last;   // what dense_last may return
  int aim;    // workgroups of one round
};

// The candidates for `total` pages are 1 << 0 .. 1 << dense_last rounds.  More are looked at only where rounding
// can cost much (at most batch / (aim - batch): a fifth at a sixth of the workgroups), and where the launch is
// long enough to win that back (some 40 us for two rounds, 120 for four).  Increasing in `total`.
constexpr int dense_last(const DenseGrid& g, int batch, int total, int least) {
  const int unit = least * g.aim;
  int last = 0;
  if (6 * batch > g.aim && total >= 8 * unit) last = 2 * batch > g.aim && total >= 24 * unit ? 2 : 1;
  while (last < 2 && g.aim << last < batch) ++last;
  return last < g.last ? last : g.last;
}

// The last candidate may also take shares of exactly total / aim, a round more of them: fewer than aim + batch.
constexpr bool dense_open(const DenseGrid& g, int batch, int last) {
  return (last == 0 ? 2 : 4) * batch > g.aim << last;
}
constexpr int dense_most(const DenseGrid& g, int batch, int last) {
  return (g.aim << last) + (dense_open(g, batch, last) ? batch : 0);
}

// `slots`: workgroups the chip runs at once; `row_len`: pages of a sequence at most; `least`: pages the
// smallest sensible share has.  Workgroups that a division leaves over come only to find that out (14
// sequences of 2048 tokens take 13.8 us, 16.9 with four times the workgroups), so the launch holds what the
// capacity can ask for and no more.
constexpr DenseGrid dense_grid(int batch, int n_kv_heads, int row_len, int slots, int least) {
  DenseGrid g = {0, 2, slots / n_kv_heads > 1 ? slots / n_kv_heads : 1};
  const int64_t total = (int64_t)batch * row_len;
  g.last = dense_last(g, batch, total < 1 << 30 ? (int)total : 1 << 30, least);
  g.limit = dense_most(g, batch, g.last);
  const int64_t most = (int64_t)batch * (row_len / least + 2);
  if (g.limit > most) g.limit = (int)most;
  return g;
}

// workgroups of a sequence for shares of c pages, rc just below 1 / c (dense_rate): whatever the
// rounding makes of the quotient, it is the same wherever it is formed, and any number of workgroups
// divides the pages
constexpr int dense_shares(int pages, float rc) {
  const float x = (float)pages * rc;
  const int w = (int)x;
  return w < 1 ? 1 : w + (int)((float)w < x);
}

// 1 / c for the lengths of a call: `total` pages in all, longest() in one sequence; count(rc) sums
// dense_shares over the sequences, rcp(x) is about 1 / x.  What R rounds of c pages cost, in pages at the
// rate of the whole chip (0.3 us, twice that at two workgroups per compute unit): an even share, or
// (R - 0.2) c if that is more (in a round that does not fill the chip the others draw up to a fifth more),
// R start-ups of some 6 us, and a twentieth of c for the drift of long shares: 16 sequences of 32768 tokens in one
// exact round of 1024 pages take 332 us, in two 322, in four 319; 31 of them 631, 631, 606.
// The loops stay loops: unrolled, the code every workgroup fetches before its first page is twice as
// long (0.3 us of 10).
template <class Longest, class Rcp, class Count>
constexpr float dense_rate(const DenseGrid& grid, int batch, int total, int last, const Longest& longest, int least,
                           const Rcp& rcp, const Count& count) {
  const auto rate = [&](float c) { return rcp(c) * 0.999998f; };  // just below, so that a share of k c is k
  const float start = 1.5f * (float)least;
  const float share = (float)total * rcp((float)grid.aim);
  const auto cost_of = [&](float rounds, float c) {
    const float stream = (rounds - 0.2f) * c;
    return (stream > share ? stream : share) + rounds * start + 0.05f * c;
  };
  float best = 0.f, best_cost = 3.0e38f;
#pragma unroll 1
  for (int i = 0; i <= last; ++i) {
    const int aim = grid.aim << i;
    const bool open = i == last && dense_open(grid, batch, i) && aim + batch <= grid.limit;
    if (aim < batch && !open) continue;
    const float even = (float)total * rcp((float)aim);
    float rounds = (float)(1 << i), c = even > (float)least ? even : (float)least;
    if (cost_of(rounds, c) >= best_cost) break;  // nothing left to win
    if (count(rate(c)) > aim) {
      // The smallest that fits lies below total / (aim - batch), which makes fewer than (aim - batch) + batch,
      // and below what gives the longest sequence an equal part of the workgroups (rounded down: aim / batch
      // is a whole number or far from the next).  A step takes about as long as half a page.
      float lo = c, hi = longest();
      if (aim >= batch) hi *= rcp((float)(int)((float)aim * rcp((float)batch))) * 1.000002f;
      if (aim > batch) {
        const float sure = (float)total * rcp((float)(aim - batch));
        hi = hi < sure ? hi : sure;
      }
#pragma unroll 1
      for (int k = 0; k < 4 && aim >= batch && hi - lo > 0.15f * (float)least; ++k) {
        const float mid = 0.5f * (lo + hi);
        if (count(rate(mid)) > aim) lo = mid; else hi = mid;
      }
      // a round more of the smaller ones instead?
      if (open && (aim < batch || cost_of(rounds + 1.0f, c) < cost_of(rounds, hi))) rounds += 1.0f;
      else c = hi;
    }
    const float cost = cost_of(rounds, c);
    if (cost < best_cost) {
      best_cost = cost;
      best = rate(c);
    }
  }
  return best;
}

}  // namespace rkv
