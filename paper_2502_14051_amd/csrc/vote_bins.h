// Bins of the pooled votes (Stage 1's select).  Keys are the ordered bits of a vote, larger vote <=> larger
// key.  Plain constexpr arithmetic that needs no device, so a host program can walk the whole key space.
#pragma once
#include <stdint.h>

namespace rkv {

constexpr int kSelBins = 4096;                         // histogram of the pooled votes, 64 bins to the octave
constexpr uint32_t kBinBase = (127u + 8u - 64u) << 6;  // bins cover 2^-56 .. 2^8; the first and the last take the rest

constexpr uint32_t vote_bin(uint32_t key) {  // monotone in the ordered bits
  if (!(key & 0x80000000u)) return 0u;
  const int x = (int)((key & 0x7fffffffu) >> 17) - (int)kBinBase;
  return x < 0 ? 0u : (x < kSelBins ? (uint32_t)x : (uint32_t)kSelBins - 1u);
}

struct KeyRange {  // the keys [lo, lo + span]
  uint32_t lo, span;
};

constexpr KeyRange bin_range(uint32_t bin) {
  const uint32_t lo = bin == 0u ? 0u : (0x80000000u | ((bin + kBinBase) << 17));
  const uint32_t last = bin == (uint32_t)kSelBins - 1u ? 0xffffffffu : (0x80000000u | ((bin + 1u + kBinBase) << 17)) - 1u;
  return {lo, last - lo};
}

// A range is divided again into at most kSelBins parts of 2^part_shift keys.  Its length need not be a
// multiple of that (bin 0 is [0, 2^-56 (1 + 1/64)), 0xa3820000 keys in parts of 2^20): the last part ends
// where the range does, not among the keys above it.
constexpr int part_shift(KeyRange r) {
  int shift = 0;
  while ((r.span >> shift) >= (uint32_t)kSelBins) ++shift;
  return shift;
}
constexpr KeyRange part_range(KeyRange r, uint32_t part, int shift) {
  const uint32_t off = part << shift, whole = (1u << shift) - 1u, left = r.span - off;
  return {r.lo + off, whole < left ? whole : left};
}

}  // namespace rkv
