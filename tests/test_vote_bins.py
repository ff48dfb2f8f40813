"""The bins that Stage 1's select narrows the votes down with (csrc/vote_bins.h), walked on the host: the bins of
the first pass and the parts a crowded bin is divided into each cover their range once, and the search they
serve finds the wanted rank of any vote, also where only the division of the lowest bin decides."""
import subprocess

import numpy as np
import pytest

from paper_2502_14051_amd import build as libbuild

DRIVER = r"""
#include <algorithm>
#include <functional>
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "vote_bins.h"
using namespace rkv;
static void fail(const char* what, unsigned a, unsigned b) { printf("%s: %#x %#x\n", what, a, b); exit(1); }
static void parts_cover(KeyRange r) {
  const int shift = part_shift(r);
  const uint32_t n = (r.span >> shift) + 1u;
  if (n > (uint32_t)kSelBins) fail("too many parts", r.lo, r.span);
  uint64_t next = r.lo;
  for (uint32_t p = 0; p < n; ++p) {
    const KeyRange x = part_range(r, p, shift);
    if (x.lo != next || ((x.lo - r.lo) >> shift) != p || ((x.lo + x.span - r.lo) >> shift) != p) fail("part", r.lo, p);
    next = (uint64_t)x.lo + x.span + 1u;
  }
  if (next != (uint64_t)r.lo + r.span + 1u) fail("the parts do not end with the range", r.lo, (unsigned)next);
}
// the select's search: the bin of the wanted rank, divided until `few` keys are left
static uint32_t kth(const std::vector<uint32_t>& keys, uint32_t k, size_t few, uint32_t* rank) {
  std::vector<uint32_t> h(kSelBins);
  const auto find = [&] {
    int b = kSelBins - 1;
    while (k > h[b]) k -= h[b--];
    return (uint32_t)b;
  };
  for (uint32_t x : keys) ++h[vote_bin(x)];
  KeyRange in = bin_range(find());
  std::vector<uint32_t> cand;
  const auto collect = [&] {
    cand.clear();
    for (uint32_t x : keys) if (x >= in.lo && x - in.lo <= in.span) cand.push_back(x);
  };
  collect();
  while (cand.size() > few && in.span != 0u) {
    const int shift = part_shift(in);
    std::fill(h.begin(), h.end(), 0u);
    for (uint32_t x : cand) ++h[(x - in.lo) >> shift];
    in = part_range(in, find(), shift);
    collect();
  }
  std::sort(cand.begin(), cand.end(), std::greater<uint32_t>());
  *rank = k;
  return k <= cand.size() ? cand[k - 1] : 0u;
}
int main(int argc, char** argv) {
  if (argc == 1) {
    uint64_t next = 0;
    for (int b = 0; b < kSelBins; ++b) {
      const KeyRange r = bin_range(b);
      if (r.lo != next || vote_bin(r.lo) != (uint32_t)b || vote_bin(r.lo + r.span) != (uint32_t)b) fail("bin", b, r.lo);
      next = (uint64_t)r.lo + r.span + 1u;
      for (KeyRange x = r; x.span != 0u; x = part_range(x, x.span >> part_shift(x), part_shift(x))) parts_cover(x);
    }
    if (next != 1ull << 32) fail("the bins do not cover the keys", (unsigned)next, 0);
    return 0;
  }
  std::vector<uint32_t> keys;
  uint32_t x;
  FILE* f = fopen(argv[1], "rb");
  while (fread(&x, 4, 1, f) == 1) keys.push_back(x);
  fclose(f);
  std::vector<uint32_t> sorted = keys;
  std::sort(sorted.begin(), sorted.end(), std::greater<uint32_t>());
  for (size_t k = 1; k <= keys.size(); k += atoi(argv[2])) {
    uint32_t rank;
    const uint32_t got = kth(keys, (uint32_t)k, 512, &rank);
    if (got != sorted[k - 1]) fail("rank", (unsigned)k, got);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("vote_bins")
    src, exe = d / "driver.cpp", d / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I" + libbuild.CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def run(*cmd):
    r = subprocess.run([str(c) for c in cmd], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_bins_and_parts_cover_their_ranges(driver):
    run(driver)


@pytest.mark.parametrize("low,high", [
    (2.0**-60, 2.0**-56 * 1.2),       # into the lowest bin, the wanted vote among smaller and slightly larger ones
    (2.0**-56, 2.0**-56 * (1 + 8 / 64)),
    (0.0, 2.0**-120),                 # all of them below the bins
    (2.0**9, 2.0**20),                # all of them above
    (0.5, 0.5 * (1 + 1 / 128)),       # one crowded bin inside
])
def test_search_finds_every_rank(driver, tmp_path, low, high):
    rng = np.random.default_rng(7)
    u = rng.random(9000)
    v = (low + u * (high - low)) if low == 0.0 else low * (high / low) ** u
    bits = v.astype(np.float32).view(np.uint32)
    keys = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000)).astype(np.uint32)
    (tmp_path / "keys").write_bytes(keys.tobytes())
    run(driver, tmp_path / "keys", 13)
