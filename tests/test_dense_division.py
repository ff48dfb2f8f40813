"""The arithmetic by which the Full-KV baseline divides sequences between workgroups (csrc/dense_division.h), swept
on the host over batch sizes, KV heads, capacities and lengths: the workgroups never exceed the launch, also
with a reciprocal that is off by a unit in the last place, and the work they get is balanced: run in order
on the workgroups the chip holds, they are done within a bounded multiple of an even share."""
import subprocess

import pytest

from paper_2502_14051_amd import build as libbuild

DRIVER = r"""
#include <algorithm>
#include <functional>
#include <queue>
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "dense_division.h"
using namespace rkv;
static uint64_t state = 1;
static uint32_t rnd(uint32_t n) {  // [0, n)
  state = state * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)((state >> 33) % n);
}
static double worst = 0;
static void check(int H, const std::vector<int>& P, int row_len, float err) {
  const int B = (int)P.size(), waves = B * H > 256 ? 4 : 8, slots = 2048 / waves, least = 2 * waves;
  const DenseGrid g = dense_grid(B, H, row_len, slots, least);
  int total = 0, longest = 0;
  for (int p : P) total += p, longest = std::max(longest, p);
  const auto count = [&](float rc) { int w = 0; for (int p : P) w += dense_shares(p, rc); return w; };
  const auto rcp = [&](float x) { return 1.0f / x * (1.0f + err); };
  const int last = dense_last(g, B, total, least);
  const float rc = dense_rate(g, B, total, last, [&] { return (float)longest; }, least, rcp, count);
  const int n = count(rc);
  bool ok = n >= B && n <= g.limit && n <= dense_most(g, B, last);
  for (int p : P) ok = ok && dense_shares(p, rc) >= 1 && dense_shares(p, rc) <= std::max(1, (p + least - 1) / least);
  if (!ok) {
    printf("B %d H %d row_len %d total %d: %d workgroups of %d launched\n", B, H, row_len, total, n, g.limit);
    exit(1);
  }
  if (err != 0.f || total < 24 * least * slots / H) return;
  // share by share, every head of it: the next workgroup goes where one ends first
  std::priority_queue<long, std::vector<long>, std::greater<long>> busy;
  for (int i = 0; i < slots; ++i) busy.push(0);
  long end = 0;
  for (int p : P) {
    const int w = dense_shares(p, rc), chunk = (p + w - 1) / w;
    for (int i = 0; i < w * H; ++i) {
      const long t = busy.top() + std::max(0, std::min(chunk, p - i / H * chunk));
      busy.pop();
      busy.push(t);
      end = std::max(end, t);
    }
  }
  const double ratio = (double)end * slots / ((double)total * H);
  if (ratio > worst) {
    worst = ratio;
    printf("%.3f of an even share: B %d H %d row_len %d total %d, %d workgroups of at most %d pages\n", ratio, B, H, row_len, total, n, (int)(1 / rc));
  }
}
int main(int argc, char** argv) {
  const int H = atoi(argv[1]);
  for (int B = 1; B <= kDenseMaxBatch; ++B)
    for (int row_len : {48, 100, 128, 257, 512, 2048, 8192})
      for (int form = 0; form < 8; ++form) {
        std::vector<int> P(B);
        for (int b = 0; b < B; ++b) {
          const int any = (int)rnd(row_len + 1);
          P[b] = form == 0 ? row_len : form == 1 ? any : form == 2 ? any * (int)rnd(2) : form == 3 ? (b == B / 2 ? row_len : (int)rnd(3))
               : form == 4 ? (int)((long)any * any / row_len) : form == 5 ? row_len - (b % 2) * (row_len / 2) : form == 6 ? any / 64 : row_len + 1;  // a last page of fewer than 16 slots
        }
        for (float err : {0.f, 1.2e-7f, -1.2e-7f}) check(H, P, row_len, err);
      }
  printf("worst %.3f\n", worst);
  return worst <= atof(argv[2]) ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("dense_division")
    src, exe = d / "driver.cpp", d / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-I" + libbuild.CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


# What the division may cost at most in this model, which gives every workgroup the same rate: rounding up, the
# fifth that the cost of a round forgives, and start-ups not spent on evening out less than they take.  Fitting
# one round whatever the rounding costs reaches 12 here.
@pytest.mark.parametrize("heads", [1, 2, 3, 4, 8, 16, 40, 96])
def test_division(driver, heads):
    r = subprocess.run([driver, str(heads), "1.6"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
