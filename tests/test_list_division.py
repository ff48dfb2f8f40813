"""The division of a page list between workgroups (csrc/list_division.h), swept on the host: every entry has
one workgroup and one wavefront, in whole pairs and never more workgroups than asked for; shares are equal to
a pair where all workgroups run at once, and as long as whole rounds of the wavefronts where some wait."""
import subprocess

from paper_2502_14051_amd import build as libbuild

DRIVER = r"""
#include <initializer_list>
#include <stdio.h>
#include "list_division.h"
using namespace rkv;
int main() {
  for (int waves : {4, 8})
    for (int n_wg = 1; n_wg <= 40; ++n_wg)
      for (int row = 1; row <= 1500; ++row)
        for (int full = 0; full < 2; ++full) {
          const ListShares s = list_shares(row, n_wg, waves, [&](int) { return full == 0; });
          const int last = row - (s.n_split - 1) * s.chunk;
          bool ok = s.n_split >= 1 && s.n_split <= n_wg && s.chunk % 2 == 0 && s.per_wave % 2 == 0 && s.per_wave * waves >= s.chunk;
          ok = ok && last >= 1 && last <= s.chunk;
          // waiting workgroups, or one pair a wavefront: whole rounds of the wavefronts
          if (full || s.per_wave == 2) ok = ok && s.chunk == s.per_wave * waves;
          // otherwise nobody has a pair more than an even share
          else ok = ok && s.chunk * s.n_split < row + 2 * s.n_split;
          if (!ok) {
            printf("waves %d n_wg %d row %d full %d: %d x %d, %d a wavefront\n", waves, n_wg, row, full, s.n_split, s.chunk, s.per_wave);
            return 1;
          }
        }
  return 0;
}
"""


def test_list_shares(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I" + libbuild.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
