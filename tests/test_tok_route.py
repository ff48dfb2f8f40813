"""The rule by which a decode step over a token-major cache with large summaries takes one launch or several
(csrc/tok_route.h), on the host: at shapes next to its lines, where both were timed on the GPU and differ by 4 % or
more, it takes the faster side."""
import subprocess

from paper_2502_14051_amd import build as libbuild

DRIVER = r"""
#include <stdio.h>
#include "tok_route.h"
using namespace rkv;
int main() {
  int v[9];
  while (scanf("%d %d %d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7, v + 8) == 9)
    printf("%d\n", (int)tok_one_launch({v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8] != 0}));
}
"""

# units, pages of the cache, channels; wavefronts, workgroups a unit, entries a workgroup, entries of the attention's
# plan; through an index; us a layer in one launch, and otherwise
TIMED = [
    (320, 2032, 90, 4, 1, 46, 45, False, 74.4, 81.0), (264, 2024, 90, 4, 2, 64, 128, False, 129.4, 123.7),
    (320, 1256, 120, 4, 2, 64, 128, False, 125.8, 135.7), (128, 744, 120, 4, 2, 10, 18, False, 33.6, 32.2),
    (4, 704, 96, 4, 6, 8, 45, False, 25.6, 27.2), (200, 2048, 32, 4, 2, 10, 18, False, 39.6, 37.1),
    (144, 712, 96, 4, 2, 12, 24, False, 37.2, 39.2), (172, 1544, 81, 4, 1, 16, 15, False, 33.4, 30.2),
    (96, 3584, 32, 8, 2, 24, 45, False, 31.3, 29.8), (8, 1496, 90, 8, 3, 16, 45, False, 21.2, 23.2),
    (32, 2520, 60, 8, 1, 16, 8, False, 23.1, 20.5), (8, 1496, 90, 8, 1, 16, 8, False, 17.7, 19.0),
    (256, 4056, 90, 8, 1, 46, 45, False, 72.1, 76.5), (72, 984, 90, 8, 4, 32, 128, False, 48.6, 43.2),
    (96, 984, 90, 8, 3, 48, 128, False, 52.1, 49.0), (72, 1496, 90, 8, 4, 32, 100, False, 40.4, 44.0),
    (136, 984, 90, 8, 2, 64, 128, False, 71.7, 67.0), (240, 1496, 60, 8, 2, 32, 45, False, 53.2, 51.1),
    (136, 2520, 60, 8, 2, 32, 56, False, 55.1, 58.4), (136, 3032, 90, 8, 2, 32, 45, False, 62.2, 66.2),
    (296, 4992, 32, 4, 1, 28, 28, False, 65.9, 81.7), (264, 2424, 40, 4, 2, 64, 128, False, 123.9, 118.3),
    (24, 4280, 16, 4, 7, 16, 108, False, 42.5, 33.8), (24, 3288, 81, 4, 1, 8, 8, False, 51.6, 23.4),
    (148, 2256, 96, 4, 3, 36, 103, False, 90.5, 75.3), (216, 2960, 128, 4, 1, 16, 15, False, 77.1, 62.7),
    (232, 3176, 48, 4, 4, 32, 126, False, 129.1, 106.4), (48, 4240, 24, 8, 2, 16, 22, False, 30.5, 26.0),
    (64, 4288, 24, 8, 1, 16, 13, False, 28.4, 24.0), (112, 4328, 48, 8, 3, 32, 77, False, 74.5, 62.2),
    (320, 1496, 120, 4, 1, 46, 45, True, 71.7, 83.5), (416, 1688, 64, 4, 2, 56, 105, True, 125.7, 139.5),
    (16, 2024, 90, 4, 3, 8, 18, True, 37.4, 35.2), (4, 2024, 60, 4, 3, 8, 18, True, 31.1, 32.7),
    (200, 1512, 60, 4, 2, 10, 18, True, 42.0, 46.3), (32, 4056, 60, 8, 2, 16, 18, True, 34.3, 32.2),
    (8, 2520, 120, 8, 3, 16, 45, True, 30.5, 34.2), (32, 3824, 64, 8, 1, 16, 16, True, 34.4, 32.1),
    (8, 2624, 81, 8, 1, 16, 15, True, 23.4, 30.5), (256, 4056, 90, 8, 1, 46, 45, True, 73.8, 80.3),
    (88, 3760, 32, 8, 3, 32, 91, True, 56.3, 50.1), (96, 3032, 90, 8, 3, 48, 128, True, 73.3, 66.8),
    (96, 1496, 120, 8, 3, 32, 93, True, 50.3, 53.6), (120, 712, 128, 8, 3, 32, 82, True, 49.7, 55.8),
    (136, 4096, 32, 8, 2, 64, 128, True, 82.8, 77.0), (192, 3032, 90, 8, 2, 32, 45, True, 75.5, 68.5),
    (136, 1496, 120, 8, 2, 48, 93, True, 61.8, 66.9), (136, 4096, 32, 8, 2, 32, 45, True, 50.9, 54.6),
    (408, 2400, 81, 4, 1, 20, 19, True, 74.2, 69.8), (320, 2424, 60, 4, 1, 46, 45, True, 76.3, 80.1),
    (272, 2072, 48, 4, 2, 56, 111, True, 106.9, 102.5), (4, 2424, 32, 4, 6, 8, 45, True, 35.5, 32.0),
    (8, 4168, 40, 8, 3, 16, 45, True, 32.5, 31.2), (8, 4168, 32, 8, 3, 16, 45, True, 28.8, 31.5),
    (112, 4688, 128, 8, 1, 16, 9, True, 72.7, 59.8), (152, 4560, 64, 8, 1, 16, 9, True, 48.1, 43.9),
    (256, 4168, 32, 8, 1, 46, 45, True, 52.3, 62.2), (96, 4168, 20, 8, 3, 48, 128, True, 65.7, 62.3),
    (136, 4168, 20, 8, 2, 64, 128, True, 81.4, 76.1), (192, 4168, 32, 8, 2, 32, 45, True, 67.3, 62.7),
]


def test_the_faster_side(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I" + libbuild.CSRC, str(src), "-o", str(exe)], check=True)
    ask = []
    for units, pages, k1, waves, n_split, chunk, entries, indexed, _, _ in TIMED:
        rounds = -(-pages // (64 * waves))
        ask.append(f"{units} {pages} {k1} {rounds if rounds <= 8 else 0} {waves} {n_split} {chunk} {entries} {int(indexed)}")
    r = subprocess.run([str(exe)], input="\n".join(ask), capture_output=True, text=True, check=True)
    got = [x == "1" for x in r.stdout.split()]
    assert len(got) == len(TIMED)
    wrong = [t for t, one in zip(TIMED, got) if one != (t[-2] < t[-1])]
    assert not wrong, wrong
