// Whether a decode step over a token-major cache with large summaries runs as one launch.  Plain constexpr arithmetic that
// needs no device, so a host program can sweep it.
#pragma once

namespace rkv {

struct TokRoute {
  int units;      // (sequence, KV head) pairs
  int pages_cap;  // of the cache Step 2 works on
  int k1;         // picked channels
  int rounds;     // pages a thread holds in registers (0: scores through LDS)
  int waves, n_split, chunk;  // of the attention's plan
  int entries;    // 16-token entries it divides
  bool indexed;
};

// In one launch every workgroup of a unit reads all of its picked summary rows for itself; otherwise they are divided between
// workgroups, for a launch boundary and the hand-over of the scores (through an index an append launch more, and the scores
// and the top-k apart).  What the rows cost in one launch goes by `steps`: rounds of pages a thread walks, times its batches
// of 32 rows and one for what a round costs whatever the rows.  How many steps are worth a launch depends on how the
// workgroups fill the chip.  us a layer in one launch / otherwise, 8 KV heads a sequence, as many layers as exceed the
// last-level cache (32 of one sequence), by rounds x batches, at a budget of 734 tokens if none is given (over 2169 shapes the
// side taken is 0.35 % behind the faster one on average):
//  - all workgroups run at once: 12 steps.
//      1 sequence   3x3 21.2 / 23.2, 4x2 21.2 / 23.2, 6x1 21.0 / 22.8, 8x1 23.5 / 23.2, 5x2 22.8 / 23.1 (2048 tokens 25.0 / 23.4)
//      4            3x3 24.5 / 24.9, 4x2 24.4 / 24.7, 6x1 23.6 / 24.6, 7x1 25.0 / 24.8, 5x2 26.7 / 24.7
//      8            3x3 26.1 / 26.4, 4x2 25.8 / 26.1, 6x1 25.6 / 25.6, 7x1 26.9 / 26.1, 5x2 28.0 / 26.5
//      14           3x3 30.8 / 31.8, 4x2 30.6 / 30.5, 5x2 34.2 / 32.9, 3x4 34.8 / 34.0, 5x3 39.3 / 36.3
//    Through an index 25; 21 with more than five rounds in two to eight sequences.  Pages of 3: one 7x2 27.4 / 30.4, 6x3
//    29.5 / 31.9, 8x2 30.0 / 30.2; four 31.6 / 32.6, 33.9 / 34.0, 34.1 / 33.0; eight at 300 32.9 / 34.1, 35.9 / 36.0, 35.7 /
//    34.8; sixteen 40.1 / 44.3, 44.5 / 47.7, 43.1 / 46.2.  Of one token, 8x3: one 37.4 / 33.3, sixteen 53.8 / 55.6.
//  - more than 128 units, one workgroup each: as many steps as were measured, 32.  17 sequences of 400 tokens 6x3 43.9 / 51.0,
//    28 6x3 51.2 / 57.1; 32 8x3 72.2 / 76.5; 64 8x3 90.2 / 104.8; 72 8x3 120.4 / 133.7; index, 32 8x3 73.8 / 80.3.
//  - several workgroups a unit, some of which wait for their turn and select then: mostly two launches.  9 sequences of 2048
//    tokens 2x3 48.6 / 43.2, 17 71.7 / 67.0; 17 of 1024 51.4 / 47.9, 24 of 900 4x2 56.9 / 51.5; 24 4x2 53.2 / 51.3, 6x3 74.8 / 70.3.
//    With more than 128 units of more than 2048 pages the score launch, two workgroups of 1024 threads a unit then, has them
//    wait as well: 15 steps (24 5x2 58.0 / 61.2, of 900 60.2 / 62.0, 20 of 2048 6x1 79.0 / 79.3, 5x2 84.9 / 82.7, 24 6x3 above).
//    As many through an index (17 of 2048 3x3 75.7 / 75.7, 3x4 80.5 / 77.7, 6x3 94.3 / 84.0; 24 3x4 58.5 / 62.7, 6x3 75.5 / 68.5).
//    With four wavefronts, two workgroups beside each other, 25 (33 of 2048 5x4 119.9 / 121.6, 8x3 129.4 / 123.7; 40 125.8 /
//    135.7, 136.4 / 140.1; 64 178.4 / 180.2, 197.6 / 186.4).
//    A unit's last share can be shorter than the others.  Where those that wait are no more than the last shares running
//    before them, they start behind these while the longer ones still run: 24 steps with two a unit (last share of 0.41: 17 3x3
//    44.4 / 49.0, 5x3 56.2 / 64.2, 6x3 62.2 / 66.2, 8x3 74.2 / 73.7, 20 6x3 64.2 / 68.8, 8x3 79.3 / 75.1; 0.69: 20 of 1300 3x3 59.2 /
//    60.6, 5x3 72.8 / 76.4; 0.75: 20 of 900 3x3 52.2 / 50.6), 8 where more wait (22 2x3 46.4 / 48.5, 4x2 51.0 / 50.5, 6x3 71.2 /
//    69.2; 28 50.2 / 50.8, 56.8 / 53.0, 82.0 / 72.8).  Fewer units have more of the long ones: 12 steps, and a last share of a
//    quarter (9 of 1600, 0.13, 3x3 40.4 / 44.0; 12, 0.08, 43.8 / 43.9; 12 of 1232, 0.41, 5x1 39.8 / 37.1; 12 of 1300, 0.53, 2x3
//    41.4 / 39.3).
// Four wavefronts for the size of the group, not for many units (16 query heads a KV head), change nothing while all run at once
// (4 KV heads, one sequence 3x3 25.6 / 27.4, 3x4 27.5 / 27.6, 8x1 27.6 / 27.1, 32 35.9 / 37.2, 38.0 / 37.7, 38.6 / 36.4; through an
// index one 8x2 31.4 / 33.3, sixteen 38.9 / 38.8); no rule beyond that was measured for them.
// With more pages than the register selection holds the scores go through LDS and radix passes: two launches from 128 KiB of
// rows on, and from 320 KiB for more than 256 units, where none waits (40 sequences of 2424 pages at 60 channels, 284 KiB, 76.9 /
// 81.5, at 120 99.0 / 98.5; 33 of 2048 tokens 139.7 / 122.1), and through an index (4168 pages at 32, 40, 64 channels, 260,
// 325, 521 KiB: one 28.8 / 31.5, 31.0 / 32.5, 38.5 / 33.2; four 31.9 / 34.6, 34.4 / 35.3, 42.0 / 36.5; sixteen 39.6 / 44.5, 42.7 /
// 46.7, 51.9 / 51.3; 24, some waiting, at 32 67.3 / 62.6).  (16 query heads a KV head, one sequence of 2424 pages at 32 35.9 / 27.0.)
constexpr bool tok_one_launch(const TokRoute& r) {
  const int workgroups = r.units * r.n_split, at_once = 256 * 8 / r.waves;
  const bool waits = r.n_split > 1 && workgroups > at_once, large_group = r.waves == 4 && r.units <= 256;
  if (r.rounds == 0) return (r.indexed || r.waves == 4) && !waits && !large_group && 2 * r.k1 * r.pages_cap <= 320 * 1024;
  const int steps = r.rounds * ((r.k1 + 31) / 32 + 1);
  if (r.units > 128 && r.n_split == 1 && !large_group) return steps <= 32;
  if (!waits) return steps <= (!r.indexed ? 12 : r.units <= 8 || r.units > 64 || r.rounds <= 5 ? 25 : 21);
  if (r.waves == 4) return !large_group && steps <= 25;
  int most = r.indexed || (r.units > 128 && r.rounds > 4) ? 15 : 0;
  const int last_share = r.entries - (r.n_split - 1) * r.chunk;
  const bool behind_short = 2 * (workgroups - at_once) <= r.units;
  if (r.units > 128 && 10 * last_share <= 7 * r.chunk) most = behind_short ? 24 : most > 8 ? most : 8;
  if (r.units <= 128 && 4 * last_share <= r.chunk && behind_short && most < 12) most = 12;
  return steps <= most;
}

}  // namespace rkv
