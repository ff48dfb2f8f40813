// How a page list is divided between the workgroups of its unit.  Plain constexpr arithmetic that needs no
// device, so a host program can sweep it.
#pragma once

namespace rkv {

struct ListShares {
  int n_split;   // workgroups that have a share
  int chunk;     // entries per workgroup (the last one takes what is left)
  int per_wave;  // entries per wavefront, whole pairs
};

// `row_len` entries for at most `n_wg` workgroups of `waves` wavefronts; room(n): whether all workgroups of
// the launch run at once if every unit has n of them.
//
// Whole pairs per wavefront set the number of workgroups.  Where wavefronts walk more than one pair and all
// workgroups run at once, they then take equal shares (49 entries: 26 and 23, not 32 and 17; 13 ragged
// sequences at a budget of 777: 21.9 -> 21.4 us a layer, 4 x 32 heads at 700: 22.2 -> 21.3).  With one pair
// each there is no round to save, and a short share that is done early costs nothing (19 entries as 16 and
// 3 rather than 10 and 9: 17.0 against 17.3 us).  Nor is there with workgroups waiting for their turn: the
// longest wavefront walks the same pairs either way, and a short last share lets the next workgroup
// start early (20 sequences x 8 KV heads at a budget of 700, 320 workgroups: 32 + 12 entries 31.0 us, 22 + 22
// 35.9; 12 at 2048 over token-major V: 48 + 48 + 32 43.2, 44 + 44 + 40 47.2).
template <class Room>
constexpr ListShares list_shares(int row_len, int n_wg, int waves, const Room& room) {
  const auto pairs_of = [&](int entries) { return ((entries + waves - 1) / waves + 1) / 2 * 2; };
  ListShares s = {1, 0, pairs_of((row_len + n_wg - 1) / n_wg)};
  s.chunk = s.per_wave * waves;
  s.n_split = (row_len + s.chunk - 1) / s.chunk;
  if (s.n_split < 1) s.n_split = 1;
  if (s.per_wave > 2 && room(s.n_split)) {
    s.chunk = ((row_len + s.n_split - 1) / s.n_split + 1) / 2 * 2;
    s.per_wave = pairs_of(s.chunk);
    s.n_split = (row_len + s.chunk - 1) / s.chunk;
  }
  return s;
}

}  // namespace rkv
