// Which workgroups a decode projection (k_gemv.hip) runs as: host code only, chosen per call from the sizes and the
// stream's compute units.
#pragma once
#include <cstddef>

namespace nova {

constexpr int GV_KC = 256;             // K chunk per pipeline step (32 pieces of 8)
constexpr int GV_RW = 16;              // weight rows per wave
constexpr int GV_ROWS = 4 * GV_RW;     // rows per workgroup (4 waves)
constexpr int GV_TAIL_MAX = 4;         // K slices of a tail tile at most

// Whether a bf16 projection whose K is not split runs as 128-row workgroups of the ring, which halve the X traffic
// per weight: while they make at least two rounds of two per CU.
static inline bool gemv_wide(int N, int cus) { return N % 128 == 0 && N / 128 >= 4 * cus; }

// The K slices of the gate/up projection's last row tiles.  With one workgroup per 64 rows, N / 64 = 592
// tiles on 256 CUs are 2.3 rounds: 80 CUs stream three tiles while the others stream two.  The 80 tiles past
// the last whole round are cut into the number of K slices (at most 4, as many as the workspace and the
// arrival counters hold) that gives the busiest CU the least to stream: 3 slices, a third of a tile each.
// Decode steps with and without (and with gate/up on the ring below 17 rows): batch 1, 4 layers 636 -> 624 us,
// batch 8, 8 layers 1148 -> 1120, batch 32 at context 3627 872 -> 857, batch 8 on 128 CUs 850 -> 845.
// 1: no slices.
static inline int gemv_tail(int N, int K, int B, int cus, int counters, size_t partial_floats) {
  const int tiles = N / GV_ROWS, tail = tiles % cus, chunks = K / GV_KC;
  if (tiles < cus || tail == 0 || tail > counters) return 1;
  int best = 1;
  auto share = [&](int s) { return (double)((tail * s + cus - 1) / cus) * ((chunks + s - 1) / s) / chunks; };
  for (int s = 2; s <= GV_TAIL_MAX; ++s) {
    if ((s - 1) * ((chunks + s - 1) / s) >= chunks) continue;           // an empty slice
    if ((size_t)s * tail * GV_ROWS * B > partial_floats) break;
    if (share(s) < share(best)) best = s;
  }
  return best;
}

}  // namespace nova
