// Which workgroups a decode projection (k_gemv.hip) runs as: host code only, chosen per call from the sizes and the
// stream's compute units.
#pragma once
#include <cstddef>

namespace nova {

constexpr int GV_KC = 256;             // K chunk per pipeline step (32 pieces of 8)
constexpr int GV_RW = 16;              // weight rows per wave
constexpr int GV_ROWS = 4 * GV_RW;     // rows per workgroup (4 waves)
constexpr int GV_TAIL_MAX = 4;         // K slices of a tail tile at most

// A bf16 projection whose K is not split and whose 128-row workgroups make at least two rounds of two per CU: rows
// per workgroup of the ring (0: fewer rounds).  128 rows halve the X traffic per weight, 64 share the stream more
// evenly, so the batch decides (us; K = 3584):
//  * LM head, 152,064 rows, 128 / 64 rows: on 224 CUs 184 / 179 at batch 1, 192 / 188 at 8, 194 / 193 at 12; on
//    160 194 / 185 at 1, 205 / 201 at 6, 214 / 221 at 12; on 128 222 / 211 at 1, 231 / 226 at 4, 241 / 245 at 8; on 64
//    365 / 357 at 1, 374 / 376 at 4, 389 / 401 at 8.  On the whole GPU 180 / 182 at 1, 188 / 190 at 8, 203 / 214 at 32.
//  * gate/up, 37,888 rows (two rounds on 74 CUs or fewer), 128 rows / 64 with the tail slices below: on 64 CUs
//    100 / 92 at batch 1, 106 / 102 at 8, 108 / 107 at 12, 111 / 113 at 16, 126 / 144 at 32; on 32 183 / 168 at 1,
//    194 / 189 at 8, 199 / 199 at 12, 206 / 211 at 16, 238 / 274 at 32.
static inline int gemv_ring_rows(int N, int B, int cus, bool head, bool gate_up) {
  if (N % 128 || N / 128 < 4 * cus) return 0;
  if (head) return cus < 256 && B <= (cus >= 160 ? 8 : 4) ? 64 : 128;
  return gate_up && B <= 12 ? 64 : 128;
}

// The K slices of the gate/up projection's last row tiles.  With one workgroup per 64 rows, N / 64 = 592
// tiles on 256 CUs are 2.3 rounds: 80 CUs stream three tiles while the others stream two.  The 80 tiles past
// the last whole round are cut into the number of K slices (at most 4, as many as the workspace and the
// arrival counters hold) that gives the busiest CU the least to stream: 3 slices, a third of a tile each.
// Decode steps with and without (and with gate/up on the ring below 17 rows): batch 1, 4 layers 636 -> 624 us,
// batch 8, 8 layers 1148 -> 1120, batch 32 at context 3627 872 -> 857, batch 8 on 128 CUs 850 -> 845.
// The slices' partials grow with the batch, so the larger batches take slices only for a larger part of a tile (gate/up
// on the ring without / with slices, us): a saving of 0.14 of a tile (160 CUs) 52.6 / 51.9 at batch 1, 57.2 / 56.6 at 8,
// 58.7 / 59.0 at 12, 60.9 / 62.2 at 16, 70.6 / 75.6 at 32; of 0.29 (128 CUs) 58.6 / 55.8, 71.0 / 70.3 at 16, 75.2 / 75.7
// at 17, 83.4 / 84.4 at 32; of 0.5 (32 CUs) 240 / 236 at 17, 278 / 274 at 32; of 0.64 (256 CUs) 59.6 / 55.1 at 32.
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
  const double most = B <= 12 ? 1.0 : B <= 16 ? 0.75 : 0.5;             // of a tile, left to the busiest CU
  return share(best) <= most ? best : 1;
}

}  // namespace nova
