// Which tiles an M x N x K bf16 problem of the encode and prefill GEMM (k_gemm.hip) runs as: host code only,
// chosen per call from the sizes by estimated time.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>

namespace nova {

// The tiles a problem may run as, and the coefficients of a launch's estimated time in us, fitted to
// 2900 timings (bf16 normal data, weights from HBM; M 16..5184 on the encoder's and decoder's nine
// projection shapes, 1..12 K slices; 80% of the timings lie within 12% of the fit): with at most one
// workgroup per CU, step1 per 64-wide K step + fixed1; with more, step2 per K step + round2 per round
// of workgroup slots, + fixed2.
struct GemmTile {
  int bm, bn, per_cu;       // workgroups per CU
  float step1, fixed1, step2, round2, fixed2;
};
static constexpr GemmTile kGemmTiles[] = {
    {32, 64, 2, 0.205f, 2.4f, 0.292f, 0.0f, 4.5f},    {64, 64, 2, 0.264f, 2.8f, 0.388f, 0.1f, 4.6f},
    {64, 128, 1, 0.408f, 3.6f, 0.390f, 2.0f, 3.0f},   {128, 128, 1, 0.520f, 4.6f, 0.523f, 3.4f, 1.9f},
    {256, 128, 1, 0.810f, 6.0f, 0.854f, 6.3f, -1.2f}, {128, 256, 1, 0.840f, 6.0f, 0.855f, 6.5f, -0.3f},
    {128, 128, 2, 0.860f, 4.4f, 0.937f, 3.2f, 4.0f},  {256, 256, 1, 1.280f, 9.5f, 1.344f, 12.2f, -2.4f}};
constexpr int kGemmTileCount = (int)(sizeof(kGemmTiles) / sizeof(kGemmTiles[0]));
constexpr int kGemmTile256 = kGemmTileCount - 1;
constexpr int kGemmStepK = 64;

struct GemmProblem {
  int M, N, K;
  bool pos;                 // the position epilogue
  int max_slices;           // K slices the epilogue allows, their partials within ws_floats
  size_t ws_floats;
  bool split_rows, split_cols;   // whether the problem may run as two launches over its rows or columns
};

// One launch of `tile` with K in `slices`; or two: the first `rows` rows (or `cols` columns), unsliced, with
// `tile`, and the rest with tile2 and slices2.
struct GemmPlan {
  int tile = -1, slices = 1;
  int rows = 0, cols = 0;
  int tile2 = -1, slices2 = 1;
  double us = 1e30;         // estimated time
};

// Estimated time of `wgs` workgroups of tile t with `steps` K steps each, over weights of `bytes` (read
// from HBM at 5 TB/s; the two bounds add as squares, which the timings near both fit best).
static inline double gemm_tile_us(const GemmTile& t, long wgs, int steps, double bytes) {
  const long slots = 256L * t.per_cu;
  // a last round that is partly empty costs a whole one after a single round, and only its share
  // after eight, when the workgroups have drifted apart (the 8-image QKV's 9.5 rounds take 9.5)
  const double part = (double)wgs / (double)slots, whole = std::ceil(part);
  const double rounds = whole - (whole - part) * std::min(1.0, (whole - 1.0) / 8.0);
  const double us = wgs <= 256 ? steps * t.step1 + t.fixed1 : rounds * (steps * t.step2 + t.round2) + t.fixed2;
  const double hbm = bytes / 5.0e6 + 2.0;
  return std::sqrt(us * us + hbm * hbm);
}

// The one launch with the least estimated time: a tile and K slices.
static inline GemmPlan plan_one_launch(const GemmProblem& p) {
  GemmPlan best;
  for (int i = 0; i < kGemmTileCount; ++i) {
    const GemmTile& t = kGemmTiles[i];
    if (p.N % t.bn) continue;
    const long tiles = (long)((p.M + t.bm - 1) / t.bm) * (p.N / t.bn);
    for (int sl = 1; sl <= p.max_slices; ++sl) {
      const int ksteps = p.K / kGemmStepK, steps = (ksteps + sl - 1) / sl;
      if (sl > 1 && (ksteps - (sl - 1) * steps < 2 || (size_t)sl * p.M * p.N > p.ws_floats)) continue;
      double us = gemm_tile_us(t, tiles * sl, steps, (double)p.N * p.K * 2);
      if (sl > 1) {        // one more launch; the partials written and read, from the caches while they are few
        const double bytes = (double)sl * p.M * p.N * 8;
        us += 3.5 + bytes / (bytes < 64e6 ? 10.0e6 : 5.0e6);
      }
      if (us < best.us) {
        best = GemmPlan();
        best.tile = i, best.slices = sl, best.us = us;
      }
    }
  }
  return best;
}

// `first` us of one tile's launch, then the rest as planned by itself.
static inline GemmPlan gemm_two_launches(int tile, int rows, int cols, double first, const GemmPlan& rest) {
  GemmPlan r;
  r.tile = tile, r.rows = rows, r.cols = cols, r.tile2 = rest.tile, r.slices2 = rest.slices;
  r.us = first + 2.0 + rest.us;
  return r;
}

// The columns of whole rounds of one tile first and the leftover columns, which would leave most of a last
// round idle, with another (tile < 0: none).
static inline GemmPlan plan_columns(const GemmProblem& p) {
  GemmPlan best;
  if (!p.split_cols) return best;
  for (int i = 0; i < kGemmTileCount; ++i) {
    const GemmTile& t = kGemmTiles[i];
    if (p.N % t.bn) continue;
    const int nm = (p.M + t.bm - 1) / t.bm;
    const long tiles = (long)nm * (p.N / t.bn), slots = 256L * t.per_cu;
    if (tiles <= slots || tiles % slots == 0) continue;
    const int n1 = (int)(tiles / slots * slots / nm) * t.bn;
    if (n1 <= 0 || n1 >= p.N) continue;
    GemmProblem q = p;
    q.N = p.N - n1;
    const GemmPlan r = gemm_two_launches(
        i, 0, n1, gemm_tile_us(t, (long)nm * (n1 / t.bn), p.K / kGemmStepK, (double)n1 * p.K * 2), plan_one_launch(q));
    if (r.us < best.us) best = r;
  }
  return best;
}

// Rows run as 256x256 tiles ahead of the rest (tile < 0: none): with more than 16 row tiles and a last round
// of 256x256 tiles (one workgroup per CU) that would leave part of the GPU idle, the rows of whole rounds go
// first and the leftover rows are planned by themselves.  The results are bit-identical to one launch when
// the rest runs unsplit (the same K order per output).  The screenshot encode (53 row tiles): QKV 4 -> 3.5
// rounds, MLP up 5 -> 4.5, O and down 2 -> 1.5; the 8-image MLP down (162 x 5): 4 -> 3.5.
static inline GemmPlan plan_rows(const GemmProblem& p) {
  const int nm = (p.M + 255) / 256, nn = p.N / 256;
  if (!p.split_rows || p.N % 256 || nm <= 16) return GemmPlan();
  const long full = (long)nm * nn / 256;
  if (full < 1) return GemmPlan();
  const int m1 = (int)(full * 256 / nn);
  if (m1 < 1 || m1 >= nm) return GemmPlan();
  GemmProblem q = p;
  q.M = p.M - m1 * 256;
  return gemm_two_launches(kGemmTile256, m1 * 256, 0,
                           gemm_tile_us(kGemmTiles[kGemmTile256], (long)m1 * nn, p.K / kGemmStepK, (double)p.N * p.K * 2),
                           plan_one_launch(q));
}

// The plan of a problem (tile < 0: none fits, N is no multiple of 64).
static inline GemmPlan plan_gemm(const GemmProblem& p) {
  // the position epilogue writes fp32 and reads the table: over many rows 256-wide tiles pay (41,472
  // patches: 110 us against 122 us with 128x128 tiles)
  if (p.pos && p.M > 4096 && p.N % 256 == 0) {
    GemmPlan r;
    r.tile = kGemmTile256, r.us = 0;
    return r;
  }
  // one comparison of everything that may run: a row split set against a plan that may use neither slices nor
  // columns won at one size in six of the 1280-wide residual projections, up to 14% behind the plan it replaced
  GemmPlan best = plan_one_launch(p);
  const GemmPlan rows = plan_rows(p), cols = plan_columns(p);
  if (rows.us < best.us) best = rows;
  if (cols.us < best.us) best = cols;
  return best;
}

}  // namespace nova
