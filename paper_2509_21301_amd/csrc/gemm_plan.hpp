// Which tiles an M x N x K bf16 problem of the encode and prefill GEMM (k_gemm.hip) runs as: host code only,
// chosen per call from the sizes and the stream's compute units by estimated time.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>

namespace nova {

// The tiles a problem may run as, and the coefficients of a launch's estimated time in us: with at most one
// workgroup per CU step1 per 64-wide K step + fixed1; with one round of two per CU step2 + fixed2; with more,
// step per K step + round per round of workgroup slots, + fixed; and the epilogue's term per round.  (At K = 5120
// the smaller tiles take 3 to 15% longer per step: 256 x 1280 x 5120 unsliced in 32x64 tiles 20.7 us.)  Fitted to
// 8355 timings (bf16 normal data, weights from HBM, M 1..41472 on the encoder's and decoder's ten projections
// with their own epilogues, 1..16 K slices, 32..256 CUs): 88% of the timings lie within 10% of the fit, and the
// tile and slices it picks take 0.5% longer than the fastest ones on average, at most 15%.  Planned for 256 CUs
// on a partition they took 15% longer on average, up to twice as long.
struct GemmTile {
  int bm, bn, per_cu;       // workgroups per CU
  float step1, fixed1, step2, fixed2, step, round, fixed;
  float pitch;              // share that step1 and step2 grow by where rows of K lie a multiple of 2 KB apart
};
static constexpr GemmTile kGemmTiles[] = {
    {32, 64, 2, 0.185f, 3.2f, 0.361f, 3.7f, 0.288f, 1.2f, 3.0f, 0.15f},
    {64, 64, 2, 0.250f, 3.6f, 0.444f, 4.1f, 0.372f, 1.3f, 3.3f, 0.10f},
    {64, 128, 1, 0.382f, 4.7f, 0.f, 0.f, 0.381f, 2.3f, 2.6f, 0.08f},
    {128, 128, 1, 0.495f, 5.0f, 0.f, 0.f, 0.508f, 2.7f, 2.5f, 0.03f},
    {256, 128, 1, 0.795f, 6.2f, 0.f, 0.f, 0.827f, 4.1f, 1.4f, 0.f},
    {128, 256, 1, 0.813f, 6.4f, 0.f, 0.f, 0.838f, 3.7f, 3.1f, 0.f},
    {128, 128, 2, 0.891f, 5.2f, 0.908f, 6.9f, 0.895f, 1.5f, 7.5f, 0.f},
    {256, 256, 1, 1.260f, 10.2f, 0.f, 0.f, 1.268f, 7.1f, 3.8f, 0.f}};
constexpr int kGemmTileCount = (int)(sizeof(kGemmTiles) / sizeof(kGemmTiles[0]));
constexpr int kGemmTile256 = kGemmTileCount - 1;
constexpr int kGemmStepK = 64;

// What an epilogue adds to a 256x256 tile over the bf16 store, in us (Epi order: store, GELU, residual, position,
// SwiGLU), and the fp32 partial store of a K slice.
static constexpr float kGemmEpiUs[] = {0.0f, 7.5f, 3.8f, 2.5f, 5.4f};
constexpr float kGemmPartialUs = -1.0f;
// Bytes per output that the sum of the K slices reads and writes besides the partials, by epilogue.
static constexpr float kGemmSumBytes[] = {2.f, 2.f, 8.f, 4.f, 1.f};

struct GemmProblem {
  int M, N, K;
  int epi;                  // Epi
  int cus;                  // compute units of the stream: its partition's, or the whole GPU's
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

// Estimated time of `wgs` workgroups of tile t, `steps` K steps each, over p's first `cols` weight rows (read from
// HBM; the two bounds add as squares, which the timings near both fit best).
static inline double gemm_tile_us(const GemmProblem& p, const GemmTile& t, long wgs, int steps, bool partials,
                                  int cols) {
  const int cus = p.cus;
  const long slots = (long)cus * t.per_cu;
  // a last round that is partly empty costs a whole one after a single round, and only its share
  // after ten, when the workgroups have drifted apart (the 8-image QKV's 9.5 rounds take 9.5)
  const double part = (double)wgs / (double)slots, whole = std::ceil(part);
  const double rounds = whole - (whole - part) * std::min(1.0, (whole - 1.0) / 10.0);
  const double epi = (partials ? kGemmPartialUs : kGemmEpiUs[p.epi]) * t.bm * t.bn / 65536.0;
  const double first = steps * (p.K * 2 % 2048 ? 1.0 : 1.0 + t.pitch);
  const double us = wgs <= cus    ? first * t.step1 + t.fixed1 + epi
                    : whole <= 1 ? first * t.step2 + t.fixed2 + epi * t.per_cu
                                 : rounds * (steps * t.step + t.round + epi * t.per_cu) + t.fixed;
  const double hbm = (double)cols * p.K * 2 / 7.3e6;
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
      double us = gemm_tile_us(p, t, tiles * sl, steps, sl > 1, p.N);
      if (sl > 1) {        // one more launch; the partials written and read
        const double bytes = (8.0 * sl + kGemmSumBytes[p.epi]) * p.M * p.N;
        us += 3.1 + 0.2 * sl + bytes / 8.6e6;
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
    const long tiles = (long)nm * (p.N / t.bn), slots = (long)p.cus * t.per_cu;
    if (tiles <= slots || tiles % slots == 0) continue;
    const int n1 = (int)(tiles / slots * slots / nm) * t.bn;
    if (n1 <= 0 || n1 >= p.N) continue;
    GemmProblem q = p;
    q.N = p.N - n1;
    const double first = gemm_tile_us(p, t, (long)nm * (n1 / t.bn), p.K / kGemmStepK, false, n1);
    const GemmPlan r = gemm_two_launches(i, 0, n1, first, plan_one_launch(q));
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
  const long full = (long)nm * nn / p.cus;
  if (full < 1) return GemmPlan();
  const int m1 = (int)(full * p.cus / nn);
  if (m1 < 1 || m1 >= nm) return GemmPlan();
  GemmProblem q = p;
  q.M = p.M - m1 * 256;
  const double first = gemm_tile_us(p, kGemmTiles[kGemmTile256], (long)m1 * nn, p.K / kGemmStepK, false, p.N);
  return gemm_two_launches(kGemmTile256, m1 * 256, 0, first, plan_one_launch(q));
}

// The plan of a problem (tile < 0: none fits, N is no multiple of 64).
static inline GemmPlan plan_gemm(const GemmProblem& p) {
  // The position epilogue's traffic grows with narrower tiles, which the estimate does not count: from two rounds of
  // 256x256 tiles on it takes them.  N = 1280, K = 640, 256x256 against the best other tile: 41,472 rows (3.2 rounds)
  // 120 and 126 us, 10,680 on 64 CUs (3.3) 79 and 85, 13,416 on 128 CUs (2.1) 61 and 61; below, the estimate decides:
  // 13,416 (1.04) 49 and 42, 5184 (0.41) 25 and 17.
  if (p.epi == 3 && p.N % 256 == 0 && (long)((p.M + 255) / 256) * (p.N / 256) >= 2L * p.cus) {
    GemmPlan r;
    r.tile = kGemmTile256, r.us = 0;
    return r;
  }
  // One comparison of everything that may run (a row split set against a plan that may use neither slices nor
  // columns won although the plan it replaced had the lower estimate: at 896 of 4673 row counts from 4104 to
  // 41,480 of the encoder's O projection and 547 of MLP down, by up to 14%).  No margin: 711 two-launch plans
  // took 1% less than estimated, with a spread of 4%, and asking a split to save 2 to 4% more made the chosen
  // plans 0 to 0.09% slower on average over 256 CUs and 0.12 to 0.23% over partitions.
  GemmPlan best = plan_one_launch(p);
  const GemmPlan rows = plan_rows(p), cols = plan_columns(p);
  if (rows.us < best.us) best = rows;
  if (cols.us < best.us) best = cols;
  return best;
}

// fp32 activations: whether the 32x64 tiles run (gemm_f32_small_kernel) rather than the 128x128 ones, which take a
// whole round of one workgroup per CU however few tiles it holds.  32x64 / 128x128 tiles, us:
//  * 256 CUs, N and K 1280..5120: 20 tiles of 128x128 12.1 / 37.2, 180 35.9 / 45.3, but 240 47.3 / 45.9 and 250
//    (K = 5120) 179 / 160; 320 58.6 / 86.8, 720 125 / 134, but 750 136 / 129; 960 161 / 170, 1000 179 / 178; from there
//    on 1220 245 / 215, 1280 217 / 221, 1640 324 / 305, 2430 471 / 417, 4880 931 / 870: 128x128 tiles where the last of
//    their rounds is nearly full, and beyond 1000 tiles;
//  * partitions: a first round nearly full 47.5 / 37.5 (60 tiles on 64 CUs), but later ones on 128 CUs 250 80.6 / 86.1
//    and 287 / 313 (K = 5120), 750 225 / 250, on 64 CUs 320 181 / 209: 128x128 tiles for the first only.
static inline bool gemm_f32_small(int M, int N, int cus) {
  const long tiles = (long)((M + 127) / 128) * (N / 128), last = (tiles - 1) % cus + 1;
  const bool full = 8 * last >= 7L * cus;
  return tiles <= 1000 && !(full && (tiles <= cus || cus > 192));
}

}  // namespace nova
