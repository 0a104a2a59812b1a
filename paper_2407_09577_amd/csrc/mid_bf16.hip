// Middle rows: which workgroup shape of mid_kernel.h a call takes, or none (the many-row
// tiles).  The kinds are instantiated in mid_kinds_*.hip.
#include "mid_kernel.h"

namespace fn {

extern template hipError_t launch_mid_epi<EPI_RMS>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_GLU>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_LN>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_NONE>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_GLU_NOSCALE>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_REGLU>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_BILINEAR>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_GLU_DEFER>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_RELU_DEFER>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_ROWSCALE>(const PrefillArgs&, int);
extern template hipError_t launch_mid_epi<EPI_ROPE>(const PrefillArgs&, int);

// Workgroup shapes: 16-row blocks and packed column blocks of a workgroup, and its time in us
// on MI355X as a function of r = workgroups / 256 (the compute units):
//   fix max(1, r) + K / 1024 (round ceil(r) + fill min(1, r)).
// A workgroup's time per k is constant, a round ends when its last workgroup does, and units
// that share the memory slow each other down a little.  The constants are least-squares fits
// over 1423 random bf16 shapes (17..1500 rows, K 512..8192, 512..20480 columns, linear and
// GLU; shapes 16 and 17 over 1458 of 65..1536 rows), each shape of the table within 5 to 18%
// rms.  Shapes 13..15 are 2, 5 and 8 with non-temporal weight loads; shape 17's three column
// blocks per wave hold no whole gate/up pairs.  The last two took 2% off the mean over their sample
// (333 x 4096 -> 12288: 53.2 -> 48.3 us).
struct MidShape {
  int mb, blocks;
  float fix, round, fill;
};
static constexpr MidShape kMidShapes[] = {
    {2, 2, 2.34f, 1.09f, 1.41f}, {2, 4, 2.68f, 1.90f, 1.28f}, {2, 6, 2.87f, 2.82f, 1.28f},
    {3, 2, 2.71f, 1.47f, 1.32f}, {3, 4, 3.18f, 2.38f, 1.30f}, {3, 6, 3.15f, 3.16f, 1.24f},
    {4, 2, 3.59f, 2.09f, 1.02f}, {4, 4, 3.95f, 3.09f, 1.24f}, {4, 6, 4.16f, 4.00f, 1.32f},
    {6, 6, 4.70f, 4.42f, 2.05f}, {6, 16, 5.34f, 9.72f, 3.58f}, {8, 6, 5.37f, 5.44f, 2.54f},
    {8, 16, 6.02f, 11.06f, 4.30f},
    {2, 6, 3.56f, 4.16f, 2.38f}, {3, 6, 3.61f, 4.36f, 2.33f}, {4, 6, 4.21f, 4.76f, 2.10f},
    {4, 8, 3.81f, 4.45f, 1.56f}, {7, 12, 5.78f, 8.33f, 2.72f}};
constexpr int kMidShapeCount = sizeof(kMidShapes) / sizeof(kMidShapes[0]);
constexpr int kMidFirstNT = 13, kMidLastNT = 15, kMidLinearOnly = 17;

float estimate_us(float r, int K, float fix, float round, float fill) {
  return fix * fmaxf(1.0f, r) + (float)K / 1024.0f * (round * ceilf(r) + fill * fminf(1.0f, r));
}

// One row group and 96 MB of weights or more: the weights come from HBM and bound the call.  There
// the six-block shapes run with non-temporal loads (22016 columns, K 4096, caches cold: 32 rows
// 30.1 us, 31.4 cached; 48 rows 31.2 and 31.3; 64 rows 33.2 and 33.3), the 96- and 128-row ones,
// cached only, when more than 64 rows need them (65 rows: 33.6 us, two groups of 64 47.5), and the
// two- and four-block shapes when they cover the width in one round (32 x 8192 -> 8192: 25.3 us,
// six blocks 42.6; in two rounds 32 x 4096 -> 22016 40.0 against 30.1).  Over 152 calls of 32..128
// rows and 101..283 MB the choice is 2% off the best shape of each and never behind the tiles.
// Fewer bytes may stay in the 256 MB cache between calls, where cached loads win (the same
// 100 MB in every call, 32 rows: 18.6 us, non-temporal 24.4).  Otherwise the shape of the least
// estimated time, if that is below 0.9 of the tile kernel's: over the shapes of the fit the
// rule takes 0.62 of the tiles' time (geometric mean; the best choice at each shape 0.60).  More
// than 1536 rows and fewer than 256 packed columns were not in the fit's sample and keep the tiles,
// though single shapes are faster there (2048 x 5120 -> 576: tiles 35.0 us, shape 8 25.3;
// 4096 x 5120 -> 576: 42.6 and, shape 11, 42.2; 64 x 8192 -> 128: 43.4 and, shape 0, 12.8).
//
// Below the fit's least K the estimates miss what a call is made of: prologue, epilogue and the
// output's stores.  A second round pays the fixed part again; so do the 12- and 16-block shapes at
// any K, as their LDS leaves a compute unit room for one workgroup (1392 x 744 -> 2 x 8904 with
// 770 of them: 65.8 us, the tiles 55.3).  Nothing hides those wide shapes' epilogue: at short K
// they compete only in three rounds (two below K = 64) and only where the tiles would be 256 x 256
// (532 x 64 -> 17822: 17.1 us, 128-row tiles 9.6; 797 x 128 -> 19542: 21.0, 256-row tiles 28.5;
// 1527 x 16 -> 2 x 10143 in four rounds: 31.7 and 22.9).
//
// Held to the tiles on 3000 fresh random shapes, the rule takes 0.83 of their time at K 8..511
// (1000 shapes; 0.6% run over 5% slower, at worst 14%: 1155 x 296 -> 17958, 36.5 us and 32.2) and
// 0.61 at K 512..8192 (2000; 0.4%, at worst 13%: 130 x 4544 -> 12494, 47.6 and 42.2).  The
// estimates alone ran 11.5% of the short ones over 5% slower, at worst 94%.
constexpr int kMidFitMinK = 512;

int mid_shape(int M, int K, int NP, bool glu) {
  if (M > kMidMaxM || NP < 256) return -1;
  const int npb = NP / 16;
  const bool stream = (int64_t)K * NP * 2 >= 96 * 1000 * 1000;
  const bool big = prefill_fills_256x256(M, NP);
  int best = -1;
  float best_us = 0.9f * prefill_estimate_us(M, K, NP, glu);
  for (int i = 0; i < kMidShapeCount; ++i) {
    const MidShape& s = kMidShapes[i];
    const int groups = (M + 16 * s.mb - 1) / (16 * s.mb);
    const bool nt = i >= kMidFirstNT && i <= kMidLastNT;
    if (glu && i == kMidLinearOnly) continue;
    const int64_t wgs = (int64_t)groups * ((npb + s.blocks - 1) / s.blocks);
    if (!stream || groups > 1) {
      if (nt) continue;
    } else if (s.blocks == 6 ? !nt && (s.mb <= 4 || M <= 64) : s.blocks > 6 || wgs > 256) {
      continue;
    }
    const bool wide = s.blocks > 8;
    const float r = (float)wgs / 256.0f;
    if (wide && K < kMidFitMinK && (!big || r > (K < 64 ? 2.0f : 3.0f))) continue;
    float us = estimate_us(r, K, s.fix, s.round, s.fill);
    if (K < kMidFitMinK || wide) us += s.fix * (ceilf(r) - fmaxf(1.0f, r));
    if (us < best_us) {
      best_us = us;
      best = i;
    }
  }
  return best;
}

hipError_t launch_mid_bf16(const PrefillArgs& p, int shape) {
  switch (p.epi) {
    case EPI_RMS: return launch_mid_epi<EPI_RMS>(p, shape);
    case EPI_GLU: return launch_mid_epi<EPI_GLU>(p, shape);
    case EPI_LN: return launch_mid_epi<EPI_LN>(p, shape);
    case EPI_NONE: return launch_mid_epi<EPI_NONE>(p, shape);
    case EPI_GLU_NOSCALE: return launch_mid_epi<EPI_GLU_NOSCALE>(p, shape);
    case EPI_REGLU: return launch_mid_epi<EPI_REGLU>(p, shape);
    case EPI_BILINEAR: return launch_mid_epi<EPI_BILINEAR>(p, shape);
    case EPI_GLU_DEFER: return launch_mid_epi<EPI_GLU_DEFER>(p, shape);
    case EPI_RELU_DEFER: return launch_mid_epi<EPI_RELU_DEFER>(p, shape);
    case EPI_ROWSCALE: return launch_mid_epi<EPI_ROWSCALE>(p, shape);
    case EPI_ROPE: return launch_mid_epi<EPI_ROPE>(p, shape);
  }
  return hipErrorInvalidValue;
}

}  // namespace fn
