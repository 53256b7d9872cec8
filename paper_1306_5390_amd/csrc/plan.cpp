// plan.cpp -- the rules of plan.hpp: which launches a pass loop by deep
// launches has, and when one-pass launches are as fast.
#include "plan.hpp"

#include <algorithm>

namespace phg {

bool deep_fits(const phgrms_params& p) { return p.rows < (1 << 30) && p.cols < (1 << 30); }

// A deep launch tests its tiles' halo too while every pixel has to be tested,
// and pays that back only in the passes that follow what changed; one-pass
// launches test each pixel once a pass.  On images whose rows start on dword
// boundaries, from 2^21 pixels on, the first few passes are therefore faster
// by one-pass launches; on others their misaligned rows cost them more (1201 x
// 1601, beta 1, k 2: 31 us by one-pass launches, 19 by deep ones).  Measured
// in us per call, by one-pass and by deep launches only, a tenth and two
// fifths of the pixels noise:
//   2048^2: beta 1, k 3: 30, 30 and 36, 41; beta 2, k 3: 40, 44 and 38, 43;
//     beta 3, k 2: 33, 45 and 30, 29, k 3: 47, 58 and 43, 31; beta 4, k 3: 59,
//     82 and 44, 35, k 5: 96, 107 and 48, 40
//   8192^2: beta 1, k 4: 199, 200 and 278, 312; beta 2, k 3: 272, 291 and 252,
//     270; beta 3, k 3: 390, 520 and 357, 214; beta 4, k 4: 852, 1005 and 562, 310
// (the noise decides, which a rule cannot know; the line lies where deep
// launches lose more on little noise than they gain on much).  A single pass
// is never faster by a deep launch, save in 2^20 .. 2^22 misaligned pixels.
// Without change maps, on images of few tile columns, deep launches need more
// passes to pay (8192 x 256, a tenth noise, beta 3, k 6: 67 and 89 us; beta 4,
// k 10: 132 and 166).  Images with no interior pixel change in no pass.
// Of 25 sizes, every beta, k up to 32 and noise from 5 to 60 %, one-pass
// launches are still faster by more than a tenth, and by a fifth at most, in
// loops of 3 to 6 passes at beta 4 where much noise is gone after two or three
// of them (1448^2, k 6, three fifths noise: 24 and 28 us, but 112 and 56 .. 104
// with less), and without maps in a few passes more (16384 x 480, beta 1, k 8:
// 124 and 148 us there, 81 and 46 with a twentieth noise).
int deep_few_passes(const phgrms_params& p, bool maps) {
  const int64_t n = (int64_t)p.rows * p.cols;
  if (std::min(p.rows, p.cols) <= 2 * p.beta) return p.k;
  if ((p.cols & 3) != 0) {
    if (p.beta == 4 && n >= (1 << 22)) return 2;
    return n >= (1 << 20) && n < (1 << 22) ? 0 : 1;
  }
  const bool mid = n >= (1 << 21), large = n >= (1 << 24), narrow = p.cols <= 256;
  switch (p.beta) {
    case 1: return !mid ? 1 : !maps && (narrow || n >= (1 << 22)) ? 6 : large ? 4 : 3;
    case 2: return !mid ? 1 : !maps && narrow ? 4 : 3;
    case 3: return !mid ? 1 : !maps ? 6 : 3;
    default:
      if (mid) return !maps ? 10 : n <= (1 << 22) ? 5 : 4;
      return n < (1 << 20) ? 2 : maps ? 4 : 6;
  }
}

// `lead` dense launches of one pass come first where every pixel has to be
// tested and the image is large: the dense kernel tests it with no halo
// (2048^2, beta 2, k 32: 105 us with two, 115 with none; 8192^2 433 and 463),
// while on smaller images the launches cost more than the halo (1024^2: 80 and
// 73).  At beta 1 the dense pass is cheaper, so that this pays from 2^25
// pixels (8192^2: 1176 and 1234; 4099 x 4001: 396 and 378), on dword rows from
// 2^24 (4096^2, k 8, three fifths noise: 190 us, 217 with none, 199 by
// one-pass launches).  At beta 3 one launch, from 2^24 pixels (4096^2, k 5: 187
// us at a tenth noise, 215 with none, 191 by one-pass launches) and for the
// shortest loops from 2^21 (2048^2, k 5: 70, 89 and 75); at beta 4 only there
// (2048^2, k 6: 103, 133 and 116).  The last launches have an even number of
// passes, so that tiles that only alternate need not run.
LaunchPlan deep_plan(const phgrms_params& p, bool maps) {
  const int64_t n = (int64_t)p.rows * p.cols;
  if (p.k <= deep_few_passes(p, maps)) return LaunchPlan{p.k, 1, 1};
  const bool dwords = (p.cols & 3) == 0;
  const int most = p.beta == 1 ? 16 : p.beta == 2 ? 8 : 4;
  LaunchPlan pl{0, most, most};
  if (p.beta == 1 && n >= (1 << 22)) pl.first = 8;
  if ((p.beta == 1 && n >= (1 << (dwords ? 24 : 25))) || (p.beta == 2 && n >= (1 << 22))) {
    pl.lead = 2;
    pl.first = 6;
  }
  if (dwords && p.beta == 3 && n >= (1 << (p.k <= 5 ? 21 : 24))) pl.lead = 1;
  if (dwords && p.beta == 4 && n >= (1 << 21) && n <= (1 << 22) && p.k <= 7) pl.lead = 1;
  pl.lead = std::min(pl.lead, p.k);
  pl.first = std::max(1, std::min(pl.first, p.k - pl.lead));
  if (((p.k - pl.lead - pl.first) & 1) != 0 && pl.first > 1) --pl.first;
  return pl;
}

// In a large batch two dense one-pass launches come first, since its images
// fill the device and the halo of a deep tile is all cost while every pixel is
// tested, and at beta 1 the later launches take 16 passes (150 images of 192
// Mpixel, k 32: 2.39 ms; without the dense launches 2.99, with 8 passes 2.48).
// A small batch is latency-bound, and takes fewer launches of smaller halo (12
// images of 1.5 Mpixel, k 16: 176 us against 204; 48 images of 20 Mpixel: 413
// against 379).  Images of up to three passes have dense launches only, from
// 2^22 pixels on (us per run, a tenth noise, with deep launches, with dense ones, and before
// there were deep ones: 8 images of 8 Mpixel, beta 3, k 2: 86, 68, 72; 12 of 50
// Mpixel, beta 4, k 3: 746, 549, 557; 4 of 17 Mpixel, beta 2, k 3: 130, 102,
// 115); at beta 4 the shortest already from 2^21 (12 of 3 Mpixel, k 2: 71, 60,
// 64).  Those of four (beta 4) and of four and five (beta 3) have one dense
// launch first (12 of 50 Mpixel, beta 3, k 5: 652, 541, 561); longer ones lose
// by it on much noise what they gain on little (k 16: 776 and 721, two fifths
// noise 403 and 418).
LaunchPlan deep_batch_plan(int beta, int k, int64_t batch_px) {
  const bool most = batch_px >= (1 << 22);
  if ((k <= 3 && most) || (beta == 4 && k <= 2 && batch_px >= (1 << 21))) return LaunchPlan{3, 1, 1};
  if (beta >= 3) return LaunchPlan{most && k <= (beta == 3 ? 5 : 4) ? 1 : 0, 4, 4};
  if (batch_px < kLargeBatch) return LaunchPlan{0, 8, 8};
  return LaunchPlan{2, 6, beta == 1 ? 16 : 8};
}

int deep_rows(int rows, int cols, int beta, int depth, int cus) {
  const int most = kDeepH - 2 * (depth - 1) * beta;
  const int tiles_x = deep_tiles_x(cols);
  const int tiles_y = cus / std::max(tiles_x, 1);
  if (tiles_y < 1 || rows / tiles_y >= most) return most;
  return std::max(std::min((rows + tiles_y - 1) / tiles_y, most), std::min(4, most));
}

size_t deep_map_words(int rows, int cols) {
  return size_t(std::max(rows, 0)) * size_t(deep_tiles_x(std::max(cols, 0)));
}

// Launches after the first run an odd number of passes: their stored image is
// an even number of passes on, so that tiles that alternate are idle.  Large
// images have the shorter first launch: its passes test every pixel of the
// halo too (k 20, us per call, with the longer first launch and with the
// shorter: 8192^2: 1062 and 877 at beta 1, 719 and 648 at beta 2, 431 and 386
// at beta 3; 2048^2: 131 and 116, 92 and 79, 64 and 64; but 1023 x 1537, k 8,
// beta 2: 44 and 52).
CyclePlan cycle_plan(const phgrms_params& p) {
  const bool large = (int64_t)p.rows * p.cols >= (1 << 22);
  return p.beta == 1   ? CyclePlan{p.k, large ? 8 : 16, 15}
         : p.beta == 2 ? CyclePlan{p.k, large ? 6 : 8, 7}
         : p.beta == 3 ? CyclePlan{p.k, large ? 3 : 4, 5} : CyclePlan{p.k, 4, 3};
}

// One-pass launches are as fast, with their smaller halo and a finish of one
// launch, for the first few passes of a large image whose rows start on dword
// boundaries, and more so at the larger betas (us per call, one-pass and deep,
// a tenth of the pixels noise or, at beta 1,
// four tenths; 512^2, beta 1, k 2: 21 and 23; 4096^2: beta 1, k 4: 103 and
// 120, k 6: 145 and 147, a tenth noise 118 and 81; beta 2, k 3: 106 and 110,
// k 4: 144 and 120; beta 3, k 6: 239 and 278, k 10: 392 and 349; 2048^2, beta
// 4, k 6: 122 and 148, k 10: 199 and 183; 8192^2, beta 1, k 10: 667 and 691,
// k 12: 786 and 739).  At beta 4 large images are faster by the one or by the
// other, as their noise is (4096^2, k 32: 905 and 674, four tenths noise 193
// and 296), and stay with the one-pass launches; so do small ones of a few
// passes, where much noise is gone after two of them and the launches after
// those end at once (k 5, a tenth noise and two fifths: 720 x 1280: 72 and 67,
// 21 and 29; 1448^2: 100 and 103, 37 and 38; 321 x 481, k 2: 45 and 35, 21 and 23).
bool cycle_plan_pays(const phgrms_params& p) {
  const int64_t n = (int64_t)p.rows * p.cols;
  if (p.k <= 1 || n <= 0 || !deep_fits(p)) return false;
  if (std::min(p.rows, p.cols) <= 2 * p.beta) return false;   // (no pass changes anything)
  const bool huge = n >= (1 << 25);
  if ((p.cols & 3) != 0) return p.beta < 4 || (!huge && p.k > 2);
  if (n < (1 << 21)) return p.beta == 4 ? p.k > 6 : p.k > 2 || n < (1 << 18);
  switch (p.beta) {
    case 1: return p.k > (huge ? 10 : 4);
    case 2: return p.k > 3;
    case 3: return p.k > 8;
    default: return p.k > 8 && n < (1 << 23);
  }
}

}  // namespace phg
