// plan.hpp -- how a pass loop by deep launches (deep_kernel.hpp) is cut into
// launches and tiles.  Plain C++, so that its rules also build with an
// ordinary host compiler; the structs and constants serve the kernels too.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "phgrms.h"

namespace phg {

constexpr int kDeepH = 64;                         // rows computed: WAVES strips of R rows, R <= 8 (R rows x
                                                   // 8 words of bits, one lane each)
constexpr int kDeepHalo = 16;                      // halo columns on each side: passes * BETA fit in it
constexpr int kDeepCols = 256 - 2 * kDeepHalo;     // owned columns of a tile

// Most passes of one launch at `beta`.
constexpr int deep_max_passes(int beta) { return kDeepHalo / beta; }

constexpr int deep_tiles_x(int cols) { return int((static_cast<long long>(cols) + kDeepCols - 1) / kDeepCols); }

// How a pass loop of k passes is cut into launches: `lead` launches of one
// pass, one launch of `first`, then launches of `rest` each.
struct LaunchPlan {
  int lead, first, rest;
  constexpr int start(int j) const {   // first pass of launch j
    return j <= lead ? j : lead + first + (j - lead - 1) * rest;
  }
  // (no launch has 256 passes; a shape that is not deep has lead 0)
  constexpr int packed() const { return lead | first << 8 | rest << 16; }
  constexpr static LaunchPlan unpacked(int v) { return LaunchPlan{v & 255, (v >> 8) & 255, (v >> 16) & 255}; }
  constexpr int launch_of(int pass) const {
    return pass < lead ? pass : pass < lead + first ? lead : lead + 1 + (pass - lead - first) / rest;
  }
};

// The launches of a deep loop with the period-2 stop: a pass can be compared
// with the image two passes before only if the launch has that one, so every
// launch but the first begins with the last pass of the launch before, which
// stores the image as it was before that pass (the last launch: after it).
// `first` passes in launch 0, `rest` in the others.
struct CyclePlan {
  int k, first, rest;
  constexpr int start(int j) const { return j == 0 ? 0 : first - 1 + (j - 1) * (rest - 1); }
  constexpr int passes(int j) const {
    const int n = j == 0 ? first : rest, left = k - start(j);
    return n < left ? n : left;
  }
  constexpr bool last(int j) const { return start(j) + passes(j) >= k; }
  // passes after which launch j's stored image is taken
  constexpr int advance(int j) const { return last(j) ? passes(j) : passes(j) - 1; }
};

// A tile's row and column arithmetic stays inside an int.
bool deep_fits(const phgrms_params& p);
// The launches of the pass loop of one image.  maps: the workspace has room
// for its change maps.
LaunchPlan deep_plan(const phgrms_params& p, bool maps);
// The longest loop (in passes) of an image that runs by one-pass launches
// only.
int deep_few_passes(const phgrms_params& p, bool maps);
// The launches of an image's loop in a batch of batch_px pixels.
LaunchPlan deep_batch_plan(int beta, int k, int64_t batch_px);
constexpr int64_t kLargeBatch = 1 << 24;   // pixels
// The launches of a loop with the period-2 stop, and whether it runs by them
// where the change maps fit (else by one-pass launches).
CyclePlan cycle_plan(const phgrms_params& p);
bool cycle_plan_pays(const phgrms_params& p);
// Owned rows of a tile of an image alone on the device: the fewest (but 4)
// that give every CU at most one tile, else the most that a tile can own.
// (997 x 1031, beta 3: 46 us with 250 tiles, 51 with 125 or with 315.)
int deep_rows(int rows, int cols, int beta, int depth, int cus);
// Words of a change map (a map has a word and a count byte per image row and
// tile column).
size_t deep_map_words(int rows, int cols);

}  // namespace phg
