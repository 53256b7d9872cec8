// phgrms_internal.hpp -- declarations shared by the host-side sources of the
// library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "phgrms.h"
#include "host_common.hpp"

namespace phg {

constexpr int kDefaultShape = 3;   // (1, 8, 4): one pass, 8 rows per wave, 4 waves
// Launches at the start of a change-tracking pass loop that run the dense
// kernel of kDefaultShape (no change maps).  At most 2: the list-building
// launch of a skipping shape is launch 2.
constexpr int kDenseFirstLaunches = 2;
// The launches of a deep loop with the period-2 stop: a pass can be compared
// with the image two passes before only if the launch has that one, so every
// launch but the first begins with the last pass of the launch before, which
// stores the image as it was before that pass (the last launch: after it).
// `first` passes in launch 0, `rest` in the others.
struct CyclePlan {
  int k, first, rest;
  __host__ __device__ int start(int j) const { return j == 0 ? 0 : first - 1 + (j - 1) * (rest - 1); }
  __host__ __device__ int passes(int j) const {
    const int n = j == 0 ? first : rest, left = k - start(j);
    return n < left ? n : left;
  }
  __host__ __device__ bool last(int j) const { return start(j) + passes(j) >= k; }
  // passes after which launch j's stored image is taken
  __host__ __device__ int advance(int j) const { return last(j) ? passes(j) : passes(j) - 1; }
};

// Workgroups of a launch over listed tiles, in multiples of the grid that
// fits on the device at once.
constexpr int kListedOversubscription = 4;
// A launch with a change map over more tiles than twice what fits on the
// device at once: that many workgroups, each looking at several tiles (8192^2
// at beta 2, nearly all of 8436 tiles idle: 23 us, 64 with one workgroup per
// tile; 4 or 8 times what fits: 33 and 58).
constexpr int kDeepOversubscription = 2;
// Largest grid (in workgroups of `threads` lanes) of a launch: fewer than
// 2^31 work-items per dispatch (the dispatch size stays a positive 32-bit
// count), a multiple of 16.  Only images near 2^31 pixels reach it; the
// tile-walking kernels take the tiles beyond the grid in strides.
inline long long max_workgroups(int threads) { return (0x7fffffffll / threads) / 16 * 16; }

struct TileGeom {
  int T;             // passes per launch
  int TH, TW;        // owned tile rows and columns
  int tiles_x, tiles_y;
  long long ntiles;
};
// For a deep shape: tiles laid out for `depth` passes (0: the shape's T), of
// the rows that spread one image over the device (alone: the image has the
// launch to itself) or of the most rows they can own.
TileGeom tile_geom(const phgrms_params& p, int shape, int depth = 0, bool alone = false);

// How a pass loop of k passes is cut into launches: `lead` launches of one
// pass, one launch of `first`, then launches of `rest` each.
struct LaunchPlan {
  int lead, first, rest;
  __host__ __device__ int start(int j) const {   // first pass of launch j
    return j <= lead ? j : lead + first + (j - lead - 1) * rest;
  }
  // (no launch has 256 passes; a shape that is not deep has lead 0)
  __host__ __device__ int packed() const { return lead | first << 8 | rest << 16; }
  __host__ __device__ static LaunchPlan unpacked(int v) { return LaunchPlan{v & 255, (v >> 8) & 255, (v >> 16) & 255}; }
  __host__ __device__ int launch_of(int pass) const {
    return pass < lead ? pass : pass < lead + first ? lead : lead + 1 + (pass - lead - first) / rest;
  }
};

struct WsLayout {
  size_t state_off;    // int32 iteration count
  size_t counts_off;   // uint64 count slots, kCountSlots per pass
  size_t diff_off;     // uint64 slots of the period-2 stop, right after the counts
  size_t changed_off;  // uint64 changed[max(k,1)] totals
  size_t img_off;      // rows*cols bytes, the second ping-pong image
  size_t map_off;      // two change maps of map_bytes / 2 each
  size_t map_bytes;
  size_t total;
};
// Change maps of one-pass launches: one byte per (row, 256-column tile
// column), two of them (alternating by pass parity), then (256-aligned) the
// tile lists of the skipping shapes (TileLists, for at least 16 owned rows
// per tile).
size_t map_half_bytes(int rows, int cols);
int list_capacity(int rows, int cols);
size_t list_state_offset(int rows, int cols);
long long list_clear_u64(int rows, int cols);   // uint64 words cleared before a sequence
size_t change_map_bytes(int rows, int cols);
WsLayout ws_layout(const phgrms_params& p);

int hip_fail(hipError_t e, const char* what);
int validate_params(const phgrms_params& p);
int check_buffers(const uint8_t* d_in, const uint8_t* d_out, const phgrms_params& p,
                  const void* d_ws, size_t ws_bytes);
int size_class(long long npx);
int fused_shape(int beta, long long npx);
int set_grid_mode(int mode);
int grid_mode();
int set_fused_shape(int beta, int cls, int shape);   // cls -1: every class
// Shape of the batch path's multi-image launches (its own table: many
// images per launch favour other shapes than one image per launch).
int batch_shape(int beta, long long npx);
int set_batch_shape(int beta, int cls, int shape);   // cls -1: every class
TuneTables current_tuning();
void apply_tuning(const TuneTables& t);
// multi_pass_kernel<beta, shape> (batch.hip).
// maps: the kernel keeps change maps per image (tracking shapes only).
const void* multi_kernel_ptr(int beta, int shape, bool maps = false);
// Deep shapes (deep_kernel.hpp, deep.hip): kernels of one image and of many.
inline bool is_deep(int shape) { return kShapes[shape].track == 3; }
constexpr int kDeepShape = 13;
constexpr int kDeepWaves = 8;      // waves of a workgroup
constexpr int kDeepWideWaves = 16; // the same where no CU has more than one (beta 1 .. 3)
const void* deep_kernel_ptr(int beta, bool wide);
const void* deep_cycle_ptr(int beta, bool wide);   // the period-2 variant
const void* multi_deep_ptr(int beta, bool wide = false);
// A tile's row and column arithmetic stays inside an int.
bool deep_fits(const phgrms_params& p);
// The launches of the pass loop.  `lead` dense launches of one pass come
// first where every pixel has to be tested and the image is large: the dense
// kernel tests it with no halo (2048^2, beta 2, k 32: 105 us with two,
// 115 with none; 8192^2 433 and 463), while on smaller images the launches
// cost more than the halo (1024^2: 80 and 73).  At beta 1 the dense pass is
// cheaper, so that this pays from 2^25 pixels (8192^2: 1176 and 1234; 4099 x
// 4001: 396 and 378).  The last launches have an even number of passes, so
// that tiles that only alternate need not run.
LaunchPlan deep_plan(const phgrms_params& p);
// Owned rows of a tile of an image alone on the device: the fewest (but 4)
// that give every CU at most one tile, else the most that a tile can own.
// (997 x 1031, beta 3: 46 us with 250 tiles, 51 with 125 or with 315.)
int deep_rows(int rows, int cols, int beta, int depth, int cus);
// Words of a change map (a map has a word and a count byte per image row and
// tile column).
size_t deep_map_words(int rows, int cols);
int device_cus();                  // of the current device, or -1
// The one-pass shape that stands in for a deep one.
int one_pass_shape(int beta, long long npx, bool tracking);
// Grid size for a pass kernel shape over `ntiles` tiles: one workgroup per
// tile, or at most the resident grid (CUs x resident workgroups) in grid
// mode 1.  persistent (a launch over listed tiles): kListedOversubscription
// resident grids, whatever the grid mode.  cycle: the launch runs the
// period-2 variant (its listed kernel's occupancy may differ).
int pass_grid(int beta, int shape, long long ntiles, bool persistent = false, bool cycle = false);
int enqueue_denoise(const uint8_t* d_in, uint8_t* d_out, const phgrms_params& p, int shape,
                    uint8_t* ws_img, unsigned long long* counts, unsigned long long* changed,
                    int* iterations, uint8_t* maps, hipStream_t s,
                    unsigned long long* diff2 = nullptr);

}  // namespace phg
