// deep.hip -- instances of the kernels of deep_kernel.hpp, and how a deep
// shape's pass loop is cut into launches and tiles.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "phgrms_internal.hpp"
#include "deep_kernel.hpp"

namespace phg {

template <int WAVES, bool CYC>
static const void* deep_ptr(int beta) {
  switch (beta) {
    case 1: return reinterpret_cast<const void*>(&deep_kernel<1, WAVES, CYC>);
    case 2: return reinterpret_cast<const void*>(&deep_kernel<2, WAVES, CYC>);
    case 3: return reinterpret_cast<const void*>(&deep_kernel<3, WAVES, CYC>);
    case 4: return reinterpret_cast<const void*>(&deep_kernel<4, kDeepWaves, CYC>);
    default: return nullptr;
  }
}

const void* deep_kernel_ptr(int beta, bool wide) {
  return wide ? deep_ptr<kDeepWideWaves, false>(beta) : deep_ptr<kDeepWaves, false>(beta);
}

const void* deep_cycle_ptr(int beta, bool wide) {
  return wide ? deep_ptr<kDeepWideWaves, true>(beta) : deep_ptr<kDeepWaves, true>(beta);
}

template <int WAVES>
static const void* multi_ptr(int beta) {
  switch (beta) {
    case 1: return reinterpret_cast<const void*>(&multi_deep_kernel<1, WAVES>);
    case 2: return reinterpret_cast<const void*>(&multi_deep_kernel<2, WAVES>);
    case 3: return reinterpret_cast<const void*>(&multi_deep_kernel<3, WAVES>);
    case 4: return reinterpret_cast<const void*>(&multi_deep_kernel<4, kDeepWaves>);
    default: return nullptr;
  }
}

const void* multi_deep_ptr(int beta, bool wide) {
  return wide ? multi_ptr<kDeepWideWaves>(beta) : multi_ptr<kDeepWaves>(beta);
}

bool deep_fits(const phgrms_params& p) { return p.rows < (1 << 30) && p.cols < (1 << 30); }

LaunchPlan deep_plan(const phgrms_params& p) {
  const long long npx = (long long)p.rows * p.cols;
  const int most = p.beta == 1 ? 16 : p.beta == 2 ? 8 : 4;
  LaunchPlan pl{0, most, most};
  if (p.beta == 1 && npx >= (1ll << 22)) pl.first = 8;
  if ((p.beta == 1 && npx >= (1ll << 25)) || (p.beta == 2 && npx >= (1ll << 22))) {
    pl.lead = 2;
    pl.first = 6;
  }
  pl.lead = std::min(pl.lead, p.k);
  pl.first = std::max(1, std::min(pl.first, p.k - pl.lead));
  if (((p.k - pl.lead - pl.first) & 1) != 0 && pl.first > 1) --pl.first;
  return pl;
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

}  // namespace phg
