// deep.hip -- instances of the kernels of deep_kernel.hpp.
#include <hip/hip_runtime.h>

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

}  // namespace phg
