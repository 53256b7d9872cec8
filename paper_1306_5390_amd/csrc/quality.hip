// quality.hip -- the steps around the pass loop in the paper's experiments
// (Section 3): salt-and-pepper noise at a given density, the input the
// method is measured on (Tables 1-2), and the sum of squared differences
// behind the peak signal-to-noise ratio, the restoration measure of Table 2.
//
// Both are streams (1 B read + 1 B written, or 2 B read, per pixel); they are
// not part of the pass loop.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "phgrms.h"
#include "phgrms_internal.hpp"

using namespace phg;

namespace {

constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;   // SplitMix64 increment

// Output i (0-based) of a SplitMix64 generator seeded with `seed`: its
// state after i+1 steps is seed + (i+1)*gamma, and an output is that state
// through the generator's two xor-shift-multiply rounds and a final
// xor-shift (Steele, Lea and Flood's generator, with the mixing constants of
// its reference implementation).  Random access by pixel index makes the
// noise independent of the launch shape.  Here: the top 32 bits of the output
// for state z.
__device__ __forceinline__ uint32_t splitmix64_top(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return uint32_t((z ^ (z >> 31)) >> 32);
}

// A pixel becomes pepper (0) if u < t_pepper, salt (255) if
// t_pepper <= u < t_salt, else keeps its value.
__device__ __forceinline__ uint32_t noisy(uint32_t v, uint32_t u, uint32_t t_pepper, uint32_t t_salt) {
  return u < t_pepper ? 0u : u < t_salt ? 255u : v;
}

// u = the top 32 bits of output i.  Each thread reads and writes only its own
// pixels, so in place is fine.  Where both images start at the same place
// within 4 bytes a thread takes whole words (4096^2: 16.8 us; 20.7 by bytes).
// The generator's six 32-bit multiplies a pixel, at a quarter of the issue
// rate, bound it.
__global__ __launch_bounds__(256) void salt_pepper_kernel(const uint8_t* in, uint8_t* out, long long n, uint64_t seed,
                                                          uint32_t t_pepper, uint32_t t_salt) {
  const long long me = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long step = (long long)gridDim.x * blockDim.x;
  auto bytes = [&](long long from, long long to) {
    for (long long i = from + me; i < to; i += step)
      out[i] = uint8_t(noisy(in[i], splitmix64_top(seed + uint64_t(i + 1) * kGamma), t_pepper, t_salt));
  };
  const uintptr_t ui = reinterpret_cast<uintptr_t>(in), uo = reinterpret_cast<uintptr_t>(out);
  if (((ui ^ uo) & 3u) != 0) {
    bytes(0, n);
    return;
  }
  const long long lead = (long long)((4u - (ui & 3u)) & 3u);
  const long long head = lead < n ? lead : n;
  const long long nw = (n - head) / 4;
  const uint32_t* wi = reinterpret_cast<const uint32_t*>(in + head);
  uint32_t* wo = reinterpret_cast<uint32_t*>(out + head);
  for (long long i = me; i < nw; i += step) {
    const uint32_t v = wi[i];
    uint64_t z = seed + uint64_t(head + 4 * i + 1) * kGamma;
    uint32_t r = 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b, z += kGamma)
      r |= noisy((v >> (8 * b)) & 255u, splitmix64_top(z), t_pepper, t_salt) << (8 * b);
    wo[i] = r;
  }
  bytes(0, head);
  bytes(head + 4 * nw, n);
}

__global__ void zero_one_kernel(unsigned long long* p) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *p = 0ull;
}

// (a - b)^2 summed over the four bytes of a word: a^2 + b^2 - 2ab, at most
// 4 * 255^2.
__device__ __forceinline__ uint32_t sq_diff4(uint32_t a, uint32_t b) {
  const uint32_t squares = __builtin_amdgcn_udot4(a, a, __builtin_amdgcn_udot4(b, b, 0u, false), false);
  return squares - 2u * __builtin_amdgcn_udot4(a, b, 0u, false);
}

// Sum over i of (a[i] - b[i])^2 into *sum (zeroed beforehand): a per-thread
// partial, a wave reduction, a workgroup reduction in LDS, one atomic per
// workgroup.  Where both images start at the same place within 16 bytes, a
// thread takes 16-byte vectors, kSumUnroll of each image in flight, and a
// word's four squares take three dot products; otherwise bytes.  Two reads
// of memory bound it (4096^2: 33.6 MB in 8.5 us, 3.9 TB/s; by bytes with a
// 64-bit multiply each and 8192 atomics it took 101).  By bytes the loads in
// flight bound it, so that large images need every wave the device holds
// (a byte apart, with 256 and with 512 workgroups: 2^28 pixels 471 and 270 us,
// 287 with the 8192 small ones; 2^24: 22 and 18, 104; 2^22: 8 and 11, 102).
constexpr int kSumUnroll = 4;
constexpr int kSumThreads = 1024;
constexpr int kSumGroups = 256;    // one atomic each, 20 ns apart on the one address
constexpr int kSumByteGroups = 512;
constexpr long long kSumManyBytes = 1ll << 24;
__global__ __launch_bounds__(kSumThreads) void sq_diff_kernel(const uint8_t* a, const uint8_t* b,
                                                      long long n, unsigned long long* sum) {
  unsigned long long s = 0;
  const long long me = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long step = (long long)gridDim.x * blockDim.x;
  auto bytes = [&](long long from, long long to) {
    for (long long i = from + me; i < to; i += step) {
      const int d = int(a[i]) - int(b[i]);
      s += uint32_t(d * d);
    }
  };
  const uintptr_t ua = reinterpret_cast<uintptr_t>(a), ub = reinterpret_cast<uintptr_t>(b);
  if (((ua ^ ub) & 15u) != 0) {
    bytes(0, n);
  } else {
    const long long lead = (long long)((16u - (ua & 15u)) & 15u);
    const long long head = lead < n ? lead : n;
    const long long nv = (n - head) / 16;
    const uint4* va = reinterpret_cast<const uint4*>(a + head);
    const uint4* vb = reinterpret_cast<const uint4*>(b + head);
    auto add = [&](const uint4& x, const uint4& y) {
      s += sq_diff4(x.x, y.x) + sq_diff4(x.y, y.y) + sq_diff4(x.z, y.z) + sq_diff4(x.w, y.w);
    };
    long long i = me;
    for (; i + (kSumUnroll - 1) * step < nv; i += kSumUnroll * step) {
      uint4 x[kSumUnroll], y[kSumUnroll];
#pragma unroll
      for (int u = 0; u < kSumUnroll; ++u) {
        x[u] = va[i + u * step];
        y[u] = vb[i + u * step];
      }
#pragma unroll
      for (int u = 0; u < kSumUnroll; ++u) add(x[u], y[u]);
    }
    for (; i < nv; i += step) add(va[i], vb[i]);
    bytes(0, head);
    bytes(head + nv * 16, n);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off);
  __shared__ unsigned long long part[kSumThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) part[w] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
#pragma unroll
    for (int k = 0; k < kSumThreads / 64; ++k) t += part[k];
    if (t != 0ull) atomicAdd(sum, t);
  }
}

int grid_for(long long n) {
  const long long g = (n + 255) / 256;
  return int(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

}  // namespace

extern "C" {

int phgrms_salt_pepper(const uint8_t* d_in, uint8_t* d_out, int64_t n, uint64_t seed,
                       uint32_t t_pepper, uint32_t t_salt, void* stream) {
  if (n < 0) return fail(PHGRMS_EINVAL, "negative pixel count");
  if (t_pepper > t_salt) return fail(PHGRMS_EINVAL, "t_pepper %u > t_salt %u", t_pepper, t_salt);
  if (n == 0) return PHGRMS_OK;
  if (d_in == nullptr || d_out == nullptr) return fail(PHGRMS_EINVAL, "null image pointer");
  const uintptr_t a = reinterpret_cast<uintptr_t>(d_in), b = reinterpret_cast<uintptr_t>(d_out);
  if (a != b && a < b + uintptr_t(n) && b < a + uintptr_t(n))
    return fail(PHGRMS_EINVAL, "input and output overlap without being the same buffer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(salt_pepper_kernel, dim3(grid_for(n)), dim3(256), 0, s, d_in, d_out,
                     (long long)n, seed, t_pepper, t_salt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "noise launch");
  return PHGRMS_OK;
}

int phgrms_sq_diff_sum(const uint8_t* d_a, const uint8_t* d_b, int64_t n, int64_t* d_sum,
                       void* stream) {
  if (n < 0) return fail(PHGRMS_EINVAL, "negative pixel count");
  if (d_sum == nullptr) return fail(PHGRMS_EINVAL, "null result pointer");
  if (n > 0 && (d_a == nullptr || d_b == nullptr)) return fail(PHGRMS_EINVAL, "null image pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto* sum = reinterpret_cast<unsigned long long*>(d_sum);
  hipLaunchKernelGGL(zero_one_kernel, dim3(1), dim3(64), 0, s, sum);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "zero launch");
  if (n > 0) {
    const bool bytes = ((reinterpret_cast<uintptr_t>(d_a) ^ reinterpret_cast<uintptr_t>(d_b)) & 15u) != 0;
    const int groups = bytes && n >= kSumManyBytes ? kSumByteGroups : kSumGroups;
    hipLaunchKernelGGL(sq_diff_kernel, dim3(std::min(grid_for(n), groups)), dim3(kSumThreads), 0, s, d_a, d_b,
                       (long long)n, sum);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "sum launch");
  }
  return PHGRMS_OK;
}

}  // extern "C"
