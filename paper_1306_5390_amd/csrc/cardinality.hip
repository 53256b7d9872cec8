// cardinality.hip -- Algorithm 1 by gathering, as a call of its own: the
// cardinality of a pixel is the number of image pixels of its window whose
// grey level lies strictly within alpha of its own.
//
// The band test runs four pixels per lane in bytes, as in pass_kernel.hpp
// (the strict band is [x - alpha + 1, x + alpha - 1]), and the counts, at most
// 81, stay in bytes until they are stored.  A wave takes 256 columns of 8
// rows and keeps the window's rows, shifted, in registers, so that a row is
// loaded once per strip and nothing goes through LDS.  What bounds it: the
// stores, 4 B per pixel, and the band test, 5 VALU instructions per window
// pixel and lane (2048^2, beta 2: 21 MB and about 2 M wave-instructions in
// 10.5 us; a thread per pixel and byte loads took 52, and the caller two more
// passes over the counts to widen them).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "phgrms.h"
#include "phgrms_internal.hpp"
#include "pass_kernel.hpp"

using namespace phg;

namespace {

constexpr int kCardRows = 8;       // rows per wave
constexpr int kCardWaves = 4;

// Four counts, stored at any alignment of their type.
template <class Out> struct Four;
template <> struct Four<uint32_t> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Four<uint16_t> { typedef uint16_t type __attribute__((ext_vector_type(4), aligned(2))); };

template <int BETA, class Out>
__global__ __launch_bounds__(kCardWaves * 64) void card_kernel(const uint8_t* img, int rows, int cols, int alpha,
                                                               int tiles_x, int ntiles, Out* card) {
  constexpr int NW = 2 * BETA + 1;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // range-checked loads over the image's dwords: rows outside it read as 0
  // (and are not counted)
  const uintptr_t sb = reinterpret_cast<uintptr_t>(img);
  const uintptr_t se = sb + uintptr_t(rows) * uintptr_t(cols);
  const uintptr_t base = sb & ~uintptr_t(3);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>(base), 0, int(uint32_t(((se + 3) & ~uintptr_t(3)) - base)), kBufferWord3);
  const uint32_t head = uint32_t(sb & 3u);
  const bool aligned = head == 0 && (cols & 3) == 0;
  const uint32_t am1_16 = uint32_t(alpha > 0 ? alpha - 1 : 0) * 0x01000100u;

  for (int tile = blockIdx.x * kCardWaves + w; tile < ntiles; tile += gridDim.x * kCardWaves) {
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    const int r0 = ty * kCardRows;
    const int c = tx * 256 + 4 * lane;               // the lane's first column
    // per column offset: the lane's pixels with such a neighbour in the image
    uint32_t ok[NW];
#pragma unroll
    for (int dc = -BETA; dc <= BETA; ++dc) {
      uint32_t m = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (c + b + dc >= 0 && c + b + dc < cols) m |= 0x80u << (8 * b);
      ok[dc + BETA] = m;
    }
    uint32_t win[NW][NW];                            // window rows, shifted by -BETA .. BETA
    auto load_row = [&](int r, uint32_t (&wr)[NW]) {
      const uint32_t g = head + uint32_t(r) * uint32_t(cols) + uint32_t(c);   // modulo 2^32
      const uint32_t a = g & ~3u;
      uint32_t d0 = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(a - 4u), 0, 0);
      uint32_t d1 = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(a), 0, 0);
      uint32_t d2 = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(a + 4u), 0, 0);
      if (!aligned) {
        const uint32_t d3 = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(a + 8u), 0, 0);
        d0 = __builtin_amdgcn_alignbyte(d1, d0, g & 3u);
        d1 = __builtin_amdgcn_alignbyte(d2, d1, g & 3u);
        d2 = __builtin_amdgcn_alignbyte(d3, d2, g & 3u);
      }
#pragma unroll
      for (int dc = -BETA; dc <= BETA; ++dc)
        wr[dc + BETA] = dc == 0 ? d1 : dc == -4 ? d0 : dc == 4 ? d2
            : dc < 0 ? __builtin_amdgcn_alignbyte(d1, d0, 4 + dc) : __builtin_amdgcn_alignbyte(d2, d1, dc);
    };
#pragma unroll
    for (int i = 0; i < 2 * BETA; ++i) load_row(r0 - BETA + i, win[i]);
#pragma unroll 1
    for (int j0 = 0; j0 < kCardRows; j0 += NW) {
#pragma unroll
      for (int jj = 0; jj < NW; ++jj) {
        const int r = r0 + j0 + jj;
        if (j0 + jj < kCardRows && r < rows) {       // (uniform)
          load_row(r + BETA, win[(jj + 2 * BETA) % NW]);
          const uint32_t nx = ~win[(jj + BETA) % NW][BETA];
          const uint32_t nlo = sat_add_u8x4(nx, am1_16);   // 255 - (lowest level of the band)
          const uint32_t nhi = sat_sub_u8x4(nx, am1_16);   // 255 - (its highest)
          uint32_t n = 0u;
#pragma unroll
          for (int dr = -BETA; dr <= BETA; ++dr) {
            if (r + dr < 0 || r + dr >= rows) continue;    // (uniform)
#pragma unroll
            for (int dc = -BETA; dc <= BETA; ++dc) {
              const uint32_t y = win[(jj + BETA + dr + NW) % NW][dc + BETA];
              const uint32_t in = (__builtin_amdgcn_lerp(y, nlo, 0x01010101u) ^ __builtin_amdgcn_lerp(y, nhi, 0u)) &
                                  ok[dc + BETA];
              n += in >> 7;
            }
          }
          if (alpha <= 0) n = 0u;                          // an empty band
          Out* o = card + size_t(r) * size_t(cols) + size_t(c);
          if (c + 3 < cols) {
            typename Four<Out>::type v = {Out(n & 255u), Out((n >> 8) & 255u), Out((n >> 16) & 255u), Out(n >> 24)};
            *reinterpret_cast<typename Four<Out>::type*>(o) = v;
          } else {
#pragma unroll
            for (int b = 0; b < 3; ++b)
              if (c + b < cols) o[b] = Out((n >> (8 * b)) & 255u);
          }
        }
      }
    }
  }
}

// One thread per pixel, bytes read from memory: for images narrower than
// kCardNarrow columns, where most lanes of a wave above would have no pixel,
// for sides near 2^31, which its column arithmetic does not hold, and for small
// images, which have too few waves above to hide the chain of 8 rows that each
// of them goes through (us, a thread per pixel and a wave per strip: 128^2:
// beta 1: 3.7 and 3.9, 2: 4.2 and 5.5, 3: 6.4 and 7.5, 4: 9.2 and 9.5; 321 x
// 481: 3.6 and 5.3, 5.0 and 7.0, 7.5 and 9.0, 10.6 and 11.3; 512^2: 3.6 and
// 4.0, 5.4 and 5.6, 8.2 and 7.6, 11.6 and 9.6; 2048 x 200: 3.9 and 4.2, 6.1 and
// 5.7, 9.0 and 7.7, 12.8 and 9.8).
constexpr int kCardNarrow = 64;
constexpr long long card_small(int beta) {         // pixels
  return beta == 1 ? 6 << 16 : beta == 2 ? 5 << 16 : beta == 3 ? 4 << 16 : 1 << 16;
}
template <class Out>
__global__ void card_pixel_kernel(const uint8_t* __restrict__ img, int rows, int cols, int alpha, int beta,
                                  Out* __restrict__ card) {
  const long long n = (long long)rows * cols;
  for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < n;
       p += (long long)gridDim.x * blockDim.x) {
    const int r = int(p / cols);
    const int c = int(p - (long long)r * cols);
    const int x = img[p];
    int cnt = 0;
    // the window clipped to the image (in 64 bits: r + beta may pass INT_MAX)
    const int i0 = r - beta < 0 ? 0 : r - beta;
    const int i1 = int((long long)r + beta < rows ? (long long)r + beta : rows - 1);
    const int j0 = c - beta < 0 ? 0 : c - beta;
    const int j1 = int((long long)c + beta < cols ? (long long)c + beta : cols - 1);
    for (int i = i0; i <= i1; ++i) {
      for (int j = j0; j <= j1; ++j) {
        const int y = img[(long long)i * cols + j];
        cnt += (y < x + alpha && y > x - alpha) ? 1 : 0;
      }
    }
    card[p] = Out(cnt);
  }
}

template <int BETA, class Out>
void launch_card(const uint8_t* img, int rows, int cols, int alpha, Out* card, hipStream_t s) {
  const int tiles_x = (cols + 255) / 256;
  const int ntiles = tiles_x * ((rows + kCardRows - 1) / kCardRows);
  const int grid = int(std::min<long long>((ntiles + kCardWaves - 1) / kCardWaves, max_workgroups(kCardWaves * 64)));
  hipLaunchKernelGGL((card_kernel<BETA, Out>), dim3(grid), dim3(kCardWaves * 64), 0, s, img, rows, cols, alpha,
                     tiles_x, ntiles, card);
}

template <class Out>
int cardinality(const uint8_t* d_img, int32_t rows, int32_t cols, int32_t alpha, int32_t beta, Out* d_card,
                void* stream) {
  phgrms_params p{rows, cols, alpha, beta, 0};
  const int rc = validate_params(p);
  if (rc != PHGRMS_OK) return rc;
  const long long n = (long long)rows * cols;
  if (n == 0) return PHGRMS_OK;
  if (d_img == nullptr || d_card == nullptr) return fail(PHGRMS_EINVAL, "null pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (cols < kCardNarrow || cols >= (1 << 30) || n < card_small(beta)) {
    const int blocks = int(std::min<long long>((n + 255) / 256, 65536));
    hipLaunchKernelGGL(card_pixel_kernel<Out>, dim3(blocks), dim3(256), 0, s, d_img, rows, cols, alpha, beta, d_card);
  } else {
    switch (beta) {
      case 1: launch_card<1, Out>(d_img, rows, cols, alpha, d_card, s); break;
      case 2: launch_card<2, Out>(d_img, rows, cols, alpha, d_card, s); break;
      case 3: launch_card<3, Out>(d_img, rows, cols, alpha, d_card, s); break;
      default: launch_card<4, Out>(d_img, rows, cols, alpha, d_card, s); break;
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "cardinality launch");
  return PHGRMS_OK;
}

}  // namespace

extern "C" {

int phgrms_cardinality(const uint8_t* d_img, int32_t rows, int32_t cols, int32_t alpha, int32_t beta,
                       uint16_t* d_card, void* stream) {
  return cardinality<uint16_t>(d_img, rows, cols, alpha, beta, d_card, stream);
}

int phgrms_cardinality_u32(const uint8_t* d_img, int32_t rows, int32_t cols, int32_t alpha, int32_t beta,
                           uint32_t* d_card, void* stream) {
  return cardinality<uint32_t>(d_img, rows, cols, alpha, beta, d_card, stream);
}

}  // extern "C"
