// deep_kernel.hpp -- several passes of the P-HGRMS pass loop per launch, each
// after the first following only what the pass before it changed.
//
// A pixel can change in a pass only if a pixel of its window changed in the
// pass before (otherwise it sees the window it was left unchanged with).
// After the first one to four passes of a noisy image a tenth of the pixels
// or fewer have such a neighbour, and soon one in a hundred; a pass over
// every pixel is then work for nothing, and one launch per pass is mostly
// launch, tile load and tile store.  So a workgroup holds its tile in LDS for
// up to 16 / BETA passes (the tile carries that many passes' halo, and the
// region that is still exact shrinks by BETA a pass, as in pass_kernel.hpp),
// keeps one change bit per pixel, and takes every pass one of these ways:
//   * by list, where at most kDeepListMost pixels of the tile changed: every
//     pixel of their windows is evaluated exactly, one lane each, the items
//     shared by all waves;
//   * by strips of 8 rows (4 with 16 waves), one per wave: a strip without an active pixel
//     (within BETA of a change) does nothing; one with at most kDeepWords
//     active words (4 pixels) takes the band test on those words alone, one
//     lane each, and evaluates the candidates; any other one takes the band
//     test on all its rows, as pass_kernel.hpp does.
// Only dense strips copy rows through: the destination buffer holds the image
// two passes back, which differs from the source only where the last pass
// changed a pixel, and every such pixel is active and is written.
//
// Where a pass leaves nothing other than it was two passes before, the tile
// goes on alternating between its two buffers (its pixels' windows repeat),
// so the remaining passes are not run: each changes as many pixels as the
// last one did, and their parity says which buffer is the result.  Noisy
// images end in such an alternation at region boundaries almost everywhere.
//
// Between launches the image's change map carries, per image row and tile
// column, the last pass's changes (see kMapGroups) and their number.  A tile
// in whose reach nothing moves any more (kMapMoves) is not loaded, and rows
// that did not change in the previous launch or in this one are not stored
// (the destination holds the output of the launch before the previous one).
//
// With the period-2 stop (CYC, see CyclePlan) every pass from a launch's second
// on also tells exactly whether a pixel became other than two passes before.
//
// What bounds it: dense strips the VALU issue (1600 VALU instructions a strip
// of 8 rows at beta 2, 1270 in pass_kernel.hpp); late passes the chain of LDS
// latencies (about 1.1 us a pass); small images three launches' latency.
// Measured against the one-pass launches it takes the place of (us per call):
// 321 x 481, beta 1, k 10: 47 against 149; 2048^2, k 32: 106 against 270 at
// beta 1, 109 against 367 at beta 2; 4099 x 4001, beta 1: 387 against 1052;
// 8192^2, beta 2, half its pixels noise: 451 against 994; 1023 x 1537, beta 2,
// with the period-2 stop: 90 against 335.
#pragma once

#include "pass_kernel.hpp"

namespace phg {

constexpr int kDeepMaxPasses = 16;
constexpr int kDeepWords = 256;                    // most active words (of 4 pixels) of a strip tested one by one
constexpr int kDeepListMost = 64;                  // most changed pixels of a tile followed by list

struct DeepTile {
  const uint8_t* src;
  uint8_t* dst;
  int rows, cols, alpha;
  int depth;                 // passes the tile geometry is laid out for
  int npasses;               // passes to run, 1..depth
  int advance;               // passes after which the stored image and the map are taken (period-2
                             // launches; else npasses)
  int th;                    // owned rows of a tile
  int tiles_x;
  const uint32_t* map_in;    // change map of the previous launch, or null: the first pass
                             // tests every pixel
  uint32_t* map_out;         // change map of this launch, or null
  const uint8_t* cnt_in;     // with the maps: pixels of each map word's segment that the
  uint8_t* cnt_out;          // launch's last pass changed
  int full_store;            // 1: the destination does not hold the image of two launches back
};

// ---- pieces of both kernels --------------------------------------------------------

__device__ __forceinline__ void sync_wave() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Bits of b below this lane's.
__device__ __forceinline__ int bits_below(unsigned long long b) {
  return int(__builtin_amdgcn_mbcnt_hi(uint32_t(b >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(b), 0u)));
}

// OR over the 8 lanes that share a row of bits (lane = 8 * row + word).
__device__ __forceinline__ uint32_t or8(uint32_t v) {
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x141, 0xF, 0xF, true));  // row_half_mirror
  return v;
}

// Sum over the same 8 lanes.
__device__ __forceinline__ uint32_t add8(uint32_t v) {
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0xB1, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x4E, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x141, 0xF, 0xF, true));
  return v;
}

// alpha as the band test takes it (see sat_add_u8x4).
struct Band {
  int alpha;
  uint32_t am1_16, a_16;
  __device__ __forceinline__ explicit Band(int al)
      : alpha(al), am1_16(uint32_t(al > 0 ? al - 1 : 0) * 0x01000100u), a_16(uint32_t(al) * 0x01000100u) {}
};

// A tile's place: LDS row i holds image row row_first + i, computed row i is
// LDS row i + BETA, computed column c is LDS byte 4 + c of its row and image
// column col_first + c; computed rows own .. own + TH - 1 are the owned ones.
struct DeepGeom {
  int tx, c0, r0, own, TH, row_first, col_first;
  bool aligned;
  template <int BETA>
  __device__ __forceinline__ static DeepGeom of(const DeepTile& a, int tile) {
    DeepGeom g;
    const int ty = tile / a.tiles_x;
    g.tx = tile - ty * a.tiles_x;
    g.own = (a.depth - 1) * BETA;
    g.TH = a.th;
    g.r0 = ty * g.TH;
    g.c0 = g.tx * kDeepCols;
    g.row_first = g.r0 - g.own - BETA;
    g.col_first = g.c0 - kDeepHalo;
    // rows start on dword boundaries: loads and stores move whole dwords
    g.aligned = ((reinterpret_cast<uintptr_t>(a.src) | reinterpret_cast<uintptr_t>(a.dst)) & 3u) == 0 &&
                (a.cols & 3) == 0;
    return g;
  }
};

// What pass t must get right: the interior pixels among the owned region and
// as much around it as the passes after t still read.
struct DeepBounds {
  int row_lo, row_hi, col_lo, col_hi;   // computed rows and columns
  template <int BETA>
  __device__ __forceinline__ static DeepBounds of(const DeepTile& a, const DeepGeom& g, int t) {
    const int rest = (a.npasses - 1 - t) * BETA;
    DeepBounds b;
    b.row_lo = max(g.own - rest, -g.row_first);
    b.row_hi = min(g.own + g.TH + rest, a.rows - 2 * BETA - g.row_first);
    b.col_lo = max(kDeepHalo - rest, BETA - g.col_first);
    b.col_hi = min(kDeepHalo + kDeepCols + rest, a.cols - BETA - g.col_first);
    return b;
  }
};

// A change map's word: bit g: one of the pixels 8g .. 8g+7 changed in the
// launch's last pass; kMapMoves: the segment may differ from two passes
// before the launch's end; kMapAny: it changed in some pass of the launch.
constexpr uint32_t kMapGroups = 0x0FFFFFFFu;
constexpr uint32_t kMapMoves = 1u << 30;
constexpr uint32_t kMapAny = 1u << 31;

// The previous launch's map words of the LDS rows, one row per lane (and
// round of 64 rows): of the tile's own column and of its neighbours'.
template <int BROWS>
struct DeepMap {
  static constexpr int NCH = (BROWS + 63) / 64;
  uint32_t mc[NCH];                // the tile's own words
  uint32_t gr[NCH];                // groups of 8 computed columns (bit j: 8j .. 8j+7) with a change
  unsigned long long stale[NCH];   // LDS rows that the destination does not hold
  // false: the tile ends this launch as it starts it
  __device__ __forceinline__ bool read(const DeepTile& a, const DeepGeom& g, int lane) {
    uint32_t ml[NCH], mr[NCH];
#pragma unroll
    for (int h = 0; h < NCH; ++h) {
      mc[h] = ml[h] = mr[h] = 0u;
      stale[h] = ~0ull;
    }
    if (a.map_in == nullptr) return true;
#pragma unroll
    for (int h = 0; h < NCH; ++h) {
      const int i = h * 64 + lane;
      const int r = g.row_first + i;
      if (i < BROWS && r >= 0 && r < a.rows) {
        const uint32_t* m = a.map_in + size_t(r) * size_t(a.tiles_x) + size_t(g.tx);
        mc[h] = m[0];
        ml[h] = g.tx > 0 ? m[-1] : 0u;
        mr[h] = g.tx + 1 < a.tiles_x ? m[1] : 0u;
      }
    }
    uint32_t moves = 0u, groups = 0u;
#pragma unroll
    for (int h = 0; h < NCH; ++h) {
      gr[h] = ((mc[h] & kMapGroups) << 2) | ((ml[h] >> 26) & 3u) | (mr[h] << 30);
      moves |= (mc[h] | ml[h] | mr[h]) & kMapMoves;
      groups |= gr[h];
      if (!a.full_store) stale[h] = __builtin_amdgcn_ballot_w64((mc[h] & kMapAny) != 0u);
    }
    // Where no pixel in reach differs from two passes before, the region
    // goes on alternating between its last two images, and an even number
    // of passes ends where it began.
    return __builtin_amdgcn_ballot_w64((a.advance & 1 ? groups : moves) != 0u) != 0ull;
  }
  __device__ __forceinline__ bool row_stale(int lr) const {
    return ((stale[NCH > 1 && lr >= 64 ? NCH - 1 : 0] >> (lr & 63)) & 1ull) != 0ull;
  }
  // The rows i with mine(i), as change bits (every pixel of a marked group).
  template <class Mine>
  __device__ __forceinline__ void spread(uint32_t* chg, int lane, Mine mine) const {
#pragma unroll
    for (int h = 0; h < NCH; ++h) {
      const int i = h * 64 + lane;
      if (i < BROWS && mine(i)) {
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const uint32_t n = (gr[h] >> (4 * d)) & 15u;
          chg[i * 8 + d] = ((n | (n << 7) | (n << 14) | (n << 21)) & 0x01010101u) * 255u;
        }
      }
    }
  }
  // The number of marked groups; if there are at most `most`, their entries
  // (LDS row << 8 | first computed column) in list (where write).
  __device__ __forceinline__ int list_groups(uint16_t* list, int lane, int most, bool write) const {
    int total = 0, pos[NCH];
#pragma unroll
    for (int h = 0; h < NCH; ++h) {
      const uint32_t c = uint32_t(__builtin_popcount(gr[h]));
      pos[h] = total;
#pragma unroll
      for (int b = 0; b < 6; ++b) {
        const unsigned long long bm = __builtin_amdgcn_ballot_w64((c >> b) & 1u);
        pos[h] += bits_below(bm) << b;
        total += int(__builtin_popcountll(bm)) << b;
      }
    }
    if (write && total <= most) {
#pragma unroll
      for (int h = 0; h < NCH; ++h)
        for (uint32_t m = gr[h]; m != 0u; m &= m - 1u)
          list[pos[h]++] = uint16_t((h * 64 + lane) << 8 | __builtin_ctz(m) << 3);
    }
    return total;
  }
};

// Loads of NROWS LDS rows (first, first + step, ...): range-checked raw
// buffer loads over the image's dwords, as in pass_kernel.hpp, all issued
// before the first use.  put(i - first, dword of lane's columns) takes row i.
template <int NROWS, int step, class Put>
__device__ __forceinline__ void load_rows(const DeepTile& a, const DeepGeom& g, int lane, int first,
                                          Put put) {
  const uintptr_t sb = reinterpret_cast<uintptr_t>(a.src);
  const uintptr_t se = sb + uintptr_t(a.rows) * uintptr_t(a.cols);
  const uintptr_t base = sb & ~uintptr_t(3);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>(base), 0, int(uint32_t(((se + 3) & ~uintptr_t(3)) - base)), kBufferWord3);
  // byte of the row's computed column 0, from the first dword (modulo 2^32)
  const uint32_t origin = uint32_t(sb & 3u) + uint32_t(g.row_first) * uint32_t(a.cols) + uint32_t(g.col_first);
  uint32_t d0[NROWS];
  if (g.aligned) {
#pragma unroll
    for (int u = 0; u < NROWS; ++u) {
      const uint32_t o = origin + uint32_t(first + u * step) * uint32_t(a.cols);
      d0[u] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(o + 4u * uint32_t(lane)), 0, 0);
    }
#pragma unroll
    for (int u = 0; u < NROWS; ++u) put(u * step, d0[u]);
  } else {
    // two dwords per lane, the second for the bytes past the first's end
    uint32_t d1[NROWS];
#pragma unroll
    for (int u = 0; u < NROWS; ++u) {
      const uint32_t o = origin + uint32_t(first + u * step) * uint32_t(a.cols);
      const uint32_t a0 = (o & ~3u) + 4u * uint32_t(lane);
      d0[u] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(a0), 0, 0);
      d1[u] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(a0 + 4u), 0, 0);
    }
#pragma unroll
    for (int u = 0; u < NROWS; ++u) {
      const uint32_t o = origin + uint32_t(first + u * step) * uint32_t(a.cols);
      put(u * step, __builtin_amdgcn_alignbyte(d1[u], d0[u], o & 3u));
    }
  }
}

// Store the owned segment of image row r; row: its owned dwords in LDS.
__device__ __forceinline__ void store_row(const DeepTile& a, const DeepGeom& g, int lane, int r,
                                          const uint32_t* row) {
  uint8_t* const d = a.dst + size_t(r) * size_t(a.cols) + size_t(g.c0);
  if (g.aligned) {
    if (lane < kDeepCols / 4 && g.c0 + 4 * lane < a.cols) reinterpret_cast<uint32_t*>(d)[lane] = row[lane];
    return;
  }
  const int len = (a.cols - g.c0) < kDeepCols ? (a.cols - g.c0) : kDeepCols;
  const uintptr_t b = reinterpret_cast<uintptr_t>(d), e = b + uintptr_t(len);
  const uintptr_t ad = (b & ~uintptr_t(3)) + 4u * uintptr_t(lane);
  if (ad >= e) return;
  if (ad >= b && ad + 4 <= e) {
    const int off = int(ad - b);
    *reinterpret_cast<uint32_t*>(ad) =
        __builtin_amdgcn_alignbyte(row[(off >> 2) + 1], row[off >> 2], uint32_t(off) & 3u);
  } else {
    const uint8_t* rb = reinterpret_cast<const uint8_t*>(row);
    for (uintptr_t p = ad > b ? ad : b; p < ad + 4 && p < e; ++p) *reinterpret_cast<uint8_t*>(p) = rb[p - b];
  }
}

// Copy the owned segment of image row r from the source.
__device__ __forceinline__ void copy_row(const DeepTile& a, const DeepGeom& g, int lane, int r) {
  const size_t o = size_t(r) * size_t(a.cols) + size_t(g.c0);
  if (g.aligned) {
    if (lane < kDeepCols / 4 && g.c0 + 4 * lane < a.cols)
      reinterpret_cast<uint32_t*>(a.dst + o)[lane] = reinterpret_cast<const uint32_t*>(a.src + o)[lane];
    return;
  }
#pragma unroll
  for (int u = 0; u < (kDeepCols + 63) / 64; ++u) {
    const int c = 64 * u + lane;
    if (c < kDeepCols && g.c0 + c < a.cols) a.dst[o + c] = a.src[o + c];
  }
}

// Algorithm 2 for the pixel at LDS (row bc, byte bb) of src, exactly: its
// value x and what it becomes (see pass_kernel.hpp for the byte arithmetic).
// It is replaced if at most 2 window pixels lie in its band; with alpha > 0
// one of them is the pixel itself, so the band's sum of grey levels gives the
// other's, and the outside pixels' squares are the window's less those two.
template <int BETA>
__device__ __forceinline__ uint32_t pass_value(const uint32_t* src, int bc, int bb, const Band& band,
                                               uint32_t& x) {
  constexpr int NW = 2 * BETA + 1, N = NW * NW, NG = (NW + 3) / 4;
  x = reinterpret_cast<const uint8_t*>(src)[bc * kRowBytes + bb];
  const uint32_t nx4 = ~(x * 0x01010101u);
  const uint32_t nlo4 = sat_add_u8x4(nx4, band.am1_16);
  const uint32_t nhi4 = sat_sub_u8x4(nx4, band.a_16);
  uint32_t S = 0, K = 0, in = 0;
#pragma unroll
  for (int dr = -BETA; dr <= BETA; ++dr) {
    const int A = (bc + dr) * kRowBytes + bb - BETA;
    const uint32_t* wp = src + (A >> 2);
    const uint32_t sh = uint32_t(A) & 3u;
    uint32_t d[NG + 1];
#pragma unroll
    for (int g = 0; g <= NG; ++g) d[g] = wp[g];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      uint32_t y = __builtin_amdgcn_alignbyte(d[g + 1], d[g], sh);
      const int nvalid = (NW - 4 * g) < 4 ? (NW - 4 * g) : 4;
      if (nvalid < 4) y &= 0xFFFFFFFFu >> (8 * (4 - nvalid));
      uint32_t in7 = __builtin_amdgcn_lerp(y, nlo4, 0x01010101u) ^ __builtin_amdgcn_lerp(y, nhi4, 0u);
      in7 &= 0x80808080u >> (8 * (4 - nvalid));
      K += uint32_t(__builtin_popcount(in7));
      in = __builtin_amdgcn_udot4(in7 >> 7, y, in, false);
      S = __builtin_amdgcn_udot4(y, y, S, false);
    }
  }
  if (band.alpha <= 0) K = in = 0u;                // an empty band
  uint32_t v = x;
  if (K <= 2u) {
    const uint32_t other = in - x;                 // (K 1: 0)
    if (K != 0u) S -= x * x + other * other;
    v = isqrt_small(udiv_small(S, uint32_t(N) - K));
  }
  return v;
}

// The active pixels of up to 8 computed rows from `strip` on, as bits: lane 8
// ri + wd has word wd of row strip + ri.  cur: the last pass's change bits.
template <int BETA>
__device__ __forceinline__ uint32_t active_word(const uint32_t* cur, int strip, int ri, int wd,
                                                const DeepBounds& b) {
  const uint32_t* c = cur + (strip + ri + BETA) * 8 + wd;
  uint32_t v = 0u;
#pragma unroll
  for (int dr = -BETA; dr <= BETA; ++dr) v |= c[8 * dr];
  // the neighbouring words of the row (at a row's ends the lane next door has
  // another row's: such columns are outside what a pass must get right)
  const uint32_t vl = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));  // row_shr:1
  const uint32_t vr = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x101, 0xF, 0xF, true));  // row_shl:1
  uint32_t act = v;
#pragma unroll
  for (int s = 1; s <= BETA; ++s)
    act |= __builtin_amdgcn_alignbit(v, vl, 32 - s) | __builtin_amdgcn_alignbit(vr, v, s);
  const int lo = b.col_lo - 32 * wd, hi = b.col_hi - 32 * wd, i = strip + ri;
  uint32_t m = hi <= 0 ? 0u : (hi >= 32 ? ~0u : (1u << hi) - 1u);
  m &= lo >= 32 ? 0u : (lo <= 0 ? ~0u : ~((1u << lo) - 1u));
  return i >= b.row_lo && i < b.row_hi ? act & m : 0u;
}

// Queue the words with an active pixel (row of the strip << 10 | word << 4 |
// active pixels) if there are at most kDeepWords; their number either way.
__device__ __forceinline__ int queue_words(uint32_t act, uint16_t* wq, int ri, int wd) {
  if (__builtin_amdgcn_ballot_w64(act != 0u) == 0ull) return 0;
  uint32_t z = act | (act >> 1);
  z = (z | (z >> 2)) & 0x11111111u;                // bit 4d: word d has an active pixel
  const uint32_t c = uint32_t(__builtin_popcount(z));
  int pos = 0, total = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const unsigned long long bm = __builtin_amdgcn_ballot_w64((c >> b) & 1u);
    pos += bits_below(bm) << b;
    total += int(__builtin_popcountll(bm)) << b;
  }
  if (total <= kDeepWords) {
    const uint32_t ent = (uint32_t(ri) << 10) | (uint32_t(wd) << 7);
    while (z != 0u) {
      const uint32_t k = uint32_t(__builtin_ctz(z));
      wq[pos++] = uint16_t(ent | (k << 2) | ((act >> k) & 15u));
      z &= z - 1u;
    }
    sync_wave();
  }
  return total;
}

// The band test of the 4 pixels of word `word` of LDS row lr: bit 7 of each
// byte is set where at least two other pixels of the window are in the band.
template <int BETA>
__device__ __forceinline__ uint32_t word_settled(const uint32_t* src, int lr, int word, const Band& band,
                                                 uint32_t& X) {
  constexpr int NW = 2 * BETA + 1;
  const uint32_t* p = src + lr * kRowWords + word;
  uint32_t rows[NW][3];
#pragma unroll
  for (int r = 0; r < NW; ++r)
#pragma unroll
    for (int k = 0; k < 3; ++k) rows[r][k] = p[(r - BETA) * kRowWords + k];
  X = rows[BETA][1];
  if (band.alpha <= 0) return 0u;
  const uint32_t nlo = sat_add_u8x4(~X, band.am1_16);
  const uint32_t nhi = sat_sub_u8x4(~X, band.a_16);
  uint32_t t1 = 0, t2 = 0;
#pragma unroll
  for (int g = 0; g < BETA * (BETA + 1); ++g) {
    uint32_t m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      int dr = 0, dc = 0;
      ring_offset(4 * g + u, dr, dc);
      const uint32_t (&R)[3] = rows[BETA + dr];
      const uint32_t Y = dc == 0 ? R[1] : dc < 0 ? (dc == -4 ? R[0] : __builtin_amdgcn_alignbyte(R[1], R[0], 4 + dc))
                                                 : (dc == 4 ? R[2] : __builtin_amdgcn_alignbyte(R[2], R[1], dc));
      m[u] = __builtin_amdgcn_lerp(Y, nlo, 0x01010101u) ^ __builtin_amdgcn_lerp(Y, nhi, 0u);
    }
    const uint32_t cg = bitop3_maj(m[0], m[1], m[2]);
    const uint32_t sg = bitop3_xor3(m[0], m[1], m[2]);
    const uint32_t ug = bitop3_maj(t1, sg, m[3]);
    t2 = bitop3_or3(t2, cg, ug);
    t1 = bitop3_or3(t1, sg, m[3]);
  }
  return t2;
}

// Append one entry per candidate byte (bit 7 of cand's bytes; the lane's
// first entry `ent`) to the ring q.
__device__ __forceinline__ void push_candidates(uint32_t cand, uint32_t ent, uint16_t* q, int& qtail) {
  const uint32_t c = uint32_t(__builtin_popcount(cand));
  const unsigned long long b0 = __builtin_amdgcn_ballot_w64(c & 1u);
  const unsigned long long b1 = __builtin_amdgcn_ballot_w64(c & 2u);
  const unsigned long long b2 = __builtin_amdgcn_ballot_w64(c & 4u);
  int pos = qtail + bits_below(b0) + 2 * bits_below(b1) + 4 * bits_below(b2);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if ((cand >> (8 * k + 7)) & 1u) {
      q[pos & (kQueueCap - 1)] = uint16_t(ent + uint32_t(k));
      ++pos;
    }
  }
  qtail += __builtin_popcountll(b0) + 2 * __builtin_popcountll(b1) + 4 * __builtin_popcountll(b2);
  sync_wave();
}

// The band test on every pixel of R computed rows from `strip` on, as in
// pass_kernel.hpp.  Candidates go to the ring q (through dq) and to
// evaluate(valid, LDS row << 8 | column) in rounds of 64; those left over are
// entries [qhead, qtail) of q.  row(LDS row, lane's dword, candidates, pixels
// that the pass must get right) takes every row.
template <int BETA, int R, class Eval, class Row>
__device__ __forceinline__ void dense_rows(const uint32_t* src, int strip, int lane, const DeepBounds& b,
                                           const Band& band, uint16_t* q, uint32_t* dq, int& qhead,
                                           int& qtail, Eval evaluate, Row row) {
  constexpr int NW = 2 * BETA + 1;
  int dhead = 0, dtail = 0;
  uint32_t colmask = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = 4 * lane + k;
    if (c >= b.col_lo && c < b.col_hi) colmask |= 0x80u << (8 * k);
  }
  auto expand = [&](int n) {
    const uint32_t e = lane < n ? dq[(dhead + lane) & (kLaneQueueCap - 1)] : 0u;
    dhead += n;
    push_candidates(e & 0x80808080u, (e & 0x7F00u) | ((e & 63u) << 2), q, qtail);   // row << 8 | first column
  };
  uint32_t win[NW][NW];
  auto load_row = [&](int i, uint32_t (&wr)[NW]) {
    const uint32_t* rp = src + (strip + i) * kRowWords + lane;
    const uint32_t L = rp[0], C = rp[1], Rr = rp[2];
#pragma unroll
    for (int dc = -BETA; dc <= BETA; ++dc) {
      if (dc < 0)
        wr[dc + BETA] = (dc == -4) ? L : __builtin_amdgcn_alignbyte(C, L, 4 + dc);
      else if (dc == 0)
        wr[BETA] = C;
      else
        wr[dc + BETA] = (dc == 4) ? Rr : __builtin_amdgcn_alignbyte(Rr, C, dc);
    }
  };
#pragma unroll
  for (int i = 0; i < 2 * BETA; ++i) load_row(i, win[i]);
#pragma unroll 1
  for (int j0 = 0; j0 < R; j0 += NW) {
#pragma unroll
    for (int jj = 0; jj < NW; ++jj) {
      const int jc = j0 + jj;
      if (jc < R) {
        load_row(jc + 2 * BETA, win[(jj + 2 * BETA) % NW]);
        const int i = strip + jc;
        const uint32_t X = win[(jj + BETA) % NW][BETA];
        const bool test = i >= b.row_lo && i < b.row_hi;
        const uint32_t tested = test ? colmask : 0u;
        uint32_t cand = tested;
        if (test && band.alpha > 0) {
          const uint32_t nx = ~X;
          const uint32_t nlo = sat_add_u8x4(nx, band.am1_16);
          const uint32_t nhi = sat_sub_u8x4(nx, band.a_16);
          uint32_t t1 = 0, t2 = 0;
          auto group = [&](int g) {
            uint32_t m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              int dr = 0, dc = 0;
              ring_offset(4 * g + u, dr, dc);
              const uint32_t Y = win[(jj + BETA + dr + NW) % NW][dc + BETA];
              m[u] = __builtin_amdgcn_lerp(Y, nlo, 0x01010101u) ^ __builtin_amdgcn_lerp(Y, nhi, 0u);
            }
            const uint32_t cg = bitop3_maj(m[0], m[1], m[2]);
            const uint32_t sg = bitop3_xor3(m[0], m[1], m[2]);
            const uint32_t ug = bitop3_maj(t1, sg, m[3]);
            t2 = bitop3_or3(t2, cg, ug);
            t1 = bitop3_or3(t1, sg, m[3]);
          };
          group(0);
          cand = colmask & ~t2;
          bool more = __builtin_amdgcn_ballot_w64(cand != 0u) != 0ull;
          if (more) {
            group(1);
            cand = colmask & ~t2;
            more = __builtin_amdgcn_ballot_w64(cand != 0u) != 0ull;
          }
#pragma unroll
          for (int d = 2; d <= BETA; ++d) {
            if (more) {
#pragma unroll
              for (int g = d * (d - 1); g < d * (d + 1); ++g) group(g);
              cand = colmask & ~t2;
              if (d < BETA) more = __builtin_amdgcn_ballot_w64(cand != 0u) != 0ull;
            }
          }
        }
        row(i + BETA, X, cand, tested);
        const unsigned long long hb = __builtin_amdgcn_ballot_w64(cand != 0u);
        if (hb != 0ull) {
          const int pos = dtail + bits_below(hb);
          if (cand != 0u)
            dq[pos & (kLaneQueueCap - 1)] = cand | uint32_t(lane) | (uint32_t(i + BETA) << 8);
          dtail += __builtin_popcountll(hb);
          if (dtail - dhead >= 64) {
            sync_wave();
            expand(64);
            while (qtail - qhead >= 64) {
              evaluate(true, q[(qhead + lane) & (kQueueCap - 1)]);
              qhead += 64;
            }
          }
        }
      }
    }
  }
  if (dtail > dhead) {
    sync_wave();
    expand(dtail - dhead);
  }
}

// Bits of a word's 32 pixels as its 4 groups of 8.
__device__ __forceinline__ uint32_t groups4(uint32_t x) {
  x |= x >> 4;
  x |= x >> 2;
  x |= x >> 1;
  return ((x & 0x01010101u) * 0x10204080u) >> 28;
}

// ---- a tile ---------------------------------------------------------------------------
//
// 8 waves of 8 rows; or 16 waves of 4 rows, where a launch leaves every CU at
// most one tile and a pass takes as long as a strip (1024^2, beta 2, k 32: 64
// us against 72; 128^2, k 5: 19 against 22; at beta 4 the window's registers
// spill, and 8 waves are faster, 31 us against 33 at 500 x 700, k 12).

template <int BETA, int WAVES>
struct DeepSmem {
  static constexpr int R = kDeepH / WAVES;                 // rows of a strip
  static constexpr int BROWS = kDeepH + 2 * BETA;          // rows per LDS buffer
  static_assert(R <= 8 && R * WAVES == kDeepH, "a lane has one word of bits");
  uint32_t buf0[BROWS * kRowWords + 1];
  uint32_t buf1[BROWS * kRowWords + 1];
  uint32_t chg[2][BROWS * 8];       // change bits: word d of a row, bit i: computed column 32d + i
  uint16_t queue[WAVES][kQueueCap];
  uint32_t lanes[WAVES][kLaneQueueCap];   // a dense strip's lane queue, or a sparse one's words
  uint16_t list[2][kDeepListMost];  // pixels the last pass changed, and this one's (alternating):
                                    // LDS row << 8 | computed column
  unsigned nlist[3];                // how many there are: the last pass's, this one's, the next one's
  int runs[WAVES];                  // of the tiles looked at: which run
  unsigned fill;                    // entries of a list built from the change bits
  unsigned moves[3];                // the same of: a pixel became other than two passes before
  unsigned count[kDeepMaxPasses];   // owned pixels each pass changed
  unsigned moved[kDeepMaxPasses];   // (period-2 launches) whether a pass left a pixel other than two
                                    // passes before; over the tiles of the workgroup
  unsigned row_any[(BROWS + 31) / 32];               // LDS rows changed before list passes
  unsigned changed[kDeepMaxPasses];
};

// A tile that ends the launch as it starts it, by `waves` waves of which this
// is number w: rows the destination does not hold yet are copied, and every
// pass changes as many pixels as the last one did.  Wave 0 returns how many.
template <int BETA, int BROWS>
__device__ __forceinline__ unsigned idle_tile(const DeepTile& a, const DeepGeom& g, const DeepMap<BROWS>& map,
                                              int lane, int w, int waves) {
  static_assert(BROWS - 2 * BETA <= 64, "one lane per owned row");
  unsigned c = 0u;
  if (w == 0) {
    const bool in = lane < g.TH && g.r0 + lane < a.rows;
    const size_t at = size_t(g.r0 + lane) * size_t(a.tiles_x) + size_t(g.tx);
    c = in ? a.cnt_in[at] : 0u;
    if (in && a.map_out != nullptr) {
      a.map_out[at] = a.map_in[at] & kMapGroups;
      a.cnt_out[at] = uint8_t(c);
    }
    if (__builtin_amdgcn_ballot_w64(c != 0u) != 0ull) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    }
  }
  for (int o = w; o < g.TH && g.r0 + o < a.rows; o += waves)
    if (map.row_stale(g.own + BETA + o)) copy_row(a, g, lane, g.r0 + o);
  return c;
}

// Run the tile's passes and add its per-pass changed counts to sm.changed
// (threads 0 .. npasses - 1, one pass each).  Called by every thread of the
// workgroup.
template <int BETA, int WAVES, bool CYC = false>
__device__ __forceinline__ void run_deep_tile(DeepSmem<BETA, WAVES>& sm, const DeepTile& a, int tile) {
  constexpr int NW = 2 * BETA + 1;
  constexpr int N = NW * NW;
  constexpr int R = kDeepH / WAVES;
  constexpr int BROWS = kDeepH + 2 * BETA;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const DeepGeom g = DeepGeom::of<BETA>(a, tile);
  const Band band(a.alpha);
  const bool has_map = a.map_in != nullptr;
  uint16_t* q = sm.queue[w];

  // Every wave reads the words of all LDS rows, so that all of them decide
  // alike whether the tile runs, without a barrier.
  DeepMap<BROWS> map;
  if (!map.read(a, g, lane)) {
    const unsigned c = idle_tile<BETA>(a, g, map, lane, w, WAVES);
    if (tid < a.npasses) sm.changed[tid] += c;
    return;
  }
  if (tid < 3) sm.nlist[tid] = sm.moves[tid] = 0u;
  if (tid == 0) sm.fill = 0u;
  if (tid < kDeepMaxPasses) sm.count[tid] = 0u;
  if (tid < int(sizeof(sm.row_any) / sizeof(unsigned))) sm.row_any[tid] = 0u;
  for (int m = tid; m < 2 * BROWS * 8; m += WAVES * 64) (&sm.chg[0][0])[m] = 0u;
  // Both buffers start as the image: only dense strips copy rows through.
  load_rows<(BROWS + WAVES - 1) / WAVES, WAVES>(a, g, lane, w, [&](int k, uint32_t d) {
    if (k + WAVES <= BROWS || w + k < BROWS) {
      sm.buf0[(w + k) * kRowWords + 1 + lane] = d;
      sm.buf1[(w + k) * kRowWords + 1 + lane] = d;
    }
  });
  // The first pass follows the map's marked groups of 8 pixels, by list where
  // they are few.
  unsigned n = ~0u;
  bool groups = false;                             // the list is of groups
  if (has_map) {
    n = unsigned(map.list_groups(sm.list[0], lane, kDeepListMost, w == 0));
    groups = n <= unsigned(kDeepListMost);
    if (!groups) {
      __syncthreads();   // the clearing above
      map.spread(sm.chg[0], lane, [&](int i) { return ((i >> 3) % WAVES) == w; });
    }
  }
  __syncthreads();

  const int ri = lane >> 3, wd = lane & 7;         // this lane's row of the strip and word of bits
  const bool has_word = R == 8 || ri < R;
  const int strip = w * R;                         // this wave's first computed row
  const int mine = (strip + ri + BETA) * 8 + wd;
  uint32_t any_bits = 0u;                          // changes of the strip's passes (not of list passes)
  uint32_t* src = sm.buf0;
  uint32_t* dst = sm.buf1;
  bool listed = has_map;                           // sm.list holds the last pass's changes, chg[cb ^ 1] is clear
  bool periodic = false;
  int cb = 0;                                      // chg[cb]: the last pass's changes
  int t = 0;
  // owned pixels: LDS rows own_r .. , computed columns kDeepHalo ..
  const unsigned own_r = unsigned(g.own + BETA), own_h = unsigned(min(g.TH, a.rows - g.r0));
  const unsigned own_w = unsigned(min(kDeepCols, a.cols - g.c0));
#pragma unroll 1
  for (; t < a.npasses; ++t) {
    if (t > 0) n = unsigned(__builtin_amdgcn_readfirstlane(int(sm.nlist[t % 3])));
    // Nothing changed: nor will any later pass.  Nothing other than two
    // passes before: the tile goes on alternating between its two buffers.
    if (n == 0u || (t > 1 && __builtin_amdgcn_readfirstlane(int(sm.moves[t % 3])) == 0)) {
      periodic = true;
      break;
    }
    if (tid == 0) sm.nlist[(t + 2) % 3] = sm.moves[(t + 2) % 3] = 0u;
    uint32_t* cur = sm.chg[cb];
    uint32_t* nxt = sm.chg[cb ^ 1];
    uint16_t* list = sm.list[t & 1];
    unsigned wave_changed = 0, wave_fresh = 0;
    bool moved = false;
    const DeepBounds b = DeepBounds::of<BETA>(a, g, t);

    // The pixel at e (LDS row << 8 | computed column): evaluated and written
    // to the destination.  True if it changed.
    auto step = [&](unsigned e) {
      const int lr = int(e >> 8), c = int(e & 255u);
      uint32_t x;
      uint8_t* d = reinterpret_cast<uint8_t*>(dst) + lr * kRowBytes + 4 + c;
      const uint32_t before = *d;
      const uint32_t v = pass_value<BETA>(src, lr, 4 + c, band, x);
      if (v != before) {
        *d = uint8_t(v);
        moved = true;
      }
      return v != x;
    };
    auto owned = [&](unsigned e) { return (e >> 8) - own_r < own_h && (e & 255u) - unsigned(kDeepHalo) < own_w; };

    if (n <= unsigned(kDeepListMost)) {
      // ---- few changes: every pixel of every changed pixel's window -----------
      // Shared by all waves; a pixel may come more than once, and its change
      // bit tells which came first.
      if (!listed) {
        // the list, from the change bits; and the bits of two passes back go
        uint32_t m = has_word ? cur[mine] : 0u;
        if (has_word) nxt[mine] = 0u;
        any_bits |= m;
        if (m != 0u) {
          unsigned at = atomicAdd(&sm.fill, unsigned(__builtin_popcount(m)));
          for (; m != 0u; m &= m - 1u, ++at)
            if (at < unsigned(kDeepListMost))
              list[at] = uint16_t((strip + ri + BETA) << 8 | wd << 5 | __builtin_ctz(m));
        }
        __syncthreads();
        if (tid == 0) sm.fill = 0u;
      }
      // chg[cb] is cleared behind the list for the pass after this (not where
      // the map is taken before the last pass)
      if (!groups && tid < int(n)) {
        const unsigned e = list[tid];
        const int lr = int(e >> 8);
        if (!CYC || t + 1 < a.npasses || a.advance == a.npasses) cur[lr * 8 + (int(e & 255u) >> 5)] = 0u;
        atomicOr(&sm.row_any[lr >> 5], 1u << (lr & 31));
      }
      const int span = groups ? NW + 7 : NW;       // window columns of an entry
      const int items = int(n) * span * NW;
      for (int m0 = w * 64; m0 < items; m0 += WAVES * 64) {
        const int m = m0 + lane;
        const int p = groups ? m / ((NW + 7) * NW) : m / N, k = m - p * (span * NW);
        const int dr = groups ? k / (NW + 7) : k / NW, dc = k - dr * span;
        const unsigned le = list[m < items ? p : 0];
        const int lr = int(le >> 8) + dr - BETA, c = int(le & 255u) + dc - BETA;
        const unsigned e = unsigned(lr) << 8 | unsigned(c);
        bool fresh = false;
        if (m < items && lr >= b.row_lo + BETA && lr < b.row_hi + BETA && c >= b.col_lo && c < b.col_hi && step(e)) {
          const uint32_t bit = 1u << (c & 31);
          fresh = (atomicOr(&nxt[lr * 8 + (c >> 5)], bit) & bit) == 0u;
        }
        const unsigned long long fm = __builtin_amdgcn_ballot_w64(fresh);
        if (fm != 0ull) {
          wave_changed += __builtin_popcountll(__builtin_amdgcn_ballot_w64(fresh && owned(e)));
          // listed while they fit
          unsigned at = 0u;
          if (lane == 0) at = atomicAdd(&sm.nlist[(t + 1) % 3], unsigned(__builtin_popcountll(fm)));
          at = unsigned(__builtin_amdgcn_readfirstlane(int(at))) + unsigned(bits_below(fm));
          if (fresh && at < unsigned(kDeepListMost)) sm.list[(t & 1) ^ 1][at] = uint16_t(e);
        }
      }
      listed = true;
    } else {
      // ---- by strips -------------------------------------------------------------
      const bool live = strip < b.row_hi && strip + R > b.row_lo;   // some row counts in this pass
      const bool all = t == 0 && !has_map;           // no change bits yet: every pixel is active
      if (!all && has_word) any_bits |= t > 0 ? cur[mine] : 0u;
      if (has_word) nxt[mine] = 0u;
      sync_wave();                                 // cleared before this wave sets bits
      if (live) {
        int qhead = 0, qtail = 0;
        auto evaluate = [&](bool valid, unsigned e) {
          const bool ch = valid && step(e);
          if (ch) atomicOr(&nxt[(e >> 8) * 8 + ((e & 255u) >> 5)], 1u << (e & 31u));
          const unsigned long long cm = __builtin_amdgcn_ballot_w64(ch);
          if (cm == 0ull) return;
          wave_fresh += __builtin_popcountll(cm);
          wave_changed += __builtin_popcountll(__builtin_amdgcn_ballot_w64(ch && owned(e)));
        };
        uint16_t* wq = reinterpret_cast<uint16_t*>(sm.lanes[w]);
        const int words = all ? kDeepWords + 1 : queue_words(has_word ? active_word<BETA>(cur, strip, ri, wd, b) : 0u, wq, ri, wd);
        if (words > kDeepWords) {
          dense_rows<BETA, R>(src, strip, lane, b, band, q, sm.lanes[w], qhead, qtail, evaluate,
                           [&](int lr, uint32_t X, uint32_t cand, uint32_t tested) {
                             uint32_t* d = dst + lr * kRowWords + 1 + lane;
                             if constexpr (CYC) {
                               // candidates keep the destination's byte until they are evaluated
                               const uint32_t x = (X ^ *d) & ~((cand >> 7) * 255u);
                               moved = moved || (x & ((tested >> 7) * 255u)) != 0u;
                               *d ^= x;
                             } else {
                               *d = X;
                             }
                           });
          if (!CYC) moved = true;                  // (not looked at)
        } else {
          for (int m0 = 0; m0 < words; m0 += 64) {
            uint32_t cand = 0u, ent = 0u;
            if (m0 + lane < words) {
              const uint32_t e = wq[m0 + lane];
              const int lr = strip + BETA + int(e >> 10), wi = int(e >> 4) & 63;
              const uint32_t act = e & 15u;
              uint32_t X;
              cand = word_settled<BETA>(src, lr, wi, band, X);
              cand = ~cand & (((act | (act << 7) | (act << 14) | (act << 21)) & 0x01010101u) << 7);
              ent = uint32_t(lr) << 8 | uint32_t(wi) << 2;
              // pixels that stay, where the destination holds something else
              // (candidates are written when they are evaluated)
              uint32_t* d = dst + lr * kRowWords + 1 + wi;
              const uint32_t x = X ^ *d;
              const uint32_t other = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & ~cand & 0x80808080u;
              if (other != 0u) {
                const uint32_t full = (other >> 7) * 255u;
                *d = (*d & ~full) | (X & full);
                // (beside the region that this pass must get right, what the
                // destination holds says nothing)
                bool counts = !CYC;
                if constexpr (CYC) {
#pragma unroll
                  for (int k = 0; k < 4; ++k)
                    counts = counts || (((other >> (8 * k + 7)) & 1u) != 0u && 4 * wi + k >= b.col_lo && 4 * wi + k < b.col_hi);
                }
                moved = moved || counts;
              }
            }
            push_candidates(cand, ent, q, qtail);
            while (qtail - qhead >= 64) {
              evaluate(true, q[(qhead + lane) & (kQueueCap - 1)]);
              qhead += 64;
            }
          }
        }
        for (; qhead < qtail; qhead += 64) evaluate(qhead + lane < qtail, q[(qhead + lane) & (kQueueCap - 1)]);
      }
      if (lane == 0 && wave_fresh != 0u) atomicAdd(&sm.nlist[(t + 1) % 3], wave_fresh);
      listed = false;
    }
    groups = false;
    if (lane == 0 && wave_changed != 0u) atomicAdd(&sm.count[t], wave_changed);
    if (__builtin_amdgcn_ballot_w64(moved) != 0ull && lane == 0) {
      sm.moves[(t + 1) % 3] = 1u;
      if (CYC) sm.moved[t] = 1u;
    }
    __syncthreads();
    uint32_t* tmp = src;
    src = dst;
    dst = tmp;
    cb ^= 1;
  }
  // (a tile that alternates ends in the other buffer after an odd number of passes)
  if ((a.advance - t) & 1) src = dst;
  // the map's changes: those before the last pass, where the image is taken before it
  if (CYC && t == a.npasses && a.advance < t) cb ^= 1;
  if (tid < a.npasses) sm.changed[tid] += sm.count[tid < t ? tid : max(t - 1, 0)];

  // The strip's map words and owned rows.
  {
    const uint32_t last = has_word ? sm.chg[cb][mine] : 0u;
    // owned columns only: half of the first and of the last word
    const uint32_t ownm = wd == 0 ? 0xFFFF0000u : (wd == 7 ? 0x0000FFFFu : ~0u);
    const int i = strip + ri;
    const uint32_t any = or8((any_bits | last) & ownm) |
                         (has_word ? (sm.row_any[(i + BETA) >> 5] >> ((i + BETA) & 31)) & 1u : 0u);
    if (a.map_out != nullptr) {
      const uint32_t nib = groups4(last & ownm);
      const uint32_t word = or8(wd == 0 ? nib >> 2 : nib << (4 * wd - 2));
      const uint32_t c = add8(uint32_t(__builtin_popcount(last & ownm)));
      const int r = g.row_first + BETA + i;
      if (wd == 0 && has_word && i >= g.own && i < g.own + g.TH && r < a.rows) {
        // (one pass does not tell how the image was two passes before)
        const bool moves = a.advance < 2 || (any != 0u && !periodic);
        const size_t at = size_t(r) * size_t(a.tiles_x) + size_t(g.tx);
        a.map_out[at] = word | (any != 0u ? kMapAny : 0u) | (moves ? kMapMoves : 0u);
        a.cnt_out[at] = uint8_t(c);
      }
    }
    const unsigned long long put = __builtin_amdgcn_ballot_w64(any != 0u);   // bit 8s: row s of the strip
    const bool everything = a.full_store || !has_map;
#pragma unroll 1
    for (int s = 0; s < R; ++s) {
      const int is = strip + s;
      const int r = g.row_first + BETA + is;
      if (is < g.own || is >= g.own + g.TH || r >= a.rows) continue;
      if (!everything && !map.row_stale(is + BETA) && ((put >> (8 * s)) & 1ull) == 0ull) continue;
      store_row(a, g, lane, r, src + (is + BETA) * kRowWords + 1 + kDeepHalo / 4);
    }
  }
  // the next tile's load overwrites what the store reads
  __syncthreads();
}

// ---- one image ---------------------------------------------------------------------

struct DeepArgs {
  DeepTile t;
  unsigned long long* changed;   // count slots, kCountSlots per pass, zeroed beforehand
  int pass0;                     // index of this launch's first pass
  int ntiles;
  int check;                     // 1: a workgroup looks at several tiles at once
  // Period-2 launches: the slots of the passes that moved a pixel (as
  // `changed`; pass 0's say nothing).  The first pass of every launch but the
  // first is the last one of the launch before, which says what its second
  // pass is compared with: it is not counted again.
  unsigned long long* diff2;
  // Or, where fix is not null, the one pass that may be missing after the stop
  // (see CyclePlan): run unless *fix is negative, with source and destination,
  // and the two maps, exchanged where it is odd.
  const int* fix;
  const uint32_t* fix_map1;
};

// Waves per SIMD asked of the register allocator: what LDS lets run.
template <int BETA, int WAVES>
constexpr int deep_min_waves() {
  return WAVES > 8 || BETA > 2 ? 4 : 6;
}

// With `check`, a workgroup has several tiles, most of them idle: each wave
// looks at one (looks(tile, wave) deals with an idle one and returns false),
// and the workgroup runs those that are not.
template <int WAVES, class Looks, class Run>
__device__ __forceinline__ void walk_tiles(int* runs, int ntiles, int check, Looks looks, Run run) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TileRange tr = xcd_range(blockIdx.x, gridDim.x, ntiles);
  const int batch = check ? WAVES : 1;
  for (int first = tr.first; first < tr.end; first += batch * tr.stride) {
    unsigned todo = 1u;
    if (check) {
      const int mine = first + w * tr.stride;
      const bool r = mine < tr.end && looks(mine);
      if (lane == 0) runs[w] = r ? 1 : 0;
      __syncthreads();
      todo = 0u;
#pragma unroll
      for (int u = 0; u < WAVES; ++u) todo |= unsigned(__builtin_amdgcn_readfirstlane(runs[u])) << u;
      __syncthreads();   // runs is rewritten
    }
#pragma unroll 1
    for (; todo != 0u; todo &= todo - 1u) run(first + __builtin_ctz(todo) * tr.stride);
  }
}

template <int BETA, int WAVES, bool CYC = false>
__global__ __launch_bounds__(WAVES * 64, (deep_min_waves<BETA, WAVES>())) void deep_kernel(DeepArgs a) {
  __shared__ DeepSmem<BETA, WAVES> sm;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  if (tid < kDeepMaxPasses) sm.changed[tid] = sm.moved[tid] = 0u;
  if (CYC && a.fix != nullptr) {
    const int f = __builtin_amdgcn_readfirstlane(*a.fix);
    if (f < 0) return;
    const uint8_t* const s = a.t.src;
    uint8_t* const d = a.t.dst;
    a.t.map_in = f & 1 ? a.fix_map1 : a.t.map_in;
    a.t.src = f & 1 ? d : s;
    a.t.dst = f & 1 ? const_cast<uint8_t*>(s) : d;
  }
  // After a pass without a change the image is a fixed point, and so every
  // later pass has no change either: the last pass of the previous launch
  // tells (a launch that does not run leaves its counts at zero).  The load
  // of the vote is in flight with those of the map words.
  // (Period-2 launches: the pass that this launch does again; and a pass that
  // moved nothing ends the run too.)
  const int vp = CYC ? a.pass0 : a.pass0 - 1;
  const int vs = vp * kCountSlots + lane * kCountStride;
  const unsigned long long v = a.pass0 <= 0 ? 1ull : lane < kCountShards ? a.changed[vs] : 0ull;
  const unsigned long long v2 = !CYC || a.pass0 <= 0 ? 1ull : lane < kCountShards ? a.diff2[vs] : 0ull;
  auto converged = [&] {
    return __builtin_amdgcn_ballot_w64(v != 0ull) == 0ull || __builtin_amdgcn_ballot_w64(v2 != 0ull) == 0ull;
  };
  auto looks = [&](int tile) {
    const DeepGeom g = DeepGeom::of<BETA>(a.t, tile);
    DeepMap<kDeepH + 2 * BETA> map;
    const bool runs = map.read(a.t, g, lane);
    if (converged()) return false;
    if (!runs) {
      const unsigned c = idle_tile<BETA>(a.t, g, map, lane, 0, 1);
      if (c != 0u && lane < a.t.npasses) atomicAdd(&sm.changed[lane], c);
    }
    return runs;
  };
  if (a.check)
    __syncthreads();   // the counts are cleared before any wave adds an idle tile's
  else if (converged())
    return;
  walk_tiles<WAVES>(sm.runs, a.ntiles, a.check, looks, [&](int tile) { run_deep_tile<BETA, WAVES, CYC>(sm, a.t, tile); });
  __syncthreads();
  if (CYC && a.fix != nullptr) return;             // (its counts are not wanted)
  const int shard = (blockIdx.x % kCountShards) * kCountStride;
  if (CYC && tid == 0 && a.pass0 > 0) return;      // (counted by the launch before)
  if (CYC && tid < a.t.npasses && sm.moved[tid] != 0u)
    atomicAdd(a.diff2 + (a.pass0 + tid) * kCountSlots + shard, 1ull);
  if (tid < a.t.npasses && sm.changed[tid] != 0u)
    atomicAdd(a.changed + (a.pass0 + tid) * kCountSlots + shard, (unsigned long long)sm.changed[tid]);
}

// ---- many images per launch ------------------------------------------------------------

// The tile parameters of an image of a multi-image launch.
__device__ __forceinline__ DeepTile deep_tile(const ImageDesc& d) {
  DeepTile t;
  t.src = d.src;
  t.dst = d.dst;
  t.rows = d.rows;
  t.cols = d.cols;
  t.alpha = d.alpha;
  t.depth = d.deep & 255;
  t.npasses = t.advance = d.npasses;
  t.th = (d.deep >> 8) & 255;
  t.tiles_x = d.tiles_x;
  t.map_in = reinterpret_cast<const uint32_t*>(d.map_in);
  t.map_out = reinterpret_cast<uint32_t*>(d.map_out);
  // the count bytes follow both maps of words
  const size_t n = size_t(d.rows) * size_t(d.tiles_x), odd = size_t(d.seq & 1);
  uint8_t* bytes = d.map_out + (2 - odd) * sizeof(uint32_t) * n;
  t.cnt_in = bytes + (1 - odd) * n;
  t.cnt_out = bytes + odd * n;
  t.full_store = (d.deep >> 16) & 1;
  return t;
}

// As deep_kernel, over a table of tiles of many images, each with its own
// parameters, pass index, pass count and convergence (see multi_pass_kernel).
template <int BETA, int WAVES>
__global__ __launch_bounds__(WAVES * 64, (deep_min_waves<BETA, WAVES>())) void multi_deep_kernel(MultiArgs a) {
  __shared__ DeepSmem<BETA, WAVES> sm;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int shard = (blockIdx.x % kCountShards) * kCountStride;
  // Whether the image runs in this launch; the workgroup of its tile 0 says
  // whether it had converged before.
  auto live = [&](const ImageDesc& d, int tile, bool first) {
    const bool zero = d.prev_passes > 0 && pass_zero_wave(d.counts, d.pass0 - 1, lane) != 0;
    if (tile == 0 && first && d.status != nullptr) *d.status = zero ? 1 : 0;
    return !zero;
  };
  auto looks = [&](int t) {
    const TileRef ref = a.tiles[t];
    const ImageDesc d = a.images[ref.image];
    if (d.npasses <= 0 || !live(d, ref.tile, lane == 0)) return false;
    const DeepTile dt = deep_tile(d);
    const DeepGeom g = DeepGeom::of<BETA>(dt, ref.tile);
    DeepMap<kDeepH + 2 * BETA> map;
    if (map.read(dt, g, lane)) return true;
    const unsigned c = idle_tile<BETA>(dt, g, map, lane, 0, 1);
    if (c != 0u && lane < d.npasses)
      atomicAdd(d.counts + (d.pass0 + lane) * kCountSlots + shard, (unsigned long long)c);
    return false;
  };
  auto run = [&](int t) {
    const TileRef ref = a.tiles[t];
    const ImageDesc d = a.images[ref.image];
    if (!a.check && (d.npasses <= 0 || !live(d, ref.tile, tid == 0))) return;
    if (tid < kDeepMaxPasses) sm.changed[tid] = 0u;
    run_deep_tile<BETA, WAVES>(sm, deep_tile(d), ref.tile);
    if (tid < d.npasses && sm.changed[tid] != 0u)
      atomicAdd(d.counts + (d.pass0 + tid) * kCountSlots + shard, (unsigned long long)sm.changed[tid]);
  };
  walk_tiles<WAVES>(sm.runs, a.ntiles, a.check, looks, run);
}

}  // namespace phg
