// Packed-byte arithmetic for the 8-bit frame actors of the motion-detection
// pipeline (Sec. 4.1): four pixels per 32-bit word, split into two words of
// 16-bit lanes (even pixels 0 and 2, odd pixels 1 and 3) so that sums and
// comparisons of up to 16 bits never carry into the neighbouring pixel.
// Host-compilable so the same code can be checked on the CPU.
#pragma once

#include <stdint.h>

#ifndef __HIPCC__
#define __host__
#define __device__
#endif

namespace dfh {
namespace swar {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kLo = 0x00FF00FFu;

// Low 32 bits of the 64-bit value hi:lo shifted right by s (0 <= s < 32).
__host__ __device__ inline uint32_t funnel(uint32_t hi, uint32_t lo, int s) {
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> s);
}

// Byte permute: byte i of the result is byte sel[i] (0..7) of the 8-byte
// pool lo (bytes 0..3) : hi (bytes 4..7); a selector byte of 0x0C gives 0.
__host__ __device__ inline uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_perm(hi, lo, sel);
#else
  const uint64_t pool = ((uint64_t)hi << 32) | lo;
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = (sel >> (8 * i)) & 0xFF;
    const uint32_t v = s < 8 ? (uint32_t)((pool >> (8 * s)) & 0xFF) : s == 0x0C ? 0u : 0xFFu;
    r |= v << (8 * i);
  }
  return r;
#endif
}

// Selectors for perm() building horizontal windows of the 4 pixels p0..p3
// of word m from its neighbour words l and r.  With `edge` set the pixels
// beyond the frame edge repeat the edge pixel (p-1 = p-2 = p0 on the left,
// p4 = p5 = p3 on the right).
//   perm(m, l, win2_left(e))  = (p-2, p-1, p0, p1)
//   perm(r, m, win2_right(e)) = (p2, p3, p4, p5)
//   perm(m, l, win1_left(e))  = (p-1, p0, p1, p2)
//   perm(r, m, win1_right(e)) = (p1, p2, p3, p4)
__host__ __device__ inline uint32_t win2_left(bool edge) { return edge ? 0x05040404u : 0x05040302u; }
__host__ __device__ inline uint32_t win2_right(bool edge) { return edge ? 0x03030302u : 0x05040302u; }
__host__ __device__ inline uint32_t win1_left(bool edge) { return edge ? 0x06050404u : 0x06050403u; }
__host__ __device__ inline uint32_t win1_right(bool edge) { return edge ? 0x03030201u : 0x04030201u; }

// The right selectors with `avail` in-frame pixels to the right of p3.  With
// 1..3 of them r is the row's last word, in which p4 is byte 4 - avail.
__host__ __device__ inline uint32_t win2_right_avail(int avail) {
  if (avail <= 0 || avail >= 4) return win2_right(avail <= 0);
  const uint32_t p4 = 8u - (uint32_t)avail, p5 = avail > 1 ? p4 + 1 : p4;
  return 0x0302u | (p4 << 16) | (p5 << 24);
}
__host__ __device__ inline uint32_t win1_right_avail(int avail) {
  if (avail <= 0 || avail >= 4) return win1_right(avail <= 0);
  return 0x00030201u | ((8u - (uint32_t)avail) << 24);
}

// Horizontal 5-tap binomial sums (1,4,6,4,1) of four pixels p0..p3 given
// the 8-byte window X = (p-2, p-1, p0, p1, p2, p3, p4, p5) as lo (bytes
// 0..3) and hi (bytes 4..7).  Returns the sums of (p0, p2) in *even and of
// (p1, p3) in *odd, one per 16-bit lane (each at most 255*16 = 4080).
__host__ __device__ inline void hsum5(uint32_t lo, uint32_t hi, uint32_t *even, uint32_t *odd) {
  // u[k]: bytes k and k+2 of X in the two 16-bit lanes, one byte permute
  // each (selector 0x0C writes a zero byte)
  const uint32_t u0 = lo & kLo;
  const uint32_t u1 = perm(hi, lo, 0x0C030C01u);
  const uint32_t u2 = perm(hi, lo, 0x0C040C02u);
  const uint32_t u3 = perm(hi, lo, 0x0C050C03u);
  const uint32_t u4 = hi & kLo;
  const uint32_t u5 = perm(hi, lo, 0x0C070C05u);
  *even = u0 + u4 + 4u * (u1 + u3) + 6u * u2;
  *odd = u1 + u5 + 4u * (u2 + u4) + 6u * u3;
}

// Vertical 5-tap binomial sum of horizontal sums, rounded (s + 128) >> 8,
// back to one byte per 16-bit lane.  Lanes stay below 65536: 4080*16 + 128.
__host__ __device__ inline uint32_t vround5(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e) {
  // 6c as 4c + 2c: c exceeds 24 bits, and a full 32-bit multiply is slow
  const uint32_t s = a + e + ((b + d + c) << 2) + (c << 1) + 0x00800080u;
  return (s >> 8) & kLo;
}

// The same filter with the vertical pass first: per 16-bit lane the
// unrounded 5-tap sum of five pixels (at most 255 * 16 = 4080) ...
__host__ __device__ inline uint32_t vsum5(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e) {
  return (a + e) + ((b + d + c) << 2) + (c << 1);
}

// ... and the horizontal pass over vertical sums v0..v3 of a word's pixels,
// E = (v0, v2) and O = (v1, v3), with l = (v-2, v-1) and r = (v4, v5) of the
// neighbours: rounded (s + 128) >> 8, the bytes of pixels 0, 2 in *even and
// of 1, 3 in *odd.  Lanes stay below 65536 as in vround5.
__host__ __device__ inline void hround5(uint32_t E, uint32_t O, uint32_t l, uint32_t r, uint32_t *even, uint32_t *odd) {
  const uint32_t A = perm(E, l, 0x05040100u);   // (v-2, v0)
  const uint32_t B = perm(O, l, 0x05040302u);   // (v-1, v1)
  const uint32_t F = perm(r, E, 0x05040302u);   // (v2, v4)
  const uint32_t G = perm(r, O, 0x07060302u);   // (v3, v5)
  const uint32_t se = (A + F + 0x00800080u) + ((B + O + E) << 2) + (E << 1);
  const uint32_t so = (B + G + 0x00800080u) + ((E + F + O) << 2) + (O << 1);
  *even = perm(se, se, 0x0C030C01u);
  *odd = perm(so, so, 0x0C030C01u);
}

// A word's own pairs as its neighbours take them: (v2, v3) for the word on
// the right, (v0, v1) for the one on the left; and the selectors that keep
// such a pair p, or at a frame edge repeat the edge pixel's sum instead:
//   perm(E, p, pair_left(edge))  = l above, (v0, v0) at the left edge
//   perm(O, p, pair_right(edge)) = r above, (v3, v3) at the right edge
__host__ __device__ inline uint32_t pair_hi(uint32_t E, uint32_t O) { return perm(O, E, 0x07060302u); }
__host__ __device__ inline uint32_t pair_lo(uint32_t E, uint32_t O) { return perm(O, E, 0x05040100u); }
__host__ __device__ inline uint32_t pair_left(bool edge) { return edge ? 0x05040504u : 0x03020100u; }
__host__ __device__ inline uint32_t pair_right(bool edge) { return edge ? 0x07060706u : 0x03020100u; }

// Re-interleave even-pixel and odd-pixel lanes into one word of 4 pixels.
__host__ __device__ inline uint32_t interleave(uint32_t even, uint32_t odd) { return even | (odd << 8); }

// 0xFF in every byte lane where |a - b| > t, else 0 (t in 0..255).
__host__ __device__ inline uint32_t absdiff_gt(uint32_t a, uint32_t b, uint32_t t) {
  const uint32_t bias = (255u - t) * 0x00010001u;
  uint32_t m[2];
  for (int k = 0; k < 2; ++k) {
    const uint32_t x = (a >> (8 * k)) & kLo, y = (b >> (8 * k)) & kLo;
    // each lane: 256 + x - y (1..511), and 256 + y - x; + (255 - t) reaches
    // 512 (bit 9) exactly when the difference exceeds t
    const uint32_t p = ((x | 0x01000100u) - y + bias) >> 9;
    const uint32_t q = ((y | 0x01000100u) - x + bias) >> 9;
    m[k] = ((p | q) & 0x00010001u) * 0xFFu;
  }
  return interleave(m[0], m[1]);
}

__host__ __device__ inline u16x2 as_u16x2(uint32_t v) {
  u16x2 r;
  r.x = (unsigned short)(v & 0xFFFFu);
  r.y = (unsigned short)(v >> 16);
  return r;
}
__host__ __device__ inline uint32_t from_u16x2(u16x2 v) { return (uint32_t)v.x | ((uint32_t)v.y << 16); }

__host__ __device__ inline u16x2 vmin(u16x2 a, u16x2 b) { return __builtin_elementwise_min(a, b); }
__host__ __device__ inline u16x2 vmax(u16x2 a, u16x2 b) { return __builtin_elementwise_max(a, b); }

// Median of five values per 16-bit lane: the median of e and the two middle
// candidates max(min(a,b), min(c,d)) and min(max(a,b), max(c,d)).
__host__ __device__ inline u16x2 med5(u16x2 a, u16x2 b, u16x2 c, u16x2 d, u16x2 e) {
  const u16x2 f = vmax(vmin(a, b), vmin(c, d));
  const u16x2 g = vmin(vmax(a, b), vmax(c, d));
  return vmax(vmin(e, f), vmin(vmax(e, f), g));
}

// Threshold of pixels given in split form (even pixels 0, 2 in the 16-bit
// lanes of *E, odd pixels 1, 3 in *O, values 0..255): 0x01 in every byte
// where |cur - prev| > t (t in 0..255), else 0.  |d| + (255 - t) stays below
// 512, so bit 8 of each lane is the comparison.
__host__ __device__ inline uint32_t thres_split(uint32_t cE, uint32_t cO, uint32_t pE, uint32_t pO, uint32_t t) {
  const uint32_t bias = (255u - t) * 0x00010001u;
  const u16x2 ce = as_u16x2(cE), co = as_u16x2(cO), pe = as_u16x2(pE), po = as_u16x2(pO);
  const uint32_t dE = from_u16x2(vmax(ce, pe) - vmin(ce, pe)) + bias;
  const uint32_t dO = from_u16x2(vmax(co, po) - vmin(co, po)) + bias;
  return ((dE >> 8) & 0x00010001u) | (dO & 0x01000100u);
}

// Median of five words of 0x00/0x01 bytes, as 0x00/0xFF: with only two values
// the median is the majority, and a byte's sum of five (at most 5) plus 5
// reaches 8 exactly from three on.
__host__ __device__ inline uint32_t med5_ones(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e) {
  const uint32_t s = (a + b + c) + d + e;
  const uint32_t y = ((s + 0x05050505u) >> 3) & 0x01010101u;
  return (y << 8) - y;                      // x 255, modulo 2^32
}

// Median of five words of four pixels each, per pixel.
__host__ __device__ inline uint32_t med5_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e) {
  uint32_t r[2];
  for (int k = 0; k < 2; ++k) {
    const int s = 8 * k;
    const u16x2 m = med5(as_u16x2((a >> s) & kLo), as_u16x2((b >> s) & kLo), as_u16x2((c >> s) & kLo),
                         as_u16x2((d >> s) & kLo), as_u16x2((e >> s) & kLo));
    r[k] = from_u16x2(m);
  }
  return interleave(r[0], r[1]);
}

}  // namespace swar
}  // namespace dfh
