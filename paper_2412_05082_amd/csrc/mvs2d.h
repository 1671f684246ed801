// Numbering of the patches of one colour of the 2D multiplicative smoother.
// Colour c = px + 2 py + 4 rb holds the vertices v = (2a + px, 2b + py) in
// [1, N-1]^2 with (a + b) mod 2 = rb; they are numbered row by row of b, and
// rows alternate between two lengths.
#pragma once

#include <hip/hip_runtime.h>

namespace c0ip {
namespace {

struct ColourRows {
  int a_lo, a_hi, b_lo, nb;  // lattice ranges of a and b
  int rb;
  int cnt0, cnt1;            // patches in rows b_lo + 2i and b_lo + 2i + 1
  int total;
};

__host__ __device__ inline int colour_row_count(int a_lo, int a_hi, int b, int rb) {
  const int af = a_lo + (((rb - a_lo - b) % 2) + 2) % 2;
  return af <= a_hi ? (a_hi - af) / 2 + 1 : 0;
}

inline ColourRows colour_rows(int N, int c) {
  const int px = c & 1, py = (c >> 1) & 1;
  ColourRows cr;
  cr.rb = (c >> 2) & 1;
  cr.a_lo = px == 0 ? 1 : 0;
  cr.a_hi = (N - 1 - px) / 2;
  cr.b_lo = py == 0 ? 1 : 0;
  const int b_hi = (N - 1 - py) / 2;
  cr.nb = b_hi >= cr.b_lo ? b_hi - cr.b_lo + 1 : 0;
  cr.cnt0 = colour_row_count(cr.a_lo, cr.a_hi, cr.b_lo, cr.rb);
  cr.cnt1 = colour_row_count(cr.a_lo, cr.a_hi, cr.b_lo + 1, cr.rb);
  cr.total = (cr.nb / 2) * (cr.cnt0 + cr.cnt1) + (cr.nb % 2) * cr.cnt0;
  return cr;
}

// vertex (vx, vy) of the patch with number q of the colour
__device__ __forceinline__ void colour_vertex(const ColourRows& cr, int px, int py, int q, int& vx, int& vy) {
  const int pair = cr.cnt0 + cr.cnt1;
  const int i = q / pair, rem = q - i * pair;
  const int b = cr.b_lo + 2 * i + (rem >= cr.cnt0 ? 1 : 0);
  const int t = rem >= cr.cnt0 ? rem - cr.cnt0 : rem;
  const int af = cr.a_lo + (((cr.rb - cr.a_lo - b) % 2) + 2) % 2;
  vx = 2 * (af + 2 * t) + px;
  vy = 2 * b + py;
}

}  // namespace
}  // namespace c0ip
