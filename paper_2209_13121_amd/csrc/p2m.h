// p2m.h -- the sums of P2M over one box, by a group of lanes.
//
// What bounds it: FP64 issue (about 4 operations per coefficient and particle)
// once the chip is full; with one lane per box, as it was, the serial chain of
// the box's particles, a chip that a few thousand boxes leave nearly idle, and
// loads and stores a row apart between lanes.  A group of lanes per box shares
// the particles and then the coefficients: its loads are consecutive and its
// stores one run.  The sum over the group costs about as much as two particles
// (some 10 instructions per coefficient, half of them through the LDS unit),
// so a group should have about 4 particles per lane, unless the chip is not
// full otherwise.  Alone, one lane per box -> now, us: 2^20 particles, depth 4
// (4096 boxes), p = 8: 279 -> 26; depth 5: 55 -> 27; 262 144, depth 4, p = 8:
// 83 -> 14; depth 5: 28 -> 21; 100 003, depth 4, p = 6: 30 -> 10; 4096, depth 3,
// p = 4: 12 -> 6; adaptive, p = 10: 300 000 in clusters, FP64: 114 -> 39; 3 10^6
// mixed: 324 -> 302 (11 particles a box).
#pragma once
#include <type_traits>

#include "fmm_internal.h"

namespace fmm {

// Sum over the lanes of an aligned group of lanes (a power of two of them,
// 2 W being the distance still to halve) of N values per lane, N a multiple of
// the group, by halving: at each step the lanes exchange half of what they
// still hold with the partner lane W apart, the lanes with bit W set keeping
// the upper half.  Afterwards lane L of a group of G holds in v[0 .. N/G) the
// sums of the values N/G L .. N/G L + N/G - 1.  About N shuffles instead of
// N log2 G, in a fixed order.
template <int H, int W, typename T>
__device__ __forceinline__ void halve_exchange(T* v) {
  const bool up = (threadIdx.x & W) != 0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const T send = up ? v[i] : v[i + H];
    const T keep = up ? v[i + H] : v[i];
    v[i] = keep + __shfl_xor(send, W);
  }
}
template <int N, int G, typename T>
__device__ __forceinline__ void group_sum_split(T* v) {
  static_assert(G >= 1 && G <= 64 && (G & (G - 1)) == 0 && N % G == 0, "group of lanes");
  if constexpr (G > 1) {
    halve_exchange<N / 2, G / 2>(v);
    group_sum_split<N / 2, G / 2>(v);
  }
}

// The multipole of the particles src[b .. e) about their box centre, by the
// group of G lanes to which the thread belongs (g: its index in the group),
// which takes the particles G apart; written as a row of mstride_of(NC) values,
// the pad zero, at row of mult64 and / or mult32.
template <int P, int G>
__device__ __forceinline__ void p2m_box(const Rec<double>* __restrict__ src, uint32_t b, uint32_t e, int g,
                                        int64_t row, double* __restrict__ mult64,
                                        float* __restrict__ mult32) {
  constexpr int NC = (P + 1) * (P + 1);
  constexpr int MS = mstride_of(NC);
  constexpr int NT = (P + 1) * (P + 2) / 2;
  constexpr int R = (MS + G - 1) / G;  // values per lane after the sum
  double acc[R * G];
#pragma unroll
  for (int c = 0; c < R * G; ++c) acc[c] = 0.0;
  for (uint32_t s = b + g; s < e; s += G) {
    double re[NT], im[NT];
    const Rec<double> r = src[s];
    regular_harmonics<P, double>(r.x, r.y, r.z, re, im);
    const double qq = r.q;
#pragma unroll
    for (int nn = 0; nn <= P; ++nn) {
      acc[cidx_re(nn, 0)] += qq * re[tri(nn, 0)];
#pragma unroll
      for (int m = 1; m <= nn; ++m) {
        acc[cidx_re(nn, m)] += qq * re[tri(nn, m)];
        acc[cidx_im(nn, m)] -= qq * im[tri(nn, m)];
      }
    }
  }
  group_sum_split<R * G, G>(acc);
  // (tests of the arguments alone, so that the stores stay whole vectors)
  if (mult64) {
    double* o = mult64 + row * MS + R * g;
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (R * G == MS || R * g + i < MS) o[i] = acc[i];
  }
  if (mult32) {
    float* o = mult32 + row * MS + R * g;
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (R * G == MS || R * g + i < MS) o[i] = (float)acc[i];
  }
}

// Lanes per box for n particles in nbox boxes: one for the smallest (2^20
// particles, depth 6, 4 per leaf, p = 8: 1 / 2 / 4 lanes 49 / 52 / 62 us), then a
// third to a quarter of the mean box up to 16 (6 per leaf, 32 768 leaves, p = 12:
// 61 / 41 / 45; adaptive, 8.3 per box, p = 8: 70 / 60 / 66; 13 per box, p = 10:
// 1 / 2 / 4 / 16 lanes 114 / 60 / 39 / 54; 32 per leaf: 2 / 4 / 8 / 16 lanes 41 / 27 /
// 27 / 37; 256 per leaf: 16 / 32 / 64 lanes 26 / 30 / 40), and more where that leaves
// SIMDs without a wave (4096 leaves of 24: 4 / 16 lanes 12.8 / 9.6; adaptive, 6208
// boxes of 23: 22 / 14; 512 leaves of 2048: 16 / 64 lanes 120 / 38; but 10 952 boxes
// of 7: 4 / 16 lanes 10.5 / 13.4; where most boxes hold about one particle more lanes
// lose a little, 4096 leaves of 0.7, p = 8: 1 / 16 lanes 8.5 / 9.4, and where few of
// them hold all they win by far, so the rule stays with the mean).
inline int p2m_lanes(int64_t n, int64_t nbox) {
  constexpr int64_t kFullLanes = 40000;
  const int steps[5] = {1, 2, 4, 16, 64};
  int k = n >= 64 * nbox ? 3 : (n >= 10 * nbox ? 2 : (n >= 6 * nbox ? 1 : 0));
  while (k < 4 && nbox * steps[k] < kFullLanes) ++k;
  return steps[k];
}

// Calls f(std::integral_constant<int, G>) for g = 1, 2, 4, 16 or 64 lanes per box.
template <typename F>
inline void with_p2m_lanes(int g, F&& f) {
  if (g == 1) f(std::integral_constant<int, 1>{});
  else if (g == 2) f(std::integral_constant<int, 2>{});
  else if (g == 4) f(std::integral_constant<int, 4>{});
  else if (g == 16) f(std::integral_constant<int, 16>{});
  else f(std::integral_constant<int, 64>{});
}

}  // namespace fmm
