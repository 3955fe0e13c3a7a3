// m2l_sym.h -- tables of the reflection-reduced M2L (m2l_sym_kernel.h): the parity
// classes of the packed real coefficients, the order of rows and columns they
// give, and the offsets grouped into orbits.
//
// Reflecting an axis maps every packed real solid harmonic to itself or its
// negative (parities kappa below), so with S_e the diagonal +-1 matrix of the
// reflections e the unit-box operators satisfy T_{e d} = S_e T_d S_e.  The
// offsets of a class that differ only in the signs of reflected axes (an
// orbit, up to 8 of them) therefore share one operator, and the sum over the
// orbit splits by the parity class sigma of the output row:
//   sum_e T_{e d} M_e  restricted to rows of class sigma
//     = T_d[sigma, :] X_sigma,  X_sigma[k] = sum_e (-1)^{(sigma ^ kappa(k)) . e} M_e[k].
// One product of T_d's rows then serves the whole orbit: per axis the six
// offsets of a class become the four magnitudes 0 (rows and columns of unlike
// parity are zero: half a product), 1 and 2 (pairs) and 3 (single), so 189
// products become 39.5.
#pragma once

#include "fmm_internal.h"
#include "m2l_form.h"

namespace fmm {
namespace sym {

// Parity of packed coefficient c = (n, m, re / im) under reflection of z (bit
// 0), y (bit 1) and x (bit 2): cos(m f) P_n^m and sin(m f) P_n^m get (-1)^{n+m}
// under z, sin changes sign under y, and x -> -x (f -> pi - f) gives (-1)^m
// for cos, (-1)^{m+1} for sin.
__host__ __device__ constexpr int parity_of(int c) {
  const int n = isqrt_c(c), r = c - n * n, m = (r + 1) / 2;
  const int im = r != 0 && r % 2 == 0 ? 1 : 0;
  return ((n + m) & 1) | im << 1 | ((m + im) & 1) << 2;
}

constexpr int kNumOps = 56;  // orbits of the 316 offsets = items of a target's loop

constexpr int kMaxKs = (((FMM_P_MAX + 1) * (FMM_P_MAX + 1)) + 3) / 4;  // k steps of 4 at p = FMM_P_MAX
constexpr int kMaxBlk = 15;                                            // 16-row blocks at p = FMM_P_MAX

// Row and column order of one p: coefficients sorted by class (columns in
// Gray-code order of the classes, so that a k step of 4 that spans two classes
// mixes one axis only; each class's rows padded to 16-row blocks).
struct Tab {
  int16_t kcoef[4 * kMaxKs];    // coefficient of column rank r (k step r / 4, lane group r % 4), -1 pad
  int16_t rcoef[16 * kMaxBlk];  // coefficient of row 16 b + i, -1 pad
  uint64_t kbits[3][4];         // per axis and lane group: bit ks = parity of column 4 ks + group
  uint64_t has[3][2];           // per axis and parity: bit ks = k step ks holds such a column
  int nb;                       // row blocks
  int8_t bcls[kMaxBlk];         // class of each row block
};

constexpr Tab make_tab(int p) {
  Tab t{};
  const int nc = (p + 1) * (p + 1), ncls = 8;
  for (int i = 0; i < 4 * kMaxKs; ++i) t.kcoef[i] = -1;
  for (int i = 0; i < 16 * kMaxBlk; ++i) t.rcoef[i] = -1;
  int r = 0;
  for (int g = 0; g < ncls; ++g) {
    const int cls = g ^ (g >> 1);
    for (int c = 0; c < nc; ++c)
      if (parity_of(c) == cls) t.kcoef[r++] = (int16_t)c;
  }
  for (int i = 0; i < nc; ++i) {
    const int par = parity_of(t.kcoef[i]);
    for (int a = 0; a < 3; ++a) {
      const int b = (par >> a) & 1;
      if (b) t.kbits[a][i % 4] |= (uint64_t)1 << (i / 4);
      t.has[a][b] |= (uint64_t)1 << (i / 4);
    }
  }
  for (int cls = 0; cls < ncls; ++cls) {
    int n = 0;
    for (int c = 0; c < nc; ++c)
      if (parity_of(c) == cls) {
        if (n % 16 == 0) t.bcls[t.nb++] = (int8_t)cls;
        t.rcoef[16 * (t.nb - 1) + n % 16] = (int16_t)c;
        ++n;
      }
  }
  return t;
}

// Shape for order P and type T.
template <int P, typename T>
struct Shape {
  static constexpr Tab TAB = make_tab(P);
  static constexpr int NC = (P + 1) * (P + 1);
  static constexpr int NCLS = 8;              // parity classes = largest orbit
  static constexpr int NB = TAB.nb;           // 16-row blocks
  static constexpr int KS = (NC + 3) / 4;     // k steps of 4
  static constexpr int V = 16 / (int)sizeof(T);  // k steps per chunk: one 16-byte vector per lane
  static constexpr int NCH = (KS + V - 1) / V;   // chunks
  static constexpr int NT = KS - V * (NCH - 1);  // k steps of the last chunk
  static constexpr int STR = 4 * KS;             // elements of a source row (= mstride_of(NC))
  static constexpr int CHUNK = NB * 64 * V;      // operator elements per chunk
  static constexpr int OP = NCH * CHUNK;         // operator elements
  static constexpr int NI = kNumOps;
  static_assert(STR == mstride_of(NC), "the permuted rows take the space of a multipole row");
};
// Elements of one operator (run-time p, element size).
inline size_t op_elems(int p, int elem) {
  const int v = 16 / elem, ks = (ncoef(p) + 3) / 4;
  return (size_t)((ks + v - 1) / v) * make_tab(p).nb * 64 * v;
}

// Position in a source row of column rank r = 4 ks + g: chunk, lane group,
// k step within the chunk (the last chunk holds nt k steps).
__host__ __device__ constexpr int row_slot(int r, int ks_total, int v) {
  const int ks = r / 4, g = r % 4, ch = ks / v, s = ks % v, nch = (ks_total + v - 1) / v;
  const int w = ch == nch - 1 ? ks_total - v * (nch - 1) : v;
  return 4 * v * ch + w * g + s;
}

// Operators: the offsets 0 <= d_a <= 3, max d_a >= 2, in runs of the same zero
// axes (those with fewer of them, more products, first).  Every class walks its
// items in operator order.
__host__ __device__ constexpr bool near_offset(int x, int y, int z) {
  return x >= -1 && x <= 1 && y >= -1 && y <= 1 && z >= -1 && z <= 1;
}
// Axis types of an orbit: |d_a| = 0, a pair (+-1 or +-2: both offsets exist in
// the class's range [pi - 3, pi + 2]), or single (magnitude 3: d_a = 3 for
// pi_a = 1, -3 for pi_a = 0).
enum : int { kZero = 0, kPair = 1, kSingle = 2 };
struct Orbits {
  int8_t d[56][3];
  int ngroups;   // runs of operators with the same zero axes: 7
  int start[8];  // first operator of each run
  int zeros[7];  // zero axes of the run, bit 0 z .. bit 2 x
};
constexpr Orbits make_orbits() {
  Orbits o{};
  int n = 0;
  constexpr int order[7] = {0, 1, 2, 4, 3, 5, 6};
  for (int g = 0; g < 7; ++g) {
    o.zeros[g] = order[g];
    o.start[g] = n;
    for (int x = 0; x <= 3; ++x)
      for (int y = 0; y <= 3; ++y)
        for (int z = 0; z <= 3; ++z) {
          if (near_offset(x, y, z) || ((x == 0) << 2 | (y == 0) << 1 | (z == 0)) != order[g]) continue;
          o.d[n][0] = (int8_t)x;
          o.d[n][1] = (int8_t)y;
          o.d[n][2] = (int8_t)z;
          ++n;
        }
  }
  o.ngroups = 7;
  o.start[7] = n;
  return o;
}

// Whether an item of this type has a source with the axis kept / negated
__host__ __device__ constexpr bool source_on_axis(int type, int pa, bool neg) {
  return type == kPair || neg == (type == kSingle && !pa);
}
// Items of class pi: op | (d_a + 4) << 9, 13, 17 (x, y, z) | type << 21, 23,
// 25 (z, y, x), d_a >= 0; source e has d_a negated on the axes of its bits (bit
// 2: x).
struct Items {
  uint32_t v[8][kNumOps];
};
constexpr Items make_items() {
  Items t{};
  const Orbits orb = make_orbits();
  for (int pi = 0; pi < 8; ++pi)
    for (int i = 0; i < kNumOps; ++i) {
      uint32_t code = (uint32_t)i;
      for (int a = 0; a < 3; ++a) {
        const int m = orb.d[i][a], type = m == 0 ? kZero : (m == 3 ? kSingle : kPair);
        code |= (uint32_t)(m + 4) << (9 + 4 * a) | (uint32_t)type << (25 - 2 * a);
      }
      t.v[pi][i] = code;
    }
  return t;
}
// every class's items hold its 189 interaction-list offsets once each
constexpr bool items_ok(const Items& t) {
  for (int pi = 0; pi < 8; ++pi) {
    bool seen[216] = {};
    int n = 0;
    for (int i = 0; i < kNumOps; ++i) {
      const uint32_t c = t.v[pi][i];
      for (int e = 0; e < 8; ++e) {
        int cell = 0;
        bool have = true;
        for (int a = 0; a < 3; ++a) {
          const bool neg = (e >> (2 - a)) & 1;
          int d = (int)((c >> (9 + 4 * a)) & 15u) - 4;
          have = have && source_on_axis((int)((c >> (25 - 2 * a)) & 3u), (pi >> (2 - a)) & 1, neg);
          if (neg) d = -d;
          const int u = d - (((pi >> (2 - a)) & 1) - 3);
          if (have && (u < 0 || u > 5)) return false;
          cell = cell * 6 + u;
        }
        if (!have) continue;
        if (seen[cell]) return false;
        seen[cell] = true;
        ++n;
      }
    }
    if (n != kIL) return false;
  }
  return true;
}
static_assert(items_ok(make_items()), "orbits cover the interaction lists");
// Offset of operator op
__host__ __device__ inline void op_offset(int op, int d[3]) {
  constexpr Orbits orb = make_orbits();
  for (int i = 0; i < kNumOps; ++i)
    if (i == op)
      for (int a = 0; a < 3; ++a) d[a] = orb.d[i][a];
}

}  // namespace sym

hipError_t launch_m2l_sym_f64(fmm_plan_s* P, hipStream_t s);  // m2l_sym_f64.hip
hipError_t launch_m2l_sym_f32(fmm_plan_s* P, hipStream_t s);  // m2l_sym_f32.hip
}  // namespace fmm
