// m2l_form.h -- which kernel the FP64 / FP32 M2L takes: the plain one (m2l.hip,
// a product per offset) or the reflection-reduced one (m2l_sym.h, a product per
// orbit of offsets).  Arithmetic on counts only, no HIP.
#pragma once
#include <stdint.h>

namespace fmm {
namespace sym {

// The orders the plain kernel is built for; up to kPlainOnlyP it always serves.
constexpr int kPlainOnlyP = 3;
constexpr int kPlainMaxP = 7;

// Fewest work-groups of the wide reflection forms (16 parents, all classes
// each): with fewer the small form is used, its 8 x more work-groups then fill
// the chip better.
constexpr int64_t kWideGroups = 200;

// groups16, groups128: the (class, level, tile) work-groups with tiles of 16 and
// of 128 parents (m2l_common.h make_args).
//
// The reflections make 39.5 products of 189, but of rows padded to 16 per class:
// 8 row blocks at every p from 4 to 9, where the plain form has ceil(ncoef / 16)
// (p = 6: a last row on the vector unit) = 1 .. 7, and they skip an orbit only
// if none of its up to 8 sources exists.  The plain form has one work-group per
// tile of 128, so that a tree of few tiles leaves CUs idle: the time of both is
// the number of rounds of the 256 CUs times that of one.  Measured, us a round,
// FP64 / FP32 (adaptive):
//                      p = 4      p = 5      p = 6      p = 7
//   plain             210 / 143  411 / 272  590 / 323  810 / 440
//   small reflections  70 /  47   84 /  59  115 /  74  109 /  69
//   wide reflections  486 / 291  591 / 392  800 / 497  781 / 461
// so a wide round counts as 7 small ones and a plain round as 3 to 6.  M2L of
// adaptive trees, us, plain / reflections: a sphere of 120 000, p 4, 5, 6, FP64
// 210 / 425, 413 / 511, 578 / 681; 250 000 uniform charges, 24 a leaf: 380 / 939,
// 847 / 1150, 1216 / 1567; 256 systems of 1e3 .. 65 536, 64 a leaf, p 6: FP64
// 5392 / 7329, FP32 2920 / 4627; p 7 FP32: 64 systems 1329 / 1367, a sphere of
// 500 000 1609 / 1813; p 7 FP64: 2456 / 2271 and 3031 / 3071.  p = 8, FP64,
// nine trees: reflections 0.95 to 1.04 of plain, FP32 0.88 to 1.00; from p = 9
// 0.58 to 0.73.
// Uniform tree: the block form needs 0.62 of the plain time from p = 5, at p = 4
// 0.98 to 1.02 in FP32 but in FP64 1.06 (depth 5) to 1.10 (depth 7).
constexpr bool serves(int p, bool fp64, bool adaptive, int64_t groups16, int64_t groups128) {
  if (p <= kPlainOnlyP) return false;
  if (p > kPlainMaxP || (p == kPlainMaxP && fp64)) return true;
  const bool wide = groups16 >= 8 * kWideGroups;
  if (!adaptive) return !(p == 4 && fp64 && wide);
  const int64_t plain_rounds = (groups128 + 255) / 256;
  const int64_t small_rounds = wide ? 7 * ((groups16 / 8 + 255) / 256) : (groups16 + 255) / 256;
  // small rounds that one plain round is worth
  const int worth = p == 4 ? 3 : (p == 5 ? 4 : (p == 6 ? (fp64 ? 5 : 4) : 6));
  return small_rounds <= worth * plain_rounds;
}

}  // namespace sym
}  // namespace fmm
