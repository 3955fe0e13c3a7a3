// upward.hip -- charges into Hilbert order, P2M at the leaves, M2M up to
// level 2.
//
// P2M (p2m.h): M~_n^m = sum_j q_j conj(R_n^m(u_j)) with u_j the box-unit offset of
// particle j from its leaf centre (computed by the tree pass), accumulated in
// FP64 in both precision modes from the FP64 offsets.  (An FP32 sum of
// neutral clusters of charges, one cluster after another, rounds every
// cluster's partial sums the same way, so the leaf monopoles would drift by an
// amount proportional to the particle count: a smooth, density-shaped error
// charge.  FP64 adds cost the same issue slots as FP32 ones here.)  The mixed
// mode stores the sum rounded to FP32 only, read by the M2L pass and,
// converted back, by the M2M pass: one rounding of the final value, with no
// drift.
// M2M (shift.hip): M~p = sum over the 8 children of A[octant] M~c with the
// level-free octant matrices, always in FP64; in the mixed mode each parent is
// also stored rounded to FP32 for the M2L pass.
#include "p2m.h"

namespace fmm {
namespace {

template <typename T>
__global__ void k_gather_q(const double* __restrict__ q, const int32_t* __restrict__ perm, int64_t n,
                           double* __restrict__ q64, Rec<T>* __restrict__ src,
                           Rec<double>* __restrict__ src64) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const double v = q[perm[s]];
  q64[s] = v;
  src[s].q = (T)v;
  if (src64) src64[s].q = v;
}

template <int P, int G>
__global__ __launch_bounds__(64) void k_p2m(const uint32_t* __restrict__ start,
                                            const Rec<double>* __restrict__ src, int64_t nleaf,
                                            double* __restrict__ mult64, float* __restrict__ mult32) {
  const int64_t leaf = (int64_t)blockIdx.x * (64 / G) + threadIdx.x / G;
  if (leaf >= nleaf) return;  // the whole group
  p2m_box<P, G>(src, start[leaf], start[leaf + 1], threadIdx.x % G, leaf, mult64, mult32);
}

template <int P>
struct P2MRun {
  static hipError_t run(fmm_plan_s* Pl, hipStream_t s) {
    const Layout& lay = Pl->lay;
    const int64_t nleaf = lay.nleaf, row0 = lay.lvl_off[Pl->L] * mstride(Pl->p);
    with_p2m_lanes(p2m_lanes(Pl->n, nleaf), [&](auto g) {
      constexpr int G = decltype(g)::value;
      k_p2m<P, G><<<grid_for(nleaf * G, 64), 64, 0, s>>>(
          wsp<uint32_t>(Pl, lay.leaf_start), wsp<Rec<double>>(Pl, Pl->mixed ? lay.src64 : lay.src), nleaf,
          Pl->mixed ? nullptr : wsp<double>(Pl, lay.mult64) + row0,
          Pl->mixed ? wsp<float>(Pl, lay.mult32) + row0 : nullptr);
    });
    return hipGetLastError();
  }
};

}  // namespace

hipError_t launch_upward(fmm_plan_s* P, const double* d_q, hipStream_t s) {
  const Layout& lay = P->lay;
  const int64_t n = P->n;
  if (d_q) {  // NULL: reuse the sorted charges of the last evaluation (adjoint)
    if (P->mixed)
      k_gather_q<float><<<grid_for(n, kBlock), kBlock, 0, s>>>(
          d_q, wsp<int32_t>(P, lay.perm), n, wsp<double>(P, lay.q64), wsp<Rec<float>>(P, lay.src),
          wsp<Rec<double>>(P, lay.src64));
    else
      k_gather_q<double><<<grid_for(n, kBlock), kBlock, 0, s>>>(
          d_q, wsp<int32_t>(P, lay.perm), n, wsp<double>(P, lay.q64), wsp<Rec<double>>(P, lay.src),
          nullptr);
  }
  if (P->adaptive) return launch_adaptive_upward(P, s);
  if (P->L < 2) return hipGetLastError();
  prof_begin(P, FMM_PHASE_P2M, s);
  hipError_t e = dispatch_p<P2MRun>(P->p, P, s);
  prof_end(P, s);
  if (e != hipSuccess) return e;
  prof_begin(P, FMM_PHASE_M2M, s);
  e = launch_m2m(P, s);
  prof_end(P, s);
  return e;
}

}  // namespace fmm
