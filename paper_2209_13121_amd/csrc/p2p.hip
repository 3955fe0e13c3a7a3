// p2p.hip -- P2P near field on source tiles staged in LDS, combination with
// the far field, return to the caller's particle order, and the FP64 energy.
//
// One wave per target leaf t.  The sources of t are the particles of its
// neighbour leaves (uniform tree: the 27 leaves at Chebyshev distance <= 1;
// adaptive tree: the leaves of U(t), t included).  They are staged in LDS in
// tiles of TILE (kTile by default, 128 or 512 by schedule), each source as its
// offset from t's centre in t's box units,
// s_j = o_c + sc_c u_j (o_c the source leaf's centre offset, sc_c its size in
// t's units, u_j the particle's offset in its own leaf, all exact in FP64),
// then the leaf's targets take the tile in groups (target_group):
//   * whole sets of 64 targets: every lane holds K <= kKMax of them (lane + 64
//     m) and reads every source (one LDS broadcast read serves K pairs);
//   * the remaining r < 64: L = ceil(r / K) lanes hold K targets each and G =
//     64 / L copies of them split the sources (copy g takes sources g, g + G,
//     ... of the leaf's list), K chosen for the fullest wave; the copies' sums
//     are combined by shuffles, halving G, in a fixed order.
// Pair offsets u_i - s_j are taken in FP64 in both precisions (one instruction
// an axis: the FP64 vector rate is the FP32 one); mixed rounds them to FP32,
// so they keep FP32 relative accuracy however close the pair, and r^2, 1/r and
// the sums run in FP32.  The target's own leaf is staged first: its pairs at
// distance 0 (the target itself, or a coincident point, which always shares
// the leaf) contribute nothing, and more than one per target raises the
// coincident flag; pairs with the other leaves skip that check.
// Then phi_i = phi_near + phi_far, F_i = -q_i grad phi_i (FP64), written at
// the particle's user index.  In the adjoint form the same pass writes
// g dE/dq_i = g phi_i and g dE/dx_i = g q_i grad phi_i: with every
// (local <= p, multipole <= p) pair kept, the FMM energy is a symmetric
// quadratic form in q, and while no particle crosses a box face its gradient
// in x_i is q_i grad phi_i.  E = 1/2 sum q_i phi_i is reduced in FP64 in a
// fixed tree order over the per-particle terms.
//
// Bound: vector issue.  A mixed pair is 17 instructions (3 FP64 subtractions,
// 3 conversions, 1 / r at half rate), 19 with the loop and idle lanes: 80 cycles for
// 64 pairs, 90 % of the launch (FP64: 19 and 21, 96 cycles, 73 %; counters).
// Measured (uniform): 2^20 charges, depth 4 (256 a leaf), mixed
// 3.87 ms (FP32 hi + lo pair
// offsets and a lane layout of one target per lane up to 32 targets, K = 1, 2,
// 4 above: 4.65 ms), FP64 5.8 ms (1 / sqrt by square root and division, 2 waves
// per SIMD: 13.9 ms); 10^5 charges, depth 4 (24 a leaf), mixed 96 -> 67 us;
// 4096 charges, depth 3, FP64 125 -> 15 us (a wave per leaf instead of one per
// parent box: 512 waves instead of 64).
#include <math.h>

#include <type_traits>

#include "fmm_internal.h"

namespace fmm {
namespace {

constexpr int kTile = 256;   // sources per staged tile (FMM_SCHED_P2P_TILE: 128, 256, 512)
constexpr int kNbBatch = 64;  // neighbour leaves handled per batch (one per lane)
constexpr int kKMax = 4;      // targets per lane, at most
// occupancy the register budget is held to (waves per SIMD)
template <typename T>
constexpr int waves_per_simd() { return sizeof(T) == 4 ? 4 : 3; }

// Staged source: its offset from the target leaf's centre (box units) and its
// charge.
template <typename T>
struct alignas(16) SSrc {
  double x, y, z;
  T q;
};

// A target in registers: its offset from its leaf centre (box units).
struct Tgt {
  double x, y, z;
};

template <typename T>
struct Acc {
  T f, gx, gy, gz;
  int nz;  // pairs at distance 0 (the target itself included)
};

__device__ __forceinline__ Tgt make_tgt(const Rec<double>& r) { return Tgt{r.x, r.y, r.z}; }

__device__ __forceinline__ float inv_sqrt(float x) { return __builtin_amdgcn_rsqf(x); }
// FP64: the hardware estimate y (relative error up to 2^-24.2 over 4 10^6 values)
// and one step of third order: with e = 1 - x y^2, below 2^-23.2,
// x^(-1/2) = y (1 + e / 2 + 3 e^2 / 8 + ...), the dropped term 5 e^3 / 16 below
// 2^-71.  Relative error at most 1.25 2^-53, 0.41 in the mean, against 1.49 and 0.50
// of 1 / sqrt(x); 6 instructions instead of the 30 of a square root and a division
// (and 3 waves per SIMD instead of 2).
__device__ __forceinline__ double inv_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// One pair.  SELF: the source may be the target itself or coincide with it
// (sources of the target's own leaf: coincident points share a leaf), so a
// zero distance contributes nothing and is counted; otherwise no check (a
// zero distance there would make the sums non-finite, which finish_particle
// flags).
template <typename T, bool SELF>
__device__ __forceinline__ void pair(Acc<T>& a, const Tgt& t, const SSrc<T>& s) {
  const T dx = (T)(t.x - s.x), dy = (T)(t.y - s.y), dz = (T)(t.z - s.z), q = s.q;
  const T r2 = dx * dx + dy * dy + dz * dz;
  T rinv;
  if constexpr (SELF) {
    const bool z = r2 == T(0);
    rinv = z ? T(0) : inv_sqrt(r2);
    a.nz += z ? 1 : 0;
  } else {
    rinv = inv_sqrt(r2);
  }
  const T qr = q * rinv;
  const T qr3 = qr * rinv * rinv;
  a.f += qr;
  a.gx -= qr3 * dx;
  a.gy -= qr3 * dy;
  a.gz -= qr3 * dz;
}

// One neighbour leaf: particle range and its centre offset / scale in the
// target's box units.
struct Nb {
  uint32_t start, count;
  double ox, oy, oz, sc;
};

struct FinishArgs {
  int64_t n;
  const double* q64;
  const int32_t* perm;
  int has_far;
  const double* far_phi;
  const double* far_grad;
  double* phi_out;
  double* force_out;
  const double* adj_g;
  double* dEdq;
  double* dEdx;
  int32_t* flags;
  double* eterm;  // q_i phi_i per sorted particle (energy), or NULL
};

// phi_i = near + far, F_i = -q_i grad phi_i (or the adjoint outputs), at the
// particle's user index; q_i phi_i into the energy terms.
template <typename T>
__device__ __forceinline__ void finish_particle(const FinishArgs& fa, int64_t i, double inv_h,
                                                const Acc<T>& acc) {
  if (acc.nz > 1 || !isfinite((double)acc.f)) atomicOr(fa.flags, kFlagCoincident);
  double phi = inv_h * (double)acc.f;
  double g[3] = {inv_h * inv_h * (double)acc.gx, inv_h * inv_h * (double)acc.gy,
                 inv_h * inv_h * (double)acc.gz};
  const int64_t n = fa.n;
  if (fa.has_far) {
    phi += fa.far_phi[i];
    for (int a = 0; a < 3; ++a) g[a] += fa.far_grad[a * n + i];
  }
  const double qi = fa.q64[i];
  const int64_t u = fa.perm[i];
  if (fa.phi_out) fa.phi_out[u] = phi;
  if (fa.force_out)
    for (int a = 0; a < 3; ++a) fa.force_out[3 * u + a] = -qi * g[a];
  if (fa.adj_g) {  // adjoint: dE/dq_i = phi_i, dE/dx_i = q_i grad phi_i, times g
    const double gs = fa.adj_g[0];
    if (fa.dEdq) fa.dEdq[u] = gs * phi;
    if (fa.dEdx)
      for (int a = 0; a < 3; ++a) fa.dEdx[3 * u + a] = gs * (qi * g[a]);
  }
  if (fa.eterm) fa.eterm[i] = qi * phi;
}

// Neighbour leaves of a target leaf.
struct UniformNbs {
  int L;
  const uint32_t* start;  // leaf particle ranges (Hilbert slot order), 8^L + 1
  const uint32_t* c2s;    // leaf level: lexicographic cell -> slot
  const uint32_t* s2c;    // leaf level: slot -> packed cell
  // Target leaf b: its particle range and level; false for no particles.
  __device__ bool target(int64_t b, uint32_t& t0, uint32_t& nt, int& lt) const {
    t0 = start[b];
    nt = start[b + 1] - t0;
    lt = L;
    return nt > 0;
  }
  __device__ int count(int64_t) const { return 27; }
  // neighbour k: the leaf itself first (k = 0), then the other 26
  __device__ Nb get(int64_t b, int k) const {
    int cx, cy, cz;
    unpack_coord(s2c[b], cx, cy, cz);
    const int kk = k == 0 ? 13 : (k <= 13 ? k - 1 : k);  // 13 = (0, 0, 0)
    const int dx = kk / 9 - 1, dy = (kk / 3) % 3 - 1, dz = kk % 3 - 1;
    const int sx = cx + dx, sy = cy + dy, sz = cz + dz, nb = 1 << L;
    Nb r{0, 0, (double)dx, (double)dy, (double)dz, 1.0};
    if (sx >= 0 && sy >= 0 && sz >= 0 && sx < nb && sy < nb && sz < nb) {
      const uint32_t sl = c2s[lex_index(sx, sy, sz, L)];
      r.start = start[sl];
      r.count = start[sl + 1] - r.start;
    }
    return r;
  }
};

// Adaptive tree: boxes in compact order; a leaf's sources are the leaves of
// U(b).  A source leaf c sits at (c_c - c_t) / h_t = (cc + 1/2) 2^(lt - lc) -
// (ct + 1/2) from t in t's units, its offsets scaled by 2^(lt - lc) (exact).
struct AdaptiveNbs {
  const int32_t* level;
  const uint32_t* coord;
  const uint32_t* range;  // {first sorted particle, count} per box
  const int32_t* child0;  // -1 for a leaf
  const uint32_t* uoff;
  const uint32_t* uidx;
  __device__ bool target(int64_t b, uint32_t& t0, uint32_t& nt, int& lt) const {
    if (child0[b] >= 0) return false;
    t0 = range[2 * b];
    nt = range[2 * b + 1];
    lt = level[b];
    return nt > 0;
  }
  __device__ int count(int64_t b) const { return (int)(uoff[b + 1] - uoff[b]); }
  // entry k of U(b) with b itself moved to the front (swapped with entry 0)
  __device__ Nb get(int64_t b, int k) const {
    uint32_t c = uidx[uoff[b] + k];
    if (k == 0)
      c = (uint32_t)b;
    else if (c == (uint32_t)b)
      c = uidx[uoff[b]];
    const int lt = level[b], lc = level[c];
    int ct[3], cc[3];
    unpack_coord(coord[b], ct[0], ct[1], ct[2]);
    unpack_coord(coord[c], cc[0], cc[1], cc[2]);
    const double sc = lt >= lc ? (double)(1 << (lt - lc)) : 1.0 / (double)(1 << (lc - lt));
    Nb r;
    r.start = range[2 * c];
    r.count = range[2 * c + 1];
    r.ox = ((double)cc[0] + 0.5) * sc - ((double)ct[0] + 0.5);
    r.oy = ((double)cc[1] + 0.5) * sc - ((double)ct[1] + 0.5);
    r.oz = ((double)cc[2] + 0.5) * sc - ((double)ct[2] + 0.5);
    r.sc = sc;
    return r;
  }
};

template <typename T>
__device__ __forceinline__ SSrc<T> stage_one(const Rec<double>& r, const Nb& nb) {
  return SSrc<T>{fma(nb.sc, r.x, nb.ox), fma(nb.sc, r.y, nb.oy), fma(nb.sc, r.z, nb.oz), (T)r.q};
}

// Pairs of a lane's K targets with sources j0, j0 + G, .. < ns of the tile, the
// first nself of them from the target's own leaf; returns the first j >= ns.
template <typename T, int K>
__device__ __forceinline__ int tile_pairs(Acc<T> (&acc)[kKMax], const Tgt (&tg)[kKMax], const SSrc<T>* sS, int j0,
                                           int G, int nself, int ns) {
  int j = j0;
  for (; j < nself; j += G) {
    const SSrc<T> s = sS[j];
#pragma unroll
    for (int m = 0; m < K; ++m) pair<T, true>(acc[m], tg[m], s);
  }
  for (; j < ns; j += G) {
    const SSrc<T> s = sS[j];
#pragma unroll
    for (int m = 0; m < K; ++m) pair<T, false>(acc[m], tg[m], s);
  }
  return j;
}

// How the next targets of a leaf (rem of them left) lie over the wave: n
// targets, K per lane, L lanes per copy, G copies.  For the last rem < 64 the
// K of the fewest instructions for 27 rem sources: 20 K + 6 per source of a
// copy, 20 K per round of the combination (24 targets: 2 x 12 lanes x 5 copies,
// 94 % of the lanes busy, against 75 % for 24 x 2).
struct Group {
  int n, K, L, G;
};
// K | L << 3 | G << 10 | ceil(2^14 / L) << 17 for rem = 1 .. 63
struct GroupTable {
  uint32_t v[64];
};
constexpr GroupTable make_groups() {
  GroupTable t{};
  for (int rem = 1; rem < 64; ++rem) {
    int least = 1 << 30;
    for (int K = 1; K <= kKMax; ++K) {
      const int L = (rem + K - 1) / K, G = 64 / L;
      int rounds = 0;
      while ((1 << rounds) < G) ++rounds;
      const int cost = (27 * rem + G - 1) / G * (20 * K + 6) + 20 * K * rounds;
      if (cost < least) {
        least = cost;
        t.v[rem] = (uint32_t)(K | L << 3 | G << 10 | ((1 << 14) + L - 1) / L << 17);
      }
    }
  }
  return t;
}
static __constant__ GroupTable kGroups = make_groups();
// The next group, and this lane's copy gi and first target tl in it
__device__ __forceinline__ Group target_group(int rem, int lane, int& gi, int& tl) {
  if (rem >= 64) {
    const int K = rem / 64 < kKMax ? rem / 64 : kKMax;
    gi = 0;
    tl = lane;
    return Group{64 * K, K, 64, 1};
  }
  const uint32_t c = kGroups.v[rem];
  const Group g{rem, (int)(c & 7u), (int)(c >> 3 & 127u), (int)(c >> 10 & 127u)};
  gi = (int)((uint32_t)lane * (c >> 17) >> 14);  // lane / L, exact for lane < 64
  tl = lane - gi * g.L;
  return g;
}

// LDS of one wave's leaf (TILE sources per staged tile).
template <typename T, int TILE>
struct P2PShared {
  SSrc<T> sS[TILE];
  Nb sNb[kNbBatch];
  uint32_t sPre[kNbBatch + 1];
};

// The near field of target leaf b (one wave).
template <typename T, typename NBS, int TILE>
__device__ __forceinline__ void p2p_leaf(const NBS& nbs, int64_t b, P2PShared<T, TILE>& sh,
                                         const DevParams* __restrict__ dp,
                                         const Rec<double>* __restrict__ src, const FinishArgs& fa) {
  SSrc<T>* sS = sh.sS;
  Nb* sNb = sh.sNb;
  uint32_t* sPre = sh.sPre;
  const int lane = threadIdx.x;
  uint32_t t0, nt;
  int lt;
  if (!nbs.target(b, t0, nt, lt)) return;  // uniform over the wave
  const int nn = nbs.count(b);
  const double inv_h = (double)(1 << lt) / dp->side;
  Acc<T> acc[kKMax];
  Tgt tg[kKMax];
  for (uint32_t g0 = 0; g0 < nt;) {
    int gi, tl;  // this lane's copy and first target
    const Group gr = target_group((int)__builtin_amdgcn_readfirstlane((int)(nt - g0)), lane, gi, tl);
    const int K = gr.K, G = gr.G;
#pragma unroll
    for (int m = 0; m < kKMax; ++m) {
      acc[m] = Acc<T>{T(0), T(0), T(0), T(0), 0};
      const int t = tl + gr.L * m;
      if (m < K) tg[m] = make_tgt(src[t0 + g0 + (t < gr.n ? t : 0)]);
    }
    for (int n0 = 0; n0 < nn; n0 += kNbBatch) {
      // neighbour batch: one leaf per lane, the inclusive scan of counts
      const int k = n0 + lane;
      Nb me{0, 0, 0.0, 0.0, 0.0, 1.0};
      if (k < nn) me = nbs.get(b, k);
      uint32_t c = me.count;
#pragma unroll
      for (int w = 1; w < 64; w <<= 1) {
        const uint32_t v = __shfl_up(c, w, 64);
        if (lane >= w) c += v;
      }
      __syncthreads();  // the previous batch's tables and tile are no longer read
      sNb[lane] = me;
      sPre[lane + 1] = c;
      if (lane == 0) sPre[0] = 0;
      const uint32_t total = __shfl(c, 63, 64);
      __syncthreads();
      int first = gi;  // this copy's first source in the tile
      for (uint32_t c0 = 0; c0 < total; c0 += TILE) {
        const int ns = (int)(total - c0 < (uint32_t)TILE ? total - c0 : (uint32_t)TILE);
        // stage: lane stages sources c0 + lane + 64 m of the batch
        for (int m = lane; m < ns; m += 64) {
          const uint32_t q = c0 + m;
          int lo = 0, hi = kNbBatch;  // sPre[lo] <= q < sPre[hi]
          while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (sPre[mid] <= q)
              lo = mid;
            else
              hi = mid;
          }
          const Nb& nb = sNb[lo];
          sS[m] = stage_one<T>(src[nb.start + (q - sPre[lo])], nb);
        }
        __syncthreads();
        // the target leaf's own sources lead batch 0 (neighbour 0)
        int nself = 0;
        if (n0 == 0 && c0 < nt) nself = nt - c0 < (uint32_t)ns ? (int)(nt - c0) : ns;
        // copy gi takes the batch's sources c0 + j = gi modulo G (whatever the
        // tile); the lanes past the last copy none
        const int j0 = gi >= G ? ns : first;
        int last = j0;
        if (K == 1)
          last = tile_pairs<T, 1>(acc, tg, sS, j0, G, nself, ns);
        else if (K == 2)
          last = tile_pairs<T, 2>(acc, tg, sS, j0, G, nself, ns);
        else if (K == 3)
          last = tile_pairs<T, 3>(acc, tg, sS, j0, G, nself, ns);
        else
          last = tile_pairs<T, kKMax>(acc, tg, sS, j0, G, nself, ns);
        first = last - ns;  // past this tile's end, within the next
        __syncthreads();
      }
    }
    // the copies' sums: the upper half's onto the lower half's, until one is left
    for (int g = G; g > 1; g = (g + 1) / 2) {
      const int h = (g + 1) / 2, from = lane + gr.L * h;
      const bool take = gi + h < g;
#pragma unroll
      for (int m = 0; m < kKMax; ++m) {
        if (m >= K) break;
        const T f = __shfl(acc[m].f, from, 64), gx = __shfl(acc[m].gx, from, 64);
        const T gy = __shfl(acc[m].gy, from, 64), gz = __shfl(acc[m].gz, from, 64);
        const int nz = __shfl(acc[m].nz, from, 64);
        if (take) {
          acc[m].f += f;
          acc[m].gx += gx;
          acc[m].gy += gy;
          acc[m].gz += gz;
          acc[m].nz += nz;
        }
      }
    }
#pragma unroll
    for (int m = 0; m < kKMax; ++m)
      if (m < K && gi == 0 && tl + gr.L * m < gr.n)
        finish_particle<T>(fa, (int64_t)t0 + g0 + tl + gr.L * m, inv_h, acc[m]);
    g0 += gr.n;
  }
}

// One wave per box (boxes that are no leaf, or empty, return at once).
template <typename T, typename NBS, int TILE>
__global__ __launch_bounds__(64, waves_per_simd<T>()) void k_p2p(NBS nbs, int64_t nbox, const DevParams* __restrict__ dp,
                                            const Rec<double>* __restrict__ src, FinishArgs fa) {
  __shared__ P2PShared<T, TILE> sh;
  if ((int64_t)blockIdx.x >= nbox) return;
  p2p_leaf<T, NBS, TILE>(nbs, blockIdx.x, sh, dp, src, fa);
}

// Persistent form over a work-list: the non-empty leaves in order of
// decreasing pair count (built at plan time by k_p2p_worklist), taken one at a
// time by resident waves through a ticket counter (zeroed before the launch),
// so the costliest leaves start first and no wave waits for an empty box.
// Every wave leaves once the tickets pass the list's length.  Each leaf's
// outputs are written by its one task in a fixed order, so the result does
// not depend on which wave takes it.
template <typename T, typename NBS, int TILE>
__global__ __launch_bounds__(64, waves_per_simd<T>()) void k_p2p_persistent(
    NBS nbs, const uint32_t* __restrict__ worklist, const uint32_t* __restrict__ ntasks,
    uint32_t* __restrict__ ticket, const DevParams* __restrict__ dp, const Rec<double>* __restrict__ src,
    FinishArgs fa) {
  __shared__ P2PShared<T, TILE> sh;
  const uint32_t n = ntasks[0];
  for (;;) {
    uint32_t t = 0;
    if (threadIdx.x == 0) t = atomicAdd(ticket, 1u);
    t = __shfl(t, 0, 64);
    if (t >= n) break;  // uniform over the wave
    p2p_leaf<T, NBS, TILE>(nbs, worklist[t], sh, dp, src, fa);
    __syncthreads();  // the tile of this leaf is no longer read
  }
}

// Work-list of the adaptive tree's non-empty leaves by decreasing pair count
// n_b sum_{c in U(b)} n_c: a leaf's bucket is the bit length of its count
// (64 buckets, costliest first).  Counts and positions are taken per
// work-group in LDS and reserved in the global buckets by one atomic per
// (work-group, bucket); the order within a bucket only steers the schedule.
__global__ void k_p2p_cost(AdaptiveNbs nbs, int64_t nbox, uint8_t* __restrict__ bucket,
                           uint32_t* __restrict__ hist) {
  __shared__ uint32_t sh[64];
  if (threadIdx.x < 64) sh[threadIdx.x] = 0;
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint8_t k = 255;  // not a task
  uint32_t t0, nt;
  int lt;
  if (b < nbox && nbs.target(b, t0, nt, lt)) {
    uint64_t ns = 0;
    const int nn = nbs.count(b);
    for (int j = 0; j < nn; ++j) ns += nbs.range[2 * nbs.uidx[nbs.uoff[b] + j] + 1];
    const uint64_t cost = (uint64_t)nt * ns;
    k = (uint8_t)(63 - __clzll(cost | 1ull));
    atomicAdd(&sh[63 - k], 1u);  // bucket 63 - k: the costliest first
  }
  if (b < nbox) bucket[b] = k;
  __syncthreads();
  if (threadIdx.x < 64 && sh[threadIdx.x]) atomicAdd(&hist[threadIdx.x], sh[threadIdx.x]);
}

// Exclusive scan of the 64 bucket counts (one wave) and the list length.
__global__ void k_p2p_hist_scan(uint32_t* __restrict__ hist, uint32_t* __restrict__ ntasks) {
  const int lane = threadIdx.x;
  uint32_t c = hist[lane];
#pragma unroll
  for (int w = 1; w < 64; w <<= 1) {
    const uint32_t v = __shfl_up(c, w, 64);
    if (lane >= w) c += v;
  }
  hist[lane] = c - hist[lane];  // exclusive
  if (lane == 63) ntasks[0] = c;
}

__global__ void k_p2p_worklist(int64_t nbox, const uint8_t* __restrict__ bucket,
                               uint32_t* __restrict__ hist, uint32_t* __restrict__ worklist) {
  __shared__ uint32_t cnt[64], base[64];
  if (threadIdx.x < 64) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int k = b < nbox && bucket[b] != 255 ? 63 - bucket[b] : -1;
  const uint32_t r = k >= 0 ? atomicAdd(&cnt[k], 1u) : 0u;
  __syncthreads();
  if (threadIdx.x < 64) base[threadIdx.x] = cnt[threadIdx.x] ? atomicAdd(&hist[threadIdx.x], cnt[threadIdx.x]) : 0u;
  __syncthreads();
  if (k >= 0) worklist[base[k] + r] = (uint32_t)b;
}

// Uniform tree with small leaves: one wave per parent box P (level L - 1),
// the targets being the particles of its 8 children (consecutive Hilbert
// slots 8P .. 8P + 7, so a contiguous particle range).  The sources of all 8
// are the 4 x 4 x 4 leaves around P, staged once in LDS (tiles of
// kGroupTile) as offsets from P's centre in leaf units, leaf by leaf in
// lexicographic order; each target reads the 27 leaves around its own as 9
// runs of 3 leaves adjacent in z, each run's sources contiguous in LDS.  With
// at most 32 targets, lanes t and t + 32 share a target, taking runs 0..4 and
// 5..8, combined by one xor shuffle.  Tiles of 256 sources (8 KB
// of LDS in mixed mode) leave the occupancy to the registers (4 waves per
// SIMD); tiles of 512 held all 64 leaves of a typical block at once but
// limited it to 9 waves per CU: 0.37 -> 0.26 ms at 2^20 charges, depth 6.
constexpr int kGroupTile = 256;
constexpr int64_t kGroupParents = 4096;  // fewer leave SIMDs without a wave: a wave per leaf then
template <typename T>
__global__ __launch_bounds__(64, waves_per_simd<T>()) void k_p2p_group(
    int L, const uint32_t* __restrict__ start, const uint32_t* __restrict__ c2s,
    const uint32_t* __restrict__ s2c, const uint32_t* __restrict__ sorted_leaf,
    const DevParams* __restrict__ dp, const Rec<double>* __restrict__ src, FinishArgs fa) {
  __shared__ SSrc<T> sS[kGroupTile];
  __shared__ uint32_t sPre[65];  // staged order: block leaf k holds [sPre[k], sPre[k + 1])
  __shared__ uint32_t sStart[64];
  const int64_t P = blockIdx.x;
  const int lane = threadIdx.x;
  const uint32_t t0 = start[8 * P], nt = start[8 * P + 8] - t0;
  if (nt == 0) return;  // uniform over the wave
  int px, py, pz;
  unpack_coord(s2c[8 * P], px, py, pz);
  px >>= 1;
  py >>= 1;
  pz >>= 1;
  const int nb = 1 << L;
  // block leaf k = 16 a + 4 b + c at cell (2 px - 1 + a, ...), centre offset
  // from P's centre (a - 1.5, b - 1.5, c - 1.5) leaf units
  const int ba = lane >> 4, bb = (lane >> 2) & 3, bc = lane & 3;
  {
    const int sx = 2 * px - 1 + ba, sy = 2 * py - 1 + bb, sz = 2 * pz - 1 + bc;
    uint32_t st = 0, cnt = 0;
    if (sx >= 0 && sy >= 0 && sz >= 0 && sx < nb && sy < nb && sz < nb) {
      const uint32_t sl = c2s[lex_index(sx, sy, sz, L)];
      st = start[sl];
      cnt = start[sl + 1] - st;
    }
    uint32_t c = cnt;
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) {
      const uint32_t v = __shfl_up(c, w, 64);
      if (lane >= w) c += v;
    }
    sStart[lane] = st;
    sPre[lane + 1] = c;
    if (lane == 0) sPre[0] = 0;
  }
  __syncthreads();
  const uint32_t total = sPre[64];
  const bool split = nt <= 32;
  for (uint32_t g0 = 0; g0 < nt; g0 += (split ? 32u : 64u)) {
    const int t = split ? (lane & 31) : lane;
    const int h = split ? (lane >> 5) : 0;
    const bool live = g0 + t < nt;
    const int64_t i = (int64_t)t0 + g0 + (live ? t : 0);
    // this target's leaf in the block and its offset from P's centre
    int lx, ly, lz;
    unpack_coord(s2c[sorted_leaf[i]], lx, ly, lz);
    lx -= 2 * px - 1;
    ly -= 2 * py - 1;
    lz -= 2 * pz - 1;
    Rec<double> r = src[i];
    r.x += (double)lx - 1.5;
    r.y += (double)ly - 1.5;
    r.z += (double)lz - 1.5;
    const Tgt tg = make_tgt(r);
    const int kown = 16 * lx + 4 * ly + lz;
    Acc<T> acc = {T(0), T(0), T(0), T(0), 0};
    for (uint32_t c0 = 0; c0 < total; c0 += kGroupTile) {
      const uint32_t ns = total - c0 < (uint32_t)kGroupTile ? total - c0 : (uint32_t)kGroupTile;
      __syncthreads();  // the previous tile is no longer read
      for (uint32_t m = lane; m < ns; m += 64) {
        const uint32_t q = c0 + m;
        int lo = 0, hi = 64;  // sPre[lo] <= q < sPre[hi]
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (sPre[mid] <= q)
            lo = mid;
          else
            hi = mid;
        }
        const Nb nbk{0, 0, (double)(lo >> 4) - 1.5, (double)((lo >> 2) & 3) - 1.5, (double)(lo & 3) - 1.5, 1.0};
        sS[m] = stage_one<T>(src[sStart[lo] + (q - sPre[lo])], nbk);
      }
      __syncthreads();
      if (live) {
        // the 27 neighbour leaves as 9 runs of 3 consecutive block leaves (dz =
        // -1, 0, 1 for each (dx, dy)), whose sources are contiguous in the
        // staged order; split lanes take runs 0..4 and 5..8
        const int r0 = split ? 5 * h : 0, r1 = split ? (h ? 9 : 5) : 9;
        for (int r = r0; r < r1; ++r) {
          const int k = kown + 16 * (r / 3 - 1) + 4 * (r % 3 - 1) - 1;  // first leaf of the run
          // the run's sources within this tile: [a, e) (empty when e <= a)
          const int a = (int)(sPre[k] > c0 ? sPre[k] : c0) - (int)c0;
          const int e = (int)(sPre[k + 3] < c0 + ns ? sPre[k + 3] : c0 + ns) - (int)c0;
          if (r == 4)  // the run through the target's own leaf (zero distances only there)
            for (int j = a; j < e; ++j) pair<T, true>(acc, tg, sS[j]);
          else
            for (int j = a; j < e; ++j) pair<T, false>(acc, tg, sS[j]);
        }
      }
    }
    if (split) {
      acc.f += __shfl_xor(acc.f, 32, 64);
      acc.gx += __shfl_xor(acc.gx, 32, 64);
      acc.gy += __shfl_xor(acc.gy, 32, 64);
      acc.gz += __shfl_xor(acc.gz, 32, 64);
      acc.nz += __shfl_xor(acc.nz, 32, 64);
    }
    if (live && h == 0) finish_particle<T>(fa, i, (double)nb / dp->side, acc);
  }
}

// E = 1/2 sum q_i phi_i: per-block sums of 4 * kBlock consecutive terms in a
// fixed tree order, then one block over the block sums (or, of few terms, over
// the terms).
__global__ void k_energy_blocks(const double* __restrict__ eterm, int64_t n, double* __restrict__ part) {
  __shared__ double red[kBlock];
  double s = 0.0;
  const int64_t base = (int64_t)blockIdx.x * 4 * kBlock;
  for (int r = 0; r < 4; ++r) {
    const int64_t i = base + r * kBlock + threadIdx.x;
    if (i < n) s += eterm[i];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void k_energy(const double* __restrict__ part, int64_t nparts, double* __restrict__ e) {
  __shared__ double red[kBlock];
  double s = 0.0;
  for (int64_t b = threadIdx.x; b < nparts; b += kBlock) s += part[b];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) e[0] = 0.5 * red[0];
}

}  // namespace

namespace {
AdaptiveNbs adaptive_nbs(fmm_plan_s* P) {
  const Layout& lay = P->lay;
  return AdaptiveNbs{wsp<int32_t>(P, lay.a_level), wsp<uint32_t>(P, lay.a_coord),
                     wsp<uint32_t>(P, lay.a_range), wsp<int32_t>(P, lay.a_child0),
                     wsp<uint32_t>(P, lay.a_off), wsp<uint32_t>(P, lay.a_uidx)};
}
// Calls f with std::integral_constant<int, TILE> for the plan's P2P tile.
template <typename F>
void launch_tile(int tile, F&& f) {
  if (tile == 128)
    f(std::integral_constant<int, 128>{});
  else if (tile == 512)
    f(std::integral_constant<int, 512>{});
  else
    f(std::integral_constant<int, kTile>{});
}
}  // namespace

// Plan time (adaptive tree, after its lists): the P2P work-list of the
// persistent form.  Device work only; no read-back.
hipError_t launch_p2p_worklist(fmm_plan_s* P, hipStream_t s) {
  const Layout& lay = P->lay;
  const int64_t nbox = P->ce_off[P->Ld + 1];
  uint32_t* ctl = wsp<uint32_t>(P, lay.a_p2p_ctl);  // [64] bucket counts, [64] tasks, [65] ticket
  uint8_t* bucket = wsp<uint8_t>(P, lay.a_p2p_bucket);
  hipError_t e = fill_u32(ctl, 66, 0u, s);
  if (e != hipSuccess) return e;
  if (nbox > 0) k_p2p_cost<<<grid_for(nbox, kBlock), kBlock, 0, s>>>(adaptive_nbs(P), nbox, bucket, ctl);
  k_p2p_hist_scan<<<1, 64, 0, s>>>(ctl, ctl + 64);
  if (nbox > 0)
    k_p2p_worklist<<<grid_for(nbox, kBlock), kBlock, 0, s>>>(nbox, bucket, ctl,
                                                               wsp<uint32_t>(P, lay.a_p2p_list));
  return hipGetLastError();
}

hipError_t launch_near_and_finish(fmm_plan_s* P, double* d_phi, double* d_force,
                                  double* d_energy, const double* adj_g, double* dEdq,
                                  double* dEdx, hipStream_t s) {
  const Layout& lay = P->lay;
  const int64_t n = P->n;
  const int L = P->L;
  double* eterm = d_energy ? wsp<double>(P, lay.energy_part) : nullptr;
  prof_begin(P, FMM_PHASE_P2P, s);
  FinishArgs fa;
  fa.n = n;
  fa.q64 = wsp<double>(P, lay.q64);
  fa.perm = wsp<int32_t>(P, lay.perm);
  fa.has_far = (P->adaptive || L >= 2) ? 1 : 0;  // the adaptive L2P pass always writes far_*
  fa.far_phi = wsp<double>(P, lay.far_phi);
  fa.far_grad = wsp<double>(P, lay.far_grad);
  fa.phi_out = d_phi;
  fa.force_out = d_force;
  fa.adj_g = adj_g;
  fa.dEdq = dEdq;
  fa.dEdx = dEdx;
  fa.flags = wsp<int32_t>(P, lay.flags);
  fa.eterm = eterm;
  const DevParams* dp = wsp<DevParams>(P, lay.params);
  const Rec<double>* src = wsp<Rec<double>>(P, P->mixed ? lay.src64 : lay.src);
  if (P->adaptive) {
    const AdaptiveNbs nb = adaptive_nbs(P);
    const int64_t nbox = P->ce_off[P->Ld + 1];
    if (P->p2p_persistent) {
      // resident waves over the work-list (16 per CU cover the occupancy of
      // both forms; surplus waves find no ticket and leave)
      uint32_t* ticket = wsp<uint32_t>(P, lay.a_p2p_ctl) + 65;
      hipError_t e = fill_u32(ticket, 1, 0u, s);
      if (e != hipSuccess) return e;
      const uint32_t* wl = wsp<uint32_t>(P, lay.a_p2p_list);
      const uint32_t* nt = wsp<uint32_t>(P, lay.a_p2p_ctl) + 64;
      launch_tile(P->p2p_tile, [&](auto tile) {
        constexpr int TL = decltype(tile)::value;
        const unsigned grid = 256 * 16;
        if (P->mixed)
          k_p2p_persistent<float, AdaptiveNbs, TL><<<grid, 64, 0, s>>>(nb, wl, nt, ticket, dp, src, fa);
        else
          k_p2p_persistent<double, AdaptiveNbs, TL><<<grid, 64, 0, s>>>(nb, wl, nt, ticket, dp, src, fa);
      });
    } else {
      launch_tile(P->p2p_tile, [&](auto tile) {
        constexpr int TL = decltype(tile)::value;
        if (P->mixed)
          k_p2p<float, AdaptiveNbs, TL><<<(unsigned)nbox, 64, 0, s>>>(nb, nbox, dp, src, fa);
        else
          k_p2p<double, AdaptiveNbs, TL><<<(unsigned)nbox, 64, 0, s>>>(nb, nbox, dp, src, fa);
      });
    }
  } else {
    UniformNbs nb{L, wsp<uint32_t>(P, lay.leaf_start), wsp<uint32_t>(P, lay.coord2slot) + lay.lvl_off[L],
                  wsp<uint32_t>(P, lay.slot2coord) + lay.lvl_off[L]};
    const int64_t nleaf = lay.nleaf;
    const int64_t npar = nleaf / 8;
    if (npar >= kGroupParents && n <= 8 * nleaf) {
      // small leaves (at most 8 particles on average): a wave per parent box
      const uint32_t* sl = wsp<uint32_t>(P, lay.sorted_leaf);
      if (P->mixed)
        k_p2p_group<float><<<(unsigned)npar, 64, 0, s>>>(L, nb.start, nb.c2s, nb.s2c, sl, dp, src, fa);
      else
        k_p2p_group<double><<<(unsigned)npar, 64, 0, s>>>(L, nb.start, nb.c2s, nb.s2c, sl, dp, src, fa);
    } else {
      launch_tile(P->p2p_tile, [&](auto tile) {
        constexpr int TL = decltype(tile)::value;
        if (P->mixed)
          k_p2p<float, UniformNbs, TL><<<(unsigned)nleaf, 64, 0, s>>>(nb, nleaf, dp, src, fa);
        else
          k_p2p<double, UniformNbs, TL><<<(unsigned)nleaf, 64, 0, s>>>(nb, nleaf, dp, src, fa);
      });
    }
  }
  prof_end(P, s);
  if (d_energy) {
    prof_begin(P, FMM_PHASE_ENERGY, s);
    const int64_t nparts = (n + 4 * kBlock - 1) / (4 * kBlock);
    double* part = eterm + n;
    // few terms: one block sums them alone (us between events, one / two launches:
    // 700 terms 6.0 / 8.0, 3000 6.8 / 8.1, 4096 8.0 / 8.2, 5000 8.7 / 8.1, 8192
    // 11.9 / 8.2).  A last block that adds the block sums in one launch was slower: the
    // fences of 1024 blocks took 9 to 27 us.
    if (n <= 16 * kBlock) {
      k_energy<<<1, kBlock, 0, s>>>(eterm, n, d_energy);
    } else {
      k_energy_blocks<<<(unsigned)nparts, kBlock, 0, s>>>(eterm, n, part);
      k_energy<<<1, kBlock, 0, s>>>(part, nparts, d_energy);
    }
    prof_end(P, s);
  }
  return hipGetLastError();
}

}  // namespace fmm
