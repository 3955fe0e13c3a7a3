// m2l_sym_kernel.h -- the reflection-reduced multipole-to-local translation on
// the FP64 / FP32 matrix cores (m2l_sym.h has the method; instantiated in
// m2l_sym_f64.hip and m2l_sym_f32.hip).
//
// A wave owns 16 targets of one parity class pi (lane = column c = lane % 16,
// lane group g = lane / 16) and walks the class's items (orbits of offsets).
// Per item and chunk of k steps (one 16-byte vector of every source row per
// lane) it
//   1. turns the orbit's source vectors into the signed sums X_sigma by one
//      butterfly stage per pair axis, (x0 + s x1, x0 - s x1) with s = +-1 the
//      parity of the lane's column under that axis (so that the four columns
//      of a k step may be of different classes), and by +-1 factors on single
//      axes;
//   2. multiplies: row block b of class sigma takes v_mfma_*_16x16x4 of the
//      operator's rows with X_sigma; blocks whose parity under a zero axis no
//      column of the k step shares are skipped.
// Forms:
//  * k_m2l_block (uniform tree): a work-group owns the 128 children of 16
//    parents (16 aligned Hilbert slots: a 4 x 2 x 2 block), wave w the class w
//    children.  All classes walk the same 56 operators, so they share each
//    staged one.  The chunk of every source the work-group reads (a 12 x 8 x 8
//    halo) lies in LDS, copied there once per chunk while the previous one is
//    used; an orbit's sources are LDS reads at uniform displacements.
//  * k_m2l_gather (adaptive tree): the same 16 parents per work-group, sources
//    read from global memory through the source table.  (Many targets at p 4 to 6,
//    FP32 also 7: the plain form, m2l_form.h.)
//  * k_m2l_gather, small (few targets, where the others leave most of the
//    chip idle): the waves of a work-group share 16 targets of one
//    class and split the items (wave w takes w, w + W, ...), operators are read
//    from L2 by each wave, no barriers; the waves' sums are added pairwise
//    through LDS in a fixed order.  With very few targets two work-groups share
//    them (small_parts).
// Sources outside the domain (or absent) read row 0, which is zero.
//
// Bound (FP64, 2^20 charges, depth 6, p = 8): the matrix cores and the vector
// unit, which share the FP64 pipe: 1.30e8 v_mfma_f64_16x16x4 (64 cycles each;
// 128 padded rows of 81 real) are 3.8 ms and the signed sums 1.2 ms of the
// block form's 5.9 ms (0.83 of its cycles, counters); the kernel with a product per offset took 13.2 ms
// (depth 5: 2.70 -> 1.20 ms; 2 x 10^5 charges, depth 5, p = 12: 17.5 -> 4.2
// ms; depth 4, small form: 1.31 -> 0.32 ms; clusters, 3 x 10^5 sites, p = 10:
// 3.2 -> 1.6 ms).  Operators through LDS with a barrier per step: 9.1 ms (the
// waves of a SIMD wait together); operators from L2 without a register set
// ahead: 7.9 ms.
// FP32: chains of a few items are added to the total with Kahan compensation
// (one chain over all items loses accuracy); FP64: one chain.
#pragma once

#include <type_traits>
#include <utility>

#include "m2l_common.h"
#include "m2l_sym.h"

namespace fmm {
namespace sym {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

template <typename T>
struct Mfma;
// Accumulator lane layout (measured on gfx950): lane l holds column l % 16;
// its four values are rows 4 (l / 16) + i for the f32 form and (l / 16) + 4 i
// for the f64 form.
template <>
struct Mfma<float> {
  typedef f32x4 acc_t;
  typedef f32x4 vec_t;
  static constexpr bool kChain = true;  // per-item chains, compensated sum
  static __device__ __forceinline__ int row(int kg, int i) { return 4 * kg + i; }
  static __device__ __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float unit(uint32_t neg) { return __uint_as_float(0x3F800000u | neg); }
};
template <>
struct Mfma<double> {
  typedef f64x4 acc_t;
  typedef f64x2 vec_t;
  static constexpr bool kChain = false;  // one FP64 chain over all items
  static __device__ __forceinline__ int row(int kg, int i) { return kg + 4 * i; }
  static __device__ __forceinline__ acc_t step(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // +-1 by the sign bit
  static __device__ __forceinline__ double unit(uint32_t neg) {
    return __hiloint2double((int)(0x3FF00000u | neg), 0);
  }
};

constexpr int kSymThreads = 512;  // block form: 8 waves, one per class
// Waves per work-group of the gather form: 8 (256 registers per lane), 4 (512)
// at p >= 11, whose accumulators leave too few of 256 for the orbit.
constexpr int gather_waves(int p) { return p <= 10 ? 8 : 4; }

template <int P>
static __constant__ Tab kTab = make_tab(P);
static __constant__ Items kItems = make_items();

// Position of offset d in the class-pi interaction list (the order of the
// adaptive tree's source table: lexicographic, the near offsets skipped).
__device__ __forceinline__ int il_index(int pi, const int* d) {
  const int p[3] = {(pi >> 2) & 1, (pi >> 1) & 1, pi & 1};
  int u[3], v[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u[a] = d[a] + 3 - p[a];       // 0 .. 5
    v[a] = clamp03(d[a] + 1);     // near offsets below, on this axis
  }
  int before = 9 * v[0];
  if (d[0] >= -1 && d[0] <= 1) {
    before += 3 * v[1];
    if (d[1] >= -1 && d[1] <= 1) before += v[2];
  }
  return u[0] * 36 + u[1] * 6 + u[2] - before;
}

// Signed sums of one k step over the axes not in Z: x[e] (e over their bits;
// absent sources are zero) -> w[sigma].  s: the columns' signs.
template <int Z, typename T>
__device__ __forceinline__ void butterfly(T* w, const T* s) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (!(Z & (1 << a))) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((i & (Z | 1 << a)) == 0) {
          const T u = w[i], v = w[i | (1 << a)];
          w[i] = fma(v, s[a], u);
          w[i | (1 << a)] = fma(-v, s[a], u);
        }
    }
}

// Calls f(std::integral_constant<int, zeros>) for the run-time zero axes.
template <typename F>
__device__ __forceinline__ void with_zeros(uint32_t zeros, F&& f) {
  switch (zeros) {
      case 1: f(std::integral_constant<int, 1>{}); break;
      case 2: f(std::integral_constant<int, 2>{}); break;
      case 3: f(std::integral_constant<int, 3>{}); break;
      case 4: f(std::integral_constant<int, 4>{}); break;
      case 5: f(std::integral_constant<int, 5>{}); break;
      case 6: f(std::integral_constant<int, 6>{}); break;
      default: f(std::integral_constant<int, 0>{}); break;
  }
}

// Whether source e (bit a: the reflected partner on axis a, a = 0: z) of the
// item exists: both on pair axes; on single axes the one of the offset's sign.
__device__ __forceinline__ bool has_source(uint32_t code, int pi, int e) {
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ok = ok && source_on_axis((int)(code >> (21 + 2 * a) & 3u), (pi >> a) & 1, (e >> a) & 1);
  }
  return ok;
}
__device__ __forceinline__ uint32_t zero_axes(uint32_t code) {
  uint32_t z = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) z |= (code >> (21 + 2 * a) & 3u) == kZero ? 1u << a : 0u;
  return z;
}
// Offset of source e
__device__ __forceinline__ void item_offset(uint32_t code, int e, int* d) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    d[a] = (int)((code >> (9 + 4 * a)) & 15u) - 4;
    if (e & (4 >> a)) d[a] = -d[a];
  }
}

// A wave's arithmetic: the lane's column parities, the sums and the products.
template <int P, typename T>
struct Core {
  typedef Shape<P, T> S;
  typedef Mfma<T> M;
  typedef typename M::acc_t acc_t;
  typedef typename M::vec_t vec_t;
  typedef typename std::conditional<(S::KS > 32), uint64_t, uint32_t>::type bits_t;
  static constexpr int NAX = 3, NCLS = S::NCLS, NB = S::NB, V = S::V, KS = S::KS, NCH = S::NCH, NT = S::NT;
  static constexpr int NBC = M::kChain ? NB : 1;
  bits_t kb[NAX];
  acc_t acc[NB], sum[NBC], comp[NBC];

  __device__ __forceinline__ void init(int kg) {
#pragma unroll
    for (int x = 0; x < NAX; ++x) kb[x] = (bits_t)kTab<P>.kbits[x][kg];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < NBC; ++b) sum[b] = comp[b] = acc_t{0, 0, 0, 0};
  }
  // Chunk c of an item with zero axes Z: the signed sums of the orbit's
  // vectors xv and their products with the operator's row blocks av; mid()
  // runs once xv is no longer needed, before the last products.
  template <int Z, typename F>
  __device__ __forceinline__ void chunk(int c, const vec_t* xv, const vec_t* av, F&& mid) {
    const bool tail = NT < V && c == NCH - 1;  // the shorter last chunk
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int ks = c * V + v;
      const bool past = tail && v >= NT;
      T w[NCLS];
      if (!past) {
        T s[NAX];
#pragma unroll
        for (int x = 0; x < NAX; ++x) s[x] = M::unit((uint32_t)((kb[x] >> ks) & 1u) << 31);
#pragma unroll
        for (int e = 0; e < NCLS; ++e) w[e] = xv[e][v];
        butterfly<Z, T>(w, s);
      }
      if (v == V - 1) mid();
      if (past) continue;
      if constexpr (Z == 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = M::step(av[b][v], w[S::TAB.bcls[b]], acc[b]);
      } else {
        // rows of parity q under the zero axes meet columns of parity q only
#pragma unroll
        for (int q = 0; q < NCLS; ++q) {
          if (q & ~Z) continue;
          bool need = true;
#pragma unroll
          for (int x = 0; x < NAX; ++x)
            if (Z & (1 << x)) need = need && ((bits_t)S::TAB.has[x][(q >> x) & 1] >> ks & 1u);
          if (need) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
              if ((S::TAB.bcls[b] & Z) == q) acc[b] = M::step(av[b][v], w[S::TAB.bcls[b] & ~Z], acc[b]);
          }
        }
      }
    }
  }
  // The same with the zero axes known at run time only.  The sources absent on
  // them are zero, so both partners of a pair hold the one vector.
  __device__ __forceinline__ void chunk_any(uint32_t zeros, int c, const vec_t* xv, const vec_t* av) {
    constexpr uint32_t kOdd[3] = {0xAAu, 0xCCu, 0xF0u};  // classes odd under each axis
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if (NT < V && v >= NT && c == NCH - 1) return;  // the shorter last chunk
      const int ks = c * V + v;
      T w[NCLS], s[NAX];
#pragma unroll
      for (int x = 0; x < NAX; ++x) s[x] = M::unit((uint32_t)((kb[x] >> ks) & 1u) << 31);
#pragma unroll
      for (int e = 0; e < NCLS; ++e) w[e] = xv[e][v];
      butterfly<0, T>(w, s);
      uint32_t meets = 0xFFu;  // classes that share a column of the k step
#pragma unroll
      for (int x = 0; x < NAX; ++x)
        if (zeros & (1u << x))
          meets &= ((bits_t)S::TAB.has[x][0] >> ks & 1u ? ~kOdd[x] : 0u) |
                   ((bits_t)S::TAB.has[x][1] >> ks & 1u ? kOdd[x] : 0u);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (meets >> S::TAB.bcls[b] & 1u) acc[b] = M::step(av[b][v], w[S::TAB.bcls[b]], acc[b]);
    }
  }
  // FP32: the running chain joins the compensated total
  __device__ __forceinline__ void flush() {
    if constexpr (M::kChain) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const acc_t y = acc[b] - comp[b];
        const acc_t t = sum[b] + y;
        comp[b] = (t - sum[b]) - y;
        sum[b] = t;
        acc[b] = acc_t{0, 0, 0, 0};
      }
    }
  }
  // The waves' sums added pairwise, in a fixed order, through LDS (room for
  // waves / 2 waves); true for the wave that holds the total.
  __device__ __forceinline__ bool add_waves(acc_t* red, int wave, int lane, int waves) {
    acc_t* tot = M::kChain ? sum : acc;
    for (int h = waves / 2; h > 0; h >>= 1) {
      __syncthreads();
      if (wave >= h && wave < 2 * h) {
#pragma unroll
        for (int b = 0; b < NB; ++b) red[((wave - h) * NB + b) * 64 + lane] = tot[b];
      }
      __syncthreads();
      if (wave < h) {
#pragma unroll
        for (int b = 0; b < NB; ++b) tot[b] += red[(wave * NB + b) * 64 + lane];
      }
    }
    return wave == 0;
  }
  // add: one of two shares onto zeroed results, by the hardware's atomic add.  On
  // gfx950 it holds on coarse- and fine-grained device memory (measured equal to
  // the bit), which is what a workspace may be; an exchange with zero by
  // compare-and-swap, valid on any memory, took 1 to 8 us more (4096 charges, p 4:
  // 49 -> 50; 100 003, depth 4, p 10: 468 -> 476).
  __device__ __forceinline__ void store(int kg, T* o, bool add = false) const {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rc = kTab<P>.rcoef[16 * b + M::row(kg, i)];
        if (rc < 0) continue;
        const T v = M::kChain ? sum[b < NBC ? b : 0][i] : acc[b][i];
        if (add) unsafeAtomicAdd(o + rc, v);
        else o[rc] = v;
      }
  }
};

constexpr Orbits kOrbits = make_orbits();
template <typename F, int... G>
__device__ __forceinline__ void for_groups(F&& f, std::integer_sequence<int, G...>) {
  (f(std::integral_constant<int, G>{}), ...);
}

// Block form.  LDS halo: cell (i along the block's long axis A, j, k along the
// others) of lane group g at 16-byte unit g kPlane + 84 i + 10 j + k.  A 16-byte
// read serves 32 lanes (two lane groups) at a time: the 16 targets lie at
// 2 (84 a + 10 b + c), a < 4, b, c < 2 -- 16 distinct even units modulo 32 --
// and the odd plane stride puts the second group on the odd ones, so the
// reads are free of bank conflicts.
constexpr int kHaloA = 12, kHaloB = 8, kStrA = 84, kStrB = 10;
constexpr int kHaloUnits = kHaloA * kStrA;  // units of a plane in use
constexpr int kPlane = 1025;                // 16 copies of 64 units, and odd
// a cell past the block's edge, above every cell in use: it holds the zero row
constexpr int kZeroUnit = (kHaloA - 1) * kStrA + (kHaloB - 1) * kStrB + kHaloB;
constexpr int kNoSource = 1 << 28;  // displacement of an absent source
static_assert(kHaloUnits <= 2 * kSymThreads && 2 * kSymThreads <= kPlane, "two cells per thread");

template <int P, typename T>
__global__ __launch_bounds__(kSymThreads, 2) void k_m2l_block(m2l::Args a, const T* __restrict__ rows,
                                                           const T* __restrict__ ops, T* __restrict__ out) {
  typedef Core<P, T> C;
  typedef typename C::S S;
  typedef typename C::vec_t vec_t;
  constexpr int NB = S::NB, V = S::V, NCH = S::NCH, NT = S::NT, STR = S::STR, NI = S::NI;
  constexpr int NCLS = S::NCLS;
  __shared__ vec_t sH[2][4 * kPlane];
  __shared__ int sD[8][NI][8];  // per class and item: the sources' displacements in units
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 15, kg = lane >> 4, pi = wave;

  // group -> level and parents (XCD-aware: each XCD a contiguous range)
  const int64_t per_xcd = (a.ngroups + 7) / 8;
  const int64_t lg = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (lg >= a.ngroups) return;
  int l = 2;
  while (l < a.L && lg >= a.group_off[l + 1]) ++l;
  const int64_t ps = (lg - a.group_off[l]) * 16 + col;
  const bool col_ok = ps < ((int64_t)1 << (3 * (l - 1)));
  const int nbx = 1 << l;
  const uint32_t* c2s = a.c2s + a.lvl_off[l];
  const int64_t row0 = a.exp_off[l];
  int pc[3], lo[3], hi[3];
  unpack_coord(a.s2c[a.lvl_off[l - 1] + (col_ok ? ps : 0)], pc[0], pc[1], pc[2]);
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    lo[x] = hi[x] = pc[x];
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
      lo[x] = min(lo[x], __shfl_xor(lo[x], m));
      hi[x] = max(hi[x], __shfl_xor(hi[x], m));
    }
    lo[x] = __builtin_amdgcn_readfirstlane(lo[x]);
    hi[x] = __builtin_amdgcn_readfirstlane(hi[x]);
  }
  const int A = hi[2] - lo[2] == 3 ? 2 : (hi[1] - lo[1] == 3 ? 1 : 0);  // the long axis
  int str[3];  // units per cell step along x, y, z
  str[0] = A == 0 ? kStrA : kStrB;
  str[1] = A == 1 ? kStrA : (A == 0 ? kStrB : 1);
  str[2] = A == 2 ? kStrA : 1;
  const int hp[3] = {(pi >> 2) & 1, (pi >> 1) & 1, pi & 1};
  // unit of this lane's target in the halo (which starts two cells below lo)
  int base = kg * kPlane;
#pragma unroll
  for (int x = 0; x < 3; ++x) base += (2 * (pc[x] - lo[x]) + hp[x] + 2) * str[x];

  // the two halo cells this thread copies: their rows (0 outside the domain)
  uint32_t hrow[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int u = j * kSymThreads + (int)threadIdx.x;
    const int i0 = u / kStrA, i1 = (u % kStrA) / kStrB, i2 = u % kStrA % kStrB;
    const int x = 2 * lo[0] - 2 + (A == 0 ? i0 : i1);
    const int y = 2 * lo[1] - 2 + (A == 1 ? i0 : (A == 0 ? i1 : i2));
    const int z = 2 * lo[2] - 2 + (A == 2 ? i0 : i2);
    const bool ok = i0 < kHaloA && i1 < kHaloB && i2 < kHaloB && x >= 0 && y >= 0 && z >= 0 && x < nbx &&
                    y < nbx && z < nbx;
    hrow[j] = ok ? (uint32_t)row0 + c2s[lex_index(x, y, z, l)] : 0u;
  }
  // chunk c of the halo's cells j: lane group g's vectors copied straight into
  // LDS; the shorter last chunk (NT < V) all at once through registers
  auto copy_halo = [&](int c, int j, int g) {
    const T* r = rows + (size_t)hrow[j] * STR + c * 4 * V;
    __builtin_amdgcn_global_load_lds(
        (__attribute__((address_space(1))) void*)(r + g * V),
        (__attribute__((address_space(3))) void*)(&sH[c & 1][g * kPlane + j * kSymThreads + wave * 64]), 16, 0, 0);
  };
  auto copy_tail = [&]() {
    constexpr int c = NCH - 1;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const T* r = rows + (size_t)hrow[j] * STR + c * 4 * V;
      const int u = j * kSymThreads + (int)threadIdx.x;
      T t[4 * NT];
#pragma unroll
      for (int k = 0; k < 4 * NT; ++k) t[k] = r[k];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        vec_t v;
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = k < NT ? t[g * NT + (k < NT ? k : 0)] : T(0);
        sH[c & 1][g * kPlane + u] = v;
      }
    }
  };
  for (int e = threadIdx.x; e < 8 * NI * 8; e += kSymThreads) {
    const int cls = e / (8 * NI), src = e % 8;
    const uint32_t code = kItems.v[cls][e / 8 % NI];
    int d[3];
    item_offset(code, src, d);
    sD[cls][e / 8 % NI][src] =
        has_source(code, cls, src) ? -(d[0] * str[0] + d[1] * str[1] + d[2] * str[2]) : kNoSource;
  }
  // the operator of the next step arrives during this one in a second set of
  // registers, up to 9 row blocks (p = 9).  VGPRs spilled of 256: FP64 none to p = 10,
  // then 28 and 54 without the second set; FP32, whose chains have their own sums,
  // 9 to 16 at p 4 .. 9, then 51, 110 and 501 without it
  constexpr int AHEAD = NB <= 9 ? 1 : 0;
  vec_t xv[NCLS], av[1 + AHEAD][NB];
  int disp[NCLS];
  const uint32_t zero_at = kg * kPlane + kZeroUnit;
  auto read_disp = [&](int it) {
#pragma unroll
    for (int e = 0; e < NCLS; ++e) disp[e] = sD[pi][it][e];
  };
  // The orbit's vectors
  auto read_x = [&](int hb) {
#pragma unroll
    for (int e = 0; e < NCLS; ++e) xv[e] = sH[hb][min((uint32_t)(base + disp[e]), zero_at)];
  };
  const T* opl = ops + lane * V;
  auto load_a = [&](const T* r, vec_t* to) {
#pragma unroll
    for (int b = 0; b < NB; ++b) to[b] = *reinterpret_cast<const vec_t*>(r + b * 64 * V);
  };

  C core;
  core.init(kg);
  if (NT < V && NCH == 1) {
    copy_tail();
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) copy_halo(0, k / 4, k % 4);
  }
  load_a(opl, av[0]);
  // Item it of chunk c with the operator in cur; the next step's operator is
  // on its way to nxt and its sources to xv meanwhile.
  auto step = [&](auto zc, int c, int it, const vec_t* cur, vec_t* nxt) {
    const bool last = it + 1 == NI;
    const T* na =
        opl + (size_t)(last ? 0 : it + 1) * S::OP + (size_t)(last && c + 1 < NCH ? c + 1 : c) * S::CHUNK;
    if (AHEAD) load_a(na, nxt);
    core.template chunk<decltype(zc)::value>(c, xv, cur, [&]() {
      if (!last) read_x(c & 1);
      read_disp(it + 2 < NI ? it + 2 : 0);
    });
    if (!AHEAD) load_a(na, nxt);
    if (C::M::kChain && (it % 4 == 3 || last)) core.flush();
  };
#pragma unroll 1
  for (int c = 0; c < NCH; ++c) {
    // this wave's copies have landed, then every wave's; the buffer of chunk
    // c - 1 is no longer read
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    read_disp(0);
    read_x(c & 1);
    read_disp(1);
    auto run = [&](auto gc) {  // the items of one set of zero axes, two at a time
      constexpr int G = decltype(gc)::value;
      static_assert((kOrbits.start[G + 1] - kOrbits.start[G]) % 2 == 0, "runs of even length");
      typedef std::integral_constant<int, kOrbits.zeros[G]> Z;
#pragma unroll 1
      for (int it = kOrbits.start[G]; it < kOrbits.start[G + 1]; it += 2) {
        if constexpr (G == 0) {  // the next chunk's halo, a copy per lane group and pair of items
          if (c + 1 < NCH) {
            if (NT < V && c + 1 == NCH - 1) {
              if (it == 0) copy_tail();
            } else if (it < 16) {
              copy_halo(c + 1, it >> 3, it >> 1 & 3);
            }
          }
        }
        step(Z{}, c, it, av[0], av[AHEAD]);
        step(Z{}, c, it + 1, av[AHEAD], av[0]);
      }
    };
    for_groups(run, std::make_integer_sequence<int, kOrbits.ngroups>{});
  }
  if (!col_ok) return;
  const int tx = 2 * pc[0] + hp[0], ty = 2 * pc[1] + hp[1], tz = 2 * pc[2] + hp[2];
  core.store(kg, out + (row0 + c2s[lex_index(tx, ty, tz, l)]) * S::NC);
}

// A lane's target: number ps of the class-pi children of level l's parents.
struct Target {
  bool ok, ad;
  int x, y, z;
  int64_t row;         // row within the level
  const uint32_t* vt;  // adaptive: the target's column of the source table
  __device__ __forceinline__ Target(const m2l::Args& a, int l, int pi, int64_t ps)
      : ad(a.vtab != nullptr), x(0), y(0), z(0), row(0), vt(nullptr) {
    if (ad) {
      ok = ps < a.ndiv[l];
      if (ok) row = a.tgt[a.tgt_off[l] + pi * a.ndiv[l] + ps];
      vt = a.vtab + a.vt_off[l] +
           ((ps / m2l::kTargetsPerGroup) * 8 + pi) * (int64_t)kIL * m2l::kTargetsPerGroup +
           ps % m2l::kTargetsPerGroup;
    } else {
      ok = ps < ((int64_t)1 << (3 * (l - 1)));
      if (ok) {
        unpack_coord(a.s2c[a.lvl_off[l - 1] + ps], x, y, z);
        x = 2 * x + ((pi >> 2) & 1);
        y = 2 * y + ((pi >> 1) & 1);
        z = 2 * z + (pi & 1);
        row = a.c2s[a.lvl_off[l] + lex_index(x, y, z, l)];
      }
    }
  }
  // Row of the source at offset d, 0 (the zero row) where there is none
  __device__ __forceinline__ uint32_t source(const m2l::Args& a, int l, int pi, const int* d) const {
    if (ad) {
      const uint32_t v = vt[(int64_t)il_index(pi, d) * m2l::kTargetsPerGroup];
      return (v & m2l::kAbsent) ? 0u : (uint32_t)a.exp_off[l] + v;
    }
    const int nb = 1 << l, sx = x - d[0], sy = y - d[1], sz = z - d[2];
    const bool in = ok && sx >= 0 && sy >= 0 && sz >= 0 && sx < nb && sy < nb && sz < nb;
    const uint32_t v = a.c2s[a.lvl_off[l] + (in ? lex_index(sx, sy, sz, l) : 0)];
    return in ? (uint32_t)a.exp_off[l] + v : 0u;
  }
};

// Whether a chunk's zero axes stay a run-time value: one body instead of seven,
// some 50 registers fewer (FP64: none spilled; with seven, 15 at p = 10, 361 at
// p = 12).  FP64, ms, seven bodies -> one: 262 144 charges, depth 4, p = 4 / 8 / 10 /
// 12: 0.138 / 0.331 / 0.495 / 3.61 -> 0.132 / 0.321 / 0.463 / 1.12; adaptive, 10^6,
// p = 10: 4.22 -> 3.98.  FP32 spills little up to p = 10 (15 at p = 4, 8 at p = 10),
// and there the products that a known axis leaves out by class weigh more (10^6,
// p = 10: 2.00 against 2.22); p = 12: 0.72 -> 0.67.
template <int P, typename T>
constexpr bool any_zeros() {
  return sizeof(T) == 8 || P >= 11;
}

// Gather form (see the head of the file).  parts > 0, the small form: the waves
// of parts work-groups (1 or 2) share 16 targets.
template <int P, typename T>
__global__ __launch_bounds__(64 * gather_waves(P), gather_waves(P) / 4) void k_m2l_gather(m2l::Args a, int parts, const T* __restrict__ rows,
                                                            const T* __restrict__ ops, T* __restrict__ out) {
  typedef Core<P, T> C;
  typedef typename C::S S;
  typedef typename C::acc_t acc_t;
  typedef typename C::vec_t vec_t;
  constexpr int W = gather_waves(P), NCLS = S::NCLS, NB = S::NB, V = S::V, NCH = S::NCH, NT = S::NT;
  constexpr int STR = S::STR, NI = S::NI;
  __shared__ acc_t red[(W / 2) * NB * 64];          // small: the sums of W / 2 waves
  __shared__ uint32_t sRow[2][64 * W * NCLS];  // rows of the current and the next item's sources
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 15, kg = lane >> 4;

  // group -> level, parents and (small) class (XCD-aware: each XCD a contiguous
  // range of groups; small: the 8 classes of the same parents consecutive)
  const bool small = parts > 0;
  const int64_t per_xcd = (a.ngroups + 7) / 8;
  int64_t lg = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (lg >= a.ngroups) return;
  int first = small ? wave : 0;  // item of the wave
  if (parts == 2) {
    first += W * (int)(lg & 1);
    lg >>= 1;
  }
  int l = 2;
  while (l < a.L && lg >= a.group_off[l + 1]) ++l;
  const int64_t idx = lg - a.group_off[l];
  const int pi = small ? (int)(idx % 8) : (int)(idx % (8 / W)) * W + wave;
  const Target t(a, l, pi, idx / (small ? 8 : 8 / W) * 16 + col);

  uint32_t nrow[NCLS];  // rows of the next item's sources, on their way to LDS
  // Rows of the item's sources (0, the zero row, where there is none)
  auto lookup = [&](uint32_t code) {
#pragma unroll
    for (int e = 0; e < NCLS; ++e) {
      nrow[e] = 0;
      if (!has_source(code, pi, e)) continue;
      int d[3];
      item_offset(code, e, d);
      nrow[e] = t.source(a, l, pi, d);
    }
  };
  auto keep_rows = [&](int rb) -> bool {  // nrow into LDS; whether a lane has a source
    uint32_t any = 0;
#pragma unroll
    for (int e = 0; e < NCLS; ++e) {
      sRow[rb][e * 64 * W + threadIdx.x] = nrow[e];
      any |= nrow[e];
    }
    return __any(any != 0);
  };
  vec_t xv[NCLS], av[NB];
  const T* opl = ops + lane * V;
  // chunk c of the item's sources and operator
  auto load = [&](uint32_t code, int c, int rb) {
    const bool tail = NT < V && c == NCH - 1;
    __asm__ volatile("" ::: "memory");  // the rows are read from LDS here, not kept in registers
#pragma unroll
    for (int e = 0; e < NCLS; ++e) {
      if (!has_source(code, pi, e)) {
#pragma unroll
        for (int v = 0; v < V; ++v) xv[e][v] = T(0);
        continue;
      }
      const T* r = rows + (size_t)sRow[rb][e * 64 * W + threadIdx.x] * STR + c * 4 * V;
      if (tail) {
#pragma unroll
        for (int v = 0; v < NT; ++v) xv[e][v] = r[kg * NT + v];
      } else {
        xv[e] = *reinterpret_cast<const vec_t*>(r + kg * V);
      }
    }
    const T* r = opl + (size_t)(code & 511u) * S::OP + (size_t)c * S::CHUNK;
#pragma unroll
    for (int b = 0; b < NB; ++b) av[b] = *reinterpret_cast<const vec_t*>(r + b * 64 * V);
  };

  C core;
  core.init(kg);
  const int step = small ? W * parts : 1;  // item stride of a wave
  int rb = 0;
  uint32_t code = kItems.v[pi][first];
  lookup(code);
  bool any = keep_rows(0);
  if (any) load(code, 0, 0);
#pragma unroll 1
  for (int it = first; it < NI; it += step) {
    const bool more = it + step < NI;
    const uint32_t ncode = kItems.v[pi][more ? it + step : it];
    if (more) lookup(ncode);
    if (any) {
#pragma unroll 1
      for (int c = 0; c < NCH; ++c) {
        if constexpr (any_zeros<P, T>())
          core.chunk_any(zero_axes(code), c, xv, av);
        else
          with_zeros(zero_axes(code),
                     [&](auto zc) { core.template chunk<decltype(zc)::value>(c, xv, av, []() {}); });
        if (c + 1 < NCH) load(code, c + 1, rb);
      }
      core.flush();
    }
    rb ^= 1;
    code = ncode;
    any = more && keep_rows(rb);
    if (any) load(code, 0, rb);
  }

  if (small && !core.add_waves(red, wave, lane, W)) return;
  if (t.ok) core.store(kg, out + (a.exp_off[l] + t.row) * S::NC, parts == 2);
}

// Multipole rows in the order of the columns (m2l_sym.h row_slot), row 0 zero.
// A work-group copies 64 rows; reads and writes run along the rows.  zero: the
// results of nz values per box, to which two work-groups will add.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_sym_rows(Tab tab, int str, int64_t box0, int64_t nbox,
                                                     const T* __restrict__ mult, T* __restrict__ rows,
                                                     T* __restrict__ zero, int nz) {
  __shared__ int16_t src[4 * kMaxKs];  // coefficient held by each slot
  const int ks = str / 4, v = 16 / (int)sizeof(T);
  for (int r = threadIdx.x; r < str; r += kBlock) src[row_slot(r, ks, v)] = tab.kcoef[r];
  __syncthreads();
  if (blockIdx.x == 0)
    for (int e = threadIdx.x; e < str; e += kBlock) rows[e] = T(0);
  const int64_t b0 = box0 + (int64_t)blockIdx.x * 64;
  const int64_t nb = b0 + 64 < nbox ? 64 : nbox - b0, n = nb * str;
  if (zero)
    for (int64_t e = threadIdx.x; e < nb * nz; e += kBlock) zero[b0 * nz + e] = T(0);
  for (int64_t e = threadIdx.x; e < n; e += kBlock) {
    const int64_t b = b0 + e / str;
    const int c = src[e % str];
    rows[b * str + e % str] = c < 0 ? T(0) : mult[b * str + c];
  }
}

// Work-groups that share 16 targets in the small form, with the work-groups
// (of one each) that there are.  Two, each walking half of the 56 items (4
// instead of 7 a wave) and adding to zeroed results (two terms: the order does
// not matter), where that takes fewer rounds of the 256 CUs, which hold one
// work-group each (40 work-groups, 4096 charges, depth 3, p = 4 / 8: 79 / 201 ->
// 49 / 121 us; 296, depth 4, p = 4 / 8: 146 / 350 -> 132 / 320; some 400,
// p = 8: 358 -> 423, so one).  FP32 stays at one: two rounded terms would be less
// exact than the compensated total.
inline int small_parts(int64_t groups, bool fp64) {
  auto rounds = [](int64_t g) { return (g + 255) / 256; };
  return fp64 && groups < 512 && 4 * rounds(2 * groups) < 7 * rounds(groups) ? 2 : 1;
}

template <int P, typename T>
hipError_t run(fmm_plan_s* Pl, hipStream_t s) {
  const Layout& lay = Pl->lay;
  // the rows lie in the space of the local expansions, which the downward
  // pass writes after the M2L
  T* rows = wsp<T>(Pl, lay.loc_exp64);
  const T* mult = wsp<T>(Pl, sizeof(T) == 4 ? lay.mult32 : lay.mult64);
  const T* ops = wsp<T>(Pl, sizeof(T) == 4 ? lay.op_m2l32 : lay.op_m2l64);
  T* out = wsp<T>(Pl, lay.m2l_out);
  const int64_t box0 = exp_box0(Pl), nbox = exp_nbox(Pl);
  if (nbox <= box0) return hipSuccess;
  // group_off, ngroups: 8 classes x groups of 16 parents
  m2l::Args a = m2l::make_args(Pl, 16);
  const bool wide = a.ngroups >= 8 * kWideGroups;
  const int parts = wide ? 0 : small_parts(a.ngroups, sizeof(T) == 8);
  prof_begin(Pl, FMM_PHASE_M2L, s);
  k_sym_rows<T><<<grid_for(nbox - box0, 64), kBlock, 0, s>>>(Shape<P, T>::TAB, Shape<P, T>::STR, box0, nbox,
                                                             mult, rows, parts == 2 ? out : nullptr,
                                                             Shape<P, T>::NC);
  auto share = [&](int classes) {  // work-groups of that many classes each
    for (int l = 2; l <= a.L + 1; ++l) a.group_off[l] /= classes;
    a.ngroups /= classes;
  };
  constexpr int W = gather_waves(P);
  if (wide && !Pl->adaptive) {
    if constexpr (serves(P, sizeof(T) == 8, false, INT32_MAX, 1)) {
      share(8);
      k_m2l_block<P, T><<<m2l::grid_of(a), kSymThreads, 0, s>>>(a, rows, ops, out);
    }
  } else {
    if (wide) share(W);
    if (parts == 2) a.ngroups *= 2;
    k_m2l_gather<P, T><<<m2l::grid_of(a), 64 * W, 0, s>>>(a, parts, rows, ops, out);
  }
  prof_end(Pl, s);
  return hipGetLastError();
}

}  // namespace sym
}  // namespace fmm
