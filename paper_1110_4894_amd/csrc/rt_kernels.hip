// gfx950 kernels of the ray-bundle lensing path.
//
// Method: Killedar, Lasky, Lewis & Fluke (2011).  The hot kernel is the
// persistent trace kernel: every wavefront owns 7 whole bundles (63 rays, one
// per lane) and integrates them through all RK4 steps in FP64; at every stage
// the rays' field is the direct sum over the step's particle set (Sec. 3.3,
// eq. psi, derivs), streamed in tiles through the wavefront's own LDS slice.
//
// Design notes for CDNA4:
//   * FP32 field sums work per bundle (Sec. 3.1: an anchor and a ring of 8
//     rays a few parsecs away).  The nine lanes of a bundle split the
//     particles; each (bundle, particle) pair is evaluated once, at the
//     bundle's expansion point, as the pair's potential and field and their
//     first and second derivatives (20 moments, 37 VALU instructions per pair
//     of a set of equal masses including one v_rsq_f32, i.e. 4.1 per
//     ray-particle interaction).  Every ray
//     assembles its own field in FP64 from the moments and its exact offset.
//     Ring-minus-anchor field differences, which carry the lensing signal,
//     so keep FP32 relative precision: rounding each particle-ray
//     displacement to FP32 instead would quantise the ring offset to the ulp
//     of a Mpc-scale distance, identically for every particle of a binade;
//   * plain FP32 partial sums over 256 rounds of a bundle's nine lanes (32
//     where the nearness test runs) are added with
//     Kahan compensation; FP64 is kept for the ray state, the integration and
//     the assembly of each ray's field;
//   * an RK4 step visits two planes twice each, and a plane's moments are
//     summed once (see Planes below), which halves the pairs;
//   * the pairwise sum is not a dense contraction: no matrix cores;
//   * work items (field, block of rays) are pulled from an atomic queue so that
//     fields of very different particle counts share one launch.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <map>
#include <mutex>
#include <type_traits>

#include "rt_direct.h"
#include "rt_geodesic.h"
#include "rt_internal.h"

namespace rt {

namespace {

// ---------------------------------------------------------------------------
// Lane layout shared by every kernel that holds bundles: a wavefront holds 7
// whole bundles, lane l < 63 owns ray l of the group (bundle l / 9, ray l % 9
// of it, the anchor first); lane 63 only helps to stage tiles.
// ---------------------------------------------------------------------------
constexpr int kLanes = 63;              // rays per wavefront
constexpr int kSeg = 7;                 // bundles per wavefront

__device__ __forceinline__ int lane_segment(int lane) { return lane < kLanes ? lane / 9 : kSeg - 1; }

// ===========================================================================
// FP32 field sums: bundle moments.
//
// A ray of a bundle sits at e + delta, where e is the bundle's expansion point
// (its anchor rounded to FP32 in the set's frame, at the stage's z) and delta
// = (dx, dy, 0) its own offset, a few parsecs (all rays of a field share z).
// With D = x_j - e and s = |D|^2 + eps^2, one particle's terms at the ray,
// m (s - 2 D.delta + |delta|^2)^(-1/2) and m (D - delta) (...)^(-3/2), expand
// in delta; to second order the sums over the particles are
//
//   S0(delta) = Phi + G.delta - |delta|^2 W / 2 + 3/2 delta.T.delta
//   S(delta)  = G + 3 T.delta - W delta - 3/2 |delta|^2 V - 3 delta (V.delta)
//               + 15/2 U(delta, delta)
//
// with the moments (w = s^-3/2, q = s^-5/2, r = s^-7/2, sums over j of m_j x)
//   Phi = m s^-1/2, G_i = m w D_i, W = m w, V_i = m q D_i, T_il = m q D_i D_l,
//   U_ilk = m r D_i D_l D_k   (l, k over x and y only, as delta_z = 0).
//
// The expansion variable u = (|delta|^2 - 2 D.delta) / s has |u| <= 2 |delta|
// / sqrt(s) + |delta|^2 / s; the first neglected terms are 35/16 u^3 of the
// pair's field and 5/16 u^3 of its potential, i.e. about 1.5 u^2 and 0.6 u^2 of
// the pair's ring-minus-anchor difference (its first-order term).  A pair is
// summed this way only when sqrt(s) >= 1024 |delta|max of its bundle
// (|u| < 0.002: the neglected terms stay below 7e-6 of the pair's ring
// difference, the expansion point's own distance from the anchor included, and
// 1e-8 of the pair term); closer pairs, and pairs within 1e-4
// Mpc of the expansion point (where s^-7/2 would leave the FP32 range), are
// left out of the moments and summed per ray directly in FP64.  Softened sets
// whose softening exceeds 1024 |delta|max for every bundle of a wavefront
// (boxes: 71 kpc against a few parsecs) skip the nearness test altogether.
// ===========================================================================
constexpr int kMom = 20;
constexpr int kKahanRounds = 256;        // rounds of plain FP32 sums between compensated adds, without the nearness test
constexpr int kGuardRounds = 32;         // the same where the test runs
constexpr float kNearRatio2 = 1048576.f;   // (1024)^2
constexpr float kNearFloor2 = 1e-8f;     // (1e-4 Mpc)^2
// LDS of the FP32 path, per workgroup: WPR tiles (one per wavefront index q of
// the ray groups; the NG groups of a workgroup share them), each TP float4
// (x, y in the set's frame, z relative to the stage, m, or z^2 + eps^2 for a
// set of equal masses) followed by TP float2
// (the rounding residuals of x and y).  After the last tile the same bytes hold
// the moment reduction: per wavefront [20][64] floats and [4][64] doubles.
// Beside them, kept from one field evaluation to the next: per group [20][7] double
// totals, per wavefront its list of near particles (float4, then float2) and where it stands (NearList::Mark).
constexpr int kRedBytes = kMom * 64 * 4 + 4 * 64 * 8;
static_assert(kRedBytes % 16 == 0, "reduction areas stay 16-byte aligned");
constexpr int kNearList = 62;            // particles: a halo's core holds some near ones per wavefront and stage
constexpr int kNearBytes = kNearList * 24 + 16;
static_assert(kNearBytes % 16 == 0 && kMom * kSeg * 8 % 16 == 0, "kept areas stay 16-byte aligned");
template <int NW, int WPR, int TP>
struct Lds32 {
  static_assert(TP % 9 == 0, "a tile holds whole rounds of the nine lanes of a bundle");
  static_assert(TP % 2 == 0, "the residuals start 16-byte aligned");
  static constexpr int kTileElems = TP * 24 / 16;                    // float4 per tile
  static constexpr int kTileBytes = WPR * TP * 24;
  static constexpr int kRed = NW * kRedBytes;
  static constexpr int kTotAt = (kTileBytes > kRed) ? kTileBytes : kRed;         // bytes
  static constexpr int kNearAt = kTotAt + (NW / WPR) * kMom * kSeg * 8;
  static constexpr int kElems = (kNearAt + NW * kNearBytes) / 16;
};

// LDS elements of a kernel's FP32 workgroup tiles (none for FP64 kernels).
template <bool F64, int NW, int WPR, int TP>
struct Lds32Elems {
  static constexpr int v = 1;
};
template <int NW, int WPR, int TP>
struct Lds32Elems<false, NW, WPR, TP> {
  static constexpr int v = Lds32<NW, WPR, TP>::kElems;
};

// Moment indices.
enum : int {
  M_PHI = 0, M_GX, M_GY, M_GZ, M_W, M_VX, M_VY, M_VZ, M_TXX, M_TXY, M_TYY, M_TZX, M_TZY,
  M_UXXX, M_UXXY, M_UXYY, M_UYYY, M_UZXX, M_UZXY, M_UZYY
};

// One (bundle, particle) pair.  p = (x, y, z relative to e, w) with x, y still
// in the set's frame and w = m / mref, or for a set of equal masses (whose pairs
// need no mass) w = z^2 + eps^2, staged once per particle; lo = the residuals of
// x and y; (ex, ey) = e.  GUARD: a near pair (s < thr) is left out of the moments;
// returns whether it is one.
template <bool EQUAL>
__device__ __forceinline__ float pair_s(const float4 p, float Dx, float Dy, float e2) {
  const float sz = EQUAL ? p.w : fmaf(p.z, p.z, e2);
  return fmaf(Dx, Dx, fmaf(Dy, Dy, sz));
}

template <bool EQUAL, bool GUARD>
__device__ __forceinline__ bool moment_terms(const float4 p, const float2 lo, float ex, float ey, float e2,
                                             float thr, float (&a)[kMom]) {
  const float Dx = (p.x - ex) + lo.x, Dy = (p.y - ey) + lo.y, Dz = p.z;
  const float s = pair_s<EQUAL>(p, Dx, Dy, e2);
  float ia = __builtin_amdgcn_rsqf(s);
  const bool near = GUARD && s < thr;
  if constexpr (GUARD) ia = near ? 0.f : ia;
  const float ia2 = ia * ia;
  const float mia = EQUAL ? ia : p.w * ia;
  a[M_PHI] += mia;
  const float w = mia * ia2;
  a[M_GX] = fmaf(w, Dx, a[M_GX]);
  a[M_GY] = fmaf(w, Dy, a[M_GY]);
  a[M_GZ] = fmaf(w, Dz, a[M_GZ]);
  a[M_W] += w;
  const float q = w * ia2;
  const float qx = q * Dx, qy = q * Dy;
  a[M_VX] += qx;
  a[M_VY] += qy;
  a[M_VZ] = fmaf(q, Dz, a[M_VZ]);
  a[M_TXX] = fmaf(Dx, qx, a[M_TXX]);
  a[M_TXY] = fmaf(Dx, qy, a[M_TXY]);
  a[M_TYY] = fmaf(Dy, qy, a[M_TYY]);
  a[M_TZX] = fmaf(Dz, qx, a[M_TZX]);
  a[M_TZY] = fmaf(Dz, qy, a[M_TZY]);
  // m s^-7/2 (Dx, Dy), from the s^-5/2 products
  const float rx = qx * ia2, ry = qy * ia2;
  const float rxx = rx * Dx, rxy = rx * Dy, ryy = ry * Dy;
  a[M_UXXX] = fmaf(Dx, rxx, a[M_UXXX]);
  a[M_UXXY] = fmaf(Dx, rxy, a[M_UXXY]);
  a[M_UXYY] = fmaf(Dx, ryy, a[M_UXYY]);
  a[M_UYYY] = fmaf(Dy, ryy, a[M_UYYY]);
  a[M_UZXX] = fmaf(Dz, rxx, a[M_UZXX]);
  a[M_UZXY] = fmaf(Dz, rxy, a[M_UZXY]);
  a[M_UZYY] = fmaf(Dz, ryy, a[M_UZYY]);
  return near;
}

// A near pair, summed directly at the ray e + (dx, dy, 0), in FP64 (such pairs
// are rare).  The nearness test repeats moment_terms' FP32 arithmetic exactly,
// so the bundle's nine lanes and the lane that left the pair out of the moments
// agree on every pair.
// (dz is the ray's height above the staged z: zero in the trace kernel, whose
// rays share z; points of a field evaluation may differ.)
template <bool EQUAL>
__device__ __forceinline__ bool near_pair(const float4 p, const float2 lo, float ex, float ey, float e2, float thr) {
  const float Dx = (p.x - ex) + lo.x, Dy = (p.y - ey) + lo.y;
  return pair_s<EQUAL>(p, Dx, Dy, e2) < thr;
}

template <bool EQUAL>
__device__ __forceinline__ void near_direct(const float4 p, const float2 lo, float ex, float ey, float e2,
                                            double dx, double dy, double dz, double (&d)[4]) {
  // the displacement from the particle's two-part position is exact in FP64, and the
  // term's rounding stays far below its ring-minus-anchor difference
  const double rx = (((double)p.x - ex) + lo.x) - dx, ry = (((double)p.y - ey) + lo.y) - dy;
  const double rz = (double)p.z - dz;
  const double s2 = fma(rz, rz, fma(ry, ry, fma(rx, rx, (double)e2)));
  const double ia = rsqrt_f64(s2);
  const double mia = EQUAL ? ia : (double)p.w * ia;
  const double w = mia * ia * ia;
  d[0] += mia;
  d[1] += w * rx;
  d[2] += w * ry;
  d[3] += w * rz;
}

// The near particles that a wavefront met, in the order of the sum.  (The list is filled in the moment loops, its
// terms are summed after them: no FP64 term lives in those loops' registers.)  Those that do not fit are found
// again in the tiles, from the round of nine where the list was full to the last tile that held one.
struct NearList {
  struct Mark {           // kept in LDS with the list
    int n;                // particles listed
    int first, round;     // tile (of this wavefront's) and its round of the first that did not fit; first < 0: all did
    int last;             // tile of the last one
  };
  float4* p;
  float2* lo;
  Mark* mark;
  Mark at;
  bool missed;            // in the present tile
};
static_assert(sizeof(NearList::Mark) == 16, "kNearBytes holds it");

// The listed particles' terms at the lane's ray, each where its pair is near for the lane's bundle.
template <bool EQUAL>
__device__ __forceinline__ void near_terms(const NearList& list, float ex, float ey, float e2, float thr, double dx,
                                           double dy, double dz, double (&d)[4]) {
#pragma unroll 1
  for (int j = 0; j < list.at.n; ++j) {
    const float4 p = list.p[j];
    const float2 lo = list.lo[j];
    if (near_pair<EQUAL>(p, lo, ex, ey, e2, thr)) near_direct<EQUAL>(p, lo, ex, ey, e2, dx, dy, dz, d);
  }
}

__device__ __forceinline__ void kahan_add(float& s, float& c, float v) {
  float y = v - c;
  float t = s + y;
  c = (t - s) - y;
  s = t;
}

// Round i's particles near for some bundle, of the nine (m: the lanes with one; lane 63 repeats another's pair).
__device__ __forceinline__ unsigned near_slots(unsigned long long m) {
  unsigned slots = 0;
#pragma unroll
  for (int b = 0; b < kSeg; ++b) slots |= (unsigned)(m >> (9 * b)) & 0x1ffu;
  return slots;
}

// Round i's near particles (m: the lanes with one) join the list.
__device__ __forceinline__ void near_found(unsigned long long m, const float4* tile, const float2* tlo, int i, int lane,
                                           NearList& list) {
  if (list.at.n > kNearList - 9) {
    if (list.at.first < 0 && !list.missed) list.at.round = i;
    list.missed = true;
    return;
  }
  const unsigned slots = near_slots(m);
  if (lane < 9 && (slots >> lane & 1)) {
    const int at = list.at.n + __popc(slots & ((1u << lane) - 1u));
    list.p[at] = tile[9 * i + lane];
    list.lo[at] = tlo[9 * i + lane];
  }
  list.at.n += __popc(slots);
}

// This wavefront's share of a tile, its rounds from `from` to `to`: plain FP32 moment sums; a guarded sum leaves near
// pairs out and then, where it met some, looks at its rounds again for the particles that are near for some bundle, which
// join the list.  (Looking while summing, every four rounds, kept the loads of the next rounds behind the branch: the halo
// band 13.8 ms, 13.2 so.  Summing each tile twice, with the near pairs in and then out, made the cost of one near
// pair that of a pass over its tile.)
template <bool EQUAL, bool GUARD>
__device__ __forceinline__ void tile_moments(const float4* tile, const float2* tlo, int from, int to, int l, int lane, float ex,
                                             float ey, float e2, float thr, float (&a)[kMom], NearList& list) {
  if constexpr (!GUARD) {
#pragma unroll 8
    for (int i = from; i < to; ++i) moment_terms<EQUAL, false>(tile[9 * i + l], tlo[9 * i + l], ex, ey, e2, thr, a);
  } else {
    unsigned long long some = 0;
    constexpr int U = 8;
    int i = from;
    for (; i + U <= to; i += U) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        some |= __ballot(moment_terms<EQUAL, true>(tile[9 * (i + u) + l], tlo[9 * (i + u) + l], ex, ey, e2, thr, a));
    }
#pragma unroll 1
    for (; i < to; ++i) some |= __ballot(moment_terms<EQUAL, true>(tile[9 * i + l], tlo[9 * i + l], ex, ey, e2, thr, a));
    if (some) {
#pragma unroll 1
      for (i = from; i < to; ++i) {
        const unsigned long long near = __ballot(near_pair<EQUAL>(tile[9 * i + l], tlo[9 * i + l], ex, ey, e2, thr));
        if (near) near_found(near, tile, tlo, i, lane, list);
      }
    }
  }
}

// A pointer that comes from memory is taken for a flat one, whose loads also wait on LDS: say where it points.
typedef float Vec4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) Vec4 GlobalFloat4;

// Stage one tile (the particles from base on, at least one): positions in the set's frame (two parts for x and y),
// z relative to the stage's z, and for equal masses z^2 + eps^2 in place of the mass.
// Padding past the end lies so far away that s overflows to +inf, whose
// reciprocal square root is +0.  zr_hi, zr_lo: the stage's z in two FP32 parts.
template <int TP, int NG, bool EQUAL>
__device__ __forceinline__ void stage_tile(const DevSet& s, int64_t base, float4* tile, float2* tlo, int g, int lane, float e2,
                                           float zr_hi, float zr_lo) {
  const GlobalFloat4* src = (const GlobalFloat4*)s.p32;
  const GlobalFloat4 *tsrc = src + base, *tsrc_lo = src + s.n + base;
  const int cnt = s.n - base < TP ? (int)(s.n - base) : TP;
  // (a few particles per lane at a time: their loads in flight together, then stored; one after
  // the other they took a seventh of a tile of 576)
  constexpr int kMine = (TP + NG * 64 - 1) / (NG * 64), kBatch = 3;
  const int j0 = g * 64 + lane;
#pragma unroll
  for (int k0 = 0; k0 < kMine; k0 += kBatch) {
    Vec4 p[kBatch], r[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
      if (k0 + b < kMine) {
        const int j = j0 + NG * 64 * (k0 + b), at = j < cnt ? j : cnt - 1;
        p[b] = tsrc[at];
        r[b] = tsrc_lo[at];
      }
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
      if (k0 + b < kMine) {
        const int j = j0 + NG * 64 * (k0 + b);
        const bool in = j < cnt;
        const float zs = (p[b].z - zr_hi) + (r[b].z - zr_lo);
        if (j < TP) {
          tile[j] = make_float4(in ? p[b].x : 1e30f, in ? p[b].y : 1e30f, in ? zs : 1e30f,
                                in ? (EQUAL ? fmaf(zs, zs, e2) : p[b].w) : (EQUAL ? __builtin_inff() : 0.f));
          tlo[j] = make_float2(in ? r[b].x : 0.f, in ? r[b].y : 0.f);
        }
      }
  }
}

// A value that all lanes share, in a scalar register (the FP64 state fills the vector ones, and what is
// spilled in the tile loop is reloaded for every tile).
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// The tiles of one set, walked by all wavefronts of the workgroup in the same
// number of rounds: in round it, the NG wavefronts of index q stage tile
// q + it WPR together and each sums it for its own bundles.
template <int TP, int WPR, int NG, bool EQUAL, bool GUARD>
__device__ __forceinline__ void moment_tiles(const DevSet& s, float4* tile, int q, int g, int lane, float ex, float ey, float thr,
                                             double zrel, float (&ks)[kMom], float (&kc)[kMom], NearList& list) {
  const int64_t n = s.n;
  const float e2 = s.eps2f;
  const int l = lane < kLanes ? lane % 9 : 0;
  const int64_t n_tiles = (n + TP - 1) / TP;
  const int64_t n_rounds = (n_tiles + WPR - 1) / WPR;
  float2* tlo = reinterpret_cast<float2*>(tile + TP);
  const float zr_hi = uniform((float)zrel), zr_lo = uniform((float)(zrel - (double)(float)zrel));
  // unguarded sums: plain FP32 over kKahanRounds rounds (whatever the tile size), then Kahan
  constexpr int kTilesPerKahan = (kKahanRounds * 9 + TP - 1) / TP;
  float acc[kMom];
#pragma unroll
  for (int k = 0; k < kMom; ++k) acc[k] = 0.f;
  int since = 0;
  for (int64_t it = 0; it < n_rounds; ++it) {
    const int64_t ch = q + it * WPR;
    const int64_t base = ch * TP;
    if (ch < n_tiles) stage_tile<TP, NG, EQUAL>(s, base, tile, tlo, g, lane, e2, zr_hi, zr_lo);
    __syncthreads();
    if (ch < n_tiles) {
      const int64_t left = n - base;
      // a set's last tile runs only over its particles
      const int rounds = left >= TP ? TP / 9 : (int)((left + 8) / 9);
      if constexpr (GUARD) {
        // (sums with near pairs hold larger terms: 256 plain rounds moved mu of the halo's bundles by 2.5e-7
        // against 1.0e-7, for 6% of time)
        for (int r0 = 0; r0 < rounds; r0 += kGuardRounds) {
          const int to = rounds - r0 < kGuardRounds ? rounds : r0 + kGuardRounds;
          tile_moments<EQUAL, true>(tile, tlo, r0, to, l, lane, ex, ey, e2, thr, acc, list);
#pragma unroll
          for (int k = 0; k < kMom; ++k) {
            kahan_add(ks[k], kc[k], acc[k]);
            acc[k] = 0.f;
          }
        }
        if (list.missed) {
          if (list.at.first < 0) list.at.first = (int)it;
          list.at.last = (int)it;
          list.missed = false;
        }
      } else {
        // plain sums over kKahanRounds rounds of the nine lanes, then one compensated add
        tile_moments<EQUAL, false>(tile, tlo, 0, rounds, l, lane, ex, ey, e2, thr, acc, list);
        if (++since >= kTilesPerKahan || ch + WPR >= n_tiles) {
#pragma unroll
          for (int k = 0; k < kMom; ++k) {
            kahan_add(ks[k], kc[k], acc[k]);
            acc[k] = 0.f;
          }
          since = 0;
        }
      }
    }
    __syncthreads();   // before the tile is staged again
  }
}

// The direct terms of the near pairs that did not fit a list, from tile round it0 to it1, where some
// wavefront of the workgroup has them; each looks at its own (mark).  The nine lanes of a bundle test nine
// particles at a time, as in the moment loop.  Bound: the tiles' staging and the test, about a third of a moment sum.
// (50000 particles, 129024 rays, 6 steps, lists full at every plane: 19.0 ms, 9.5 without near pairs.  A walk of every
// tile by every lane, one particle after the other, with the plane summed at both of its visits: 116.  A sum at every stage
// that walked the tiles of near pairs like that: 118.)
template <int TP, int WPR, int NG, bool EQUAL>
__device__ __forceinline__ void near_tiles(const DevSet& s, float4* tile, int q, int g, int lane, float ex, float ey, float thr,
                                           double dx, double dy, double dz, double zrel, int it0, int it1,
                                           const NearList::Mark& mark, double (&dir)[4]) {
  const int64_t n_tiles = (s.n + TP - 1) / TP;
  const float e2 = s.eps2f;
  const int l = lane < kLanes ? lane % 9 : 0;
  float2* tlo = reinterpret_cast<float2*>(tile + TP);
  const float zr_hi = uniform((float)zrel), zr_lo = uniform((float)(zrel - (double)(float)zrel));
  for (int it = it0; it <= it1; ++it) {
    const int64_t ch = q + (int64_t)it * WPR, base = ch * TP;
    if (ch < n_tiles) stage_tile<TP, NG, EQUAL>(s, base, tile, tlo, g, lane, e2, zr_hi, zr_lo);
    __syncthreads();
    if (ch < n_tiles && mark.first >= 0 && it >= mark.first && it <= mark.last) {
      const int rounds = s.n - base < TP ? (int)((s.n - base + 8) / 9) : TP / 9;
      constexpr int U = 4;   // rounds per look at their near lanes
      for (int i = it == mark.first ? mark.round : 0; i < rounds; i += U) {
        unsigned long long near[U], any = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int j = 9 * (i + u < rounds ? i + u : rounds - 1) + l;
          near[u] = __ballot(i + u < rounds && near_pair<EQUAL>(tile[j], tlo[j], ex, ey, e2, thr));
          any |= near[u];
        }
        if (any == 0) continue;
        // (a lane walks its own bundle's)
#pragma unroll 1
        for (int u = 0; u < U; ++u) {
          const unsigned long long m = u == 0 ? near[0] : (u == 1 ? near[1] : (u == 2 ? near[2] : near[3]));
          for (unsigned slots = (unsigned)(m >> (9 * lane_segment(lane))) & 0x1ffu; slots != 0; slots &= slots - 1) {
            const int j = 9 * (i + u) + __ffs(slots) - 1;
            near_direct<EQUAL>(tile[j], tlo[j], ex, ey, e2, dx, dy, dz, dir);
          }
        }
      }
    }
    __syncthreads();
  }
}

// A set of at most kSmallSet particles (point-mass lenses) is summed directly at
// every ray in FP64, with the particles read by every lane from the caller's
// array: a few FP64 pair terms per stage cost less than the moments'
// reduction, and are exact.  (Every wavefront of a workgroup takes this path for
// the same set, so it needs no barrier.)
__device__ __forceinline__ void small_set_fp64(const DevCosmo& c, const DevSet& s, double x, double y, double z,
                                               double& phi, double& gx, double& gy, double& gz);

// (Every device function on the trace path is inlined into its kernel: a large
// called function reaches its far blocks through long branches, and the
// compiler builds their targets in the register pair that holds the function's
// return address.)
//
// Planes.  RK4 visits two planes per step, each twice: the middle (its second and third
// stage) and the end (its fourth, and the next step's first).  The rays move by far less
// than a bundle's radius between the two visits, and the moments belong to the expansion
// point, not to the rays: the second visit assembles each ray's field from the first
// visit's totals (kept in LDS) at the ray's new offset, and sums the near pairs again from
// the list.  That halves the pair terms; the error stays that of the expansion, whose
// nearness test the new offsets have to pass.
//   * middle: the second visit keeps the first one's expansion points and runs if every
//     bundle's threshold still covers its offsets (otherwise it sums anew, about its own points);
//   * end: it runs only if its own expansion points and thresholds equal the kept ones
//     bit by bit, so that it gives what a sum from the start would give, and a trace resumed
//     at that node gives the same rays as one that went through.  Expansion points are
//     therefore anchors rounded to a grid of 1/8192 to 1/4096 of the softening (1.5e-5 Mpc for 71
//     kpc, where the anchors of the two visits differ by about 1e-8 Mpc), and thresholds are
//     rounded up to 5 bits of mantissa.
// Measured, against a sum at every stage: 28672 bundles x 2^20 particles x 8 steps 752 -> 435 ms,
// 16384 x 2^18 x 10 172 -> 97.5 ms (85.6 with the staging of stage_tile, the choice of split and fewer spills), 7168 bundles of a
// 1e5-particle halo x 8 33.4 -> 18.9 ms (13.5 with the near list filled in the moment loop and fewer spills).
// Next to no end plane of the 2^20 box's first 25 steps is summed twice (1.534e12 pairs counted, 51 planes
// hold 1.533e12), about one of ten further on; the error of mu against
// FP64 is that of before or lower (halo 1.0e-7 for 1.3e-7 at most, box 1.6e-7 for 1.6e-7).
struct PlaneCache {
  double z;
  float ex, ey, thr;
  int set = -1;       // index of the set, -1: nothing kept
  bool near_any = false;   // some wavefront of the workgroup has near pairs,
  bool near_lost = false;  // and more than its list holds
};
enum { VISIT_FIRST = 0, VISIT_MIDDLE = 1, VISIT_END = 2 };

// Field of one set at the lane's ray (FP32 pair terms).  The WPR wavefronts of
// a group hold the same rays and split the tiles; all wavefronts of the
// workgroup share the staged tiles.  The group's partial moments meet in LDS
// in a fixed order, so that every wavefront of the group gets identical
// results.  Every wavefront of the workgroup must call this for the same set.
// LEVEL: all rays are at height z (the trace kernel, whose work items are rays of one
// field); otherwise a wavefront with other heights than the workgroup's first sums every
// pair directly.
template <int NW, int WPR, int TP, bool LEVEL>
struct FieldEval32 {
  static constexpr int NG = NW / WPR;
  using L = Lds32<NW, WPR, TP>;

  __device__ __forceinline__ static void eval(const DevCosmo& c, const DevSet& s, int set_id, int visit, PlaneCache& kept,
                                              float4* lds, int g, int q, int lane, double x, double y, double z,
                                              double& phi, double& gx, double& gy, double& gz) {
    if (s.n <= kSmallSet) {
      small_set_fp64(c, s, x, y, z, phi, gx, gy, gz);
      kept.set = -1;
      return;
    }
    // positions in the set's frame (FP64); each bundle's expansion point is its
    // anchor rounded to the grid and to FP32
    const double X = x - s.org[0], Yv = y - s.org[1], Zl = z - s.org[2];
    const int seg = lane_segment(lane), anchor = 9 * seg;
    const double xa = __shfl(X, anchor), ya = __shfl(Yv, anchor);
    float ex = (float)(rint(xa * s.igrid) * s.grid), ey = (float)(rint(ya * s.igrid) * s.grid);
    if (s.grid == 0.0) {
      ex = (float)xa;
      ey = (float)ya;
    }
    double zwg = Zl, dz = 0.0;
    bool level = true;
    if constexpr (!LEVEL) {
      // tiles are staged with z relative to one height for the whole workgroup
      __shared__ double zshared;
      if (threadIdx.x == 0) zshared = Zl;
      __syncthreads();
      zwg = zshared;
      __syncthreads();
      dz = Zl - zwg;
      level = !__any(Zl != zwg);
    }
    // largest offset in the bundle -> nearness threshold on s
    const int l = lane < kLanes ? lane % 9 : 0;
    double dx, dy;
    float thr_min;
    auto offsets = [&](float px, float py) {
      dx = X - (double)px;
      dy = Yv - (double)py;
      const float fx = (float)dx, fy = (float)dy;
      float m2 = lane < kLanes ? fmaf(fx, fx, fy * fy) : 0.f;
#pragma unroll
      for (int off = 1; off < 9; off <<= 1) {
        const float o = __shfl(m2, (l + off < 9) ? lane + off : lane);
        m2 = fmaxf(m2, o);
      }
      m2 = __shfl(m2, anchor);
      thr_min = level ? fmaxf(kNearRatio2 * m2, kNearFloor2) : __builtin_inff();
    };
    bool again = false;
    if (LEVEL && visit == VISIT_MIDDLE) {
      offsets(kept.ex, kept.ey);
      again = __syncthreads_and(thr_min <= kept.thr);
    }
    // (points that the rays have left are no place to expand about: they would raise the threshold)
    if (!again) offsets(ex, ey);
    // rounded up to 5 bits of mantissa (a threshold that large that this overflows is infinite), and at least
    // eps^2, below which no pair lies and all thresholds are one
    float thr = fmaxf(__int_as_float((__float_as_int(thr_min) + 0x3ffff) & ~0x3ffff), s.eps2f);
    double* tot = reinterpret_cast<double*>(reinterpret_cast<char*>(lds) + L::kTotAt) + g * kMom * kSeg;   // [20][7]
    char* near_at = reinterpret_cast<char*>(lds) + L::kNearAt + (g * WPR + q) * kNearBytes;
    NearList list{reinterpret_cast<float4*>(near_at), reinterpret_cast<float2*>(near_at + kNearList * 16),
                  reinterpret_cast<NearList::Mark*>(near_at + kNearList * 24), {0, -1, 0, -1}, false};
    const bool equal = s.equal_mass && *s.equal_mass;
    char* area = reinterpret_cast<char*>(lds) + g * WPR * kRedBytes;
    float* red = reinterpret_cast<float*>(area);                                   // [WPR][20][64]
    double* dred = reinterpret_cast<double*>(area + WPR * kMom * 64 * 4);          // [WPR][4][64]
    if (LEVEL && visit == VISIT_END) {
      const bool same = __float_as_int(ex) == __float_as_int(kept.ex) && __float_as_int(ey) == __float_as_int(kept.ey) &&
                        __float_as_int(thr) == __float_as_int(kept.thr);
      again = __syncthreads_and(same);
    }
    if (again) {
      ex = kept.ex;
      ey = kept.ey;
      thr = kept.thr;
    } else {
      sum_set(s, equal, lds, g, q, lane, ex, ey, thr, zwg, list);
      if (lane == 0) *list.mark = list.at;
      kept.near_any = __syncthreads_or(list.at.n > 0);
      kept.near_lost = kept.near_any && __syncthreads_or(list.at.first >= 0);
      // ---- reduction over the nine lanes of each bundle and the group's wavefronts
      for (int t = q * 64 + lane; t < kMom * kSeg; t += WPR * 64) {
        const int k = t / kSeg, b = t - k * kSeg;
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < WPR; ++w)
#pragma unroll
          for (int j = 0; j < 9; ++j) acc += (double)red[(w * kMom + k) * 64 + 9 * b + j];
        tot[t] = acc;
      }
      __syncthreads();
      kept.z = z;
      kept.ex = ex;
      kept.ey = ey;
      kept.thr = thr;
      kept.set = set_id;
    }
    // the near pairs' direct terms of the lane's own ray, in the order of the sum
    if (kept.near_any) {
      double dir[4] = {0.0, 0.0, 0.0, 0.0};
      const NearList::Mark mark = *list.mark;   // (the same for the wavefront)
      list.at = NearList::Mark{__builtin_amdgcn_readfirstlane(mark.n), __builtin_amdgcn_readfirstlane(mark.first),
                               __builtin_amdgcn_readfirstlane(mark.round), __builtin_amdgcn_readfirstlane(mark.last)};
      if (equal) near_terms<true>(list, ex, ey, s.eps2f, thr, dx, dy, dz, dir);
      else near_terms<false>(list, ex, ey, s.eps2f, thr, dx, dy, dz, dir);
      if (kept.near_lost) {
        int it0 = list.at.first, it1 = list.at.last;
        const char* marks = reinterpret_cast<const char*>(lds) + L::kNearAt + kNearList * 24;
        for (int w = 0; w < NW; ++w) {
          const NearList::Mark m = *reinterpret_cast<const NearList::Mark*>(marks + w * kNearBytes);
          if (m.first >= 0) {
            it0 = it0 < 0 || m.first < it0 ? m.first : it0;
            it1 = m.last > it1 ? m.last : it1;
          }
        }
        it0 = __builtin_amdgcn_readfirstlane(it0);
        it1 = __builtin_amdgcn_readfirstlane(it1);
        float4* tile = lds + q * L::kTileElems;
        if (equal) near_tiles<TP, WPR, NG, true>(s, tile, q, g, lane, ex, ey, thr, dx, dy, dz, zwg, it0, it1, list.at, dir);
        else near_tiles<TP, WPR, NG, false>(s, tile, q, g, lane, ex, ey, thr, dx, dy, dz, zwg, it0, it1, list.at, dir);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) dred[(q * 4 + k) * 64 + lane] = dir[k];
      __syncthreads();
    }
    double M[kMom];
#pragma unroll
    for (int k = 0; k < kMom; ++k) M[k] = tot[k * kSeg + seg];
    double D0 = 0.0, D1 = 0.0, D2 = 0.0, D3 = 0.0;
    if (kept.near_any) {
#pragma unroll
      for (int w = 0; w < WPR; ++w) {
        D0 += dred[(w * 4 + 0) * 64 + lane];
        D1 += dred[(w * 4 + 1) * 64 + lane];
        D2 += dred[(w * 4 + 2) * 64 + lane];
        D3 += dred[(w * 4 + 3) * 64 + lane];
      }
    }
    __syncthreads();   // before the tiles are staged again
    // ---- the lane's own field from the moments (FP64)
    const double d2 = dx * dx + dy * dy;
    const double Tx = M[M_TXX] * dx + M[M_TXY] * dy;
    const double Ty = M[M_TXY] * dx + M[M_TYY] * dy;
    const double Tz = M[M_TZX] * dx + M[M_TZY] * dy;
    const double Vd = M[M_VX] * dx + M[M_VY] * dy;
    const double xx = dx * dx, xy = 2.0 * dx * dy, yy = dy * dy;
    const double Ux = M[M_UXXX] * xx + M[M_UXXY] * xy + M[M_UXYY] * yy;
    const double Uy = M[M_UXXY] * xx + M[M_UXYY] * xy + M[M_UYYY] * yy;
    const double Uz = M[M_UZXX] * xx + M[M_UZXY] * xy + M[M_UZYY] * yy;
    const double W = M[M_W];
    const double S0 = M[M_PHI] + M[M_GX] * dx + M[M_GY] * dy - 0.5 * d2 * W + 1.5 * (dx * Tx + dy * Ty) + D0;
    const double Sx = M[M_GX] + 3.0 * Tx - W * dx - 1.5 * d2 * M[M_VX] - 3.0 * dx * Vd + 7.5 * Ux + D1;
    const double Sy = M[M_GY] + 3.0 * Ty - W * dy - 1.5 * d2 * M[M_VY] - 3.0 * dy * Vd + 7.5 * Uy + D2;
    const double Sz = M[M_GZ] + 3.0 * Tz - 1.5 * d2 * M[M_VZ] + 7.5 * Uz + D3;
    // the FP32 copy holds masses in units of mref; the equal-mass loop sums unit masses
    const double gm = -c.G * (equal ? s.mass : s.mref);
    phi = gm * S0;
    gx = gm * Sx;
    gy = gm * Sy;
    gz = gm * Sz;
    if (s.background) {
      // the corners are split over the wavefronts that hold the same rays (48 logarithms and arctangents a ray
      // otherwise took longer than a small set's pairs)
      double u[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
      for (int corner = q; corner < 8; corner += WPR)
        cuboid_corner(s.lo, s.hi, corner, x, y, z, u[0], u[1], u[2], u[3]);
      if constexpr (WPR > 1) {
#pragma unroll
        for (int k = 0; k < 4; ++k) dred[(q * 4 + k) * 64 + lane] = u[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          u[k] = 0.0;
#pragma unroll
          for (int w = 0; w < WPR; ++w) u[k] += dred[(w * 4 + k) * 64 + lane];
        }
        __syncthreads();   // before the tiles are staged again
      }
      phi += c.G_rho * u[0];
      gx += c.G_rho * u[1];
      gy += c.G_rho * u[2];
      gz += c.G_rho * u[3];
    }
  }

  // The wavefront's share of the moments, left in its part of the reduction area.
  __device__ __forceinline__ static void sum_set(const DevSet& s, bool equal, float4* lds, int g, int q, int lane, float ex,
                                                 float ey, float thr, double zwg, NearList& list) {
    // Every pair has s >= eps^2: if no bundle's threshold exceeds it, no pair can
    // be near and the unguarded loop runs.
    const bool guard = __any(thr > s.eps2f);
    float ks[kMom], kc[kMom];
#pragma unroll
    for (int k = 0; k < kMom; ++k) ks[k] = kc[k] = 0.f;
    float4* tile = lds + q * L::kTileElems;
    if (equal) {
      if (guard) moment_tiles<TP, WPR, NG, true, true>(s, tile, q, g, lane, ex, ey, thr, zwg, ks, kc, list);
      else moment_tiles<TP, WPR, NG, true, false>(s, tile, q, g, lane, ex, ey, thr, zwg, ks, kc, list);
    } else {
      if (guard) moment_tiles<TP, WPR, NG, false, true>(s, tile, q, g, lane, ex, ey, thr, zwg, ks, kc, list);
      else moment_tiles<TP, WPR, NG, false, false>(s, tile, q, g, lane, ex, ey, thr, zwg, ks, kc, list);
    }
    // (the tiles are free: moment_tiles ends with a barrier)
    float* red = reinterpret_cast<float*>(reinterpret_cast<char*>(lds) + g * WPR * kRedBytes);
#pragma unroll
    for (int k = 0; k < kMom; ++k) red[(q * kMom + k) * 64 + lane] = ks[k] - kc[k];
  }
};

// ===========================================================================
// FP64 field sums: the direct sum at each ray, tiles of the caller's FP64
// particles broadcast to every lane.
// ===========================================================================
// pair_fp64 with unit mass (sets of equal masses: the caller scales the sums).
__device__ __forceinline__ void pair_fp64_unit(const double4 c, double x, double y, double z, double e2,
                                               double& a0, double& a1, double& a2, double& a3) {
  const double ex = c.x - x, ey = c.y - y, ez = c.z - z;
  double r2 = fma(ex, ex, e2);
  r2 = fma(ey, ey, r2);
  r2 = fma(ez, ez, r2);
  const double ri = rsqrt_f64(r2);
  a0 += ri;
  const double r3 = ri * ri * ri;
  a1 = fma(r3, ex, a1);
  a2 = fma(r3, ey, a2);
  a3 = fma(r3, ez, a3);
}

__device__ __forceinline__ void small_set_fp64(const DevCosmo& c, const DevSet& s, double x, double y, double z,
                                               double& phi, double& gx, double& gy, double& gz) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  const int64_t n = s.n;
  const double* __restrict__ px = s.p64;
#pragma unroll 1
  for (int64_t j = 0; j < n; ++j)
    pair_fp64(make_double4(px[j], px[n + j], px[2 * n + j], px[3 * n + j]), x, y, z, s.eps2, a0, a1, a2, a3);
  phi = -c.G * a0;
  gx = -c.G * a1;
  gy = -c.G * a2;
  gz = -c.G * a3;
  if (s.background) {
    double U, ux, uy, uz;
    cuboid_field(s.lo, s.hi, x, y, z, U, ux, uy, uz);
    phi += c.G_rho * U;
    gx += c.G_rho * ux;
    gy += c.G_rho * uy;
    gz += c.G_rho * uz;
  }
}

// UNIT: every mass equals s.mass, which multiplies the finished sums.
template <int T, int WPR, bool UNIT>
__device__ __forceinline__ void sum_fp64(const DevSet& s, double4* tile, int q, int lane, double x, double y,
                                         double z, double& S0, double& Sx, double& Sy, double& Sz) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  const int64_t n = s.n;
  const double e2 = s.eps2;
  const int64_t n_chunks = (n + T - 1) / T;
  const double* __restrict__ px = s.p64;
  for (int64_t ch = q; ch < n_chunks; ch += WPR) {
    const int64_t base = ch * T;
#pragma unroll
    for (int k = lane; k < T; k += 64) {
      const int64_t j = base + k;
      tile[k] = (j < n) ? make_double4(px[j], px[n + j], px[2 * n + j], px[3 * n + j])
                        : make_double4(1e100, 1e100, 1e100, 0.0);
    }
    wave_sync();
    const int64_t left = n - base;   // the set's last tile runs only over its particles
    if (left >= T) {
#pragma unroll 8
      for (int k = 0; k < T; ++k) {
        if constexpr (UNIT) pair_fp64_unit(tile[k], x, y, z, e2, a0, a1, a2, a3);
        else pair_fp64(tile[k], x, y, z, e2, a0, a1, a2, a3);
      }
    } else {
#pragma unroll 1
      for (int k = 0; k < (int)left; ++k) {
        if constexpr (UNIT) pair_fp64_unit(tile[k], x, y, z, e2, a0, a1, a2, a3);
        else pair_fp64(tile[k], x, y, z, e2, a0, a1, a2, a3);
      }
    }
    wave_sync();
  }
  const double m = UNIT ? s.mass : 1.0;
  S0 = m * a0;
  Sx = m * a1;
  Sy = m * a2;
  Sz = m * a3;
}

// Field of one set at the lane's point for a group of WPR wavefronts holding
// the same rays: each sums its share of the tiles and the shares meet in LDS
// in a fixed order, so every wavefront of the group gets identical results.
// UNIT selects the loop of sets whose masses are all equal; the caller picks it
// from the set's device flag.
template <int T, int WPR>
struct FieldEval64 {
  __device__ __forceinline__ static void eval(const DevCosmo& c, const DevSet& s, double4* tile, double* red, int q,
                                              int lane, double x, double y, double z, double& phi, double& gx,
                                              double& gy, double& gz) {
    double S0, Sx, Sy, Sz;
    if (s.equal_mass && *s.equal_mass)
      sum_fp64<T, WPR, true>(s, tile, q, lane, x, y, z, S0, Sx, Sy, Sz);
    else
      sum_fp64<T, WPR, false>(s, tile, q, lane, x, y, z, S0, Sx, Sy, Sz);
    if constexpr (WPR > 1) {
      // red: [WPR][4][64] for this group
      red[(q * 4 + 0) * 64 + lane] = S0;
      red[(q * 4 + 1) * 64 + lane] = Sx;
      red[(q * 4 + 2) * 64 + lane] = Sy;
      red[(q * 4 + 3) * 64 + lane] = Sz;
      __syncthreads();
      S0 = Sx = Sy = Sz = 0.0;
#pragma unroll
      for (int w = 0; w < WPR; ++w) {
        S0 += red[(w * 4 + 0) * 64 + lane];
        Sx += red[(w * 4 + 1) * 64 + lane];
        Sy += red[(w * 4 + 2) * 64 + lane];
        Sz += red[(w * 4 + 3) * 64 + lane];
      }
      __syncthreads();
    }
    phi = -c.G * S0;
    gx = -c.G * Sx;
    gy = -c.G * Sy;
    gz = -c.G * Sz;
    if (s.background) {
      double U, ux, uy, uz;
      cuboid_field(s.lo, s.hi, x, y, z, U, ux, uy, uz);
      phi += c.G_rho * U;
      gx += c.G_rho * ux;
      gy += c.G_rho * uy;
      gz += c.G_rho * uz;
    }
  }
};

// ---------------------------------------------------------------------------
// The persistent trace kernel.
// NW wavefronts per workgroup; WPR of them share 63 rays (7 bundles) and split
// the particles; T particles per tile; OCC wavefronts per SIMD requested (the
// register budget is 512 / OCC per lane).
// ---------------------------------------------------------------------------
template <bool F64, int NW, int WPR, int T, int OCC>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(OCC, OCC))) void trace_kernel(TraceParams P) {
  constexpr int NG = NW / WPR;
  // FP64: a tile per wavefront; FP32: workgroup tiles (Lds32)
  __shared__ double4 tiles64[F64 ? NW : 1][F64 ? T : 1];
  __shared__ double red_own[NG][(F64 && WPR > 1) ? WPR * 4 * 64 : 1];
  __shared__ float4 lds32[Lds32Elems<F64, NW, WPR, T>::v];
  __shared__ int s_item;

  // the wavefront index is uniform: keep it (and the tile loop counters) in SGPRs
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = wave / WPR, q = wave % WPR;
  const DevCosmo& cz = P.cosmo;

  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = s_item;
    __syncthreads();
    if (item >= P.n_items) break;

    const WorkItem wi = P.items[item];
    const DevField f = P.fields[wi.field];
    const int64_t rend = f.ray_begin + f.n_rays;
    int64_t ri = f.ray_begin + (int64_t)wi.block * (kLanes * NG) + g * kLanes + (lane < kLanes ? lane : kLanes - 1);
    const bool valid = lane < kLanes && ri < rend;
    if (ri >= rend) ri = rend - 1;
    const int64_t N = P.n_rays;
    State Y{P.rays[ri], P.rays[N + ri], P.rays[2 * N + ri], P.rays[4 * N + ri], P.rays[5 * N + ri],
            P.rays[6 * N + ri], P.rays[7 * N + ri]};
    double zpos = P.rays[3 * N + ri];
    uint8_t flag = 0;
    bool live = true;
    PlaneCache kept;
    const int sb = P.step_begin < 0 ? 0 : P.step_begin;
    const int se = P.step_end > f.n_steps ? f.n_steps : P.step_end;

    for (int s = sb; s < se; ++s) {
      const double Z0 = P.nodes[f.node_off + s], Z1 = P.nodes[f.node_off + s + 1];
      const double h = Z1 - Z0, hh = 0.5 * h;
      const int S = P.step_set[f.step_off + s];
      State acc{}, Ys{}, k;
      double psi;
#pragma unroll 1
      for (int stage = 0; stage < 4; ++stage) {
        const double xin = (stage == 0) ? Y.x : Ys.x, yin = (stage == 0) ? Y.y : Ys.y;
        const double zs = (stage == 0) ? Z0 : ((stage == 3) ? Z1 : Z0 + hh);
        double phi = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
        if (S >= 0) {
          const DevSet& set = P.sets[f.set_off + S];
          if constexpr (F64)
            FieldEval64<T, WPR>::eval(cz, set, tiles64[wave], &red_own[g][0], q, lane, xin, yin, zs, phi, gx, gy,
                                      gz);
          else
            FieldEval32<NW, WPR, T, true>::eval(
                cz, set, S, kept.set == S && kept.z == zs ? (stage == 2 ? VISIT_MIDDLE : VISIT_END) : VISIT_FIRST, kept,
                lds32, g, q, lane, xin, yin, zs, phi, gx, gy, gz);
        }
        const State& Yin = (stage == 0) ? Y : Ys;
        k = rhs(cz, Yin, phi, gx, gy, gz, psi);
        if (stage == 0) {
          if (fabs(psi) > 1e-2) flag |= 4;
          acc = k;
          Ys = axpy(Y, hh, k);
        } else if (stage == 1) {
          acc = axpy(acc, 2.0, k);
          Ys = axpy(Y, hh, k);
        } else if (stage == 2) {
          acc = axpy(acc, 2.0, k);
          Ys = axpy(Y, h, k);
        } else {
          acc = axpy(acc, 1.0, k);
        }
      }
      if (live) {
        const State Yn = axpy(Y, h / 6.0, acc);
        const bool finite = isfinite(Yn.t) && isfinite(Yn.x) && isfinite(Yn.y) && isfinite(Yn.kt) &&
                            isfinite(Yn.kx) && isfinite(Yn.ky) && isfinite(Yn.kz);
        if (!finite) {
          flag |= 1;
          live = false;
        } else if (!(Yn.kz > 0.0)) {
          flag |= 2;
          live = false;
        } else {
          Y = Yn;
          zpos = Z1;
        }
      }
    }
    if (valid) {
      P.rays[ri] = Y.t;
      P.rays[N + ri] = Y.x;
      P.rays[2 * N + ri] = Y.y;
      P.rays[3 * N + ri] = zpos;
      P.rays[4 * N + ri] = Y.kt;
      P.rays[5 * N + ri] = Y.kx;
      P.rays[6 * N + ri] = Y.ky;
      P.rays[7 * N + ri] = Y.kz;
      if (P.flags && flag) P.flags[ri] |= flag;
    }
  }
}

// Field at arbitrary points: one wavefront = 63 points, no particle split.
// Every group of 9 consecutive points is treated as a bundle: FP32 sums expand
// about the first point of the group (rounded to FP32), as the trace kernel
// does about a bundle's anchor, when the points of the workgroup share z
// (otherwise each point's sum is direct).  Wavefronts past the last point still
// take part in the workgroup's tile rounds, on a copy of the last point.
template <bool F64, int T>
__global__ __launch_bounds__(256) void field_eval_kernel(DevCosmo c, const DevSet* set_p, int64_t n,
                                                         const double* pts, double* phi, double* grad) {
  __shared__ double4 tiles64[F64 ? 4 : 1][F64 ? T : 1];
  __shared__ float4 lds32[Lds32Elems<F64, 4, 1, T>::v];
  // the wavefront index is uniform: keep it (and the tile loop counters) in SGPRs
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t w0 = ((int64_t)blockIdx.x * 4 + wave) * kLanes;
  int64_t i = w0 + (lane < kLanes ? lane : kLanes - 1);
  const bool valid = lane < kLanes && i < n;
  if (i >= n) i = n - 1;
  const DevSet set = *set_p;
  double p, gx, gy, gz;
  if constexpr (F64) {
    if (w0 >= n) return;   // whole wavefront idle (no workgroup barriers in this path)
    FieldEval64<T, 1>::eval(c, set, tiles64[wave], nullptr, 0, lane, pts[i], pts[n + i], pts[2 * n + i], p, gx, gy,
                            gz);
  } else {
    PlaneCache kept;
    FieldEval32<4, 1, T, false>::eval(c, set, 0, VISIT_FIRST, kept, lds32, wave, 0, lane, pts[i], pts[n + i],
                                      pts[2 * n + i], p, gx, gy, gz);
  }
  if (valid) {
    phi[i] = p;
    grad[i] = gx;
    grad[n + i] = gy;
    grad[2 * n + i] = gz;
  }
}

// ---------------------------------------------------------------------------
// Small kernels: queue reset, set frames, FP32 copies.
// ---------------------------------------------------------------------------
__global__ void reset_queue_kernel(int32_t* q) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *q = 0;
}

// Frame origin of each set: the cuboid centre for sets with a background,
// otherwise the first particle.
__global__ void prepare_sets_kernel(DevSet* sets, int32_t n_sets) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_sets) return;
  DevSet& s = sets[i];
  s.mass = (s.n > 0) ? s.p64[3 * s.n] : 0.0;
  s.mref = (s.mass != 0.0 && isfinite(s.mass)) ? s.mass : 1.0;
  // grid of the expansion points: the power of two in (softening / 8192, softening / 4096], none for a softening
  // outside FP32's range of such steps
  const double soft = sqrt(s.eps2);
  s.grid = soft > 1e-12 && soft < 1e12 ? ldexp(1.0, ilogb(soft) - 12) : 0.0;
  s.igrid = s.grid > 0.0 ? 1.0 / s.grid : 0.0;
  if (s.equal_mass) *s.equal_mass = 1;   // cleared by the FP32 conversion at the first other mass
  if (s.background) {
    for (int d = 0; d < 3; ++d) s.org[d] = 0.5 * (s.lo[d] + s.hi[d]);
  } else if (s.n > 0) {
    for (int d = 0; d < 3; ++d) s.org[d] = s.p64[d * s.n];
  } else {
    for (int d = 0; d < 3; ++d) s.org[d] = 0.0;
  }
}

// The FP32 copy: positions relative to the set's frame origin as an FP32 value
// and its FP32 rounding residual (so that the FP32 displacement from a ray is
// rounded once relative to the particle-ray distance, not to the particle's
// distance from the frame origin), masses in units of the set's first mass (1 if
// that is 0), which multiplies the finished sums, so that the moments' powers of
// 1/r stay inside the FP32 range for any mass scale.
__global__ void convert_set_kernel(const DevSet* set, const double* p64, float4* p32, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const double ox = set->org[0], oy = set->org[1], oz = set->org[2];
  const double m = p64[3 * n + j];
  if (p32) {   // (FP64 sets have no copy: only their masses are checked)
    const double x = p64[j] - ox, y = p64[n + j] - oy, z = p64[2 * n + j] - oz;
    const float xh = (float)x, yh = (float)y, zh = (float)z;
    p32[j] = make_float4(xh, yh, zh, (float)(m / set->mref));
    p32[n + j] = make_float4((float)(x - (double)xh), (float)(y - (double)yh), (float)(z - (double)zh), 0.f);
  }
  if (!(m == p64[3 * n])) *set->equal_mass = 0;   // (a NaN mass also takes the general path)
}

// ---------------------------------------------------------------------------
// Bundle construction (Sec. 3.1).
// ---------------------------------------------------------------------------
__constant__ double kRingCos[8] = {1.0, 0.70710678118654752440, 0.0, -0.70710678118654752440,
                                   -1.0, -0.70710678118654752440, 0.0, 0.70710678118654752440};
__constant__ double kRingSin[8] = {0.0, 0.70710678118654752440, 1.0, 0.70710678118654752440,
                                   0.0, -0.70710678118654752440, -1.0, -0.70710678118654752440};

// Potential at the observer of up to kObsFields sets, one row of workgroups per set: every
// lane sums its own particles (FP64, coalesced columns), each workgroup leaves one partial sum.
// Bound: one read of the particles (32 B each).  A field_eval_kernel launch has one lane
// per point, so that a single point left one workgroup to walk the set: rt_build_bundles of 512^2 bundles
// in front of 2^20 particles took 55.5 ms, and takes 54.5 us (38 us at the rate of a copy).
constexpr int kObsFields = 32;       // by value in the kernel's arguments (a table there needs no copy and no wait)
constexpr int kObsParts = 512;       // workgroups per set at most: two per compute unit
constexpr int kObsThreads = 256;
struct ObsSets {
  ObsSet s[kObsFields];
};

__global__ __launch_bounds__(kObsThreads) void observer_partial_kernel(ObsSets sets, double* part) {
  __shared__ double sh[kObsThreads / 64];
  const ObsSet& s = sets.s[blockIdx.y];
  const double* __restrict__ px = s.p64;
  const int64_t n = s.n, step = (int64_t)gridDim.x * kObsThreads;
  double acc = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * kObsThreads + threadIdx.x; j < n; j += step) {
    const double x = px[j], y = px[n + j], z = px[2 * n + j], m = px[3 * n + j];
    acc = fma(m, rsqrt_f64(fma(z, z, fma(y, y, fma(x, x, s.eps2)))), acc);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// The partial sums of a set in a fixed order, and its cuboid background, a corner to a lane (one after the other the
// eight were most of this kernel's 8 us).
__global__ __launch_bounds__(64) void observer_final_kernel(DevCosmo c, ObsSets sets, int n_part, const double* part,
                                                            double* phi) {
  const ObsSet& s = sets.s[blockIdx.x];
  double acc = 0.0;
  for (int k = threadIdx.x; k < n_part; k += 64) acc += part[(int64_t)blockIdx.x * n_part + k];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  double u[4] = {0.0, 0.0, 0.0, 0.0};
  if (s.background && threadIdx.x < 8) cuboid_corner(s.lo, s.hi, threadIdx.x, 0.0, 0.0, 0.0, u[0], u[1], u[2], u[3]);
#pragma unroll
  for (int off = 4; off > 0; off >>= 1) u[0] += __shfl_xor(u[0], off);
  if (threadIdx.x == 0) phi[blockIdx.x] = -c.G * acc + c.G_rho * u[0];
}

// One thread per ray; the bundles of [b0, b0 + nb_range) share the potential at the observer.
__global__ void bundles_kernel(DevCosmo c, const double* phi_obs, int64_t b0, int64_t nb_range, int64_t n_bundles,
                               const double* theta, double radius, double* rays) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 9 * nb_range) return;
  const int64_t b = b0 + i / 9;
  const int k = (int)(i % 9);
  double tx = theta[b], ty = theta[n_bundles + b];
  if (k > 0) {
    tx += radius * kRingCos[k - 1];
    ty += radius * kRingSin[k - 1];
  }
  double a0, inv_a0, adot0;
  scale_factor(c, 0.0, a0, inv_a0, adot0);
  const double ph = phi_obs ? *phi_obs : 0.0;
  const double E0 = 1.0 + 2.0 * ph / a0, F0 = a0 * a0 - 2.0 * a0 * ph;
  const double norm = sqrt(E0 / F0) / sqrt(tx * tx + ty * ty + 1.0);
  const int64_t N = 9 * n_bundles, r = 9 * b + k;
  rays[r] = 0.0;
  rays[N + r] = 0.0;
  rays[2 * N + r] = 0.0;
  rays[3 * N + r] = 0.0;
  rays[4 * N + r] = 1.0;
  rays[5 * N + r] = norm * tx;
  rays[6 * N + r] = norm * ty;
  rays[7 * N + r] = norm;
}

// ---------------------------------------------------------------------------
// Bundle reductions.  One thread per bundle; the workgroup's rays (9 per bundle, so a
// contiguous run of each coordinate) come through LDS, which turns the coalesced reads
// into one bundle per thread (stride 9 doubles: the 32 lanes of a pass fall in 32 different
// pairs of banks).  Bound: HBM, 144 B read per bundle (32 to 80 B written).  A lane per ray
// with segmented shuffle sums took 26 and 27 us for the 512^2 bundles of a map (the shuffles,
// 40 and 48 of them per wavefront, took longer than the reads); these take 9.7 and 10.1.
// ---------------------------------------------------------------------------
constexpr int kBundleThreads = 256;

__device__ __forceinline__ void load_bundle(const double* rays, int64_t nb, double (&dx)[9], double (&dy)[9]) {
  __shared__ double sx[9 * kBundleThreads], sy[9 * kBundleThreads];
  const int64_t N = 9 * nb, r0 = (int64_t)blockIdx.x * (9 * kBundleThreads);
  const int cnt = (int)(N - r0 < 9 * kBundleThreads ? N - r0 : 9 * kBundleThreads);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int i = k * kBundleThreads + threadIdx.x;
    if (i < cnt) {
      sx[i] = rays[N + r0 + i];
      sy[i] = rays[2 * N + r0 + i];
    }
  }
  __syncthreads();
  const int at = 9 * threadIdx.x < cnt ? 9 * threadIdx.x : 0;
  const double x0 = sx[at], y0 = sy[at];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    dx[k] = sx[at + k] - x0;
    dy[k] = sy[at + k] - y0;
  }
}

// Sec. 3.1, eq. lensmap, magnification: signed octagon area and least-squares Jacobian.
__global__ __launch_bounds__(kBundleThreads) void magnification_kernel(double chi_s, int64_t nb, double radius,
                                                                       const double* rays, double* mu, double* jac) {
  double dx[9], dy[9];
  load_bundle(rays, nb, dx, dy);
  const int64_t b = (int64_t)blockIdx.x * kBundleThreads + threadIdx.x;
  if (b >= nb) return;
  double area = 0.0, s11 = 0.0, s12 = 0.0, s21 = 0.0, s22 = 0.0;
#pragma unroll
  for (int k = 1; k < 9; ++k) {
    const int nx = k == 8 ? 1 : k + 1;
    area += 0.5 * (dx[k] * dy[nx] - dy[k] * dx[nx]);
    const double ux = radius * kRingCos[k - 1], uy = radius * kRingSin[k - 1];
    s11 += dx[k] * ux;
    s12 += dx[k] * uy;
    s21 += dy[k] * ux;
    s22 += dy[k] * uy;
  }
  const double hom = 2.0 * sqrt(2.0) * radius * radius * chi_s * chi_s;
  mu[b] = hom / area;
  if (jac) {
    const double nrm = 1.0 / (4.0 * radius * radius * chi_s);
    const double a11 = s11 * nrm, a12 = s12 * nrm, a21 = s21 * nrm, a22 = s22 * nrm;
    jac[b] = 1.0 - 0.5 * (a11 + a22);
    jac[nb + b] = 0.5 * (a22 - a11);
    jac[2 * nb + b] = -0.5 * (a12 + a21);
    jac[3 * nb + b] = 0.5 * (a21 - a12);
  }
}

// Bundle flexion (Sec. 6: flexion, the gradient of the shear, through ray
// bundles).  About the anchor, the ring offsets are
//   D_k = chi_s (r A e_k + 1/2 r^2 Dm(e_k, e_k)) + O(r^3),
// e_k = (cos 2 pi k / 8, sin 2 pi k / 8), Dm_ijl = d A_ij / d theta_l.  Over the
// eight ring rays the first- and third-order parts live in the harmonics 1 and
// 3 only, so the harmonics 0 and 2 hold Dm alone:
//   sum_k D_ik = 2 r^2 chi_s (Dm_i11 + Dm_i22),
//   sum_k D_ik cos 2 phi_k = r^2 chi_s (Dm_i11 - Dm_i22),
//   sum_k D_ik sin 2 phi_k = 2 r^2 chi_s Dm_i12
// (cos 2 phi_k and sin 2 phi_k are exactly 0 or +-1).  F = grad kappa and
// G = (d1 gamma1 - d2 gamma2, d2 gamma1 + d1 gamma2) with kappa, gamma read from
// A as in magnification_kernel.
__global__ __launch_bounds__(kBundleThreads) void flexion_kernel(double chi_s, int64_t nb, double radius,
                                                                 const double* rays, double* flex, double* dm) {
  double dx[9], dy[9];
  load_bundle(rays, nb, dx, dy);
  const int64_t b = (int64_t)blockIdx.x * kBundleThreads + threadIdx.x;
  if (b >= nb) return;
  double v0 = 0.0, v1 = 0.0;
#pragma unroll
  for (int k = 1; k < 9; ++k) {
    v0 += dx[k];
    v1 += dy[k];
  }
  // 2 phi_k = (k - 1) pi / 2 (mod 2 pi)
  const double v2 = (dx[1] - dx[3]) + (dx[5] - dx[7]), v3 = (dy[1] - dy[3]) + (dy[5] - dy[7]);
  const double v4 = (dx[2] - dx[4]) + (dx[6] - dx[8]), v5 = (dy[2] - dy[4]) + (dy[6] - dy[8]);
  const double u = 1.0 / (radius * radius * chi_s);
  const double tx = 0.5 * v0 * u, ty = 0.5 * v1 * u;   // Dm_x11 + Dm_x22, Dm_y11 + Dm_y22
  const double ex = v2 * u, ey = v3 * u;               // Dm_x11 - Dm_x22, Dm_y11 - Dm_y22
  const double d111 = 0.5 * (tx + ex), d122 = 0.5 * (tx - ex), d112 = 0.5 * v4 * u;
  const double d211 = 0.5 * (ty + ey), d222 = 0.5 * (ty - ey), d212 = 0.5 * v5 * u;
  // kappa = 1 - (A11 + A22) / 2, gamma1 = (A22 - A11) / 2, gamma2 = -(A12 + A21) / 2
  const double dk1 = -0.5 * (d111 + d212), dk2 = -0.5 * (d112 + d222);
  const double dg1_1 = 0.5 * (d212 - d111), dg1_2 = 0.5 * (d222 - d112);
  const double dg2_1 = -0.5 * (d112 + d211), dg2_2 = -0.5 * (d122 + d212);
  flex[b] = dk1;
  flex[nb + b] = dk2;
  flex[2 * nb + b] = dg1_1 - dg2_2;
  flex[3 * nb + b] = dg1_2 + dg2_1;
  if (dm) {
    dm[b] = d111;
    dm[nb + b] = d112;
    dm[2 * nb + b] = d122;
    dm[3 * nb + b] = d211;
    dm[4 * nb + b] = d212;
    dm[5 * nb + b] = d222;
  }
}

// ---------------------------------------------------------------------------
// Source-weighted histograms (Sec. 5.3, eq. weighthisto; the same weighting
// for the shear distribution of Sec. 5.4): every bundle with mu > 0 has
// weight 1/mu.  mode 0: value log10 mu, bins of width in mu; mode 1: value
// |gamma| from the Jacobian, bins of width in |gamma|.  Deterministic: every
// sum runs in a fixed order.
//
// Up to kHistParted bins: one pass.  Each workgroup owns a run of bundles and leaves its
// own bins and moments (hist_part_kernel); hist_join_kernel adds them up in the order of the
// workgroups.  Bound: latency and launches (the values are 8 to 24 B a bundle).
// More bins: one workgroup per bin reads everything (hist_bins_kernel, hist_final_kernel).
// That walk evaluated log10 of every bundle once per bin and the variance in one workgroup:
// 1.1 ms for 512^2 bundles and 200 bins, against 19 us; it stays where a workgroup's private
// bins no longer fit LDS beside each other.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double hist_value(int mode, const double* mu, const double* jac, int64_t n, int64_t i) {
  return mode == 0 ? log10(mu[i]) : hypot(jac[n + i], jac[2 * n + i]);
}

__device__ __forceinline__ int value_bin(double v, double lo, double hi, int nb) {
  if (v < lo) return -1;
  if (v >= hi) return nb;
  const double f = floor((v - lo) / (hi - lo) * nb);
  return f >= 1.0 ? (f < nb ? (int)f : nb - 1) : 0;   // (no number: the first bin.  The result is an index into LDS)
}

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int o = NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

constexpr int kHistParted = 1024;      // bins: four private copies in 32 KB of LDS
constexpr int kHistRow = 1024;         // bundles of a workgroup's round, four per lane
constexpr int kHistParts = 512;        // workgroups at most: two per compute unit
constexpr int kHistStats = 6;          // sum w, sum w v, second moment about the part's mean, n bad, under, over
constexpr int kHistScratch = 65536 + 8;   // doubles of scratch, whatever the bins

__host__ __device__ inline int hist_parts(int64_t n, int nb) {
  // (a quarter of a round each for up to 64 workgroups: 1000 bundles, 200 bins, 15.3 -> 12.3 us)
  const int64_t fit = kHistScratch / (nb + kHistStats), row = n <= 64 * (kHistRow / 4) ? kHistRow / 4 : kHistRow;
  const int64_t want = (n + row - 1) / row;
  const int64_t k = fit < kHistParts ? fit : kHistParts;
  return (int)(want < 1 ? 1 : (want < k ? want : k));
}

// Sum over the workgroup's 256 lanes, in a fixed order, for every lane.
__device__ __forceinline__ double sum256(double v, double* sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// bins[id] += w for the wavefront's 64 (id, w), id < 0 for none.  The lanes of equal id are
// found by ballots over the id's bits; the lowest of them adds the others' weights in lane
// order and alone touches the bin.  Few different ids, i.e. many lanes of one: a sum over the wavefront for each
// (1000 bundles in one bin: 29.9 -> 12.2 us a call).
__device__ __forceinline__ void wave_bin_add(double* bins, int id, double w, int bits) {
  const int lane = threadIdx.x & 63;
  unsigned long long same = __ballot(id >= 0);
  for (int b = 0; b < bits; ++b) {
    const bool one = (id >> b) & 1;
    const unsigned long long m = __ballot(one);
    same &= one ? m : ~m;
  }
  const bool leads = id >= 0 && (same & ((1ull << lane) - 1ull)) == 0;
  unsigned long long leaders = __ballot(leads);
  if (__popcll(leaders) <= 3) {
    for (; leaders != 0; leaders &= leaders - 1) {
      const int lead = __ffsll(leaders) - 1, its = __builtin_amdgcn_readlane(id, lead);
      double v = id == its ? w : 0.0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
      if (lane == lead) bins[its] += v;
    }
    wave_sync();
    return;
  }
  unsigned long long rest = leads ? same : 0ull;
  double sum = 0.0;
  while (__any(rest != 0)) {
    const double v = __shfl(w, rest ? __ffsll(rest) - 1 : lane);
    if (rest) {
      sum += v;
      rest &= rest - 1;
    }
  }
  if (leads) bins[id] += sum;
  wave_sync();
}

// part: [parts][nb] bin weights, then [parts][kHistStats].
__global__ __launch_bounds__(256) void hist_part_kernel(int64_t n, const double* mu, const double* jac, int mode,
                                                        int32_t nb, double lo, double hi, double* part) {
  __shared__ double bins[4 * kHistParted];
  __shared__ double sh[4];
  const int wave = threadIdx.x >> 6;
  int bits = 1;
  while ((1 << bits) < nb) ++bits;
  for (int i = threadIdx.x; i < 4 * nb; i += 256) bins[i] = 0.0;
  __syncthreads();
  const int64_t per = (((n + gridDim.x - 1) / gridDim.x + 255) / 256) * 256;
  const int64_t i0 = (int64_t)blockIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
  double sw = 0.0, swv = 0.0, m2 = 0.0, bad = 0.0, under = 0.0, over = 0.0;
  for (int64_t r0 = i0; r0 < i1; r0 += kHistRow) {
    double v[4], w[4], rw = 0.0, rwv = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = r0 + 256 * k + threadIdx.x;
      int id = -1;
      w[k] = v[k] = 0.0;
      if (r0 + 256 * k >= i1) continue;
      if (i < i1) {
        const double m = mu[i];
        if (m > 0.0) {
          const double val = hist_value(mode, mu, jac, n, i);
          w[k] = 1.0 / m;
          v[k] = mode == 0 ? m : val;
          rw += w[k];
          rwv += w[k] * v[k];
          const int b = value_bin(val, lo, hi, nb);
          under += b < 0 ? 1.0 : 0.0;
          over += b >= nb ? 1.0 : 0.0;
          id = b >= nb ? -1 : b;
        } else {
          bad += 1.0;
        }
      }
      wave_bin_add(bins + wave * nb, id, w[k], bits);
    }
    rw = sum256(rw, sh);
    rwv = sum256(rwv, sh);
    if (rw > 0.0) {
      const double mean = rwv / rw;
      double d2 = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (w[k] != 0.0) d2 += w[k] * (v[k] - mean) * (v[k] - mean);
      m2 += sum256(d2, sh);
      if (sw > 0.0) {   // the two parts' means meet
        const double d = mean - swv / sw;
        m2 += d * d * (sw / (sw + rw)) * rw;
      }
    }
    sw += rw;
    swv += rwv;
  }
  bad = sum256(bad, sh);
  under = sum256(under, sh);
  over = sum256(over, sh);
  for (int i = threadIdx.x; i < nb; i += 256)
    part[(int64_t)blockIdx.x * nb + i] = (bins[i] + bins[nb + i]) + (bins[2 * nb + i] + bins[3 * nb + i]);
  if (threadIdx.x == 0) {
    double* st = part + (int64_t)gridDim.x * nb + (int64_t)blockIdx.x * kHistStats;
    st[0] = sw;
    st[1] = swv;
    st[2] = m2;
    st[3] = bad;
    st[4] = under;
    st[5] = over;
  }
}

// Eight bins per workgroup, 32 lanes each; workgroup 0 also joins the moments.
__global__ __launch_bounds__(256) void hist_join_kernel(int parts, int mode, int32_t nb, double lo, double hi,
                                                        const double* part, double* pdf, double* moments) {
  __shared__ double sh[4];
  const double* st = part + (int64_t)parts * nb;
  double sw = 0.0;
  for (int k = threadIdx.x; k < parts; k += 256) sw += st[k * kHistStats];
  sw = sum256(sw, sh);
  const int bin = blockIdx.x * 8 + (threadIdx.x >> 5), sub = threadIdx.x & 31;
  double acc = 0.0;
  if (bin < nb)
    for (int k = sub; k < parts; k += 32) acc += part[(int64_t)k * nb + bin];
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (bin < nb && sub == 0) {
    const double e0 = lo + (hi - lo) * bin / nb, e1 = lo + (hi - lo) * (bin + 1) / nb;
    const double width = mode == 0 ? pow(10.0, e1) - pow(10.0, e0) : (hi - lo) / nb;
    pdf[bin] = sw > 0.0 ? acc / (sw * width) : 0.0;
  }
  if (blockIdx.x != 0) return;
  double swv = 0.0, bad = 0.0, under = 0.0, over = 0.0;
  for (int k = threadIdx.x; k < parts; k += 256) {
    swv += st[k * kHistStats + 1];
    bad += st[k * kHistStats + 3];
    under += st[k * kHistStats + 4];
    over += st[k * kHistStats + 5];
  }
  swv = sum256(swv, sh);
  bad = sum256(bad, sh);
  under = sum256(under, sh);
  over = sum256(over, sh);
  const double mean = sw > 0.0 ? swv / sw : 0.0;
  double var = 0.0;
  for (int k = threadIdx.x; k < parts; k += 256) {
    const double w = st[k * kHistStats];
    if (w > 0.0) {
      const double d = st[k * kHistStats + 1] / w - mean;
      var += st[k * kHistStats + 2] + w * d * d;
    }
  }
  var = sum256(var, sh);
  if (threadIdx.x == 0) {
    moments[0] = sw;
    moments[1] = mean;
    moments[2] = sw > 0.0 ? sqrt(var / sw) : 0.0;
    moments[3] = bad;
    moments[4] = under;
    moments[5] = over;
  }
}

// work layout: [n_bins] bin weights, then sum w, sum w v, n_bad, n_under, n_over.
__global__ __launch_bounds__(256) void hist_bins_kernel(int64_t n, const double* mu, const double* jac, int mode,
                                                        int32_t nb, double lo, double hi, double* work) {
  __shared__ double sh[256];
  const int bin = blockIdx.x;
  if (bin < nb) {
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
      const double m = mu[i];
      if (m > 0.0 && value_bin(hist_value(mode, mu, jac, n, i), lo, hi, nb) == bin) acc += 1.0 / m;
    }
    const double t = block_sum<256>(acc, sh);
    if (threadIdx.x == 0) work[bin] = t;
  } else {
    double sw = 0.0, swv = 0.0, bad = 0.0, under = 0.0, over = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
      const double m = mu[i];
      if (!(m > 0.0)) {
        bad += 1.0;
        continue;
      }
      const double w = 1.0 / m;
      const double v = hist_value(mode, mu, jac, n, i);
      sw += w;
      swv += w * (mode == 0 ? m : v);
      const int b = value_bin(v, lo, hi, nb);
      if (b < 0) under += 1.0;
      if (b >= nb) over += 1.0;
    }
    const double t0 = block_sum<256>(sw, sh), t1 = block_sum<256>(swv, sh), t2 = block_sum<256>(bad, sh);
    const double t3 = block_sum<256>(under, sh), t4 = block_sum<256>(over, sh);
    if (threadIdx.x == 0) {
      work[nb] = t0;
      work[nb + 1] = t1;
      work[nb + 2] = t2;
      work[nb + 3] = t3;
      work[nb + 4] = t4;
    }
  }
}

__global__ __launch_bounds__(256) void hist_final_kernel(int64_t n, const double* mu, const double* jac, int mode,
                                                         int32_t nb, double lo, double hi, const double* work,
                                                         double* pdf, double* moments) {
  __shared__ double sh[256];
  const double sw = work[nb];
  const double mean = sw > 0.0 ? work[nb + 1] / sw : 0.0;
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) {
    const double m = mu[i];
    if (m > 0.0) {
      const double v = mode == 0 ? m : hist_value(mode, mu, jac, n, i);
      acc += (1.0 / m) * (v - mean) * (v - mean);
    }
  }
  const double var = block_sum<256>(acc, sh);
  for (int i = threadIdx.x; i < nb; i += 256) {
    const double e0 = lo + (hi - lo) * i / nb, e1 = lo + (hi - lo) * (i + 1) / nb;
    const double width = mode == 0 ? pow(10.0, e1) - pow(10.0, e0) : (hi - lo) / nb;
    pdf[i] = sw > 0.0 ? work[i] / (sw * width) : 0.0;
  }
  if (threadIdx.x == 0) {
    moments[0] = sw;
    moments[1] = mean;
    moments[2] = sw > 0.0 ? sqrt(var / sw) : 0.0;
    moments[3] = work[nb + 2];
    moments[4] = work[nb + 3];
    moments[5] = work[nb + 4];
  }
}

// ---------------------------------------------------------------------------
// Plan table.
// ---------------------------------------------------------------------------
// FP32: the workgroup's tiles, its reduction area and what it keeps take at most 79 KB of LDS, so
// two workgroups of 8 wavefronts (four per SIMD, 128 registers) or three of 4
// (three per SIMD, 168 registers) fit a compute unit.
// rays != 0: trace_few_kernel with that many rays per workgroup, per_lane of them summed by a lane, and tiles of one chunk (FP64 sums, in
// the FP32 table too: there for launches whose sets are all summed in FP64 anyway).
struct PlanShape {
  int nw, wpr, tile, occ, rays, per_lane;
};
constexpr PlanShape kPlans32[] = {{8, 1, 576, 4, 0}, {8, 2, 576, 4, 0}, {8, 4, 576, 4, 0}, {8, 8, 288, 4, 0},
                                  {8, 1, 1152, 4, 0}, {8, 2, 1152, 4, 0}, {4, 1, 576, 3, 0}, {4, 4, 288, 3, 0},
                                  {8, 1, 2304, 4, 0}, {1, 1, 64, 2, 64, 1}, {8, 8, 288, 2, 0}};
constexpr PlanShape kPlans64[] = {{8, 1, 128, 4, 0}, {8, 2, 128, 4, 0}, {8, 4, 128, 4, 0},
                                  {8, 8, 64, 4, 0},  {4, 1, 128, 4, 0}, {4, 4, 128, 4, 0},
                                  {8, 8, 4096, 2, 2, 2}, {8, 8, 4096, 2, 8, 8}, {8, 8, 4096, 2, 16, 8},
                                  {8, 8, 4096, 2, 32, 8}, {1, 1, 64, 2, 64, 1}};
constexpr int kNumPlans32 = sizeof(kPlans32) / sizeof(kPlans32[0]);
constexpr int kNumPlans64 = sizeof(kPlans64) / sizeof(kPlans64[0]);

template <bool F64, int I>
struct PlanKernel {
  static constexpr PlanShape S = F64 ? kPlans64[I] : kPlans32[I];
  // the plan of few rays without a particle split has its kernel in a file of its own (launch_trace_ray)
  static constexpr bool kRay = S.rays > 0 && S.nw == 1;
  static_assert(!kRay || (S.rays == kRayPlanRays && S.tile == kRayPlanTile && S.per_lane == 1), "the kernel of launch_trace_ray");
  static auto kernel() {
    if constexpr (S.rays > 0) return &trace_few_kernel<S.rays, S.per_lane, S.nw, S.tile>;
    else return &trace_kernel<F64, S.nw, S.wpr, S.tile, S.occ>;
  }
  static const void* fn() {
    if constexpr (kRay) return trace_ray_fn();
    else return (const void*)kernel();
  }
  static hipError_t launch(const TraceParams& p, int grid, hipStream_t st) {
    if constexpr (kRay) return launch_trace_ray(p, grid, st);
    else {
      hipLaunchKernelGGL(kernel(), dim3(grid), dim3(S.nw * 64), 0, st, p);
      return hipGetLastError();
    }
  }
};

template <bool F64, int I = 0>
const void* plan_fn(int id) {
  constexpr int n = F64 ? kNumPlans64 : kNumPlans32;
  if constexpr (I + 1 < n) {
    if (id != I) return plan_fn<F64, I + 1>(id);
  }
  return PlanKernel<F64, I>::fn();
}

template <bool F64, int I = 0>
hipError_t plan_launch(int id, const TraceParams& p, int grid, hipStream_t st) {
  constexpr int n = F64 ? kNumPlans64 : kNumPlans32;
  if constexpr (I + 1 < n) {
    if (id != I) return plan_launch<F64, I + 1>(id, p, grid, st);
  }
  return PlanKernel<F64, I>::launch(p, grid, st);
}

}  // namespace

int plan_count(bool fp64) { return fp64 ? kNumPlans64 : kNumPlans32; }

rt_plan_info plan_info(bool fp64, int id) {
  const PlanShape s = fp64 ? kPlans64[id] : kPlans32[id];
  rt_plan_info r;
  r.waves_per_block = s.nw;
  r.waves_per_group = s.wpr;
  r.tile = s.tile;
  r.rays_per_block = s.rays > 0 ? s.rays : kLanes * s.nw / s.wpr;
  r.waves_per_simd = s.occ;
  return r;
}

bool plan_few(bool fp64, int id) { return (fp64 ? kPlans64[id] : kPlans32[id]).rays > 0; }

hipError_t plan_occupancy(bool fp64, int id, int* blocks_per_cu) {
  const PlanShape s = fp64 ? kPlans64[id] : kPlans32[id];
  const void* fn = fp64 ? plan_fn<true>(id) : plan_fn<false>(id);
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, s.nw * 64, 0);
}

hipError_t launch_trace(bool fp64, int id, const TraceParams& p, int grid, hipStream_t s) {
  return fp64 ? plan_launch<true>(id, p, grid, s) : plan_launch<false>(id, p, grid, s);
}

hipError_t launch_reset_queue(int32_t* q, hipStream_t s) {
  hipLaunchKernelGGL(reset_queue_kernel, dim3(1), dim3(64), 0, s, q);
  return hipGetLastError();
}

hipError_t launch_prepare_sets(DevSet* sets, int32_t n_sets, hipStream_t s) {
  if (n_sets <= 0) return hipSuccess;
  hipLaunchKernelGGL(prepare_sets_kernel, dim3((n_sets + 63) / 64), dim3(64), 0, s, sets, n_sets);
  return hipGetLastError();
}

hipError_t launch_convert_set(const DevSet* set_dev, const double* p64, float4* p32, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(convert_set_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, set_dev, p64, p32, n);
  return hipGetLastError();
}

hipError_t launch_bundles(DevCosmo c, const double* phi_obs, int64_t b0, int64_t nb_range, int64_t n_bundles,
                          const double* theta, double radius, double* rays, hipStream_t s) {
  if (nb_range <= 0) return hipSuccess;
  const int64_t n = 9 * nb_range;
  hipLaunchKernelGGL(bundles_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, c, phi_obs, b0, nb_range,
                     n_bundles, theta, radius, rays);
  return hipGetLastError();
}

int observer_max_fields() { return kObsFields; }

hipError_t launch_observer_phi(DevCosmo c, const ObsSet* sets, int n_sets, double* part, double* phi, hipStream_t s) {
  ObsSets tab{};
  int64_t n_max = 0;
  for (int i = 0; i < n_sets; ++i) {
    tab.s[i] = sets[i];
    n_max = n_max > sets[i].n ? n_max : sets[i].n;
  }
  // a few particles per lane before a second workgroup is worth its partial sum
  int64_t parts = (n_max + 4 * kObsThreads - 1) / (4 * kObsThreads);
  parts = parts < 1 ? 1 : (parts > kObsParts ? kObsParts : parts);
  hipLaunchKernelGGL(observer_partial_kernel, dim3((unsigned)parts, (unsigned)n_sets), dim3(kObsThreads), 0, s, tab,
                     part);
  hipLaunchKernelGGL(observer_final_kernel, dim3((unsigned)n_sets), dim3(64), 0, s, c, tab, (int)parts,
                     (const double*)part, phi);
  return hipGetLastError();
}

size_t histogram_scratch_doubles(int64_t n, int32_t n_bins) {
  return n_bins <= kHistParted ? (size_t)hist_parts(n, n_bins) * (n_bins + kHistStats) : (size_t)n_bins + 8;
}

size_t observer_part_doubles() { return (size_t)kObsFields * kObsParts; }

hipError_t launch_field_eval(DevCosmo c, const DevSet* set, bool fp64, int64_t n, const double* pts, double* phi,
                             double* grad, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned grid = (unsigned)((n + 4 * kLanes - 1) / (4 * kLanes));
  if (fp64)
    hipLaunchKernelGGL((field_eval_kernel<true, kPlans64[0].tile>), dim3(grid), dim3(256), 0, s, c, set, n, pts, phi,
                       grad);
  else
    hipLaunchKernelGGL((field_eval_kernel<false, kPlans32[0].tile>), dim3(grid), dim3(256), 0, s, c, set, n, pts,
                       phi, grad);
  return hipGetLastError();
}

hipError_t launch_magnification(double chi_s, int64_t nb, double radius, const double* rays, double* mu,
                                double* jac, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(magnification_kernel, dim3((unsigned)((nb + kBundleThreads - 1) / kBundleThreads)),
                     dim3(kBundleThreads), 0, s, chi_s, nb, radius,
                     rays, mu, jac);
  return hipGetLastError();
}

hipError_t launch_flexion(double chi_s, int64_t nb, double radius, const double* rays, double* flex, double* dm,
                          hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(flexion_kernel, dim3((unsigned)((nb + kBundleThreads - 1) / kBundleThreads)),
                     dim3(kBundleThreads), 0, s, chi_s, nb, radius, rays,
                     flex, dm);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch of the histogram entry point that allocates nothing
// (rt_mu_histogram_noalloc): the bin weights and the five sums of one call,
// for at most kNoAllocBins bins.  Each GPU holds its own copy of the array;
// host code uses the per-device address from hipGetSymbolAddress, never the
// array's name.
// ---------------------------------------------------------------------------
constexpr int kNoAllocBins = 65536;
static_assert(kHistScratch == kNoAllocBins + 8, "both histogram paths fit the scratch");
static __device__ __align__(256) double scratch[kNoAllocBins + 8];

hipError_t noalloc_scratch(double** out, int32_t* max_bins) {
  static std::mutex mu;
  static std::map<int, void*> addr;   // device -> address of its copy of scratch
  int dev;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    it = addr.emplace(dev, ptr).first;
  }
  *out = static_cast<double*>(it->second);
  *max_bins = kNoAllocBins;
  return hipSuccess;
}

hipError_t launch_histogram(int64_t n, const double* mu, const double* jac, int mode, int32_t n_bins, double lo,
                            double hi, double* pdf, double* moments, double* work, hipStream_t s) {
  if (n_bins <= kHistParted) {
    const int parts = hist_parts(n, n_bins);
    hipLaunchKernelGGL(hist_part_kernel, dim3(parts), dim3(256), 0, s, n, mu, jac, mode, n_bins, lo, hi, work);
    hipLaunchKernelGGL(hist_join_kernel, dim3((n_bins + 7) / 8), dim3(256), 0, s, parts, mode, n_bins, lo, hi,
                       (const double*)work, pdf, moments);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(hist_bins_kernel, dim3(n_bins + 1), dim3(256), 0, s, n, mu, jac, mode, n_bins, lo, hi, work);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(hist_final_kernel, dim3(1), dim3(256), 0, s, n, mu, jac, mode, n_bins, lo, hi, work, pdf,
                     moments);
  return hipGetLastError();
}

}  // namespace rt
