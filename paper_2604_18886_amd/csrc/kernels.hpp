// HIP kernels of the solver: coarsening (Algorithm 3), the brick stencil with
// T-junction ghosts (Section 3.1, Eq. 10), red-black Gauss-Seidel and the steps
// of the FAS-style cycle (Algorithm 4).
//
// Layout: a brick is 4x4x4 cells = one wavefront; lane m is the cell with
// local Morton index m.  Device brick ids are level-major: leaf bricks first
// (finest level first, Morton order inside a level), then inner bricks
// (finest level first, Morton order), so the bricks of one level form two
// contiguous ranges.  Per-brick arrays of 64 values are indexed
// brick * 64 + m; coefficient arrays hold [c | kx | ky | kz] per brick.
#pragma once

#include <type_traits>

#include "device.hpp"

namespace mfmg {

// One brick's topology in a single 64-byte record (one scalar load).
struct alignas(64) BrickMeta {
  int32_t nbr[6];    // >= 0 same-level brick, -1 wall, <= -2 coarser leaf (T)
  uint32_t flags;    // see kFlag*
  int32_t parent;    // parent brick, -1 at the coarsest stored level
  int32_t tplus;     // slot of plus-side T-face coefficients, -1 if none
  int32_t coord[3];  // brick coordinates at its level
  uint32_t act[2];   // active-cell mask (bit m: cell m has c != 0)
  int32_t level;     // cell level
  int32_t pad;
};
static_assert(sizeof(BrickMeta) == 64, "brick record must be 64 bytes");

// Face flags: bit d (d = 0..5) T-junction (coarser leaf beyond), bit 8 + d
// same-level neighbour is an inner brick, bit 16 + d domain wall.
constexpr uint32_t kFlagT = 0x3fu;
constexpr uint32_t kFlagInner = 0x3fu << 8;
constexpr uint32_t kFlagWall = 0x3fu << 16;

// Per brick: for each axis a, the parent brick's same-level neighbour on the
// brick's side of the parent along a (the parent's nbr[2 a + bit a of the
// brick's octant]); -1 where there is none or the brick has no parent.  The
// brick across face d of axis a has that brick as its parent when the face
// lies on the parent's face, and the brick's own parent otherwise.
struct alignas(16) ParentNbrs {
  int32_t across[3];
  int32_t pad;
};

struct Topo {
  uint32_t nlb;            // leaf bricks (device ids 0 .. nlb-1)
  uint32_t nb;             // all bricks
  const BrickMeta *meta;   // nb records
  const int32_t *child;    // 8 per brick (octant dx + 2 dy + 4 dz), -1 for leaves
  const ParentNbrs *pnb;   // nb entries (hierarchies only; null elsewhere)
};

// Bricks of one level: a leaf range followed by an inner range.
struct Range {
  uint32_t leaf_lo, n_leaf, inner_lo, n_inner;
  __device__ __forceinline__ uint32_t brick(uint32_t i) const {
    return i < n_leaf ? leaf_lo + i : inner_lo + (i - n_leaf);
  }
  __host__ __device__ uint32_t n() const { return n_leaf + n_inner; }
};

// Brick records are never written by a kernel that reads them: loading them
// through the constant address space lets a wave-uniform load be a scalar
// load even after the kernel has stored to other arrays.
__device__ __forceinline__ BrickMeta load_meta(const BrickMeta *meta, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ((const __attribute__((address_space(4))) BrickMeta *)meta)[b];
#else
  return meta[b];  // host pass: never executed
#endif
}

__device__ __forceinline__ ParentNbrs load_parent_nbrs(const ParentNbrs *pnb, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ((const __attribute__((address_space(4))) ParentNbrs *)pnb)[b];
#else
  return pnb[b];  // host pass: never executed
#endif
}

// The eight child bricks of an inner brick.
struct alignas(32) Children {
  int32_t id[8];
};
__device__ __forceinline__ Children load_children(const int32_t *child, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ((const __attribute__((address_space(4))) Children *)child)[b];
#else
  return ((const Children *)child)[b];  // host pass: never executed
#endif
}

__device__ __forceinline__ uint32_t wave_id() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}
__device__ __forceinline__ uint64_t act_mask(const BrickMeta &M) {
  return uint64_t(M.act[0]) | (uint64_t(M.act[1]) << 32);
}
__device__ __forceinline__ int octant_of(const BrickMeta &M) {
  return (M.coord[0] & 1) | ((M.coord[1] & 1) << 1) | ((M.coord[2] & 1) << 2);
}

// Coefficient arrays of one multigrid level: leaf bricks read CL values,
// inner bricks read CI values multiplied by iscale (FP16 inner coefficients
// are stored divided by the cell size of their level).
template <class V, class CL, class CI>
struct Coefs {
  const CL *leaf;
  const CI *inner;
  V iscale;
};

template <class V>
__device__ __forceinline__ V div_by(V a, V c) {
  if constexpr (std::is_same<V, float>::value) {
    return a * __builtin_amdgcn_rcpf(c);  // v_rcp_f32, 1 ulp: enough for a smoother
  } else {
    return a / c;
  }
}

// Coarse cell (local Morton index inside the coarse leaf brick J) seen from
// cell m of brick M across direction d at a T-junction: the coarse cell
// holding the fine position next to m, i.e. that position's global
// coordinates halved.  J's cells start at a multiple of 4 on every axis, so
// the local index is the halved coordinate modulo 4 and J's own record is
// not needed.
__device__ __forceinline__ int coarse_local(const BrickMeta &M, int m, int d) {
  int a = d >> 1;
  int s = (d & 1) ? 1 : -1;
  int loc[3] = {dev_cx(m), dev_cy(m), dev_cz(m)};
  int c[3];
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    int g = M.coord[ax] * 4 + loc[ax] + (ax == a ? s : 0);
    c[ax] = (g >> 1) & 3;
  }
  return dev_morton(c[0], c[1], c[2]);
}

// ---------------------------------------------------------------------------
// hierarchy build (the assembly is in face_kernels.hpp)
// ---------------------------------------------------------------------------
// The parent-neighbour table (ParentNbrs), one thread per brick.
__global__ void __launch_bounds__(kBlock) k_parent_nbrs(Topo T, ParentNbrs *out) {
  uint32_t b = blockIdx.x * kBlock + threadIdx.x;
  if (b >= T.nb) return;
  const BrickMeta &M = T.meta[b];
  ParentNbrs r;
  r.pad = 0;
  for (int a = 0; a < 3; ++a) {
    r.across[a] = -1;
    if (M.parent >= 0) {
      int side = (octant_of(M) >> a) & 1;
      r.across[a] = T.meta[M.parent].nbr[2 * a + side];
    }
  }
  out[b] = r;
}

// FP16 copy of an inner coefficient scaled to c / h_l (through FP32, round to
// nearest even).  A non-zero value that would land below FP16's normal range
// (2^-14) is stored as 2^-14 with its sign: a sliver face keeps a small
// positive coupling instead of vanishing, so no cell that is active in FP64
// gets a zero diagonal in the mixed-precision cycle.
__device__ __forceinline__ __half half_coef(double v) {
  __half q = __float2half_rn(float(v));
  if (v != 0.0 && fabsf(__half2float(q)) < 0x1p-14f)
    q = __float2half_rn(v < 0.0 ? -0x1p-14f : 0x1p-14f);
  return q;
}

// FP64 coefficients of brick b: the assembled leaves and the inner bricks of
// Algorithm 3 are in two arrays.
struct CoefPair {
  const double *leaf;
  double *inner;  // of brick nlb on
  uint32_t nlb;
  __device__ __forceinline__ const double *of(uint32_t b) const {
    return b < nlb ? leaf + uint64_t(b) * 256u : inner + uint64_t(b - nlb) * 256u;
  }
};

// One pass over the bricks of a level (levels in decreasing order): their
// active-cell masks (bit m set when c_m != 0), their FP32 or FP16 copies of
// the mixed cycle (c32, c16; null in FP64) and, by Algorithm 3, the
// coefficients of their parents' cells: one wave per brick, whose 8 sibling
// groups give 8 cells of its parent.  Bound by HBM: each coefficient is read
// once, in full lines, where one lane per parent cell read its 8 children 64
// bytes apart and the masks and copies took passes of their own (26.3M
// leaves: 1070 us for the three, 310 us in this pass).  The sums run in the children's
// order, one lane per parent cell and component, over values handed through
// LDS.
__global__ void __launch_bounds__(kBlock) k_coarsen(Range R, BrickMeta *meta, CoefPair K,
                                                    double alpha, float *c32, __half *c16) {
  __shared__ double lds[kWavesPerBlock][7][64];
  const uint32_t w = wave_id();
  const int m = threadIdx.x & (kWave - 1);
  const uint32_t i = blockIdx.x * kWavesPerBlock + w;
  if (i >= R.n()) return;
  const uint32_t b = R.brick(i);
  const BrickMeta &M = meta[b];
  const int32_t parent = M.parent;
  const int oct = octant_of(M);
  const double *src = K.of(b);
  double v[4];
#pragma unroll
  for (int comp = 0; comp < 4; ++comp) v[comp] = src[comp * 64 + m];
  const uint64_t mask = __ballot(v[0] != 0.0);
  if (c32 && b < K.nlb) {
#pragma unroll
    for (int comp = 0; comp < 4; ++comp) c32[uint64_t(b) * 256u + comp * 64 + m] = float(v[comp]);
  } else if (c16 && b >= K.nlb) {
    const double inv_h = ldexp(1.0, M.level);
#pragma unroll
    for (int comp = 0; comp < 4; ++comp)
      c16[uint64_t(b - K.nlb) * 256u + comp * 64 + m] = half_coef(v[comp] * inv_h);
  }
  if (m == 0) {
    meta[b].act[0] = uint32_t(mask);
    meta[b].act[1] = uint32_t(mask >> 32);
  }
  if (parent < 0) return;
  double(*s)[64] = lds[w];
#pragma unroll
  for (int comp = 0; comp < 4; ++comp) s[comp][m] = v[comp] / alpha;
#pragma unroll
  for (int a = 0; a < 3; ++a) s[4 + a][m] = -v[1 + a];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (m >= 32) return;
  const int q = m & 7, comp = m >> 3, base = q << 3;
  const uint32_t on = uint32_t(mask >> base) & 0xffu;
  double c = 0.0;
  if (comp == 0) {
    const double twice = 2.0 / alpha;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      if (!((on >> t) & 1u)) continue;
      c = c + s[0][base | t];
#pragma unroll
      for (int a = 0; a < 3; ++a)
        if (((t >> a) & 1) && ((on >> (t ^ (1 << a))) & 1u))
          c = fma(twice, s[4 + a][base | t], c);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (!((t >> (comp - 1)) & 1)) c = c + s[comp][base | t];
  }
  K.inner[uint64_t(uint32_t(parent) - K.nlb) * 256u + uint32_t(comp * 64 + oct * 8 + q)] = c;
}

// Number of active leaf cells (added to *n, which is zero before).
__global__ void __launch_bounds__(256) k_count_active(const BrickMeta *meta, uint32_t nlb,
                                                      unsigned long long *n) {
  __shared__ unsigned long long part[4];
  unsigned long long c = 0;
  for (uint32_t b = blockIdx.x * 256u + threadIdx.x; b < nlb; b += gridDim.x * 256u)
    c += uint32_t(__popc(meta[b].act[0]) + __popc(meta[b].act[1]));
  c = wave_sum(c);
  if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(n, part[0] + part[1] + part[2] + part[3]);
}

// Plus-face coefficients of every brick, for the level kernels: entry
// a * 16 + f is the coefficient of the face between the brick's cell on its
// +a side with face index f and what lies beyond it -- the same-level
// neighbour's k_a (in mixed precision rounded exactly as the neighbour's own
// coefficients are stored), or the T-face coefficient K_F.  At a +a domain
// wall it is the part of the cell's diagonal not carried by its other five
// faces (the wall's coefficient; 0 at a Neumann wall), so that for every cell
// the diagonal is the sum of the six face coefficients the stencil sees
// (Eq. 3; Algorithm 3 keeps this on every level).  A cell on several +walls
// carries that part on the first of them.
// pf32 (may be null): the mixed cycle's copy, with the rounding of an inner
// neighbour's store.
// The composite operator reads the same entries on leaf bricks, except next to
// an inner brick: the coarse side of a T-junction carries the fine sub-face
// coefficients' sum over 2, Algorithm 3's coefficient their sum over alpha.
// OTHER (alpha != 2; forming both in one kernel for every alpha took 292 us at
// 26.3M leaves where this one without takes 217): pfa takes the
// operator's entries, ratio = alpha / 2 times Algorithm 3's there, on leaf
// bricks; it is pf64 where the cycle does not read that (mixed precision).
template <bool OTHER>
__global__ void __launch_bounds__(kBlock) k_plus_faces(Topo T, CoefPair K, const double *tc,
                                                       double *pf64, float *pf32, double *pfa,
                                                       double ratio) {
  uint32_t b = blockIdx.x * kWavesPerBlock + wave_id();
  int e = threadIdx.x & (kWave - 1);
  if (b >= T.nb || e >= 48) return;
  int a = e >> 4, f = e & 15;
  int c[3];
  c[a] = 3;
  c[a == 0 ? 1 : 0] = f & 3;
  c[a == 2 ? 1 : 2] = f >> 2;
  int m = dev_morton(c[0], c[1], c[2]);
  const BrickMeta M = T.meta[b];
  const double *own = K.of(b);
  double kp[3];
  bool wall[3];
  bool inner_nbr = false;
  uint32_t inner = 0u;  // OTHER: bit ax
  for (int ax = 0; ax < 3; ++ax) {
    int dd = 2 * ax + 1;
    kp[ax] = 0.0;
    wall[ax] = false;
    int p = dev_partner(m, dd);
    if (!dev_outside(m, dd)) {
      kp[ax] = own[(1 + ax) * 64 + p];
      continue;
    }
    int32_t n = M.nbr[dd];
    if (n >= 0) {
      kp[ax] = K.of(uint32_t(n))[(1 + ax) * 64 + p];
      if (ax == a) inner_nbr = uint32_t(n) >= T.nlb;
      if (OTHER && uint32_t(n) >= T.nlb) inner |= 1u << ax;
    } else if ((M.flags >> dd) & 1u) {
      kp[ax] = tc[uint32_t(M.tplus) * 48u + ax * 16 + dev_face_index(m, ax)];
    } else {
      wall[ax] = true;
    }
  }
  double v = kp[a];
  if (wall[a]) {
    int first = wall[0] ? 0 : (wall[1] ? 1 : 2);
    v = first == a ? own[m] - (own[64 + m] + own[128 + m] + own[192 + m]) -
                         (kp[0] + kp[1] + kp[2])
                   : 0.0;
  }
  if (!OTHER || pf64 != pfa) pf64[b * 48u + e] = v;
  if constexpr (OTHER) {
    double sum = 0.0;
    for (int ax = 0; ax < 3; ++ax) {
      if ((inner >> ax) & 1u) kp[ax] = ratio * kp[ax];
      sum = sum + kp[ax];
    }
    double va = kp[a];
    if (wall[a]) {
      int first = wall[0] ? 0 : (wall[1] ? 1 : 2);
      va = first == a ? own[m] - (own[64 + m] + own[128 + m] + own[192 + m]) - sum : 0.0;
    }
    if (b < T.nlb) pfa[b * 48u + e] = va;
  }
  if (!pf32) return;
  if (!wall[a] && inner_nbr) {
    float hv = __half2float(half_coef(v * ldexp(1.0, M.level)));
    v = double(hv * ldexpf(1.0f, -M.level));
  }
  pf32[b * 48u + e] = float(v);
}

// ---------------------------------------------------------------------------
// multigrid cycle kernels.  A wave processes one brick at a time and loops
// over the bricks of a level; everything that depends only on the lane is
// computed once, outside the loop, and every per-brick address is scalar
// arithmetic (buffer loads with a uniform base).
// ---------------------------------------------------------------------------
template <class V, class CL, class CI>
struct LevelArgs {
  Topo T;
  Coefs<V, CL, CI> cf;
  const CL *pf;      // plus-face coefficients, 48 per brick (k_plus_faces)
  V *U;              // iterate, nb * 64
  V *B;              // right-hand side, nb * 64 (leaf part: the PCG residual)
  V *Ustar;          // FAS initial guess of inner cells, (nb - nlb) * 64
  V pscale;          // transposed cycle: beta_mg / alpha
  Range R;
  const int *done;   // skip when the solve has stopped
};

// A voffset at or above this is out of range for every buffer the level
// kernels read (all are below 2 GiB): such a load returns 0.
constexpr uint32_t kOutOfRange = 0x80000000u;

// Lane constants: the lane's cell, its partners across the six directions,
// and the byte offsets the stencil's loads use.
template <class V, class CL>
struct LaneC {
  uint32_t m;        // local Morton index
  int p[6];          // partner cell across direction d (this brick or the next)
  bool out[6];       // the partner lies in the neighbouring brick
  uint32_t poff[6];  // out[d] ? p * sizeof(V) : kOutOfRange
  uint32_t foff[3];  // plus-face slot of the cell on axis a, in bytes
  int colour;        // (x + y + z) & 1
  int esrc[6];       // fused prolongation: lane holding the correction of the
                     // parent of the neighbour across d (prolong_gather)
  // FP64 only: gathered face loads of the full stencil (see stencil_sum)
  uint32_t goff[2];  // lane k < 48 of gather h: byte offset of its value in the brick
  int gdir[2];       //   across face 3h + k / 16 (that face; 6 for k >= 48)
  int gsrc[6];       // 4 x the lane holding the value across face d (gather d / 3)
  int psrc[6];       // 4 x p[d]
  uint32_t pfoff;    // lane k < 48: byte offset of plus-face entry k
  int pfsrc[3];      // 4 x the lane holding the lane's plus-face entry of axis a
};

template <class V, class CL>
__device__ __forceinline__ LaneC<V, CL> lane_consts() {
  LaneC<V, CL> L;
  L.m = threadIdx.x & (kWave - 1);
  int m = int(L.m);
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    L.p[d] = dev_partner(m, d);
    L.out[d] = dev_outside(m, d);
    L.poff[d] = L.out[d] ? uint32_t(L.p[d]) * uint32_t(sizeof(V)) : kOutOfRange;
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
    L.foff[a] = uint32_t(a * 16 + dev_face_index(m, a)) * uint32_t(sizeof(CL));
  L.colour = (dev_cx(m) + dev_cy(m) + dev_cz(m)) & 1;
#pragma unroll
  for (int d = 0; d < 6; ++d) L.esrc[d] = (L.out[d] ? 8 * (1 + d) : 0) + (L.p[d] >> 3);
  if constexpr (sizeof(V) == 8) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      L.gdir[h] = 6;
      L.goff[h] = kOutOfRange;
      if (m < 48) {
        int d = 3 * h + (m >> 4), a = d >> 1;
        int o0 = a == 0 ? 1 : 0;
        int o1 = a == 2 ? 1 : 2;
        int f = m & 15;
        int xyz[3];
        xyz[a] = (d & 1) ? 3 : 0;
        xyz[o0] = f & 3;
        xyz[o1] = f >> 2;
        L.gdir[h] = d;
        L.goff[h] = uint32_t(dev_partner(dev_morton(xyz[0], xyz[1], xyz[2]), d)) *
                    uint32_t(sizeof(V));
      }
    }
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      L.gsrc[d] = 4 * (16 * (d % 3) + dev_face_index(m, d >> 1));
      L.psrc[d] = 4 * L.p[d];
    }
    L.pfoff = m < 48 ? uint32_t(m) * uint32_t(sizeof(CL)) : kOutOfRange;
#pragma unroll
    for (int a = 0; a < 3; ++a) L.pfsrc[a] = 4 * (a * 16 + dev_face_index(m, a));
  }
  return L;
}

// Bricks of a level range for this wave.  Workgroups are dispatched to the
// eight XCDs in turn (workgroup g on XCD g mod 8); each XCD takes one
// contiguous eighth of the range, so bricks that are close in Morton order,
// and hence mostly each other's neighbours, share that XCD's L2.  The grid
// is a multiple of 8 workgroups.
struct WaveLoop {
  uint32_t first, end, step;
};
// The loop of workgroup `block` of a grid of `blocks` (a multiple of 8).
__device__ __forceinline__ WaveLoop wave_loop_of(uint32_t n, uint32_t block, uint32_t blocks) {
  uint32_t x = block & 7u;
  uint32_t j = (block >> 3) * kWavesPerBlock + wave_id();
  uint32_t chunk = (n + 7u) >> 3;
  uint32_t lo = x * chunk;
  uint32_t hi = lo + chunk < n ? lo + chunk : n;
  return {lo + j, hi, (blocks >> 3) * kWavesPerBlock};
}
__device__ __forceinline__ WaveLoop wave_loop(uint32_t n) {
  return wave_loop_of(n, blockIdx.x, gridDim.x);
}

// CP: cache policy of the loads whose data a launch uses once (coefficient
// arrays, plus-face table, right-hand side).  On a level larger than the
// Infinity Cache these are loaded non-temporal, so that the iterate -- the
// only array read again for neighbouring bricks -- keeps the L2; on smaller
// levels everything stays cached for the next half-sweep.  kCpolStreamCoef
// streams only the coefficients: the FP32 cycle's finest level then keeps
// its iterate, right-hand side and plus-face table (216 MB on the large
// workload) in the 256 MB Infinity Cache from one half-sweep to the next.
template <class V, class CL, class CI, int CP = kCpolDefault>
struct LevelView {
  __amdgpu_buffer_rsrc_t u, b, us, cl, ci, pf;
  const BrickMeta *meta;
  const ParentNbrs *pnb;
  uint32_t nlb;
  V iscale;
  V pscale;
};

template <int CP = kCpolDefault, class V, class CL, class CI>
__device__ __forceinline__ LevelView<V, CL, CI, CP> level_view(const LevelArgs<V, CL, CI> &A) {
  LevelView<V, CL, CI, CP> X;
  uint64_t nb = A.T.nb, nlb = A.T.nlb;
  X.u = make_rsrc(A.U, nb * 64 * sizeof(V));
  X.b = make_rsrc(A.B, nb * 64 * sizeof(V));
  X.us = make_rsrc(A.Ustar, (nb - nlb) * 64 * sizeof(V));
  X.cl = make_rsrc(A.cf.leaf, nlb * 256 * sizeof(CL));
  X.ci = make_rsrc(A.cf.inner, (nb - nlb) * 256 * sizeof(CI));
  X.pf = make_rsrc(A.pf, nb * 48 * sizeof(CL));
  X.meta = A.T.meta;
  X.pnb = A.T.pnb;
  X.nlb = A.T.nlb;
  X.iscale = A.cf.iscale;
  X.pscale = A.pscale;
  return X;
}

// Coefficient comp (0 = c, 1 + a = k_a) of the lane's cell of brick b;
// INNER selects the inner-brick array (FP16 in mixed precision, stored
// divided by the cell size).
template <bool INNER, class V, class CL, class CI, int CP>
__device__ __forceinline__ V own_coef(const LevelView<V, CL, CI, CP> &X, uint32_t b, int comp,
                                      uint32_t m) {
  if constexpr (INNER) {
    V v = V(bload<CI, coef_pol(CP)>(X.ci, m, (b - X.nlb) * 256u + uint32_t(comp) * 64u));
    if constexpr (std::is_same<CL, CI>::value) return v;
    else return v * X.iscale;
  } else {
    return V(bload<CL, coef_pol(CP)>(X.cl, m, b * 256u + uint32_t(comp) * 64u));
  }
}

template <class T, int CPOL = kCpolDefault>
__device__ __forceinline__ T bload_bytes(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(
        T, __builtin_amdgcn_raw_buffer_load_b64(r, int(voff), int(soff), CPOL));
  else if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(
        T, __builtin_amdgcn_raw_buffer_load_b32(r, int(voff), int(soff), CPOL));
  else
    return __builtin_bit_cast(
        T, __builtin_amdgcn_raw_buffer_load_b16(r, int(voff), int(soff), CPOL));
}

// Neighbour sum of the level operator at the lane's cell of brick b:
//   S_m = sum_d k_d v_d,   (A u)_m = c_m u_m - S_m,
// v_d the same-level neighbour value (a lane shuffle inside the brick, a
// load from the neighbouring brick across its faces), 0 at a wall, or at a
// T-junction (Eq. 10) the ghost u_m + (u_J - mean of the active siblings)/2
// with u_J read from the coarser leaf.  k_d is the cell's own k_a on the
// minus side and the neighbour's k_a on the plus side (a shuffle inside
// the brick, the brick's plus-face array across its faces).  The loads
// across a face are issued by every lane with an offset that is out of
// range for the inner lanes and, at a wall or T-face, for all lanes, so
// the only branch is a scalar one around the T-junction ghosts.  diag
// returns c_m as the sum of the six face coefficients (see k_plus_faces),
// so the diagonal is not streamed from memory.
// Values across the six faces of the lane's cell and their coefficients:
// v[d] the same-level neighbour's entry of the vector in buffer x (0 at a
// wall or T-face, where the load is out of range), k[d] the face
// coefficient (own k_a on the minus side, the neighbour's on the plus side).
template <int CP, class V, class CL>
__device__ __forceinline__ void face_values(__amdgpu_buffer_rsrc_t x, __amdgpu_buffer_rsrc_t pf,
                                            const LaneC<V, CL> &L, uint32_t b,
                                            const BrickMeta &M, V u, V k0, V k1, V k2, V (&v)[6],
                                            V (&k)[6]) {
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    int a = d >> 1;
    V kown = a == 0 ? k0 : (a == 1 ? k1 : k2);
    int32_t n = M.nbr[d];
    uint32_t sb = n >= 0 ? uint32_t(n) * uint32_t(64 * sizeof(V)) : kOutOfRange;
    V vl = bload_bytes<V>(x, L.poff[d] + sb, 0);
    V vs = shfl(u, L.p[d]);
    v[d] = L.out[d] ? vl : vs;
    if (d & 1) {
      V kl = V(bload_bytes<CL, side_pol(CP)>(pf, L.foff[a], b * uint32_t(48 * sizeof(CL))));
      V ks = shfl(kown, L.p[d]);
      k[d] = L.out[d] ? kl : ks;
    } else {
      k[d] = kown;
    }
  }
}

// FP64 form of face_values: the brick's 96 face cells take their values
// from two gathered loads (lane k < 48 of gather h fetches the value across
// face 3h + k / 16 for the face cell with face index k % 16) and its 48
// plus-face coefficients from one (lane k: entry k), each cell reading its
// entries by lane exchange.  The face loads of face_values are full-wave
// loads with only the face lanes in range; for 8-byte values the texture
// units' per-lane work on them, not HBM, bounded the stencils.
template <int CP, class V, class CL>
__device__ __forceinline__ void face_values_gathered(__amdgpu_buffer_rsrc_t x,
                                                     __amdgpu_buffer_rsrc_t pf,
                                                     const LaneC<V, CL> &L, uint32_t b,
                                                     const BrickMeta &M, V u, V k0, V k1, V k2,
                                                     V (&v)[6], V (&k)[6]) {
  uint32_t gb0 = 0u, gb1 = 0u;  // bytes to the brick across each gather's face
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    uint32_t sb = M.nbr[d] >= 0 ? uint32_t(M.nbr[d]) * uint32_t(64 * sizeof(V)) : kOutOfRange;
    gb0 = L.gdir[0] == d ? sb : gb0;
    gb1 = L.gdir[1] == d ? sb : gb1;
  }
  V g0 = bload_bytes<V>(x, L.goff[0] + gb0, 0);
  V g1 = bload_bytes<V>(x, L.goff[1] + gb1, 0);
  CL pfv = bload_bytes<CL, side_pol(CP)>(pf, L.pfoff, b * uint32_t(48 * sizeof(CL)));
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    int a = d >> 1;
    V kown = a == 0 ? k0 : (a == 1 ? k1 : k2);
    V vl = bperm(d < 3 ? g0 : g1, L.gsrc[d]);
    V vs = bperm(u, L.psrc[d]);
    v[d] = L.out[d] ? vl : vs;
    if (d & 1) {
      V kl = V(bperm(pfv, L.pfsrc[a]));
      V ks = bperm(kown, L.psrc[d]);
      k[d] = L.out[d] ? kl : ks;
    } else {
      k[d] = kown;
    }
  }
}

// The FAS correction u_P - u*_P of the parent cell of the lane's cell
// (Algorithm 4, prolongation): the brick covers octant o of its parent
// brick, whose cells o * 8 .. o * 8 + 7 are the parents of its 2^3 blocks.
// TR: in the transposed cycle it is pscale times the parent's iterate.
template <bool TR = false, class V, class CL, class CI, int CP>
__device__ __forceinline__ V own_correction(const LevelView<V, CL, CI, CP> &X,
                                            const LaneC<V, CL> &L, const BrickMeta &M) {
  uint32_t base = uint32_t(M.parent) * 64u + uint32_t(octant_of(M)) * 8u;
  uint32_t q = L.m >> 3;
  if constexpr (TR) return X.pscale * bload<V>(X.u, q, base);
  return bload<V>(X.u, q, base) - bload<V>(X.us, q, base - X.nlb * 64u);
}

// Prolongation folded into the first post-smoothing half-sweep of a level.
// Algorithm 4 adds u_P - u*_P to every active cell of the level before the
// post-smoothing; a colour-c half-sweep reads only the colour-c cells' own
// values and their neighbours, so it can add the corrections to what it
// reads instead, and store the corrected colour-c cells it updates.  The
// other colour's cells are left uncorrected in memory: the next half-sweep
// overwrites the active ones without reading their old values, except in
// the T-junction ghosts, where it adds the correction itself (mode 2 of
// smooth_brick).  Inactive cells are not corrected (as before); their face
// coefficients are zero, so a correction added to them changes no sum.
//
// The corrections one brick needs lie in at most seven parent octants: its
// own and those of the bricks across its six faces (octant o ^ (1 << a) of
// the same parent, or of the parent's neighbour when the face lies on the
// parent's face; ParentNbrs).  Lane k < 56 fetches entry k & 7 of octant
// slot k >> 3 (0: the brick's own, 1 + d: across face d) in one load of
// each vector; a face without a same-level brick beyond it (wall,
// T-junction) is out of range and gets a zero correction.  Each lane then
// takes the correction of its own parent cell from lane m >> 3 and that of
// its neighbour across face d (in the brick or beyond it) from lane
// L.esrc[d].
// TR as in own_correction.
template <bool TR = false, class V, class CL, class CI, int CP>
__device__ __forceinline__ V prolong_gather(const LevelView<V, CL, CI, CP> &X,
                                            const LaneC<V, CL> &L, const BrickMeta &M,
                                            const ParentNbrs &PN) {
  // every brick above the coarsest level has a parent
  const bool has_parent = M.parent >= 0;
  const uint32_t P = uint32_t(M.parent);
  const uint32_t o = uint32_t(octant_of(M));
  const uint32_t slot = L.m >> 3;
  uint32_t pb = P, oc = o;
  bool valid = slot == 0u;
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    const int a = d >> 1;
    const uint32_t bit = 1u << a;
    const bool across = ((o & bit) != 0u) == ((d & 1) != 0);
    const int32_t nb = across ? PN.across[a] : int32_t(P);
    if (slot == uint32_t(1 + d)) {
      pb = uint32_t(nb);
      oc = o ^ bit;
      valid = M.nbr[d] >= 0 && nb >= 0;
    }
  }
  valid = valid && has_parent;
  const uint32_t cell = pb * 64u + oc * 8u + (L.m & 7u);
  const uint32_t ou = valid ? cell * uint32_t(sizeof(V)) : kOutOfRange;
  if constexpr (TR) return X.pscale * bload_bytes<V>(X.u, ou, 0);
  const uint32_t os = valid ? (cell - X.nlb * 64u) * uint32_t(sizeof(V)) : kOutOfRange;
  return bload_bytes<V>(X.u, ou, 0) - bload_bytes<V>(X.us, os, 0);
}

// What a T-junction adds to the neighbour sum of the transposed level
// operator: (A^T u)_m = c_m u_m - S_m - E_m with
//   E_m = kT_m u_m - (1 / n) sum over the sibling group of (kT_i / 2) u_i,
// kT the cell's coefficients on T-faces and n the group's active cells (its
// values v[d] across T-faces are 0).  The coarse leaf's row takes its share
// from face_children_sum.  PR as in stencil_sum: the own values get the
// correction first.
template <int PR, class V, class CL, class CI, int CP>
__device__ __forceinline__ V t_rows_transposed(const LevelView<V, CL, CI, CP> &X,
                                               const LaneC<V, CL> &L, const BrickMeta &M, V u,
                                               const V (&k)[6], V corr, int colour) {
  if constexpr (PR == 1) u = u + shfl(corr, int(L.m >> 3));
  if constexpr (PR == 2) u = L.colour == colour ? u + own_correction<true>(X, L, M) : u;
  V kt = V(0);
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> d) & 1u) kt += L.out[d] ? k[d] : V(0);
  const V ktu = kt * u;
  const V s = group8_sum(ktu * V(0.5));
  const int cnt = __popcll((act_mask(M) >> (L.m & 56u)) & 0xffull);
  return cnt ? ktu - div_by(s, V(cnt)) : ktu;
}

// T-junction ghosts (Eq. 10) of a brick with T-faces: across each T-face d
// the lane's value becomes u_m + (u_J - mean of the active siblings) / 2,
// u_J read from the coarser leaf.  The coarse values of all T-faces are
// requested before any is used, so a brick with several T-faces waits for
// one round trip.  PR as in stencil_sum: the own values get the FAS
// correction first (1: corr from prolong_gather; 2: the not yet stored
// correction of the colour-`colour` cells).
template <int PR, class V, class CL, class CI, int CP>
__device__ __forceinline__ void t_ghosts(const LevelView<V, CL, CI, CP> &X, const LaneC<V, CL> &L,
                                         const BrickMeta &M, V u, V (&v)[6], V corr,
                                         int colour) {
  V uJ[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    uJ[d] = V(0);
    if ((M.flags >> d) & 1u) {
      uint32_t J = uint32_t(dev_decode_coarse(M.nbr[d]));
      uJ[d] = bload<V>(X.u, uint32_t(coarse_local(M, int(L.m), d)), J * 64u);
    }
  }
  uint64_t amask = act_mask(M);
  bool act = (amask >> L.m) & 1ull;
  if constexpr (PR == 1) {
    // every lane takes part in the exchange (a lane exchange in a
    // conditional would read inactive lanes)
    const V eo = shfl(corr, int(L.m >> 3));
    u = act ? u + eo : u;
  }
  if constexpr (PR == 2) u = act && L.colour == colour ? u + own_correction(X, L, M) : u;
  V s = group8_sum(act ? u : V(0));
  int cnt = __popcll((amask >> (L.m & 56u)) & 0xffull);
  V ubar = cnt ? s / V(cnt) : V(0);
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    if ((M.flags >> d) & 1u) {
      V g = u + (uJ[d] - ubar) * V(0.5);
      v[d] = L.out[d] ? g : v[d];
    }
  }
}

// PR: 0 the plain stencil; 1 the first post-smoothing half-sweep with the
// prolongation folded in (corr from prolong_gather: every neighbour value
// gets the correction of its parent cell, the T-junction ghosts use the
// corrected own and sibling values); 2 the half-sweep after it (the
// ghosts of the colour-`colour` cells add their own, not yet stored,
// correction).  TR: the neighbour sum of the transposed operator
// (t_rows_transposed in place of the ghosts).
template <int PR = 0, bool TR = false, class V, class CL, class CI, int CP>
__device__ __forceinline__ V stencil_sum(const LevelView<V, CL, CI, CP> &X, const LaneC<V, CL> &L,
                                         uint32_t b, const BrickMeta &M, V u, V k0, V k1,
                                         V k2, V &diag, V corr = V(0), int colour = 0) {
  V v[6], k[6];
  if constexpr (sizeof(V) == 8)
    face_values_gathered<CP>(X.u, X.pf, L, b, M, u, k0, k1, k2, v, k);
  else
    face_values<CP>(X.u, X.pf, L, b, M, u, k0, k1, k2, v, k);
  if constexpr (PR == 1) {
#pragma unroll
    for (int d = 0; d < 6; ++d) v[d] = v[d] + shfl(corr, L.esrc[d]);
  }
  V extra = V(0);  // TR only
  if (M.flags & kFlagT) {
    if constexpr (TR) {
      extra = t_rows_transposed<PR>(X, L, M, u, k, corr, colour);
    } else if constexpr (sizeof(V) == 8) {
      t_ghosts<PR>(X, L, M, u, v, corr, colour);
    } else {
      // FP32: the ghosts face by face (each coarse value waited for before
      // the next is requested); the hoisted form of t_ghosts made the
      // compiler schedule the whole FP32 stencil worse (finest half-sweep
      // 114 -> 119 us), while it speeds up the FP64 one
      uint64_t amask = act_mask(M);
      bool act = (amask >> L.m) & 1ull;
      if constexpr (PR == 1) {
        // every lane takes part in the exchange (a lane exchange in a
        // conditional would read inactive lanes)
        const V eo = shfl(corr, int(L.m >> 3));
        u = act ? u + eo : u;
      }
      if constexpr (PR == 2) u = act && L.colour == colour ? u + own_correction(X, L, M) : u;
      V s = group8_sum(act ? u : V(0));
      int cnt = __popcll((amask >> (L.m & 56u)) & 0xffull);
      V ubar = cnt ? s / V(cnt) : V(0);
#pragma unroll
      for (int d = 0; d < 6; ++d) {
        if ((M.flags >> d) & 1u) {
          uint32_t J = uint32_t(dev_decode_coarse(M.nbr[d]));
          V uJ = bload<V>(X.u, uint32_t(coarse_local(M, int(L.m), d)), J * 64u);
          V g = u + (uJ - ubar) * V(0.5);
          v[d] = L.out[d] ? g : v[d];
        }
      }
    }
  }
  diag = ((k[0] + k[1]) + (k[2] + k[3])) + (k[4] + k[5]);
  V acc = V(0);
#pragma unroll
  for (int d = 0; d < 6; ++d) acc += k[d] * v[d];
  if constexpr (TR) acc += extra;
  return acc;
}

// Transposed prolongation, right-hand side: the active cells of brick b take
// D = (handed-back residual of the parent cell) / (active siblings) into
// their right-hand side and, on inner bricks, into the residual they hand back
// themselves.  The handed-back residual is what the parent's level stored plus
// the parent cell's sum of k y over its faces to same-level leaves: those
// lie across the brick's own T-faces.  Their loads are requested before any
// is used.  Returns the new right-hand side of the lane's cell.
// Taken by the first half-sweep after the coarse visit together with the
// iterate's correction; finest level of the 26.3M-leaf workload, FP32: 177 us
// for that half-sweep (a plain one 95 us and a pass of its own 100 us, 190 us
// while the sums went through the parent's record), 2.3M leaves 17 against
// 9 + 10 us.
template <bool INNER, class V, class CL, class CI, int CP>
__device__ __forceinline__ V take_residual_T(const LevelView<V, CL, CI, CP> &X,
                                             const LaneC<V, CL> &L, uint32_t b,
                                             const BrickMeta &M, V rhs) {
  const uint32_t P = uint32_t(M.parent);
  const uint32_t oc = uint32_t(octant_of(M)) * 8u;
  const uint32_t q = L.m >> 3;
  V D = bload<V>(X.us, q, (P - X.nlb) * 64u + oc);
  V sb = V(0);
  if constexpr (INNER) sb = bload<V>(X.us, L.m, (b - X.nlb) * 64u);
  if (!INNER && (M.flags & kFlagT)) {  // (an inner brick has no T-face)
    const int pc = int(oc + q);
    V y[6], k[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      const int a = d >> 1;
      y[d] = V(0);
      k[d] = V(0);
      if ((M.flags >> d) & 1u) {
        const uint32_t out = dev_outside(pc, d) ? 0u : kOutOfRange;
        y[d] = bload_bytes<V>(X.u, out + uint32_t(dev_partner(pc, d)) * uint32_t(sizeof(V)),
                              uint32_t(dev_decode_coarse(M.nbr[d])) * uint32_t(64 * sizeof(V)));
        if (d & 1)
          k[d] = V(bload<CL>(X.pf, uint32_t(a * 16 + dev_face_index(pc, a)), P * 48u));
        else
          k[d] = V(bload<CI>(X.ci, uint32_t(pc), (P - X.nlb) * 256u + uint32_t(1 + a) * 64u));
      }
    }
#pragma unroll
    for (int d = 0; d < 6; ++d)
      if ((M.flags >> d) & 1u) {
        // (the parent's cell size is twice the level's)
        if (!(d & 1) && !std::is_same<CL, CI>::value) k[d] = k[d] * (X.iscale * V(2));
        D += k[d] * y[d];
      }
  }
  const uint64_t amask = act_mask(M);
  const int cnt = __popcll((amask >> (L.m & 56u)) & 0xffull);
  if ((amask >> L.m) & 1ull) {
    D = div_by(D, V(cnt));
    rhs = rhs + D;
    bstore<V>(X.b, L.m, b * 64u, rhs);
    if constexpr (INNER) bstore<V>(X.us, L.m, (b - X.nlb) * 64u, sb + D);
  }
  return rhs;
}

// One brick of a colour half-sweep of red-black Gauss-Seidel: on the cells
// of the colour u_m = (b_m + S_m) / c_m, every read taken before the write
// (the neighbours of a cell all have the other colour).  PR = 1: the first
// post-smoothing half-sweep with the prolongation folded in; PR = 2: the
// one after it (see prolong_gather).  TR: a half-sweep for A^T.
template <bool INNER, int PR, bool TR, class V, class CL, class CI, int CP>
__device__ __forceinline__ void smooth_brick(const LevelView<V, CL, CI, CP> &X, const LaneC<V, CL> &L,
                                             uint32_t b, int colour) {
  const BrickMeta M = load_meta(X.meta, b);
  V corr = V(0);
  if constexpr (PR == 1) corr = prolong_gather<TR>(X, L, M, load_parent_nbrs(X.pnb, b));
  V k0 = own_coef<INNER>(X, b, 1, L.m);
  V k1 = own_coef<INNER>(X, b, 2, L.m);
  V k2 = own_coef<INNER>(X, b, 3, L.m);
  V u = bload<V>(X.u, L.m, b * 64u);
  V rhs = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
  if constexpr (TR && PR == 1) rhs = take_residual_T<INNER>(X, L, b, M, rhs);
  V c;
  V S = stencil_sum<PR, TR>(X, L, b, M, u, k0, k1, k2, c, corr, colour);
  bool act = (act_mask(M) >> L.m) & 1ull;
  if (act && L.colour == colour) bstore<V>(X.u, L.m, b * 64u, div_by(rhs + S, c));
}

// Gathered face loads of an FP64 colour-c half-sweep.  The loads of the
// stencil are limited by the texture units' per-lane work, and the six face
// loads of stencil_sum are full-wave loads of which only the face lanes are
// in range.  The brick's colour-c cells on its six faces need 48 values from
// the neighbouring bricks (8 per face); lane k = 8 d + j (k < 48) fetches the
// one for the j-th such cell of face d in a single load and each cell takes
// its value from that lane with a lane exchange.  Likewise one load brings
// the brick's 48 plus-face coefficients (lane k: entry k).  A face's cells
// are numbered by their face index f (dev_face_index); cells f = 2j and
// 2j + 1 have opposite colours, and the colour-c one is the j-th.  (For FP32
// the exchanges cost more than the loads they save, and the six face loads
// stay.)
struct HalfGather {
  uint32_t goff;   // k < 48: byte offset of lane k's value in the brick across face k / 8
  int gdir;        // k / 8 for k < 48, 6 (no load) otherwise
  int gsrc[6];     // 4 x the lane holding the value across face d for the lane's cell
  int psrc[6];     // 4 x the lane's partner lane across direction d
  uint32_t pfoff;  // k < 48: byte offset of plus-face entry k, else out of range
  int pfsrc[3];    // 4 x the lane holding the lane's plus-face entry of axis a
};

template <class V, class CL>
__device__ __forceinline__ HalfGather half_gather(const LaneC<V, CL> &L, int colour) {
  HalfGather G;
  int k = int(L.m);
  G.gdir = k < 48 ? k >> 3 : 6;
  G.goff = kOutOfRange;
  if (k < 48) {
    int d = k >> 3, a = d >> 1;
    int o0 = a == 0 ? 1 : 0;
    int o1 = a == 2 ? 1 : 2;
    int side = (d & 1) ? 3 : 0;
    int f = 2 * (k & 7);
    if (((side + (f & 3) + (f >> 2)) & 1) != colour) f += 1;
    int xyz[3];
    xyz[a] = side;
    xyz[o0] = f & 3;
    xyz[o1] = f >> 2;
    int p = dev_partner(dev_morton(xyz[0], xyz[1], xyz[2]), d);
    G.goff = uint32_t(p) * uint32_t(sizeof(V));
  }
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    G.gsrc[d] = 4 * (8 * d + (dev_face_index(k, d >> 1) >> 1));
    G.psrc[d] = 4 * L.p[d];
  }
  G.pfoff = k < 48 ? uint32_t(k) * uint32_t(sizeof(CL)) : kOutOfRange;
#pragma unroll
  for (int a = 0; a < 3; ++a) G.pfsrc[a] = 4 * (a * 16 + dev_face_index(k, a));
  return G;
}

// One brick of a colour half-sweep with gathered face loads: the values,
// ghosts and sums of smooth_brick, term for term.
template <bool INNER, int PR, bool TR, class V, class CL, class CI, int CP>
__device__ __forceinline__ void smooth_brick_gathered(const LevelView<V, CL, CI, CP> &X,
                                                      const LaneC<V, CL> &L, const HalfGather &G,
                                                      uint32_t b, int colour) {
  const BrickMeta M = load_meta(X.meta, b);
  V k0 = own_coef<INNER>(X, b, 1, L.m);
  V k1 = own_coef<INNER>(X, b, 2, L.m);
  V k2 = own_coef<INNER>(X, b, 3, L.m);
  V u = bload<V>(X.u, L.m, b * 64u);
  V rhs = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
  const bool act = (act_mask(M) >> L.m) & 1ull;
  V corr = V(0);
  if constexpr (PR == 1) corr = prolong_gather<TR>(X, L, M, load_parent_nbrs(X.pnb, b));
  if constexpr (TR && PR == 1) rhs = take_residual_T<INNER>(X, L, b, M, rhs);
  uint32_t gb = 0u;  // byte offset of the brick across the lane's gather face
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    uint32_t sb = M.nbr[d] >= 0 ? uint32_t(M.nbr[d]) * uint32_t(64 * sizeof(V)) : kOutOfRange;
    gb = G.gdir == d ? sb : gb;
  }
  V gv = bload_bytes<V>(X.u, G.goff + gb, 0);
  CL pfv = bload_bytes<CL, side_pol(CP)>(X.pf, G.pfoff, b * uint32_t(48 * sizeof(CL)));
  V v[6], k[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    int a = d >> 1;
    V kown = a == 0 ? k0 : (a == 1 ? k1 : k2);
    V vl = bperm(gv, G.gsrc[d]);
    V vs = bperm(u, G.psrc[d]);
    v[d] = L.out[d] ? vl : vs;
    if constexpr (PR == 1) v[d] = v[d] + shfl(corr, L.esrc[d]);
    if (d & 1) {
      V kl = V(bperm(pfv, G.pfsrc[a]));
      V ks = bperm(kown, G.psrc[d]);
      k[d] = L.out[d] ? kl : ks;
    } else {
      k[d] = kown;
    }
  }
  V extra = V(0);  // TR only
  if (M.flags & kFlagT) {
    if constexpr (TR) extra = t_rows_transposed<PR>(X, L, M, u, k, corr, colour);
    else t_ghosts<PR>(X, L, M, u, v, corr, colour);
  }
  V c = ((k[0] + k[1]) + (k[2] + k[3])) + (k[4] + k[5]);
  V S = V(0);
#pragma unroll
  for (int d = 0; d < 6; ++d) S += k[d] * v[d];
  if constexpr (TR) S += extra;
  if (act && L.colour == colour) bstore<V>(X.u, L.m, b * 64u, div_by(rhs + S, c));
}

// PR: 0 a plain half-sweep, 1 the first post-smoothing half-sweep with the
// prolongation folded in, 2 the half-sweep after it (smooth_brick).  TR: a
// half-sweep of the transposed cycle.
template <class V, class CL, class CI, int CP = kCpolDefault, int PR = 0, bool TR = false>
__global__ void __launch_bounds__(kBlock) k_smooth(LevelArgs<V, CL, CI> A, int colour) {
  if (A.done && *A.done) return;
  if constexpr (sizeof(V) == 8) {
    const LaneC<V, CL> L = lane_consts<V, CL>();
    const HalfGather G = half_gather(L, colour);
    const LevelView<V, CL, CI, CP> X = level_view<CP>(A);
    const WaveLoop W = wave_loop(A.R.n());
    for (uint32_t i = W.first; i < W.end; i += W.step) {
      if (i < A.R.n_leaf) smooth_brick_gathered<false, PR, TR>(X, L, G, A.R.leaf_lo + i, colour);
      else smooth_brick_gathered<true, PR, TR>(X, L, G, A.R.inner_lo + (i - A.R.n_leaf), colour);
    }
  } else {
    const LaneC<V, CL> L = lane_consts<V, CL>();
    const LevelView<V, CL, CI, CP> X = level_view<CP>(A);
    const WaveLoop W = wave_loop(A.R.n());
    for (uint32_t i = W.first; i < W.end; i += W.step) {
      if (i < A.R.n_leaf) smooth_brick<false, PR, TR>(X, L, A.R.leaf_lo + i, colour);
      else smooth_brick<true, PR, TR>(X, L, A.R.inner_lo + (i - A.R.n_leaf), colour);
    }
  }
}

// ---------------------------------------------------------------------------
// reductions of small solves
// ---------------------------------------------------------------------------
// Small solves: the kernel that uses a reduction adds its n <= kFoldParts
// partials itself, every workgroup, in k_finish's order (the same bits), and
// the launch between them goes.  Mixed solves, us, without -> with: 32^3 (128
// partials) 558 -> 521, 0.15 M leaves (600) 1675 -> 1600, 64^3 (1024, the
// line) 889 -> 886.  More partials would cost every workgroup what the launch
// does.  n = 0: k_finish ran.  False: the solve has stopped (one read of the
// flag per workgroup, as another may set it meanwhile).
constexpr uint32_t kFoldParts = 1024;
__device__ __forceinline__ bool fold_total(const Scalars *S, const double *partials, uint32_t n,
                                           double &tot) {
  __shared__ double red[kFoldParts / kWave];
  __shared__ int stop;
  if (threadIdx.x == 0) stop = S->done;
  const uint32_t waves = blockDim.x / kWave;
  const uint32_t chunks = (n + kWave - 1) / kWave;
  for (uint32_t c = threadIdx.x / kWave; c < chunks; c += waves) {
    const uint32_t i = c * kWave + (threadIdx.x & (kWave - 1));
    const double v = wave_sum(i < n ? partials[i] : 0.0);
    if ((threadIdx.x & (kWave - 1)) == 0) red[c] = v;
  }
  __syncthreads();
  if (stop) return false;
  tot = 0.0;
  for (uint32_t c = 0; c < chunks; ++c) tot += red[c];
  return true;
}
__device__ __forceinline__ void finish_iteration(Scalars *S, double *hist, double tot) {
  S->xpend = 1;  // the residual update of this iteration is done
  S->rr = tot;
  S->iters += 1;
  hist[S->iters] = S->rr0 > 0.0 ? sqrt(tot / S->rr0) : 0.0;
  if (!(tot < INFINITY)) {
    S->status = -5;
    S->done = 1;
  } else if (tot <= S->tol2) {
    S->done = 1;
  }
}

// The stop test of an iteration in the first kernel of the cycle that follows:
// the n partials of ||r||^2 (0: k_finish ran, and S->done tells).  Mixed solves,
// us, k_finish's launch -> this: 16^3 483 -> 469, 32^3 513 -> 501, levels 5..6
// 1573 -> 1545, 64^3 (the line) 887 -> 885.
struct StopTest {
  Scalars *S;
  const double *partials;
  double *hist;
  int *host_done;
  uint32_t n;
};
// True: the solve has stopped.
__device__ __forceinline__ bool stop_test(const StopTest &T, const int *done) {
  if (!T.n) return done && *done;
  double tot;
  if (!fold_total(T.S, T.partials, T.n, tot)) return true;
  const bool stop = !(tot < INFINITY) || tot <= T.S->tol2;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    finish_iteration(T.S, T.hist, tot);
    if (stop && T.host_done)
      __hip_atomic_store(T.host_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  return stop;
}

// First half-sweep of a level from a zero iterate (the finest level; levels in
// correction form; the transposed cycle's first visits): every neighbour, ghost
// and wall value is 0, so u = b / c on the active
// cells of the colour, 0 on all others.  The diagonal is the sum of the six face
// coefficients, as in every half-sweep.  A leaf's stored one is that sum (and a
// third of the reads), except next to an inner brick: that face's coefficient is
// Algorithm 3's (half the fine sub-faces' sum for alpha = 2 only, in FP16 in the
// mixed cycle).  It also clears the iterate.  LONE: no leaf has such a neighbour.
template <bool INNER, bool LONE, class V, class CL, class CI, int CP>
__device__ __forceinline__ void first_sweep_brick(const LevelView<V, CL, CI, CP> &X,
                                             const LaneC<V, CL> &L, uint32_t b, int colour) {
  const BrickMeta M = load_meta(X.meta, b);
  bool act = (act_mask(M) >> L.m) & 1ull;
  if (!INNER && (LONE || !(M.flags & kFlagInner))) {
    V c = own_coef<false>(X, b, 0, L.m);
    V g = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
    bstore<V>(X.u, L.m, b * 64u, act && L.colour == colour ? div_by(g, c) : V(0));
    return;
  }
  V k[6];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    V kown = own_coef<INNER>(X, b, 1 + a, L.m);
    V kl = V(bload_bytes<CL, side_pol(CP)>(X.pf, L.foff[a], b * uint32_t(48 * sizeof(CL))));
    V ks = shfl(kown, L.p[2 * a + 1]);
    k[2 * a] = kown;
    k[2 * a + 1] = L.out[2 * a + 1] ? kl : ks;
  }
  V rhs = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
  V c = ((k[0] + k[1]) + (k[2] + k[3])) + (k[4] + k[5]);
  bstore<V>(X.u, L.m, b * 64u, act && L.colour == colour ? div_by(rhs, c) : V(0));
}

// clear: the iterate of the coarser levels' leaves starts from zero too (the
// finest level's leaves are the first bricks, theirs follow).  26.3M leaves,
// FP32: 44.8 us, against 41.3 and 10.8 in a launch of its own; 2.3M leaves 7.0
// against 6.3 + 4.6.
template <class V, class CL, class CI, int CP = kCpolDefault, bool LONE = true>
__global__ void __launch_bounds__(kBlock) k_first_sweep(LevelArgs<V, CL, CI> A, int colour,
                                                        int clear, StopTest T) {
  if (stop_test(T, A.done)) return;
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI, CP> X = level_view<CP>(A);
  const WaveLoop W = wave_loop(A.R.n());
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    if (i < A.R.n_leaf) first_sweep_brick<false, LONE>(X, L, A.R.leaf_lo + i, colour);
    else first_sweep_brick<true, LONE>(X, L, A.R.inner_lo + (i - A.R.n_leaf), colour);
  }
  if (clear) {
    const WaveLoop C = wave_loop(X.nlb - A.R.n_leaf);
    for (uint32_t i = C.first; i < C.end; i += C.step)
      bstore<V>(X.u, L.m, (A.R.n_leaf + i) * 64u, V(0));
  }
}

// Residual, restriction and FAS initial guess from one brick of level l to
// its parent cells:  b_P = beta_mg (1/alpha) sum_children r,
// u_P = u*_P = mean of the active children (k_fas_rhs then adds
// A^{l-1} u* on inner cells).  CORR: level l - 1 is in correction form, where
// the iterate is u - u*: u_P = u*_P = 0, and no k_fas_rhs follows.
template <bool INNER, bool CORR, class V, class CL, class CI, int CP>
__device__ __forceinline__ void restrict_brick(const LevelView<V, CL, CI, CP> &X,
                                               const LaneC<V, CL> &L,
                                               uint32_t b, V scale) {
  const BrickMeta M = load_meta(X.meta, b);
  V k0 = own_coef<INNER>(X, b, 1, L.m);
  V k1 = own_coef<INNER>(X, b, 2, L.m);
  V k2 = own_coef<INNER>(X, b, 3, L.m);
  V u = bload<V>(X.u, L.m, b * 64u);
  V rhs = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
  V c;
  V S = stencil_sum(X, L, b, M, u, k0, k1, k2, c);
  uint64_t amask = act_mask(M);
  bool act = (amask >> L.m) & 1ull;
  V r = act ? rhs - (c * u - S) : V(0);
  V rs = group8_sum(r);
  V us = group8_sum(act ? u : V(0));
  int cnt = __popcll((amask >> (L.m & 56u)) & 0xffull);
  if ((L.m & 7u) == 0) {
    uint32_t base = uint32_t(M.parent) * 64u + uint32_t(octant_of(M)) * 8u;
    uint32_t q = L.m >> 3;
    V ust = !CORR && cnt ? div_by(us, V(cnt)) : V(0);
    bstore<V>(X.b, q, base, rs * scale);
    bstore<V>(X.u, q, base, ust);
    bstore<V>(X.us, q, base - X.nlb * 64u, ust);
  }
}

template <class V, class CL, class CI, int CP = kCpolDefault, bool CORR = false>
__global__ void __launch_bounds__(kBlock) k_restrict(LevelArgs<V, CL, CI> A, V scale) {
  if (A.done && *A.done) return;
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI, CP> X = level_view<CP>(A);
  const WaveLoop W = wave_loop(A.R.n());
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    if (i < A.R.n_leaf) restrict_brick<false, CORR>(X, L, A.R.leaf_lo + i, scale);
    else restrict_brick<true, CORR>(X, L, A.R.inner_lo + (i - A.R.n_leaf), scale);
  }
}

// FAS coarse right-hand side on inner bricks: b += A^{l-1} u*.
template <class V, class CL, class CI>
__global__ void __launch_bounds__(kBlock) k_fas_rhs(LevelArgs<V, CL, CI> A) {
  if (A.done && *A.done) return;
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI> X = level_view(A);
  const WaveLoop W = wave_loop(A.R.n_inner);
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    uint32_t b = A.R.inner_lo + i;
    const BrickMeta M = load_meta(X.meta, b);
    V k0 = own_coef<true>(X, b, 1, L.m);
    V k1 = own_coef<true>(X, b, 2, L.m);
    V k2 = own_coef<true>(X, b, 3, L.m);
    V u = bload<V>(X.u, L.m, b * 64u);
    V rhs = bload<V>(X.b, L.m, b * 64u);
    V c;
    V S = stencil_sum(X, L, b, M, u, k0, k1, k2, c);
    bool act = (act_mask(M) >> L.m) & 1ull;
    bstore<V>(X.b, L.m, b * 64u, act ? rhs + (c * u - S) : V(0));
  }
}

// A cycle's first half-sweep of a level below the finest with leaves on it,
// with the FAS right-hand side folded in.  The iterate of the leaves, here and
// on the coarser levels, is still zero, and u = u* on inner bricks.  There one
// neighbour sum S gives both b += c u* - S (stored on every cell, as k_fas_rhs)
// and, on the cells of the colour, u = (b + S) / c: it is read from the u*
// array, which this launch does not write, with 0 for the leaves (as at a
// wall), so no brick's sum can see another brick's update.  A leaf brick
// without inner neighbours sees zeros only (first_sweep_brick); the others take
// a plain half-sweep, whose cells read the other colour.  Against k_fas_rhs and
// a plain half-sweep, FP32: 45.8 us for 15.6 + 38.1 (level 9 of the 26.3M-leaf
// workload), 15.7 for 6.3 + 12.9; solves of 2.3M leaves 5.33 -> 5.24 ms, FP64
// 7.21 -> 7.04 (of 26.3M within their run-to-run spread).
template <class V, class CL, class CI, int CP = kCpolDefault>
__global__ void __launch_bounds__(kBlock) k_smooth_fas(LevelArgs<V, CL, CI> A, int colour) {
  if (A.done && *A.done) return;
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI, CP> X = level_view<CP>(A);
  LevelView<V, CL, CI, CP> Xs = X;  // u = u*, indexed by brick id - nlb
  Xs.u = X.us;
  const WaveLoop W = wave_loop(A.R.n());
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    if (i < A.R.n_leaf) {
      const uint32_t b = A.R.leaf_lo + i;
      const uint32_t flags = load_meta(X.meta, b).flags;
      if (!((flags >> 8) & 0x3fu)) {
        first_sweep_brick<false, true>(X, L, b, colour);
      } else if constexpr (sizeof(V) == 8) {
        smooth_brick_gathered<false, 0, false>(X, L, half_gather(L, colour), b, colour);
      } else {
        smooth_brick<false, 0, false>(X, L, b, colour);
      }
      continue;
    }
    const uint32_t b = A.R.inner_lo + (i - A.R.n_leaf);
    const BrickMeta M = load_meta(X.meta, b);
    BrickMeta Ms = M;
#pragma unroll
    for (int d = 0; d < 6; ++d)
      Ms.nbr[d] = M.nbr[d] >= int32_t(X.nlb) ? M.nbr[d] - int32_t(X.nlb) : -1;
    Ms.flags = M.flags & ~uint32_t(kFlagT);
    V k0 = own_coef<true>(X, b, 1, L.m);
    V k1 = own_coef<true>(X, b, 2, L.m);
    V k2 = own_coef<true>(X, b, 3, L.m);
    V u = bload<V>(X.us, L.m, (b - X.nlb) * 64u);
    V rhs = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
    V c;
    V S = stencil_sum(Xs, L, b, Ms, u, k0, k1, k2, c);
    bool act = (act_mask(M) >> L.m) & 1ull;
    V rf = act ? rhs + (c * u - S) : V(0);
    bstore<V>(X.b, L.m, b * 64u, rf);
    if (act && L.colour == colour) bstore<V>(X.u, L.m, b * 64u, div_by(rf + S, c));
  }
}

// Prolongation of the FAS correction: u += u_P - u*_P on active cells.
template <class V, class CL, class CI>
__global__ void __launch_bounds__(kBlock) k_prolong(LevelArgs<V, CL, CI> A) {
  if (A.done && *A.done) return;
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI> X = level_view(A);
  const WaveLoop W = wave_loop(A.R.n());
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    uint32_t b = A.R.brick(i);
    const BrickMeta M = load_meta(X.meta, b);
    uint32_t base = uint32_t(M.parent) * 64u + uint32_t(octant_of(M)) * 8u;
    uint32_t q = L.m >> 3;
    V corr = bload<V>(X.u, q, base) - bload<V>(X.us, q, base - X.nlb * 64u);
    V u = bload<V>(X.u, L.m, b * 64u);
    if ((act_mask(M) >> L.m) & 1ull) bstore<V>(X.u, L.m, b * 64u, u + corr);
  }
}

// Coarsest level: nu RBGS iterations in one workgroup, (R,B) for the first
// `half` iterations and (B,R) for the rest (the transposed cycle takes the
// reversed order, half = nu - nu / 2).  The level is a complete
// grid of at most kCoarsestBricks bricks (no T-junctions), so its iterate
// stays in LDS and each wave keeps the coefficients of its bricks (at most
// kCoarsestSlots) in registers for all 2 nu half-sweeps; every value read,
// and the order of every sum, is that of the global-memory half-sweep.
constexpr int kCoarsestBricks = 64;
constexpr int kCoarsestSlots = kCoarsestBricks / (1024 / kWave);

template <class V, class CL, class CI>
__global__ void __launch_bounds__(1024) k_coarsest(LevelArgs<V, CL, CI> A, int nu, int half) {
  if (A.done && *A.done) return;
  __shared__ V su[kCoarsestBricks * 64];
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI> X = level_view(A);
  const uint32_t w = wave_id();
  const uint32_t nw = blockDim.x / kWave;
  const uint32_t n = A.R.n();
  const int m = int(L.m);
  V rhs[kCoarsestSlots], kown[kCoarsestSlots][3], kpl[kCoarsestSlots][3];
  int32_t nbl[kCoarsestSlots][6];
  uint64_t amask[kCoarsestSlots];
#pragma unroll
  for (int j = 0; j < kCoarsestSlots; ++j) {
    uint32_t i = w + uint32_t(j) * nw;
    if (i >= n) continue;
    bool inner = i >= A.R.n_leaf;
    uint32_t b = A.R.brick(i);
    const BrickMeta M = load_meta(X.meta, b);
    amask[j] = act_mask(M);
    for (int a = 0; a < 3; ++a) {
      kown[j][a] = inner ? own_coef<true>(X, b, 1 + a, L.m) : own_coef<false>(X, b, 1 + a, L.m);
      kpl[j][a] = V(bload_bytes<CL>(X.pf, L.foff[a], b * uint32_t(48 * sizeof(CL))));
    }
    for (int d = 0; d < 6; ++d) {
      int32_t nb = M.nbr[d];
      nbl[j][d] = nb < 0 ? -1
                  : uint32_t(nb) < X.nlb ? nb - int32_t(A.R.leaf_lo)
                                          : int32_t(A.R.n_leaf) + nb - int32_t(A.R.inner_lo);
    }
    rhs[j] = bload<V>(X.b, L.m, b * 64u);
    su[i * 64u + uint32_t(m)] = bload<V>(X.u, L.m, b * 64u);
  }
  __syncthreads();
  for (int it = 0; it < nu; ++it) {
    for (int h2 = 0; h2 < 2; ++h2) {
      int colour = it < half ? h2 : 1 - h2;
#pragma unroll
      for (int j = 0; j < kCoarsestSlots; ++j) {
        uint32_t i = w + uint32_t(j) * nw;
        if (i >= n) continue;
        V v[6], k[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) {
          int a = d >> 1;
          int p = L.p[d];
          int32_t nbase = L.out[d] ? (nbl[j][d] >= 0 ? nbl[j][d] * 64 : -1) : int32_t(i) * 64;
          v[d] = nbase >= 0 ? su[nbase + p] : V(0);
          if (d & 1) {
            V ks = shfl(kown[j][a], p);
            k[d] = L.out[d] ? kpl[j][a] : ks;
          } else {
            k[d] = kown[j][a];
          }
        }
        V c = ((k[0] + k[1]) + (k[2] + k[3])) + (k[4] + k[5]);
        V S = V(0);
#pragma unroll
        for (int d = 0; d < 6; ++d) S += k[d] * v[d];
        bool act = (amask[j] >> m) & 1ull;
        if (act && L.colour == colour) su[i * 64u + uint32_t(m)] = div_by(rhs[j] + S, c);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int j = 0; j < kCoarsestSlots; ++j) {
    uint32_t i = w + uint32_t(j) * nw;
    if (i < n) bstore<V>(X.u, L.m, A.R.brick(i) * 64u, su[i * 64u + uint32_t(m)]);
  }
}

// ---------------------------------------------------------------------------
// The FAS step of level f = lc + 1 in one workgroup (Algorithm 4 on that
// level: FAS right-hand side, pre-smoothing, residual restriction, mu
// coarsest solves, prolongation, post-smoothing) when level f is a complete
// grid (no T-junction) of at most 16^3 cells.  Both iterates stay in LDS, so
// the dozen launches of a few microseconds each that the separate kernels
// take become one.  The sums and their order are those of k_fas_rhs,
// k_smooth, k_restrict, k_coarsest and k_prolong, and the arrays in memory
// end as those kernels leave them.  `visits` consecutive FAS steps of level f
// (the level above's mu) are taken in one launch.
// CORR: the step in correction form (level f without leaves, where the iterate
// is u - u*, and the transposed cycle): it starts from a zero iterate (fas = 0:
// from U, on later visits of the transposed W-cycle), the coarsest iterate
// starts from zero too and pscale times it is the correction; the coarsest
// level's arrays are not written.
//
// What bounds it: one CU's LDS reads, the barriers and the set-up's loads.  A
// thread holds pairs of cells that are neighbours along x, one of each colour,
// so every lane has a cell to update in every half-sweep, and neighbouring
// lanes read neighbouring LDS words.  Six face coefficients per cell, in the
// stencil's order, come from a table made with the hierarchy (k_bottom_table):
// a brick per wave with its coefficients formed at each launch took 21 us per
// FP32 V-cycle step (8.5 of it set-up, 0.75 per half-sweep of 16^3 cells with
// half of the lanes idle) and 29 us in FP64, where it spilled registers; this
// form takes 12.3 and 24.5 us (a W-cycle's two visits, FP32: 34 -> 21 us).
// ---------------------------------------------------------------------------

// Position of pair (x >> 1, y, z) of a grid of 2^f cells per axis.  The low
// bits of y and z follow the x bits, so that the four pairs of a parent cell
// are lanes of one wave and a wave's reads spread over the LDS banks.
__host__ __device__ __forceinline__ uint32_t pair_index(int f, uint32_t xh, uint32_t y,
                                                        uint32_t z) {
  return xh | ((y & 1u) << (f - 1)) | ((z & 1u) << f) | ((y >> 1) << (f + 1)) |
         ((z >> 1) << (2 * f));
}

// Table of a level (k_bottom's and k_tile's): per pair 12 face coefficients (six of the even-x cell, six
// of the odd-x one) and one unit of indices, as 16-byte units, unit q of pair
// p at q * pairs + p.  Index unit: element of the even-x cell in the level
// arrays (the odd-x cell follows it), activity bits, inner-brick bit, element
// of their parent cell.
template <class V>
struct BottomUnits {
  static constexpr int kPer = 16 / int(sizeof(V));  // coefficients per unit
  static constexpr int kCoef = 12 / kPer;
  static constexpr int kAll = kCoef + 1;
};

template <class V>
__device__ __forceinline__ V diag_of(const V (&k)[6]) {
  return ((k[0] + k[1]) + (k[2] + k[3])) + (k[4] + k[5]);
}

// tiny: set to 1 when an active cell's diagonal is below FP64's normal range,
// where bottom_div does not hold (FP64 only).
template <class V, class CL, class CI>
__global__ void __launch_bounds__(kBlock) k_bottom_table(LevelArgs<V, CL, CI> A, int f,
                                                         uint4 *tab, unsigned long long *tiny) {
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI> X = level_view(A);
  const uint32_t i = blockIdx.x * kWavesPerBlock + wave_id();
  if (i >= A.R.n()) return;
  const bool inner = i >= A.R.n_leaf;
  const uint32_t b = A.R.brick(i);
  const BrickMeta M = load_meta(X.meta, b);
  const int m = int(L.m);
  V k[6];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    V kown = inner ? own_coef<true>(X, b, 1 + a, L.m) : own_coef<false>(X, b, 1 + a, L.m);
    V kl = V(bload_bytes<CL>(X.pf, L.foff[a], b * uint32_t(48 * sizeof(CL))));
    V ks = shfl(kown, L.p[2 * a + 1]);
    k[2 * a] = kown;
    k[2 * a + 1] = L.out[2 * a + 1] ? kl : ks;
  }
  if constexpr (sizeof(V) == 8) {
    if (((act_mask(M) >> m) & 1ull) && diag_of(k) < 0x1p-1022) *tiny = 1ull;
  }
  const uint32_t x = uint32_t(M.coord[0] * 4 + dev_cx(m)), y = uint32_t(M.coord[1] * 4 + dev_cy(m)),
                 z = uint32_t(M.coord[2] * 4 + dev_cz(m));
  const uint32_t np = 1u << (3 * f - 1), p = pair_index(f, x >> 1, y, z), e = x & 1u;
  constexpr uint32_t per = uint32_t(BottomUnits<V>::kPer);
#pragma unroll
  for (uint32_t d = 0; d < 6; ++d) {
    const uint32_t q = e * 6u + d;
    reinterpret_cast<V *>(tab + (q / per) * np + p)[q % per] = k[d];
  }
  if (e == 0) {
    const uint64_t act = act_mask(M);
    const uint32_t bits = uint32_t((act >> m) & 3ull) | (inner ? 4u : 0u);
    const uint32_t parent = uint32_t(M.parent) * 64u + uint32_t(octant_of(M)) * 8u + (L.m >> 3);
    tab[uint32_t(BottomUnits<V>::kCoef) * np + p] = uint4{b * 64u + uint32_t(m), bits, parent, 0u};
  }
}

// One pair of a level in k_bottom.  The LDS iterate is one array per colour,
// indexed by pair; entry `pairs` of each holds 0, the value at a wall.  A
// cell's neighbours all lie in the other colour's array, and the y and z ones
// at the same entries for both cells of the pair.
template <class V>
struct BottomPair {
  V k[2][6];         // by colour
  V rc[2];           // 1 / diagonal
  V rhs[2];
  uint32_t x[2][2];  // entries of the -x and +x neighbours, by colour
  uint32_t y[2], z[2];
  uint32_t at;       // element of the even-x cell in the level arrays
  uint32_t parent;   // element of the parent cell
  uint32_t bits;     // 1, 2: active by colour; 4: inner brick; 8: the pair
                     // exists; 16: the colour-0 cell is the odd-x one
};
// stride between the colours' arrays
__host__ __device__ constexpr uint32_t bottom_stride(uint32_t pairs) { return pairs + 32u; }

// Coefficients, reciprocal diagonals, element and bits of pair g of a table of
// `pairs` pairs; e0: the x parity of its colour-0 cell.
template <class V>
__device__ __forceinline__ void pair_coefs(BottomPair<V> &P, const uint4 *tab, uint32_t pairs,
                                           uint32_t g, uint32_t e0) {
  uint4 unit[BottomUnits<V>::kAll];
#pragma unroll
  for (int q = 0; q < BottomUnits<V>::kAll; ++q) unit[q] = tab[uint32_t(q) * pairs + g];
  V ke[2][6];
  constexpr int per = BottomUnits<V>::kPer;
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      const int q = e * 6 + d;
      const uint4 un = unit[q / per];
      if constexpr (sizeof(V) == 4) {
        const uint32_t w = q % per == 0 ? un.x : (q % per == 1 ? un.y : (q % per == 2 ? un.z : un.w));
        ke[e][d] = __builtin_bit_cast(V, w);
      } else {
        const uint64_t w = q % per == 0 ? (uint64_t(un.y) << 32) | un.x : (uint64_t(un.w) << 32) | un.z;
        ke[e][d] = __builtin_bit_cast(V, w);
      }
    }
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    P.k[0][d] = e0 ? ke[1][d] : ke[0][d];
    P.k[1][d] = e0 ? ke[0][d] : ke[1][d];
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if constexpr (sizeof(V) == 4) P.rc[c] = __builtin_amdgcn_rcpf(diag_of(P.k[c]));
    else P.rc[c] = V(1) / diag_of(P.k[c]);
  }
  const uint32_t bits = unit[BottomUnits<V>::kCoef].y, act = bits & 3u;
  P.at = unit[BottomUnits<V>::kCoef].x;
  P.parent = unit[BottomUnits<V>::kCoef].z;
  P.bits = (e0 ? (act >> 1) | ((act & 1u) << 1) : act) | (bits & 4u) | 8u | (e0 << 4);
}

// Entries of the neighbours of pair p of a grid of 2^f cells per axis.
template <class V>
__device__ __forceinline__ void pair_neighbours(BottomPair<V> &P, int f, uint32_t p, uint32_t e0) {
  const uint32_t np = 1u << (3 * f - 1), n = 1u << f;
  const uint32_t xh = p & ((n >> 1) - 1u);
  const uint32_t y = ((p >> (f - 1)) & 1u) | (((p >> (f + 1)) & ((n >> 1) - 1u)) << 1);
  const uint32_t z = ((p >> f) & 1u) | ((p >> (2 * f)) << 1);
  const uint32_t xm = xh > 0u ? p - 1u : np, xp = xh + 1u < (n >> 1) ? p + 1u : np;
#pragma unroll
  for (uint32_t c = 0; c < 2; ++c) {  // the even-x cell's +x neighbour is in the pair
    const bool odd = (e0 ^ c) != 0u;
    P.x[c][0] = odd ? p : xm;
    P.x[c][1] = odd ? xp : p;
  }
  P.y[0] = y > 0u ? pair_index(f, xh, y - 1u, z) : np;
  P.y[1] = y + 1u < n ? pair_index(f, xh, y + 1u, z) : np;
  P.z[0] = z > 0u ? pair_index(f, xh, y, z - 1u) : np;
  P.z[1] = z + 1u < n ? pair_index(f, xh, y, z + 1u) : np;
}

template <class V>
__device__ __forceinline__ BottomPair<V> bottom_pair(const uint4 *tab, int f, uint32_t p) {
  BottomPair<V> P;
  const uint32_t np = 1u << (3 * f - 1), n = 1u << f;
  P.bits = 0;
  if (p >= np) return P;
  const uint32_t y = ((p >> (f - 1)) & 1u) | (((p >> (f + 1)) & ((n >> 1) - 1u)) << 1);
  const uint32_t z = ((p >> f) & 1u) | ((p >> (2 * f)) << 1);
  pair_coefs(P, tab, np, p, (y + z) & 1u);
  pair_neighbours(P, f, p, (y + z) & 1u);
  return P;
}

// Neighbour sum of the pair's colour-c cell, face coefficients k; s: the other
// colour's LDS array.
template <class V>
__device__ __forceinline__ V bottom_sum(const V *s, const BottomPair<V> &P, const V (&k)[6],
                                        int c) {
  V S = k[0] * s[P.x[c][0]];
  S += k[1] * s[P.x[c][1]];
  S += k[2] * s[P.y[0]];
  S += k[3] * s[P.y[1]];
  S += k[4] * s[P.z[0]];
  S += k[5] * s[P.z[1]];
  return S;
}
// a over the diagonal of the coefficients k, rc its reciprocal (FP32: as
// div_by; FP64: the quotient by the reciprocal, corrected once, which agrees
// with the division to its last bit for finite a and quotients and a diagonal
// in FP64's normal range; a hierarchy with a smaller one -- the reciprocal of a
// subnormal number overflows -- keeps the separate kernels, which divide).
template <class V>
__device__ __forceinline__ V bottom_div(const V (&k)[6], V rc, V a) {
  if constexpr (sizeof(V) == 4) return a * rc;
  const V q = a * rc;
  return fma(fma(-q, diag_of(k), a), rc, q);
}
// Sum over the four pairs of a parent cell (lane bits f - 1 and f).
template <class T>
__device__ __forceinline__ T parent_sum(T v, int f) {
  v = v + shfl_xor(v, 1 << (f - 1));
  return v + shfl_xor(v, 1 << f);
}

template <class V>
struct BottomArgs {
  const uint4 *tf, *tc;  // tables of level f and of the coarsest level
  int f;
  V *U, *B, *Ustar;
  uint32_t nlb;
  int nu_pre, nu_post, nu_coarse, half, mu, fas, visits;
  V scale, pscale;
  const int *done;
};

constexpr int kBottomLevel = 4;                            // finest f it takes
constexpr int kBottomPairs = 1 << (3 * kBottomLevel - 1);  // 2048
// Threads of the workgroup: 1024 hold two fine pairs each in FP32; FP64's
// would not fit 128 registers (112 bytes of spills per lane, 26.6 against 24.5
// us), so half the threads hold four.
template <class V>
constexpr int kBottomThreads = sizeof(V) == 8 ? 512 : 1024;

template <class V, bool CORR = false>
__global__ void __launch_bounds__(kBottomThreads<V>) k_bottom(BottomArgs<V> A) {
  if (A.done && *A.done) return;
  constexpr int kSlots = kBottomPairs / kBottomThreads<V>;
  constexpr uint32_t nt = uint32_t(kBottomThreads<V>);
  constexpr uint32_t sf = bottom_stride(kBottomPairs), sg = bottom_stride(kBottomPairs / 8);
  __shared__ V uf[2 * sf];
  __shared__ V uc[2 * sg];
  __shared__ V bc[2 * sg];  // restricted residual of the coarse cells
  __shared__ V sc[2 * sg];  // their u*
  typedef V V2 __attribute__((ext_vector_type(2)));
  const int f = A.f, fc = A.f - 1;
  const uint32_t np = 1u << (3 * f - 1), npc = 1u << (3 * fc - 1);
  const uint32_t tid = threadIdx.x;
  if (tid < 2u) {
    uf[tid * sf + np] = V(0);
    uc[tid * sg + npc] = V(0);
  }
  BottomPair<V> P[kSlots];
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const uint32_t p = tid + uint32_t(j) * nt;
    P[j] = bottom_pair<V>(A.tf, f, p);
    if (P[j].bits & 8u) {
      const bool odd = P[j].bits & 16u;
      const V2 b2 = *reinterpret_cast<const V2 *>(A.B + P[j].at);
      V2 u2 = V2{V(0), V(0)};
      if (!(CORR && A.fas)) u2 = *reinterpret_cast<const V2 *>(A.U + P[j].at);
      P[j].rhs[0] = odd ? b2.y : b2.x;
      P[j].rhs[1] = odd ? b2.x : b2.y;
      uf[p] = odd ? u2.y : u2.x;
      uf[sf + p] = odd ? u2.x : u2.y;
    }
  }
  BottomPair<V> C = bottom_pair<V>(A.tc, fc, tid);
  // the parent's entry on the coarsest level (its colour's array included)
  uint32_t par[kSlots];
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const uint32_t p = tid + uint32_t(j) * nt;
    const uint32_t xh = p & ((1u << (f - 1)) - 1u);
    const uint32_t py = (p >> (f + 1)) & ((1u << (f - 1)) - 1u), pz = p >> (2 * f);
    par[j] = ((xh + py + pz) & 1u) * sg + pair_index(fc, xh >> 1, py, pz);
  }
  __syncthreads();

  // (the colour is a type, so that its arrays' offsets are constants)
  auto half_sweep_f = [&](auto colour) {
    constexpr int c = decltype(colour)::value;
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      if (!(P[j].bits & 8u)) continue;
      const V S = bottom_sum(uf + (1 - c) * sf, P[j], P[j].k[c], c);
      if (P[j].bits & (1u << c))
        uf[c * sf + tid + uint32_t(j) * nt] =
            bottom_div(P[j].k[c], P[j].rc[c], P[j].rhs[c] + S);
    }
    __syncthreads();
  };
  auto half_sweep_c = [&](auto colour) {
    constexpr int c = decltype(colour)::value;
    if (C.bits & (1u << c)) {
      const V S = bottom_sum(uc + (1 - c) * sg, C, C.k[c], c);
      uc[c * sg + tid] = bottom_div(C.k[c], C.rc[c], C.rhs[c] + S);
    }
    __syncthreads();
  };
  const std::integral_constant<int, 0> red{};
  const std::integral_constant<int, 1> black{};
  for (int visit = 0; visit < A.visits; ++visit) {
    // FAS right-hand side of the inner bricks: b += A u*
    if (!CORR && visit == 0) {
#pragma unroll
      for (int j = 0; j < kSlots; ++j) {
        if ((P[j].bits & 12u) != 12u) continue;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const V S = bottom_sum(uf + (1 - c) * sf, P[j], P[j].k[c], c);
          const V u = uf[c * sf + tid + uint32_t(j) * nt];
          P[j].rhs[c] = P[j].bits & (1u << c) ? P[j].rhs[c] + (diag_of(P[j].k[c]) * u - S) : V(0);
        }
        const bool odd = P[j].bits & 16u;
        *reinterpret_cast<V2 *>(A.B + P[j].at) =
            V2{odd ? P[j].rhs[1] : P[j].rhs[0], odd ? P[j].rhs[0] : P[j].rhs[1]};
      }
      __syncthreads();  // every thread's reads of uf before the first writes
    }
    for (int it = 0; it < A.nu_pre; ++it) {
      half_sweep_f(red);
      half_sweep_f(black);
    }
    // residual restriction and u* to the coarsest level
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      V r[2] = {V(0), V(0)}, u[2] = {V(0), V(0)};
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (P[j].bits & (1u << c)) {
          const V S = bottom_sum(uf + (1 - c) * sf, P[j], P[j].k[c], c);
          u[c] = uf[c * sf + tid + uint32_t(j) * nt];
          r[c] = P[j].rhs[c] - (diag_of(P[j].k[c]) * u[c] - S);
        }
      const V rs = parent_sum(r[0] + r[1], f);
      const V us = parent_sum(u[0] + u[1], f);
      const int cnt = parent_sum(__popc(P[j].bits & 3u), f);
      if ((P[j].bits & 8u) && !(tid & (3u << (f - 1)))) {
        const V ust = !CORR && cnt ? div_by(us, V(cnt)) : V(0);
        bc[par[j]] = rs * A.scale;
        uc[par[j]] = ust;
        sc[par[j]] = ust;
      }
    }
    __syncthreads();
    // the coarsest level: FAS right-hand side (CORR: u = 0), mu solves
    if (C.bits & 8u) {
#pragma unroll
      for (uint32_t c = 0; c < 2; ++c) {
        const V S = bottom_sum(uc + (1 - c) * sg, C, C.k[c], int(c));
        const uint32_t own = c * sg + tid;
        C.rhs[c] = C.bits & (1u << c) ? bc[own] + (diag_of(C.k[c]) * uc[own] - S) : V(0);
      }
    }
    __syncthreads();
    for (int rep = 0; rep < A.mu; ++rep)
      for (int it = 0; it < A.nu_coarse; ++it) {
        if (it < A.half) {
          half_sweep_c(red);
          half_sweep_c(black);
        } else {
          half_sweep_c(black);
          half_sweep_c(red);
        }
      }
    // prolongation of the correction, post-smoothing
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      if (!(P[j].bits & 8u)) continue;
      const V corr = CORR ? A.pscale * uc[par[j]] : uc[par[j]] - sc[par[j]];
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (P[j].bits & (1u << c)) uf[c * sf + tid + uint32_t(j) * nt] += corr;
    }
    __syncthreads();
    for (int it = 0; it < A.nu_post; ++it) {
      half_sweep_f(black);
      half_sweep_f(red);
    }
  }

  // the arrays as the separate kernels leave them
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    if (!(P[j].bits & 8u)) continue;
    const bool odd = P[j].bits & 16u;
    const uint32_t p = tid + uint32_t(j) * nt;
    const V u0 = uf[p], u1 = uf[sf + p];
    *reinterpret_cast<V2 *>(A.U + P[j].at) = V2{odd ? u1 : u0, odd ? u0 : u1};
  }
  if (!CORR && (C.bits & 8u)) {
    const bool odd = C.bits & 16u;
    auto pair = [&](V a, V b) { return V2{odd ? b : a, odd ? a : b}; };
    *reinterpret_cast<V2 *>(A.U + C.at) = pair(uc[tid], uc[sg + tid]);
    *reinterpret_cast<V2 *>(A.B + C.at) = pair(C.rhs[0], C.rhs[1]);
    *reinterpret_cast<V2 *>(A.Ustar + (C.at - A.nlb * 64u)) = pair(sc[tid], sc[sg + tid]);
  }
}

// ---------------------------------------------------------------------------
// The visit of a complete level of 16^3 to 64^3 cells (so it has no T-junction;
// its bricks may be leaves and inner ones) in two or three launches.  The
// separate kernels take nine or ten, of 3 to 5 us each however little they do;
// here a workgroup takes a tile of 8^3 cells and the 4 cells around it, 16^3
// in all, as k_bottom takes its level, and the values that go stale at the rim
// (one cell per half-sweep) are not kept.  That is eight times the work, bound
// at 32^3 by one CU's set-up and barriers, at 64^3 by the coefficients' reads
// (eight times a table of 8.4 MB, FP32).  us, two iterations on each side, with
// the launches replaced: 32^3 FP32, zero 6.5 (15.2), up 6.1 (15.3), from and
// restrict 5.3 + 4.2 (18.5); 64^3 FP32, zero 13.7 (22), up 10 (17), from and
// restrict 9.1 + 7.8 (25).
// nu <= 2 iterations on a side:
//   kTileZero      the way down from a zero iterate: smoothing (colours 0, 1)
//                  and restriction.  From zero the first half-sweep needs no
//                  neighbours, so the residual of the tile is still exact
//                  after three more.
//   kTileFrom      the way down from U: FAS right-hand side (fas, to R),
//                  smoothing.
//   kTileRestrict  the restriction that follows it.
//   kTileUp        the parents' correction, smoothing (colours 1, 0), to U.
// Between them the iterate is in W (by pair: other tiles read U's halo).  R:
// the level's right-hand side by pair, where it is not B.
// ---------------------------------------------------------------------------
enum TileMode { kTileZero, kTileFrom, kTileRestrict, kTileUp };
constexpr int kTileMin = 4, kTileMax = 6;  // levels

template <class V>
struct TileArgs {
  const uint4 *tab;
  V *U, *B, *Ustar, *W, *R;
  uint32_t nlb;
  int l, nu;
  int fas;          // kTileFrom: form the FAS right-hand side of inner cells
  int corr;         // kTileRestrict, kTileZero: level l - 1 is in correction form
  int sub;          // kTileUp: the parents' u* is taken off
  V scale, pscale;  // of the restricted residual, of the parents' iterate
  const int *done;
  StopTest stop;    // kTileZero
};

template <class V, int MODE>
// (FP32 in 64 registers, for two workgroups per CU at 64^3; the way down from
// zero does not fit them and gained nothing there: 8.0 us at 32^3)
__global__ void __launch_bounds__(kBottomThreads<V>, sizeof(V) == 4 && MODE != kTileZero ? 8 : 2)
    k_tile(TileArgs<V> A) {
  if constexpr (MODE == kTileZero) {
    if (stop_test(A.stop, A.done)) return;
  } else {
    if (A.done && *A.done) return;
  }
  constexpr int kSlots = kBottomPairs / kBottomThreads<V>;
  constexpr uint32_t nt = uint32_t(kBottomThreads<V>);
  constexpr uint32_t np = uint32_t(kBottomPairs);
  constexpr uint32_t sf = bottom_stride(np);
  constexpr int f = kBottomLevel;  // the region's
  __shared__ V uf[2 * sf];
  typedef V V2 __attribute__((ext_vector_type(2)));
  const uint32_t tid = threadIdx.x;
  // a slab of tiles per XCD, whose L2 then holds what its tiles read twice
  const uint32_t tl = uint32_t(A.l - 3), n = 1u << A.l;
  const uint32_t tile = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t t0 = tile & ((1u << tl) - 1u), t1 = (tile >> tl) & ((1u << tl) - 1u),
                 t2 = tile >> (2u * tl);
  if (tid < 2u) uf[tid * sf + np] = V(0);
  BottomPair<V> P[kSlots];
  uint32_t pair[kSlots];  // the level's pair; bit 31: it is the tile's own
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const uint32_t p = tid + uint32_t(j) * nt;
    const uint32_t lx = p & 7u;
    const uint32_t ly = ((p >> (f - 1)) & 1u) | (((p >> (f + 1)) & 7u) << 1);
    const uint32_t lz = ((p >> f) & 1u) | ((p >> (2 * f)) << 1);
    // (outside the level: at least n, wrapped or not)
    const uint32_t x = 4u * t0 + lx - 2u, y = 8u * t1 + ly - 4u, z = 8u * t2 + lz - 4u;
    const bool own = lx - 2u < 4u && ly - 4u < 8u && lz - 4u < 8u;
    P[j].bits = 0u;
    pair[j] = 0u;
    V u0 = V(0), u1 = V(0);
    if (x < n / 2u && y < n && z < n) {
      const uint32_t g = pair_index(A.l, x, y, z);
      pair_coefs(P[j], A.tab, 1u << (3 * A.l - 1), g, (y + z) & 1u);
      pair[j] = g | (own ? 0x80000000u : 0u);
      const bool odd = P[j].bits & 16u;
      const V *rhs = A.R && !(MODE == kTileFrom && A.fas) ? A.R + 2u * g : A.B + P[j].at;
      const V2 b2 = *reinterpret_cast<const V2 *>(rhs);
      P[j].rhs[0] = odd ? b2.y : b2.x;
      P[j].rhs[1] = odd ? b2.x : b2.y;
      if constexpr (MODE != kTileZero) {
        const V *from = MODE == kTileFrom ? A.U + P[j].at : A.W + 2u * g;
        const V2 w2 = *reinterpret_cast<const V2 *>(from);
        u0 = odd ? w2.y : w2.x;
        u1 = odd ? w2.x : w2.y;
      }
      if constexpr (MODE == kTileUp) {
        V corr = A.pscale * A.U[P[j].parent];
        if (A.sub) corr = corr - A.Ustar[P[j].parent - A.nlb * 64u];
        if (P[j].bits & 1u) u0 += corr;
        if (P[j].bits & 2u) u1 += corr;
      }
    }
    pair_neighbours(P[j], f, p, (P[j].bits >> 4) & 1u);
    uf[p] = u0;
    uf[sf + p] = u1;
  }
  __syncthreads();
  auto sum = [&](int j, int c) {
    return bottom_sum(uf + (1 - c) * sf, P[j], P[j].k[c], c);
  };
  if constexpr (MODE == kTileFrom) {
    if (A.fas) {  // b += A u* on inner cells
#pragma unroll
      for (int j = 0; j < kSlots; ++j) {
        if (P[j].bits & 4u) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const V u = uf[c * sf + tid + uint32_t(j) * nt];
            const V S = sum(j, c);
            P[j].rhs[c] = P[j].bits & (1u << c) ? P[j].rhs[c] + (diag_of(P[j].k[c]) * u - S) : V(0);
          }
        }
        const bool odd = P[j].bits & 16u;
        if (pair[j] >> 31)
          *reinterpret_cast<V2 *>(A.R + 2u * (pair[j] & 0x7fffffffu)) =
              V2{odd ? P[j].rhs[1] : P[j].rhs[0], odd ? P[j].rhs[0] : P[j].rhs[1]};
      }
      __syncthreads();  // every thread's reads of uf before the first writes
    }
  }
  if constexpr (MODE != kTileRestrict) {
    auto half_sweep = [&](auto colour) {
      constexpr int c = decltype(colour)::value;
#pragma unroll
      for (int j = 0; j < kSlots; ++j)
        if (P[j].bits & (1u << c)) {
          const V S = sum(j, c);
          uf[c * sf + tid + uint32_t(j) * nt] =
              bottom_div(P[j].k[c], P[j].rc[c], P[j].rhs[c] + S);
        }
      __syncthreads();
    };
    const std::integral_constant<int, MODE == kTileUp ? 1 : 0> first{};
    const std::integral_constant<int, MODE == kTileUp ? 0 : 1> second{};
    for (int it = 0; it < A.nu; ++it) {
      half_sweep(first);
      half_sweep(second);
    }
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      const uint32_t p = tid + uint32_t(j) * nt;
      const bool odd = P[j].bits & 16u;
      if (pair[j] >> 31) {
        const V u0 = uf[p], u1 = uf[sf + p];
        V *to = MODE == kTileUp ? A.U + P[j].at : A.W + 2u * (pair[j] & 0x7fffffffu);
        *reinterpret_cast<V2 *>(to) = V2{odd ? u1 : u0, odd ? u0 : u1};
      }
    }
  }
  if constexpr (MODE == kTileZero || MODE == kTileRestrict) {
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      V r[2] = {V(0), V(0)}, u[2] = {V(0), V(0)};
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (P[j].bits & (1u << c)) {
          u[c] = uf[c * sf + tid + uint32_t(j) * nt];
          r[c] = P[j].rhs[c] - (diag_of(P[j].k[c]) * u[c] - sum(j, c));
        }
      const V rs = parent_sum(r[0] + r[1], f);
      V ust = V(0);
      if (!A.corr) {
        const V us = parent_sum(u[0] + u[1], f);
        const int cnt = parent_sum(__popc(P[j].bits & 3u), f);
        if (cnt) ust = div_by(us, V(cnt));
      }
      if ((pair[j] >> 31) && !(tid & (3u << (f - 1)))) {
        A.B[P[j].parent] = rs * A.scale;
        A.U[P[j].parent] = ust;
        A.Ustar[P[j].parent - A.nlb * 64u] = ust;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// transpose of the cycle (adjoint solves): the cycle's linear steps transposed
// and taken in reverse order, as a cycle for A^T in solution form.  On every
// level U holds the iterate y (zero at the first visit), B the right-hand
// side g and Ustar the part of a level's residual that its parent level hands
// on.  A transposed half-sweep in residual form, w = rho / c on the colour,
// rho -= A^T w, y += w, with rho = g - A^T y at all times, is one
// Gauss-Seidel half-sweep of A^T y = g: it reads and writes what a forward
// half-sweep does, where the residual form reads and writes rho and w on
// every cell besides.  Bound like the forward cycle; on the 26.3M-leaf
// workload, FP32, a finest half-sweep takes 95 us against 161 us in residual
// form and the adjoint solve and gradient 57.9 against 94.2 ms (2.3M leaves:
// 8.1 against 13.6 ms) from that alone.
//
// The residual that the transposed FAS steps hand from level l - 1 back to
// level l,  -(what was restricted) + rho + A^T (y on inner cells), is, with
// rho = g - A^T y, the change of g since the restriction plus the
// neighbour sums over the same-level leaves (leaf_neighbour_sum): no
// operator application is needed for it.
// ---------------------------------------------------------------------------

// On a leaf brick with inner same-level neighbours (record M): the sum over
// the fine cells next to the lane's cell, across all its faces to finer
// leaves, of (k_f / 2) x_f, k_f the fine cell's T-face coefficient -- the
// coarse leaf's row of the transposed T-junction coupling.  The 8 x 8 fine
// cells on a face are one per lane -- lane 4 j + s holds sub-cell s of the
// coarse face cell with interleaved in-plane index j -- so a face takes two
// loads, two exchange steps add each cell's four and one hands the sum to the
// face's lane.  Every face's child ids, then every face's values are
// requested before any is used.
template <class V, class CL>
__device__ __forceinline__ V face_children_sum(__amdgpu_buffer_rsrc_t x,
                                               __amdgpu_buffer_rsrc_t cl,
                                               __amdgpu_buffer_rsrc_t pf, const int32_t *child,
                                               const BrickMeta &M, int m) {
  const int j = m >> 2;
  const int cu = (j & 1) | ((j >> 1) & 2);
  const int cv = ((j >> 1) & 1) | ((j >> 2) & 2);
  const int fu = ((cu & 1) << 1) | (m & 1);
  const int fv = ((cv & 1) << 1) | ((m >> 1) & 1);
  uint32_t cb[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    cb[d] = 0u;
    if ((M.flags >> (8 + d)) & 1u) {
      const int a = d >> 1, o0 = a == 0 ? 1 : 0, o1 = a == 2 ? 1 : 2;
      const Children C = load_children(child, uint32_t(M.nbr[d]));
      const int c = (d & 1) ? 0 : (1 << a);
      cb[d] = uint32_t((cv & 2) ? ((cu & 2) ? C.id[c | (1 << o0) | (1 << o1)] : C.id[c | (1 << o1)])
                                : ((cu & 2) ? C.id[c | (1 << o0)] : C.id[c]));
    }
  }
  V v[6], k[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    v[d] = V(0);
    k[d] = V(0);
    if ((M.flags >> (8 + d)) & 1u) {
      const int a = d >> 1, o0 = a == 0 ? 1 : 0, o1 = a == 2 ? 1 : 2;
      int xyz[3];
      xyz[a] = (d & 1) ? 0 : 3;
      xyz[o0] = fu;
      xyz[o1] = fv;
      const uint32_t q = uint32_t(dev_morton(xyz[0], xyz[1], xyz[2]));
      v[d] = bload<V>(x, cb[d] * 64u + q, 0u);
      if (d & 1)  // the fine cells' own minus-face coefficients
        k[d] = V(bload<CL>(cl, cb[d] * 256u + uint32_t(1 + a) * 64u + q, 0u));
      else        // their plus-face entries
        k[d] = V(bload<CL>(pf, cb[d] * 48u + uint32_t(a * 16 + fu + 4 * fv), 0u));
    }
  }
  V acc = V(0);
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    if ((M.flags >> (8 + d)) & 1u) {
      const int a = d >> 1, o0 = a == 0 ? 1 : 0, o1 = a == 2 ? 1 : 2;
      V s = k[d] * V(0.5) * v[d];
      s = s + shfl_xor(s, 1);
      s = s + shfl_xor(s, 2);
      const int mu = dev_coord(m, o0), mv = dev_coord(m, o1);
      const int jm = (mu & 1) | ((mv & 1) << 1) | ((mu & 2) << 1) | ((mv & 2) << 2);
      const V r = shfl(s, 4 * jm);
      acc += dev_outside(m, d) ? r : V(0);
    }
  }
  return acc;
}

// Coupling of level l to the coarser leaves, transposed: a leaf brick b of
// level l - 1 with an inner neighbour takes g_J += sum over its fine T-face
// cells of (k_f / 2) y_f.  `prev` (null when each level is visited once)
// keeps what was added at the visit before.
template <class V, class CL, class CI, int CP>
__device__ __forceinline__ void coupling_brick(const LevelView<V, CL, CI, CP> &X,
                                               const int32_t *child, V *prev, int first,
                                               uint32_t b, int m) {
  const BrickMeta M = load_meta(X.meta, b);
  V g = bload<V>(X.b, uint32_t(m), b * 64u);
  V acc = face_children_sum<V, CL>(X.u, X.cl, X.pf, child, M, m);
  if (!((act_mask(M) >> m) & 1ull)) acc = V(0);
  if (prev) {
    V was = first ? V(0) : prev[b * 64u + uint32_t(m)];
    prev[b * 64u + uint32_t(m)] = acc;
    acc -= was;
  }
  bstore<V>(X.b, uint32_t(m), b * 64u, g + acc);
}

// Transposed prolongation: the children's residual sums become the parents'
// right-hand side; the parents' iterate and handed-back residual start from 0.
template <bool INNER, class V, class CL, class CI, int CP>
__device__ __forceinline__ void restrict_brick_T(const LevelView<V, CL, CI, CP> &X,
                                                 const LaneC<V, CL> &L, uint32_t b) {
  const BrickMeta M = load_meta(X.meta, b);
  V k0 = own_coef<INNER>(X, b, 1, L.m);
  V k1 = own_coef<INNER>(X, b, 2, L.m);
  V k2 = own_coef<INNER>(X, b, 3, L.m);
  V u = bload<V>(X.u, L.m, b * 64u);
  V rhs = bload<V, side_pol(CP)>(X.b, L.m, b * 64u);
  V c;
  V S = stencil_sum<0, true>(X, L, b, M, u, k0, k1, k2, c);
  bool act = (act_mask(M) >> L.m) & 1ull;
  V rs = group8_sum(act ? rhs - (c * u - S) : V(0));
  if ((L.m & 7u) == 0) {
    uint32_t base = uint32_t(M.parent) * 64u + uint32_t(octant_of(M)) * 8u;
    uint32_t q = L.m >> 3;
    bstore<V>(X.b, q, base, rs);
    bstore<V>(X.u, q, base, V(0));
    bstore<V>(X.us, q, base - X.nlb * 64u, V(0));
  }
}

// The restriction of level l (workgroups [0, g_restrict)) and, in the same
// launch, its coupling to the coarser leaves (the workgroups after, one wave
// per listed brick): both read the level's iterate; the former writes the
// parents' arrays, the latter the right-hand side of leaves of level l - 1.
template <class V, class CL, class CI, int CP = kCpolDefault>
__global__ void __launch_bounds__(kBlock) k_T_restrict(LevelArgs<V, CL, CI> A, V *prev, int first,
                                                       const uint32_t *list, uint32_t n,
                                                       uint32_t g_restrict) {
  if (A.done && *A.done) return;
  const LevelView<V, CL, CI, CP> X = level_view<CP>(A);
  if (blockIdx.x < g_restrict) {
    const LaneC<V, CL> L = lane_consts<V, CL>();
    const WaveLoop W = wave_loop_of(A.R.n(), blockIdx.x, g_restrict);
    for (uint32_t i = W.first; i < W.end; i += W.step) {
      if (i < A.R.n_leaf) restrict_brick_T<false>(X, L, A.R.leaf_lo + i);
      else restrict_brick_T<true>(X, L, A.R.inner_lo + (i - A.R.n_leaf));
    }
  } else {
    uint32_t i = (blockIdx.x - g_restrict) * kWavesPerBlock + wave_id();
    if (i < n) {
      uint32_t b = __builtin_amdgcn_readfirstlane(list[i]);
      coupling_brick(X, A.T.child, prev, first, b, int(threadIdx.x & (kWave - 1)));
    }
  }
}

// Sum over the faces of cell m of inner brick b to same-level leaf bricks of
// k y (M: the brick's record, iscale: of the brick's level).
template <class V, class CL, class CI, int CP>
__device__ __forceinline__ V leaf_neighbour_sum(const LevelView<V, CL, CI, CP> &X, uint32_t b,
                                                const BrickMeta &M, int m, V iscale) {
  V q = V(0);
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    const int a = d >> 1;
    const int32_t n = M.nbr[d];
    if (n < 0 || uint32_t(n) >= X.nlb || !dev_outside(m, d)) continue;
    V k;
    if (d & 1) {
      k = V(bload<CL>(X.pf, uint32_t(a * 16 + dev_face_index(m, a)), b * 48u));
    } else {
      k = V(bload<CI>(X.ci, uint32_t(m), (b - X.nlb) * 256u + uint32_t(1 + a) * 64u));
      if constexpr (!std::is_same<CL, CI>::value) k = k * iscale;
    }
    q += k * bload<V>(X.u, uint32_t(dev_partner(m, d)), uint32_t(n) * 64u);
  }
  return q;
}

// Later visits of a level by a W-cycle (its leaves' iterate is no longer
// zero): the restricted right-hand side of the inner bricks of A's level and
// the residual handed back from it start from minus the sums over its
// same-level leaves.
template <class V, class CL, class CI>
__global__ void __launch_bounds__(kBlock) k_T_revisit(LevelArgs<V, CL, CI> A) {
  if (A.done && *A.done) return;
  const LevelView<V, CL, CI> X = level_view(A);
  const int m = threadIdx.x & (kWave - 1);
  const WaveLoop W = wave_loop(A.R.n_inner);
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    uint32_t b = A.R.inner_lo + i;
    const BrickMeta M = load_meta(X.meta, b);
    V q = leaf_neighbour_sum(X, b, M, m, X.iscale);
    if (!((act_mask(M) >> m) & 1ull)) q = V(0);
    V g = bload<V>(X.b, uint32_t(m), b * 64u);
    bstore<V>(X.b, uint32_t(m), b * 64u, g - q);
    bstore<V>(X.us, uint32_t(m), (b - X.nlb) * 64u, -q);
  }
}

// After the coarse recursion, on the bricks of level l, when no half-sweep
// follows to take it along: take_residual_T, and pscale times the parent's
// iterate into the active cells' own.
template <bool INNER, class V, class CL, class CI, int CP>
__device__ __forceinline__ void prolong_brick_T(const LevelView<V, CL, CI, CP> &X,
                                                const LaneC<V, CL> &L, uint32_t b) {
  const BrickMeta M = load_meta(X.meta, b);
  V y = bload<V>(X.u, L.m, b * 64u);
  take_residual_T<INNER>(X, L, b, M, bload<V>(X.b, L.m, b * 64u));
  V corr = own_correction<true>(X, L, M);
  if ((act_mask(M) >> L.m) & 1ull) bstore<V>(X.u, L.m, b * 64u, y + corr);
}

template <class V, class CL, class CI>
__global__ void __launch_bounds__(kBlock) k_T_prolong(LevelArgs<V, CL, CI> A) {
  if (A.done && *A.done) return;
  const LaneC<V, CL> L = lane_consts<V, CL>();
  const LevelView<V, CL, CI> X = level_view(A);
  const WaveLoop W = wave_loop(A.R.n());
  for (uint32_t i = W.first; i < W.end; i += W.step) {
    if (i < A.R.n_leaf) prolong_brick_T<false>(X, L, A.R.leaf_lo + i);
    else prolong_brick_T<true>(X, L, A.R.inner_lo + (i - A.R.n_leaf));
  }
}

// flag[b] = leaf brick b has an inner (finer-refined) face neighbour
__global__ void k_couple_flag(const BrickMeta *meta, uint32_t nlb, int64_t *flag) {
  uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < nlb) flag[b] = (meta[b].flags & kFlagInner) ? 1 : 0;
}

// list[pos[b]] = b for the flagged bricks (pos: exclusive scan of the flags)
__global__ void k_couple_list(const BrickMeta *meta, uint32_t nlb, const int64_t *pos,
                              uint32_t *list) {
  uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < nlb && (meta[b].flags & kFlagInner)) list[pos[b]] = b;
}

template <class V>
__global__ void k_fill(V *x, int64_t n, V v) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

}  // namespace mfmg
