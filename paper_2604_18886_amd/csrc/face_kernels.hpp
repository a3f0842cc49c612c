// Per-face arrays without a face list.  The canonical face order is (owner
// leaf, direction), so a leaf brick's faces are one contiguous range, and
// which faces a cell owns follows from the brick's face flags alone: its
// three minus faces, except towards finer leaves, and its plus faces at walls
// and coarser leaves.  One wave per brick then finds every face of its cells
// and of its neighbours' by counting bits in six 64-bit cell masks (wave
// uniform), and values across in-brick faces are lane exchanges.
//
// 26.3M leaves, 81M faces, against one thread per face or cell through tables
// (18 bytes per face, 9 per cell) with dependent loads: divergence 950 -> 579
// us, velocity update 1276 -> 504 us, per-face gradient 1062 -> 443 us.  The
// per-face arrays alone take 240 to 350 us at the copy rate; the rest is
// instruction issue (about 800 per brick, scalar ones among them): neither
// more waves per SIMD nor fewer cache requests (faces in order through LDS,
// half of the neighbours' flows from the workgroup) changed the times much.
#pragma once

#include "kernels.hpp"

namespace mfmg {

// cells of a brick on its face d
constexpr uint64_t face_cells(int d) {
  uint64_t r = 0;
  for (int m = 0; m < 64; ++m) {
    int low = 1 << (d >> 1), both = low | (low << 3);
    if ((d & 1) ? (m & both) == both : (m & both) == 0) r |= uint64_t(1) << m;
  }
  return r;
}

// A brick without these flags is regular: every cell owns exactly its three
// minus faces.
constexpr uint32_t kFlagIrregular = 0x2au | (0x15u << 8) | (0x2au << 16);

// Lane constants for finding a cell's faces without counting bits per brick:
// a brick's faces before cell m are 3 m, less the face cells before m on each
// minus face towards finer leaves, plus those on each plus face at a wall or
// coarser leaf.  These counts (at most 16) are packed, 5 bits per face.
struct FaceLane {
  int m;
  uint32_t out;      // bit d: the cell lies on the brick's face d
  uint32_t cnt;      // of the cell
  uint32_t cntp[3];  // of the cell across plus face a, in the next brick
};
__device__ __forceinline__ uint32_t face_counts(int m) {
  uint32_t c = 0;
#pragma unroll
  for (int e = 0; e < 6; ++e)
    c |= uint32_t(__popcll(face_cells(e) & ((1ull << m) - 1ull))) << (5 * e);
  return c;
}
__device__ __forceinline__ FaceLane face_lane() {
  FaceLane L;
  L.m = threadIdx.x & (kWave - 1);
  L.out = 0;
#pragma unroll
  for (int d = 0; d < 6; ++d) L.out |= dev_outside(L.m, d) ? 1u << d : 0u;
  L.cnt = face_counts(L.m);
#pragma unroll
  for (int a = 0; a < 3; ++a) L.cntp[a] = face_counts(dev_partner(L.m, 2 * a + 1));
  return L;
}
// is the brick's plus face e (odd) one its cells own (a wall or T-junction)
__device__ __forceinline__ bool owns_plus(uint32_t flags, int e) {
  return ((flags >> e) | (flags >> (16 + e))) & 1u;
}
// Faces of the brick before the cell with index `cell` and packed counts cnt.
__device__ __forceinline__ uint32_t first_slot(uint32_t flags, uint32_t cell, uint32_t cnt) {
  uint32_t s = 3u * cell;
  if (flags & kFlagIrregular) {
    // opaque, so that the 24 unpacked counts of a kernel are not kept in
    // registers across its loop over bricks
    asm volatile("" : "+v"(cnt));
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const uint32_t n = (cnt >> (5 * e)) & 31u;
      if (e & 1) s += owns_plus(flags, e) ? n : 0u;
      else s -= (flags >> (8 + e)) & 1u ? n : 0u;
    }
  }
  return s;
}
// Faces of a cell (on the brick faces `out`) before its minus face d.
__device__ __forceinline__ uint32_t before_minus(uint32_t flags, uint32_t out, int d) {
  uint32_t s = uint32_t(d >> 1);
  if (flags & kFlagIrregular) {
#pragma unroll
    for (int e = 0; e < d; ++e) {
      const uint32_t on = (out >> e) & 1u;
      if (e & 1) s += owns_plus(flags, e) ? on : 0u;
      else s -= (flags >> (8 + e)) & 1u ? on : 0u;
    }
  }
  return s;
}
// Does the lane's cell own its face d (d even: minus).
__device__ __forceinline__ bool owns_face(uint32_t flags, uint32_t out, int d) {
  const bool on = (out >> d) & 1u;
  if (d & 1) return owns_plus(flags, d) && on;
  return !((flags >> (8 + d)) & 1u) || !on;
}

// Number of the brick's faces (at most kBrickFaces).
constexpr uint32_t kBrickFaces = 240;
constexpr uint32_t kFaceSlots = 256;  // LDS slots per wave: four full-wave accesses
static_assert(kBrickFaces <= kFaceSlots, "a brick's faces fit their slots");
__device__ __forceinline__ uint32_t face_total(uint32_t flags) {
  uint32_t n = 192u;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    n -= (flags >> (8 + 2 * a)) & 1u ? 16u : 0u;
    n += owns_plus(flags, 2 * a + 1) ? 16u : 0u;
  }
  return n;
}
// Orders a wave's own LDS stores before its loads (lanes exchange through
// LDS; a wave's LDS accesses complete in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// p[i] at a wave-uniform index, as a scalar load
template <class T>
__device__ __forceinline__ T load_uniform(const T *p, uint32_t i) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ((const __attribute__((address_space(4))) T *)p)[i];
#else
  return p[i];  // host pass: never executed
#endif
}

struct FaceTables {
  Topo T;
  const int64_t *fbase;  // per leaf brick (device order): id of its first face
  const int32_t *canon;  // device leaf brick -> canonical leaf brick
  __device__ __forceinline__ int64_t base(uint32_t b) const { return load_uniform(fbase, b); }
};

// Local Morton index, in its own brick, of the fine cell that lane m = 4 j + s
// holds on the finer side of face d: sub-cell s (bit 0 along the lower
// in-plane axis) of the coarse face cell with interleaved in-plane index j.
// octant: of the child brick it lies in.
__device__ __forceinline__ int fine_cell(int d, int m, int &octant) {
  const int a = d >> 1, o0 = a == 0 ? 1 : 0, o1 = a == 2 ? 1 : 2;
  const int j = m >> 2;
  const int cu = (j & 1) | ((j >> 1) & 2);
  const int cv = ((j >> 1) & 1) | ((j >> 2) & 2);
  octant = ((d & 1) ? 0 : (1 << a)) | ((cu >> 1) << o0) | ((cv >> 1) << o1);
  int xyz[3];
  xyz[a] = (d & 1) ? 0 : 3;
  xyz[o0] = ((cu & 1) << 1) | (m & 1);
  xyz[o1] = ((cv & 1) << 1) | ((m >> 1) & 1);
  return dev_morton(xyz[0], xyz[1], xyz[2]);
}
// Faces of a brick with these flags before face d of its cell q (a face the
// cell owns; d a constant).  Summed before it widens: the parts may be
// negative, the sum is not.
__device__ __forceinline__ uint32_t face_slot(uint32_t flags, int q, int d) {
  int s = 3 * q + ((d + 1) >> 1);
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    int n = __popcll(face_cells(e) & ((1ull << q) - 1ull));
    if (e < d) n += dev_outside(q, e) ? 1 : 0;
    const int on = int(e & 1 ? (flags >> e | flags >> (16 + e)) : flags >> (8 + e)) & 1;
    s = e & 1 ? s + on * n : s - on * n;
  }
  return uint32_t(s);
}
// Interleaved in-plane index of cell m on a face normal to axis a: its four
// sub-faces are in lanes 4 j .. 4 j + 3 (fine_face).
__device__ __forceinline__ int face_interleaved(int m, int a) {
  const int f = dev_face_index(m, a);
  return (f & 9) | ((f & 4) >> 1) | ((f & 2) << 1);
}

// Sum over the four sub-faces of the lane's face cell, in order.
__device__ __forceinline__ double fine_sum(double v, int j) {
  double s = 0.0;
#pragma unroll
  for (int n = 0; n < 4; ++n) s = s + shfl(v, 4 * j + n);
  return s;
}

// What lies across each face the lane's cell owns, for NV canonical-order leaf
// vectors: v[k][d] the other leaf's entry (the coarser leaf's at a T-junction),
// on[d] whether that leaf is active.  Faces inside the brick are lane
// exchanges of the own entries `own`.
template <int NV>
struct AcrossFaces {
  double v[NV][6];
  bool on[6];
};
template <int NV>
__device__ __forceinline__ AcrossFaces<NV> across_faces(const FaceTables &A, const BrickMeta &M,
                                                        int m, const double *const (&x)[NV],
                                                        const double (&own)[NV]) {
  AcrossFaces<NV> R;
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    R.on[d] = false;
#pragma unroll
    for (int k = 0; k < NV; ++k) R.v[k][d] = 0.0;
    const int32_t n = M.nbr[d];
    const bool coarse = n <= dCoarseBase;
    if (coarse || (!(d & 1) && n >= 0 && uint32_t(n) < A.T.nlb)) {
      const uint32_t b = uint32_t(coarse ? dev_decode_coarse(n) : n);
      const int q = coarse ? coarse_local(M, m, d) : dev_partner(m, d);
      const uint64_t amask = act_mask(load_meta(A.T.meta, b));
      const int64_t at = int64_t(load_uniform(A.canon, b)) * 64;
      R.on[d] = (amask >> q) & 1ull;
      if (dev_outside(m, d)) {
#pragma unroll
        for (int k = 0; k < NV; ++k) R.v[k][d] = (x[k] + at)[uint32_t(q)];
      }
    }
  }
  const uint64_t amask = act_mask(M);
#pragma unroll
  for (int d = 0; d < 6; d += 2) {
    const int p = dev_partner(m, d);
    const bool inside = !dev_outside(m, d);
    R.on[d] = inside ? (amask >> p) & 1ull : R.on[d];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const double t = shfl(own[k], p);
      R.v[k][d] = inside ? t : R.v[k][d];
    }
  }
  return R;
}

// Mean of x over the active cells of the lane's sibling group (0 if none).
__device__ __forceinline__ double active_mean(const BrickMeta &M, int m, double x) {
  const uint64_t amask = act_mask(M);
  const double s = group8_sum((amask >> m) & 1ull ? x : 0.0);
  const int n = __popcll((amask >> (m & 56)) & 0xffull);
  return n ? s / double(n) : 0.0;
}

// The loop of a workgroup over groups of W bricks consecutive in Morton order
// (each XCD one contiguous eighth of the groups, as wave_loop).
struct GroupLoop {
  uint32_t first, end, step;
};
template <int W>
__device__ __forceinline__ GroupLoop group_loop(uint32_t nlb) {
  const uint32_t groups = (nlb + W - 1) / W;
  const uint32_t chunk = (groups + 7u) >> 3;
  const uint32_t lo = (blockIdx.x & 7u) * chunk;
  return {lo + (blockIdx.x >> 3), lo + chunk < groups ? lo + chunk : groups, gridDim.x >> 3};
}
constexpr int kGroupWaves = 8;

// ---------------------------------------------------------------------------
// coefficient assembly
// ---------------------------------------------------------------------------
struct AssembleArgs {
  FaceTables F;
  const double *beta;  // canonical face order
  int bc[6];
  double theta;
  double *coef;        // nlb * 256
  double *tc;          // n_tplus * 48
};

// Sides towards finer leaves: per cell on such a side the sum of its 4
// sub-face coefficients over 2, left in the cell's minus-face coefficient of
// the side's axis for k_assemble (a cell lies on at most one side per axis).
// The sub-faces are one per lane (fine_cell); the dependent loads (child ids,
// their records, the faces) are requested for all sides at once.
__global__ void __launch_bounds__(kBlock) k_assemble_fine(AssembleArgs A) {
  const uint32_t b = blockIdx.x * kWavesPerBlock + wave_id();
  const int m = threadIdx.x & (kWave - 1);
  if (b >= A.F.T.nlb) return;
  const BrickMeta M = load_meta(A.F.T.meta, b);
  if (!(M.flags & kFlagInner)) return;
  uint32_t fl[6];
  int64_t f0[6];
  int q[6];
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> (8 + d)) & 1u) {
      int o;
      q[d] = fine_cell(d, m, o);
      const uint32_t cb = uint32_t(A.F.T.child[8 * int64_t(M.nbr[d]) + o]);
      fl[d] = A.F.T.meta[cb].flags;
      f0[d] = A.F.fbase[cb];
    }
  double be[6];
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> (8 + d)) & 1u) be[d] = A.beta[f0[d] + face_slot(fl[d], q[d], d ^ 1)];
  const double hf = ldexp(1.0, -(M.level + 1));
  double *cf = A.coef + uint64_t(b) * 256u;
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> (8 + d)) & 1u) {
      const double s = fine_sum(be[d] * hf * 0.5, face_interleaved(m, d >> 1));
      if (dev_outside(m, d)) cf[(1 + (d >> 1)) * 64 + m] = s;
    }
}

// Leaf coefficients (Eq. 3): per direction the face coefficient beta S / h
// (same level or the fine side of a T-junction), beta S / (theta h) at a
// Dirichlet wall, 0 at a Neumann wall, and for a finer neighbour the sum of
// its 4 sub-face coefficients over 2; c is the sum over directions.  Laid
// out as k_divergence; the sums of a side towards finer leaves are taken
// before, by k_assemble_fine.  Moves beta once and the coefficients once (1.5
// GB at 26.3M leaves, 240 us at the copy rate); one lane per cell with tables
// of 9 bytes per cell and dependent loads took 750 us, this form with the
// sub-faces in the same kernel 760 us (their code costs every brick), the two
// 561 us.
__global__ void __launch_bounds__(kGroupWaves * kWave) k_assemble(AssembleArgs A) {
  __shared__ double slots[kGroupWaves][kFaceSlots];
  const uint32_t w = wave_id();
  const FaceLane L = face_lane();
  const GroupLoop G = group_loop<kGroupWaves>(A.F.T.nlb);
  for (uint32_t g = G.first; g < G.end; g += G.step) {
    const uint32_t b0 = g * kGroupWaves, b = b0 + w;
    const bool here = b < A.F.T.nlb;
    const BrickMeta M = load_meta(A.F.T.meta, here ? b : b0);
    const double h = ldexp(1.0, -M.level);
    const uint32_t nf = here ? face_total(M.flags) : 0u;
    const int64_t own = A.F.base(here ? b : b0);
    double bo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = uint32_t(i * kWave + L.m);
      bo[i] = k < nf ? (A.beta + own)[k] : 0.0;
    }
    // beta of the leaf beyond each plus side: in this workgroup (its slot),
    // else loaded
    double bn[3];
    uint32_t at[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int d = 2 * a + 1;
      const uint32_t n = uint32_t(M.nbr[d]);
      bn[a] = 0.0;
      at[a] = 0u;
      if (n < A.F.T.nlb) {
        const uint32_t flags = load_meta(A.F.T.meta, n).flags;
        const uint32_t k = first_slot(flags, uint32_t(dev_partner(L.m, d)), L.cntp[a]) +
                           before_minus(flags, L.out, d - 1);
        if (n - b0 < uint32_t(kGroupWaves)) at[a] = (n - b0) * kFaceSlots + k;
        else if ((L.out >> d) & 1u) bn[a] = (A.beta + A.F.base(n))[k];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) slots[w][i * kWave + L.m] = bo[i];
    __syncthreads();
    uint32_t slot = w * kFaceSlots + first_slot(M.flags, uint32_t(L.m), L.cnt);
    const double *s = &slots[0][0];
    double k[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      const int a = d >> 1;
      const bool out = (L.out >> d) & 1u;
      const bool wall = M.nbr[d] == dWall;
      double x = 0.0;
      if ((d & 1) && !owns_plus(M.flags, d)) {
        const uint32_t n = uint32_t(M.nbr[d]);
        x = (n < A.F.T.nlb && n - b0 < uint32_t(kGroupWaves) ? s[at[a]] : bn[a]) * h;
      } else if (owns_face(M.flags, L.out, d)) {
        x = s[slot++];
        x = out && wall ? (A.bc[d] == 1 ? x * (h / A.theta) : 0.0) : x * h;
      }
      if (((M.flags >> (8 + d)) & 1u) && here && out)  // k_assemble_fine's
        x = (A.coef + uint64_t(b) * 256u)[uint32_t((1 + a) * 64 + L.m)];
      if ((d & 1) && here && ((M.flags >> d) & 1u) && out)
        A.tc[uint32_t(M.tplus) * 48u + uint32_t(a * 16 + dev_face_index(L.m, a))] = x;
      k[d] = x;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double t = shfl(k[2 * a], dev_partner(L.m, 2 * a + 1));
      k[2 * a + 1] = (L.out >> (2 * a + 1)) & 1u ? k[2 * a + 1] : t;
    }
    if (here) {
      double *cf = A.coef + uint64_t(b) * 256u;
      cf[L.m] = k[0] + k[1] + k[2] + k[3] + k[4] + k[5];
      cf[64 + L.m] = k[0];
      cf[128 + L.m] = k[2];
      cf[192 + L.m] = k[4];
    }
    __syncthreads();  // the slots are read before the next group's are stored
  }
}

// Faces in canonical order: owner cell, direction, the leaf cell on the other
// side (-1 at a wall) and the kind (0 wall, 1 same level, 2 coarser).  The
// cells' entries go through LDS, so that a brick's range is stored in order
// (writes 18 bytes per face; 81M faces 880 -> 354 us against one lane storing
// its cell's faces).
__global__ void __launch_bounds__(kBlock) k_oct_faces(FaceTables F, int64_t *owner, int8_t *dir,
                                                      int64_t *other, int8_t *kind) {
  __shared__ int64_t so[kWavesPerBlock][kFaceSlots];
  __shared__ uint16_t sd[kWavesPerBlock][kFaceSlots];
  int64_t *o = so[wave_id()];
  uint16_t *e = sd[wave_id()];
  const FaceLane L = face_lane();
  const WaveLoop W = wave_loop(F.T.nlb);
  for (uint32_t b = W.first; b < W.end; b += W.step) {
    const BrickMeta M = load_meta(F.T.meta, b);
    const int64_t c0 = int64_t(load_uniform(F.canon, b)) * 64;
    uint32_t slot = first_slot(M.flags, uint32_t(L.m), L.cnt);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      if ((d & 1) && !owns_plus(M.flags, d)) continue;
      const int32_t n = M.nbr[d];
      int64_t across = -1;  // beyond the brick's face d (wave uniform parts)
      int k = 0;
      if (n <= dCoarseBase) {
        across = int64_t(load_uniform(F.canon, uint32_t(dev_decode_coarse(n)))) * 64 +
                 coarse_local(M, L.m, d);
        k = 2;
      } else if (n >= 0 && uint32_t(n) < F.T.nlb) {
        across = int64_t(load_uniform(F.canon, uint32_t(n))) * 64 + dev_partner(L.m, d);
        k = 1;
      }
      if (!owns_face(M.flags, L.out, d)) continue;
      const bool out = (L.out >> d) & 1u;
      o[slot] = out ? across : c0 + dev_partner(L.m, d);
      e[slot] = uint16_t(L.m | (d << 6) | ((out ? k : 1) << 9));
      ++slot;
    }
    wave_lds_fence();
    const int64_t f0 = F.base(b);
    const uint32_t nf = face_total(M.flags);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = uint32_t(i * kWave + L.m);
      if (k < nf) {
        const uint32_t x = e[k];
        (owner + f0)[k] = c0 + int64_t(x & 63u);
        (other + f0)[k] = o[k];
        (dir + f0)[k] = int8_t((x >> 6) & 7u);
        (kind + f0)[k] = int8_t(x >> 9);
      }
    }
    wave_lds_fence();
  }
}

// Per leaf brick: its number of faces, at its canonical position.
__global__ void k_face_counts(const BrickMeta *meta, const int32_t *canon, uint32_t nlb,
                              int64_t *count) {
  const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < nlb) count[canon[b]] = int64_t(face_total(meta[b].flags));
}
// and from their exclusive scan the id of its first face
__global__ void k_face_bases(const int32_t *canon, uint32_t nlb, const int64_t *scan,
                             int64_t *fbase) {
  const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < nlb) fbase[b] = scan[canon[b]];
}

// Per-face gradient of the adjoint: dL/dbeta_f = -lambda^T (dA/dbeta_f) p
// (canonical face and leaf order), 0 at Neumann walls and where a side of the
// face is inactive.
struct GradArgs {
  FaceTables F;
  const double *lam;
  const double *p;
  int bc[6];
  double theta;
  double *g;
};

__global__ void __launch_bounds__(kBlock) k_face_gradient(GradArgs A) {
  __shared__ double slots[kWavesPerBlock][kFaceSlots];
  double *sg = slots[wave_id()];
  const FaceLane L = face_lane();
  const int m = L.m;
  const WaveLoop W = wave_loop(A.F.T.nlb);
  for (uint32_t b = W.first; b < W.end; b += W.step) {
    const BrickMeta M = load_meta(A.F.T.meta, b);
    const int64_t brick = int64_t(load_uniform(A.F.canon, b)) * 64;
    const double *const x[2] = {A.lam, A.p};
    const double own[2] = {(A.lam + brick)[uint32_t(m)], (A.p + brick)[uint32_t(m)]};
    const AcrossFaces<2> N = across_faces<2>(A.F, M, m, x, own);
    const double h = ldexp(1.0, -M.level);
    const bool act = (act_mask(M) >> m) & 1ull;
    const double pbar = (M.flags & kFlagT) ? active_mean(M, m, own[1]) : 0.0;
    double *g = A.g + A.F.base(b);
    uint32_t slot = first_slot(M.flags, uint32_t(m), L.cnt);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      if ((d & 1) && !owns_plus(M.flags, d)) continue;
      if (!owns_face(M.flags, L.out, d)) continue;
      const bool out = (L.out >> d) & 1u;
      double r = 0.0;
      if (out && M.nbr[d] == dWall) {
        if (act && A.bc[d] == 1) r = -(h / A.theta) * own[0] * own[1];
      } else if (act && N.on[d]) {
        const bool tj = out && ((M.flags >> d) & 1u);
        const double dl = own[0] - N.v[0][d];
        r = tj ? -(h / 2.0) * dl * (pbar - N.v[1][d]) : -h * dl * (own[1] - N.v[1][d]);
      }
      sg[slot++] = r;
    }
    // a brick's faces are contiguous: whole cache lines are stored
    wave_lds_fence();
    const uint32_t nf = face_total(M.flags);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = uint32_t(i * kWave + m);
      if (k < nf) g[k] = sg[k];
    }
    wave_lds_fence();
  }
}

}  // namespace mfmg
