// Projection of a face velocity field around the solve (Section 2.1's flux
// form of the pressure equation; the static projection test of Section 4.4):
// the integrated divergence of MAC face velocities weighted by the faces'
// fluid fractions (the solve's right-hand side), the velocity update with the
// operator's own face fluxes, and the volume-weighted RMS of a divergence
// (Section 4.2).
//
// Velocities u_f are normal components along the + axis of each canonical
// face; a face's fluid area is beta_f h_o^2 (h_o of its owner, the finer
// side).  With the pressure flux
//   F_f = k_f (p_o - p_t)               same level,
//   F_f = k_f (mean of p over the active siblings of o - p_t) / 2
//                                       T-junction (o the fine owner),
//   F_f = k_f p_o                       Dirichlet wall (k_f = beta h / theta),
//   F_f = 0                             Neumann wall or an inactive side,
// (A p)_i sums +F_f over the faces leaf i owns and -F_f over the others, and
// u_f <- u_f - s_o F_f / (beta_f h_o^2) (s_o = +1 where the + axis points out
// of the owner) makes div(u_new) = div(u) - A p.
#pragma once

#include "face_kernels.hpp"
#include "pcg_kernels.hpp"

namespace mfmg {

struct DivArgs {
  FaceTables F;
  const double *beta;     // canonical face order
  const double *u;        // canonical face order
  double *div;            // canonical leaf order
};

// One wave per leaf brick, one lane per cell: the outflow through each of its
// six sides except those towards finer leaves, summed in direction order.  A
// brick's own faces are loaded in order and their flows handed to the cells
// through LDS; the flow through a plus face inside the brick is the neighbour
// lane's minus face's.  A plus side reads the neighbour brick's minus faces,
// which lie in two thirds of the cache lines of its whole range, so a
// workgroup takes eight bricks consecutive in Morton order and half of these
// neighbours' flows come from its LDS.
__global__ void __launch_bounds__(kGroupWaves * kWave) k_divergence(DivArgs A) {
  __shared__ double slots[kGroupWaves][kFaceSlots];
  const uint32_t w = wave_id();
  const FaceLane L = face_lane();
  const GroupLoop G = group_loop<kGroupWaves>(A.F.T.nlb);
  for (uint32_t g = G.first; g < G.end; g += G.step) {
    const uint32_t b0 = g * kGroupWaves;
    const uint32_t b = b0 + w;
    const bool here = b < A.F.T.nlb;
    BrickMeta M = load_meta(A.F.T.meta, here ? b : b0);
    const double h = ldexp(1.0, -M.level);
    const double h2 = h * h;
    double be[3] = {0.0, 0.0, 0.0}, uu[3] = {0.0, 0.0, 0.0};
    const uint32_t nf = here ? face_total(M.flags) : 0u;
    const int64_t own = A.F.base(here ? b : b0);
    double bo[4], uo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = uint32_t(i * kWave + L.m);
      bo[i] = k < nf ? (A.beta + own)[k] : 0.0;
      uo[i] = k < nf ? (A.u + own)[k] : 0.0;
    }
    // the leaf beyond each plus side: in this workgroup (its slot), else loaded
    uint32_t at[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int d = 2 * a + 1;
      const uint32_t n = uint32_t(M.nbr[d]);
      at[a] = 0u;
      if (n < A.F.T.nlb) {
        const uint32_t flags = load_meta(A.F.T.meta, n).flags;
        const uint32_t k = first_slot(flags, uint32_t(dev_partner(L.m, d)), L.cntp[a]) +
                           before_minus(flags, L.out, d - 1);
        if (n - b0 < uint32_t(kGroupWaves)) {
          at[a] = (n - b0) * kFaceSlots + k;
        } else if ((L.out >> d) & 1u) {
          const int64_t f0 = A.F.base(n);
          be[a] = (A.beta + f0)[k];
          uu[a] = (A.u + f0)[k];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) slots[w][i * kWave + L.m] = bo[i] * h2 * uo[i];
    __syncthreads();
    double div = 0.0;
    uint32_t slot = w * kFaceSlots + first_slot(M.flags, uint32_t(L.m), L.cnt);
    const double *s = &slots[0][0];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int d = 2 * a + 1;
      const bool out = (L.out >> d) & 1u;
      double f = 0.0;
      if (owns_face(M.flags, L.out, d - 1)) f = s[slot++];
      double t = shfl(f, dev_partner(L.m, d));
      if (out) {
        const uint32_t n = uint32_t(M.nbr[d]);
        if (owns_plus(M.flags, d)) t = s[slot++];
        else if (n < A.F.T.nlb && n - b0 < uint32_t(kGroupWaves)) t = s[at[a]];
        else t = be[a] * h2 * uu[a];
      }
      div = div - f + t;
    }
    if (here) (A.div + int64_t(load_uniform(A.F.canon, b)) * 64)[uint32_t(L.m)] = div;
    __syncthreads();  // the slots are read before the next group's are stored
  }
}

// The sides towards finer leaves, added on the bricks that have any (one wave
// per leaf brick; in k_divergence itself they cost every brick their
// registers: 1125 us together): each face's 64 sub-faces are one per lane
// (fine_cell), and each face cell adds its four in order.  The dependent
// loads (child ids, their records, the faces) are requested for all sides at
// once.
__global__ void __launch_bounds__(kBlock) k_divergence_fine(DivArgs A) {
  const uint32_t b = blockIdx.x * kWavesPerBlock + wave_id();
  const int m = threadIdx.x & (kWave - 1);
  if (b >= A.F.T.nlb) return;
  const BrickMeta M = load_meta(A.F.T.meta, b);
  if (!(M.flags & kFlagInner)) return;
  uint32_t flags[6];
  int64_t f0[6];
  int q[6];
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> (8 + d)) & 1u) {
      int o;
      q[d] = fine_cell(d, m, o);
      const uint32_t cb = uint32_t(A.F.T.child[8 * int64_t(M.nbr[d]) + o]);
      flags[d] = A.F.T.meta[cb].flags;
      f0[d] = A.F.fbase[cb];
    }
  double be[6], uu[6];
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> (8 + d)) & 1u) {
      const int64_t f = f0[d] + face_slot(flags[d], q[d], d ^ 1);
      be[d] = A.beta[f];
      uu[d] = A.u[f];
    }
  double *div = A.div + int64_t(load_uniform(A.F.canon, b)) * 64 + m;
  const double hf = ldexp(1.0, -(M.level + 1));
  const double hf2 = hf * hf;
  double sum = *div;
#pragma unroll
  for (int d = 0; d < 6; ++d)
    if ((M.flags >> (8 + d)) & 1u) {
      const double s = fine_sum(be[d] * hf2 * uu[d], face_interleaved(m, d >> 1));
      sum = sum + (dev_outside(m, d) ? ((d & 1) ? s : -s) : 0.0);
    }
  *div = sum;
}

struct FluxArgs {
  FaceTables F;
  const double *beta;
  const double *p;               // canonical leaf order
  int bc[6];
  double theta;
  double *u;                     // canonical face order, updated in place
};

// One wave per leaf brick: u_f -= s_o F_f / (beta_f h_o^2) on the faces its
// cells own.  F_f is proportional to beta_f, so the step is the pressure
// difference over the cell size (a multiplication by a power of two), halved
// at a T-junction and over theta at a wall.
// The faces are loaded and stored in order, the cells' steps going through LDS.
__global__ void __launch_bounds__(kBlock) k_project_velocity(FluxArgs A) {
  __shared__ double slots[kWavesPerBlock][kFaceSlots];
  double *sq = slots[wave_id()];
  const FaceLane L = face_lane();
  const double inv_theta = 1.0 / A.theta;
  const WaveLoop W = wave_loop(A.F.T.nlb);
  for (uint32_t b = W.first; b < W.end; b += W.step) {
    const BrickMeta M = load_meta(A.F.T.meta, b);
    const double *const x[1] = {A.p};
    const double po[1] = {
        (A.p + int64_t(load_uniform(A.F.canon, b)) * 64)[uint32_t(L.m)]};
    const int64_t f0 = A.F.base(b);
    const uint32_t nf = face_total(M.flags);
    double beta[4], u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = uint32_t(i * kWave + L.m);
      beta[i] = k < nf ? (A.beta + f0)[k] : 0.0;
      u[i] = k < nf ? (A.u + f0)[k] : 0.0;
    }
    const AcrossFaces<1> N = across_faces<1>(A.F, M, L.m, x, po);
    const double inv_h = ldexp(1.0, M.level);
    const bool act = (act_mask(M) >> L.m) & 1ull;
    const double pbar = (M.flags & kFlagT) ? active_mean(M, L.m, po[0]) : 0.0;
    uint32_t slot = first_slot(M.flags, uint32_t(L.m), L.cnt);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      if ((d & 1) && !owns_plus(M.flags, d)) continue;
      const bool out = (L.out >> d) & 1u;
      double q = 0.0;
      if (act && N.on[d]) q = (po[0] - N.v[0][d]) * inv_h;
      if (M.nbr[d] == dWall) {
        const double w = act && A.bc[d] == 1 ? po[0] * inv_theta * inv_h : 0.0;
        q = out ? w : q;
      } else if ((M.flags >> d) & 1u) {
        const double w = act && N.on[d] ? (pbar - N.v[0][d]) * (0.5 * inv_h) : 0.0;
        q = out ? w : q;
      }
      if (owns_face(M.flags, L.out, d)) sq[slot++] = (d & 1) ? -q : q;
    }
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = uint32_t(i * kWave + L.m);
      if (k < nf && beta[i] > 0.0) (A.u + f0)[k] = u[i] + sq[k];
    }
    wave_lds_fence();
  }
}

// Parts of RMS_V over the active leaves of a canonical-order divergence: the
// partials of the sum of div_i^2 / V_i (= V_i (div_i / V_i)^2) go to
// P.partials, those of the sum of V_i to `vol`.
__global__ void __launch_bounds__(kBlock) k_div_rms_part(PcgArgs P, const double *div,
                                                         double *vol) {
  double part = 0.0, vpart = 0.0;
  LEAF_LOOP(P) {
    const BrickMeta M = load_meta(P.T.meta, b);
    if ((act_mask(M) >> m) & 1ull) {
      double V = ldexp(1.0, -3 * M.level);
      double x = div[int64_t(P.canon[b]) * 64 + m];
      part += x * x / V;
      vpart += V;
    }
  }
  block_partial(part, P.partials);
  __syncthreads();  // block_partial's shared slots are read before they change
  block_partial(vpart, vol);
}

}  // namespace mfmg
