// jz_node.h -- arithmetic of one node, shared by every kernel that evaluates
// the residual (the marching stage kernel, its batch form and the brick
// kernel), so that a node's result does not depend on which of them computed
// it: primitives, the three contravariant fluxes, the dissipation scales and
// pressure sensors, and the face terms.
#pragma once

#include <type_traits>
#include "jz_internal.h"

namespace jz {

namespace {

template <typename Rl>
struct Prim {
  Rl u, v, w, T, p;
};

template <typename Rl>
__device__ inline Prim<Rl> primitives(const Rl q[5], Rl gm1, Rl gamma) {
  Prim<Rl> r;
  const Rl rinv = rcp_pos(q[0]);
  r.u = q[1] * rinv;
  r.v = q[2] * rinv;
  r.w = q[3] * rinv;
  r.p = gm1 * (q[4] - Rl(0.5) * q[0] * (r.u * r.u + r.v * r.v + r.w * r.w));
  r.T = gamma * r.p * rinv;
  return r;
}

// J^(-1/3) (the filter width of a cell of volume 1/J): float seed from the
// hardware log2/exp2, then two Newton steps r <- r + r (1 - J r^3) / 3 in FP64,
// which square the relative error twice (1e-7 -> 1e-14 -> below rounding).
__device__ inline double inv_cbrt(double J) {
  const float jf = (float)J;
  double r = (double)__builtin_amdgcn_exp2f(-__builtin_amdgcn_logf(jf) * (1.0f / 3.0f));
  r = r + r * (1.0 - J * r * r * r) * (1.0 / 3.0);
  r = r + r * (1.0 - J * r * r * r) * (1.0 / 3.0);
  return r;
}

// J^(-1/3) in float: hardware log2/exp2 seed and one Newton step
__device__ inline float inv_cbrt(float J) {
  float r = __builtin_amdgcn_exp2f(-__builtin_amdgcn_logf(J) * (1.0f / 3.0f));
  return r + r * (1.0f - J * r * r * r) * (1.0f / 3.0f);
}

// Contravariant fluxes F[d] of a node (ONE: of direction only alone, if it is
// not negative; the others are left unset), the contravariant velocities Uc[d] and
// the sound speed, from its metrics m and J, its conserved variables Q and
// the primitives (u, v, w, T, p) of the node (ctr) and of its six neighbours.
template <bool ONE = false, typename Rl>
__device__ __forceinline__ void node_fluxes(const Phys& ph, const Rl m[9], double Jg, const Rl Q[5], const Rl ctr[5],
                                            const Rl nxm[5], const Rl nxp[5], const Rl nym[5], const Rl nyp[5],
                                            const Rl nzm[5], const Rl nzp[5], Rl F[3][5], Rl Uc[3], Rl& asnd,
                                            int only = -1) {
  const Rl J = (Rl)Jg;
  // chain rule d phi / d x_a = J sum_d S^d_a delta_d phi, with the 1/2 of
  // the centred difference folded into the metric factor
  Rl hm[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) hm[k] = (Rl(0.5) * J) * m[k];
  Rl gr[4][3];  // gr[q][a] = d phi_q / d x_a for phi = u, v, w, T
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const Rl dxi = nxp[q] - nxm[q];
    const Rl deta = nyp[q] - nym[q];
    const Rl dzeta = nzp[q] - nzm[q];
#pragma unroll
    for (int a = 0; a < 3; ++a) gr[q][a] = hm[a] * dxi + hm[3 + a] * deta + hm[6 + a] * dzeta;
  }
  const Rl uu[3] = {ctr[0], ctr[1], ctr[2]};
  const Rl T = ctr[3], p = ctr[4];
  asnd = sqrt_pos(T);
  const Rl mu = div_pos((Rl)ph.mu_suth * T * asnd, T + (Rl)ph.suth_s);
  // Smagorinsky: |S| = sqrt(2 S_ab S_ab), Delta = J^(-1/3)
  const Rl s01 = gr[0][1] + gr[1][0], s02 = gr[0][2] + gr[2][0], s12 = gr[1][2] + gr[2][1];
  const Rl ss2 = Rl(2) * (gr[0][0] * gr[0][0] + gr[1][1] * gr[1][1] + gr[2][2] * gr[2][2]) +
                 (s01 * s01 + s02 * s02 + s12 * s12);
  const Rl smag = ss2 > Rl(0) ? sqrt_pos(ss2) : Rl(0);
  const Rl delta = inv_cbrt(J);
  const Rl mut = Q[0] * (Rl)ph.cs2 * delta * delta * smag;
  const Rl kap = (Rl)ph.kap_lam * mu + (Rl)ph.kap_turb * mut;
  const Rl mue = mu + mut;
  const Rl div23 = (Rl(2) / Rl(3)) * (gr[0][0] + gr[1][1] + gr[2][2]);
  // Fhat^d = S^d . (E - V) for each direction d: the inviscid part through
  // the contravariant velocity U^d = S^d . u (rho U, rho u_r U + S^d_r p,
  // (e + p) U), the viscous part through the symmetric stress tensor and
  // the energy column w_a = u_r tau_ra - q_a (q_a = -kappa dT/dx_a).
  // Every multiply-add is an explicit fma and nothing else is contracted,
  // so that each instantiation of this code (shapes, stages, kernels)
  // rounds the same way and their results stay bitwise equal.
  {
#pragma clang fp contract(off)
    const Rl txx = mue * fma(Rl(2), gr[0][0], -div23), tyy = mue * fma(Rl(2), gr[1][1], -div23);
    const Rl tzz = mue * fma(Rl(2), gr[2][2], -div23);
    const Rl txy = mue * s01, txz = mue * s02, tyz = mue * s12;
    const Rl tau[3][3] = {{txx, txy, txz}, {txy, tyy, tyz}, {txz, tyz, tzz}};
    Rl wv[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
      wv[a] = fma(kap, gr[3][a], fma(uu[2], tau[2][a], fma(uu[1], tau[1][a], uu[0] * tau[0][a])));
    const Rl ep = Q[4] + p;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const Rl sx = m[3 * d], sy = m[3 * d + 1], sz = m[3 * d + 2];
      const Rl U = fma(sz, uu[2], fma(sy, uu[1], sx * uu[0]));
      Uc[d] = U;
      if (ONE && only >= 0 && only != d) continue;
      F[d][0] = Q[0] * U;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const Rl vis = fma(sz, tau[r][2], fma(sy, tau[r][1], sx * tau[r][0]));
        F[d][1 + r] = fma(Q[1 + r], U, fma(m[3 * d + r], p, -vis));
      }
      F[d][4] = fma(ep, U, -fma(sz, wv[2], fma(sy, wv[1], sx * wv[0])));
    }
  }
}

// Spectral radii and anisotropic dissipation scales.  With lambda^d = J L^d,
// L^d = |U^d| + a |S^d|, the scale sigma^d = phi^d lambda^d / J = phi^d L^d
// (phi depends only on ratios of the radii), so J drops out.  The exponent
// 1/2 (HALF) has square roots only; any other takes six calls of pow, whose
// inlined code costs a kernel registers even where it is never executed, so
// the two are separate instantiations (512 x 256 x 256: 39 SGPR
// restores less per plane of an FP64 middle stage, step with its read-back
// 10.45 -> 10.35 ms, FP32-flux 6.33 -> 6.27 ms; 3 % on a 24 x 20 x 18 block).
template <bool HALF, typename Rl>
__device__ __forceinline__ void node_scales(const Phys& ph, const Rl m[9], const Rl Uc[3], Rl asnd, Rl sig[3]) {
  Rl lam[3];  // L^d
#pragma unroll
  for (int d = 0; d < 3; ++d) {
#pragma clang fp contract(off)
    const Rl sx = m[3 * d], sy = m[3 * d + 1], sz = m[3 * d + 2];
    lam[d] = fma(asnd, sqrt_pos(fma(sz, sz, fma(sy, sy, sx * sx))), fabs(Uc[d]));
  }
  if (HALF || ph.alpha_half) {  // (the general kernel of a mixed batch serves both)
    // phi^d L^d = L^d + sum_{e != d} sqrt(L^e L^d) = sqrt(L^d) sum_e sqrt(L^e)
    const Rl r0 = sqrt_pos(lam[0]), r1 = sqrt_pos(lam[1]), r2 = sqrt_pos(lam[2]);
    const Rl rs = r0 + r1 + r2;
    sig[0] = r0 * rs;
    sig[1] = r1 * rs;
    sig[2] = r2 * rs;
  } else {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      Rl phi = 1;
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (e != d) phi += (Rl)pow((double)lam[e] / (double)lam[d], ph.tv_alpha);
      sig[d] = phi * lam[d];
    }
  }
}

// Pressure sensors |p+ - 2p + p-| / (p+ + 2p + p-) along xi, eta, zeta, the
// three divisions through one reciprocal of the product of the (positive)
// denominators.
template <typename Rl>
__device__ __forceinline__ void node_sensors(Rl p, Rl pxm, Rl pxp, Rl pym, Rl pyp, Rl pzm, Rl pzp, Rl nu[3]) {
  const Rl ax = fabs(pxp - Rl(2) * p + pxm), bx = pxp + Rl(2) * p + pxm;
  const Rl ay = fabs(pyp - Rl(2) * p + pym), by = pyp + Rl(2) * p + pym;
  const Rl az = fabs(pzp - Rl(2) * p + pzm), bz = pzp + Rl(2) * p + pzm;
  const Rl byz = by * bz, r = rcp_pos(bx * byz);
  nu[0] = ax * byz * r;
  nu[1] = ay * (bx * bz) * r;
  nu[2] = az * (bx * by) * r;
}

// Coefficients of the dissipation at the face between nodes a and b, from
// their sensors and scales: e2 (second difference), e4 (fourth), sg.
template <typename Rl>
__device__ __forceinline__ void face_coefs(Rl k2, Rl k4, Rl nua, Rl nub, Rl sga, Rl sgb, Rl& e2, Rl& e4, Rl& sg) {
  e2 = k2 * fmax(nua, nub);
  e4 = fmax(Rl(0), k4 - e2);
  sg = Rl(0.5) * (sga + sgb);
}

// Dissipation at the face between q0 and qp (qm before q0, qpp after qp).
template <typename Rl>
__device__ __forceinline__ Rl face_diss(Rl e2, Rl e4, Rl sg, Rl qm, Rl q0, Rl qp, Rl qpp) {
  return sg * (e2 * (qp - q0) - e4 * ((qpp - qm) - Rl(3) * (qp - q0)));
}

}  // namespace

}  // namespace jz
