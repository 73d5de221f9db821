// jz_brick.hip -- one Runge-Kutta stage of a small block, brick by brick.
//
// The marching stage kernel (jz_stage_kernel.h) walks the planes of a chunk
// one after another, about 2.2 us a plane, with some four planes' worth of
// warm-up and set-up: 14 us a stage even for chunks of one plane.  Here a
// workgroup takes a brick of 8 x 8 x 4 owned nodes and computes every flux it
// needs at once, one node per thread: the 256 owned nodes and the 256 nodes
// next to its faces (twice the flux work per owned node).
//   phase 1  every thread loads its node (Q, metrics) and, for 336 of them,
//            a second one that only supplies primitives and Q (the second
//            ring, and the first ring's edges); primitives and Q to LDS
//   phase 2  fluxes, dissipation scales and sensors of the thread's node; a
//            halo node keeps those of its face's direction only
//   phase 3  residual and update: the owner of a node takes two of the five
//            variables, the thread 256 above it three
// Measured, the step of a 24 x 20 x 18 block: FP64 86 us marching, 46 us in
// bricks, FP32-flux 86 and 38 us (48 x 40 x 28 FP64: 89 and 51 us, 48 x 48 x 48
// FP32-flux: 89 and 53 us).
// What bounds it: for the smallest blocks the chain of the three phases in
// one workgroup (two waves per SIMD, one workgroup per CU in FP64), for larger
// ones the doubled flux work, which is why large blocks march.
// The arithmetic of a node is the marching kernel's (jz_node.h, and the same
// order of operations here), so the states are bitwise the same.
#include "jz_node.h"

namespace jz {

namespace {

constexpr int BI = kBrickI, BJ = kBrickJ, BK = kBrickK;   // owned nodes
constexpr int SX = BI + 4, SY = BJ + 4, SZ = BK + 4;      // with the two-node halo
constexpr int NS = SX * SY * SZ;
constexpr int NOWN = BI * BJ * BK;
constexpr int NT = 2 * NOWN;
static_assert(BI == 8 && BJ == 8 && BK == 4, "the thread roles below are for 8 x 8 x 4 bricks");
static_assert(2 * (BJ * BK + BI * BK + BI * BJ) == NOWN, "one halo thread per owned node");

// A value the compiler cannot trace to its expression: multiplications and
// additions on either side of it are not contracted, as where the marching
// kernel carries the value from one step or phase to the next.
template <typename T>
__device__ __forceinline__ T opaque(T x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Slots of a node (x, y, z counted with the halo) in the rows of the fluxes,
// scales and sensors along each direction: owned nodes and that direction's
// two halo layers.
__device__ __forceinline__ int slot_x(int x, int y, int z) { return (x - 1) + (BI + 2) * ((y - 2) + BJ * (z - 2)); }
__device__ __forceinline__ int slot_y(int x, int y, int z) { return (x - 2) + BI * ((y - 1) + (BJ + 2) * (z - 2)); }
__device__ __forceinline__ int slot_z(int x, int y, int z) { return (x - 2) + BI * ((y - 2) + BJ * (z - 1)); }
constexpr int NX = (BI + 2) * BJ * BK, NY = BI * (BJ + 2) * BK, NZ = BI * BJ * (BK + 2);

// Position of owned thread o.  The rows of a 16-lane group are two apart, so
// that with 12-slot rows its 64-bit LDS accesses fall into 16 banks.
__device__ __forceinline__ void own_pos(int o, int& x, int& y, int& z) {
  const int g = (o >> 3) & 7;
  x = 2 + (o & 7);
  y = 2 + ((g & 4) | ((g & 1) << 1) | ((g >> 1) & 1));
  z = 2 + (o >> 6);
}

// MODE bits as in stage_tile: 0 norms, 1 largest spectral radius, 3 keep the
// double update of the far-field reference planes.
template <typename Rl, typename TIn, typename TOut, bool MET32, int MODE>
__global__ __launch_bounds__(NT) void brick_kernel(StageArgs A, const int* __restrict__ flag) {
  constexpr bool NORMS = (MODE & 1) != 0;
  constexpr bool LAMMAX = (MODE & 2) != 0;
  constexpr bool KEEP_REF = (MODE & 8) != 0;
  constexpr bool Q0_IN_LDS = NORMS && std::is_same<TIn, double>::value && std::is_same<Rl, double>::value;
  const int failed = *flag;  // looked at before anything is written, so that its load holds nothing up
  __shared__ __attribute__((aligned(16))) Rl sPr[5][NS];  // u, v, w, T, p; scratch of the reductions afterwards
  __shared__ Rl sQ[5][NS];
  __shared__ Rl sFx[7][NX], sFy[7][NY], sFz[7][NZ];       // five fluxes, scale, sensor
  __shared__ double sJ[NOWN];
  __shared__ int sMap[SX + SY + SZ];                      // mapped indices of the brick's columns, rows, planes

  const Phys ph = A.ph;
  const Rl gm1 = (Rl)ph.gm1, gamma = (Rl)ph.gamma, k2 = (Rl)ph.k2, k4 = (Rl)ph.k4;
  const int t = threadIdx.x;
  const int lt = xcd_remap(blockIdx.x, gridDim.x);
  const int bx = lt % A.tiles_i, byz = lt / A.tiles_i;
  const int i0 = A.in.lo[0] + bx * BI, j0 = A.in.lo[1] + (byz % A.tiles_j) * BJ, k0 = A.in.lo[2] + (byz / A.tiles_j) * BK;
  if (t < SX + SY + SZ) {
    sMap[t] = t < SX          ? map_index(i0 - 2 + t, A.ni, A.in.bnd & 1)
              : t < SX + SY   ? map_index(j0 - 2 + t - SX, A.nj, A.in.bnd & 2)
                              : map_index(k0 - 2 + t - SX - SY, A.nk, A.in.bnd & 4);
  }
  // the thread's flux node, and the node (x2, y2, z2) it also supplies
  const bool owner = t < NOWN;
  const int o = owner ? t : t - NOWN;
  int xo, yo, zo;                 // owned node this thread (or its lower half) updates
  own_pos(o, xo, yo, zo);
  int x = xo, y = yo, z = zo, x2, y2, z2;
  const int dir = owner ? -1 : o < 64 ? 0 : o < 128 ? 1 : 2;
  const int wdir = __builtin_amdgcn_readfirstlane(dir);  // (the same for a whole wave)
  if (dir < 0) {
    // edges of the first ring: along zeta 16, eta 32, xi 32
    const int e = t < 16 ? t : t < 48 ? t - 16 : t - 48;
    const int a = (e & 1), b = (e >> 1) & 1, c = e >> 2;
    x2 = t < 48 ? (a ? BI + 2 : 1) : 2 + c;
    y2 = t < 16 ? (b ? BJ + 2 : 1) : t < 48 ? 2 + c : (a ? BJ + 2 : 1);
    z2 = t < 16 ? 2 + c : (b ? BK + 2 : 1);
  } else if (dir == 0) {
    const int hi = o >> 5;
    y = y2 = 2 + (o & 7);
    z = z2 = 2 + ((o >> 3) & 3);
    x = hi ? BI + 2 : 1;
    x2 = hi ? BI + 3 : 0;
  } else if (dir == 1) {
    const int hi = (o - 64) >> 5;
    x = x2 = 2 + (o & 7);
    z = z2 = 2 + ((o >> 3) & 3);
    y = hi ? BJ + 2 : 1;
    y2 = hi ? BJ + 3 : 0;
  } else {
    const int hi = (o - 128) >> 6;
    x = x2 = 2 + (o & 7);
    y = y2 = 2 + ((o >> 3) & 7);
    z = hi ? BK + 2 : 1;
    z2 = hi ? BK + 3 : 0;
  }
  const bool two = !owner || t < 80;
  __syncthreads();

  // ---- phase 1: loads, primitives ------------------------------------------
  auto node = [&](int nx, int ny, int nz) {
    return (long long)sMap[nx] + (long long)A.ni * (sMap[SX + ny] + (long long)A.nj * sMap[SX + SY + nz]);
  };
  const TIn* __restrict__ qin = (const TIn*)A.qin;
  const long long n1 = node(x, y, z), no = node(xo, yo, zo);
  Rl Q[5], Q2[5], m[9];
  double Jg;
#pragma unroll
  for (int v = 0; v < 5; ++v) Q[v] = (Rl)qin[5 * n1 + v];
  if (two) {
    const long long n2 = node(x2, y2, z2);
#pragma unroll
    for (int v = 0; v < 5; ++v) Q2[v] = (Rl)qin[5 * n2 + v];
  }
  MetView<MET32> met;
  met.m = (decltype(met.m))A.met;
  met.jac = A.jac;
  met.load(n1, m, Jg);
  // the variables this thread updates, and their Q(0)
  const int v0 = owner ? 0 : 2, nv = owner ? 2 : 3;
  double q0v[3];
  if constexpr (!Q0_IN_LDS) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (i < nv) q0v[i] = A.q0[5 * no + v0 + i];
  }
  const double adt = A.alpha * A.clock->dt;
  const int c = x + SX * (y + SY * z);
  Rl ctr[5];
  {
    const Prim<Rl> p = primitives(Q, gm1, gamma);
    ctr[0] = opaque(p.u);
    ctr[1] = opaque(p.v);
    ctr[2] = opaque(p.w);
    ctr[3] = opaque(p.T);
    ctr[4] = opaque(p.p);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      sPr[k][c] = ctr[k];
      sQ[k][c] = Q[k];
    }
  }
  if (two) {
    const int c2 = x2 + SX * (y2 + SY * z2);
    const Prim<Rl> p = primitives(Q2, gm1, gamma);
    const Rl pr[5] = {p.u, p.v, p.w, p.T, p.p};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      sPr[k][c2] = pr[k];
      sQ[k][c2] = Q2[k];
    }
  }
  __syncthreads();

  // ---- phase 2: fluxes, scales, sensors --------------------------------------
  {
    Rl nxm[5], nxp[5], nym[5], nyp[5], nzm[5], nzp[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      nxm[k] = sPr[k][c - 1];
      nxp[k] = sPr[k][c + 1];
      nym[k] = sPr[k][c - SX];
      nyp[k] = sPr[k][c + SX];
      nzm[k] = sPr[k][c - SX * SY];
      nzp[k] = sPr[k][c + SX * SY];
    }
    Rl F[3][5], Uc[3], asnd, sig[3], nu[3];
    node_fluxes<true>(ph, m, Jg, Q, ctr, nxm, nxp, nym, nyp, nzm, nzp, F, Uc, asnd, wdir);
    node_scales<true>(ph, m, Uc, asnd, sig);
    node_sensors(ctr[4], nxm[4], nxp[4], nym[4], nyp[4], nzm[4], nzp[4], nu);
    if (dir <= 0) {
      const int q = slot_x(x, y, z);
#pragma unroll
      for (int v = 0; v < 5; ++v) sFx[v][q] = F[0][v];
      sFx[5][q] = sig[0];
      sFx[6][q] = nu[0];
    }
    if (dir < 0 || dir == 1) {
      const int q = slot_y(x, y, z);
#pragma unroll
      for (int v = 0; v < 5; ++v) sFy[v][q] = F[1][v];
      sFy[5][q] = sig[1];
      sFy[6][q] = nu[1];
    }
    if (dir < 0 || dir == 2) {
      const int q = slot_z(x, y, z);
#pragma unroll
      for (int v = 0; v < 5; ++v) sFz[v][q] = F[2][v];
      sFz[5][q] = sig[2];
      sFz[6][q] = nu[2];
    }
    if (owner) sJ[o] = Jg;
  }
  __syncthreads();

  if (failed) return;  // a failed step froze the state

  // ---- phase 3: residual and update of variables [v0, v0 + nv) ----------------
  const int co = xo + SX * (yo + SY * zo);
  const int qx = slot_x(xo, yo, zo), qy = slot_y(xo, yo, zo), qz = slot_z(xo, yo, zo);
  constexpr int DX = 1, DY = BI, DZ = BI * BJ;   // neighbours in the flux rows
  const bool mine = i0 + xo - 2 < A.in.hi[0] && j0 + yo - 2 < A.in.hi[1] && k0 + zo - 2 < A.in.hi[2];
  const double J = sJ[o];
  double qn[3] = {0, 0, 0}, rs[3] = {0, 0, 0}, rm[3] = {0, 0, 0};
  {
    Rl e2xp, e4xp, sgxp, e2xm, e4xm, sgxm, e2yp, e4yp, sgyp, e2ym, e4ym, sgym, e2zp, e4zp, sgzp, e2zm, e4zm, sgzm;
    face_coefs(k2, k4, sFx[6][qx], sFx[6][qx + DX], sFx[5][qx], sFx[5][qx + DX], e2xp, e4xp, sgxp);
    face_coefs(k2, k4, sFx[6][qx - DX], sFx[6][qx], sFx[5][qx - DX], sFx[5][qx], e2xm, e4xm, sgxm);
    face_coefs(k2, k4, sFy[6][qy], sFy[6][qy + DY], sFy[5][qy], sFy[5][qy + DY], e2yp, e4yp, sgyp);
    face_coefs(k2, k4, sFy[6][qy - DY], sFy[6][qy], sFy[5][qy - DY], sFy[5][qy], e2ym, e4ym, sgym);
    face_coefs(k2, k4, sFz[6][qz], sFz[6][qz + DZ], sFz[5][qz], sFz[5][qz + DZ], e2zp, e4zp, sgzp);
    face_coefs(k2, k4, sFz[6][qz - DZ], sFz[6][qz], sFz[5][qz - DZ], sFz[5][qz], e2zm, e4zm, sgzm);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (i >= nv) break;
      const int v = v0 + i;
      const Rl* q = &sQ[v][co];
      const Rl q0 = q[0], qxm = q[-1], qxmm = q[-2], qxp = q[1], qxpp = q[2];
      const Rl qym = q[-SX], qymm = q[-2 * SX], qyp = q[SX], qypp = q[2 * SX];
      const Rl qzm = q[-SX * SY], qzmm = q[-2 * SX * SY], qzp = q[SX * SY], qzpp = q[2 * SX * SY];
      const Rl fxm = sFx[v][qx - DX], fxp = sFx[v][qx + DX], fym = sFy[v][qy - DY], fyp = sFy[v][qy + DY];
      const Rl fzm = sFz[v][qz - DZ], fz0 = sFz[v][qz], fzp = sFz[v][qz + DZ];
      const Rl dxp = face_diss(e2xp, e4xp, sgxp, qxm, q0, qxp, qxpp);
      const Rl dxm = face_diss(e2xm, e4xm, sgxm, qxmm, qxm, q0, qxp);
      const Rl dyp = face_diss(e2yp, e4yp, sgyp, qym, q0, qyp, qypp);
      const Rl dym = face_diss(e2ym, e4ym, sgym, qymm, qym, q0, qyp);
      const Rl cx = Rl(0.5) * (fxp - fxm);
      const Rl cy = Rl(0.5) * (fyp - fym);
      const Rl Rr = (cx + cy) - ((dxp - dxm) + (dyp - dym));
      // the zeta faces below and above
      const Rl Hm = opaque(Rl(0.5) * (fzm + fz0) - face_diss(e2zm, e4zm, sgzm, qzmm, qzm, q0, qzp));
      const Rl Hp = opaque(Rl(0.5) * (fz0 + fzp) - face_diss(e2zp, e4zp, sgzp, qzm, q0, qzp, qzpp));
      const Rl acc = opaque(Rr - Hm);
      const double R = J * (double)(acc + Hp);
      if constexpr (Q0_IN_LDS) qn[i] = (double)q0 - adt * R;
      else qn[i] = q0v[i] - adt * R;
      if (mine) {
        ((TOut*)A.qout)[5 * no + v] = (TOut)qn[i];
        if (NORMS) {
          rs[i] = R * R;
          rm[i] = fabs(R);
        }
        if constexpr (KEEP_REF) {
          // a node on a far-field reference plane also keeps its double
          // update (see StageArgs::ref)
          const int ci[3] = {i0 + xo - 2, j0 + yo - 2, k0 + zo - 2};
          const int nn[3] = {A.ni, A.nj, A.nk};
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            if (A.ref_off[d] < 0) continue;
            const int e = face_e(d), f = face_f(d);
            const long long face = (long long)nn[e] * nn[f], at = ci[e] + (long long)nn[e] * ci[f];
#pragma unroll
            for (int side = 0; side < 2; ++side)
              if (ci[d] == (side ? nn[d] - 3 : 2)) A.ref[5 * (A.ref_off[d] + side * face + at) + v] = qn[i];
          }
        }
      }
    }
  }

  // ---- fixed-order reductions over the brick --------------------------------
  if constexpr (NORMS) {
    double(*red)[6] = reinterpret_cast<double(*)[6]>(&sPr[0][0]);  // a row per wave
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double sv = wave_sum(rs[i]), mv = wave_max(rm[i]);
      if ((t & 63) == 63) {
        red[t >> 6][i] = sv;
        red[t >> 6][3 + i] = mv;
      }
    }
    __syncthreads();
    if (t < 5) {
      const int w = t < 2 ? 0 : 4, i = t < 2 ? t : t - 2;
      double sv = red[w][i], mv = red[w][3 + i];
      for (int k = 1; k < 4; ++k) {
        sv += red[w + k][i];
        mv = max_nan(mv, red[w + k][3 + i]);
      }
      A.norm_part[(long long)lt * 10 + t] = sv;
      A.norm_part[(long long)lt * 10 + 5 + t] = mv;
    }
  }
  if constexpr (LAMMAX) {
    double* up = reinterpret_cast<double*>(&sPr[0][0]);   // the upper three variables' updates
    double* red = up + 3 * NOWN;
    if (!owner) {
#pragma unroll
      for (int i = 0; i < 3; ++i) up[i * NOWN + o] = qn[i];
    }
    __syncthreads();
    if (owner) {
      double lam = 0.0;
      if (mine) {
        const double qf[5] = {qn[0], qn[1], up[o], up[NOWN + o], up[2 * NOWN + o]};
        lam = lambda_sum(qf, m, J, ph.gamma);
      }
      lam = wave_max(lam);
      if ((t & 63) == 63) red[t >> 6] = lam;
    }
    __syncthreads();
    if (t == 0) A.lam_part[lt] = max_nan(max_nan(red[0], red[1]), max_nan(red[2], red[3]));
  }
}

}  // namespace

// One stage over the bricks of a block that allows the FAST form: stage 0
// writes the norm partials of its bricks, the last one (last) the spectral
// radii.  At least two stages.
hipError_t launch_brick(const StageArgs& a, bool f32, const int* flag, int stage, bool last, int nbricks, hipStream_t st) {
  const dim3 grid(nbricks), block(NT);
  if (!f32) {
    if (stage == 0) hipLaunchKernelGGL((brick_kernel<double, double, double, false, 1>), grid, block, 0, st, a, flag);
    else if (last) hipLaunchKernelGGL((brick_kernel<double, double, double, false, 2>), grid, block, 0, st, a, flag);
    else hipLaunchKernelGGL((brick_kernel<double, double, double, false, 0>), grid, block, 0, st, a, flag);
  } else if (stage == 0) {
    if (a.ref) hipLaunchKernelGGL((brick_kernel<float, double, float, true, 9>), grid, block, 0, st, a, flag);
    else hipLaunchKernelGGL((brick_kernel<float, double, float, true, 1>), grid, block, 0, st, a, flag);
  } else if (last) {
    hipLaunchKernelGGL((brick_kernel<float, float, double, true, 2>), grid, block, 0, st, a, flag);
  } else {
    if (a.ref) hipLaunchKernelGGL((brick_kernel<float, float, float, true, 8>), grid, block, 0, st, a, flag);
    else hipLaunchKernelGGL((brick_kernel<float, float, float, true, 0>), grid, block, 0, st, a, flag);
  }
  return hipGetLastError();
}

}  // namespace jz
