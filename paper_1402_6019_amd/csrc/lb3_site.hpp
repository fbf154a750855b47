// Per-site pieces of the 3-D step shared by its default kernels (lb3_march.hip, lb3_split.hip): the
// pull offsets of a site, its parameters, and the update with its outputs, operation for operation
// that of lb3_kernels.hip.
#pragma once

#include "lb3_internal.hpp"
#include "lb3_stencil.hpp"
#include "lb_step.hpp"

namespace lb355 {

// Where a site's pulls come from, relative to a z-plane: lane offsets of the source rows y - 1, y,
// y + 1 (index cy: source row y - c_y) and columns, and whether the rows beside it are walls.
struct Pull3 {
  uint32_t row[3], col[3];  // [1 + c]: source row y - c / column x - c
  bool lo, hi;
};

template <bool WALLS>
__device__ __forceinline__ Pull3 pull3_at(int x, int y, int lx, int ly, uint32_t row_b, uint32_t site_b) {
  Pull3 p;
  p.lo = WALLS && y == 0;
  p.hi = WALLS && y == ly - 1;
  p.row[1] = (uint32_t)y * row_b;
  p.row[2] = y == 0 ? (uint32_t)(ly - 1) * row_b : p.row[1] - row_b;
  p.row[0] = y == ly - 1 ? 0u : p.row[1] + row_b;
  p.col[1] = (uint32_t)x * site_b;
  p.col[2] = x == 0 ? (uint32_t)(lx - 1) * site_b : p.col[1] - site_b;
  p.col[0] = x == lx - 1 ? 0u : p.col[1] + site_b;
  return p;
}

// Pulls of a site of plane z: f_l = f*_l(x - c_l), or f*_opp(l)(x) off a wall; rz: descriptors of planes
// z + 1, z, z - 1.  Beside a wall the two links that leave it diagonally in z come from the site's
// own plane instead of a neighbouring one, which a lane offset cannot say: they are loaded apart,
// into fb (zeros without traffic for every other site), and wall_fix3 puts them in place once
// loaded.  off: a lane offset past the descriptors' range, where loads give zeros, stores are dropped and
// neither moves bytes: the bytes of a z-plane, as no constant below 4 GiB is past every plane.
template <class C, int NS, bool WALLS>
__device__ __forceinline__ void pull3(const Rsrc (&rz)[3], const Pull3 &q, uint32_t plane_b, uint32_t off,
                                      typename C::R (&f)[NS][19], typename C::R (&fb)[NS][2]) {
  using R = typename C::R;
  auto load = [&](const Rsrc &r, uint32_t vo, uint32_t so, R &f0, R &f1) {
    if (NS == 2) C::bload2(r, vo, so, f0, f1);
    else f0 = C::bload(r, vo, so);
  };
  const uint32_t here = q.row[1] + q.col[1];
#pragma unroll
  for (int l = 0; l < 19; ++l) {
    const int cx = d3::cx(l), cy = d3::cy(l), cz = d3::cz(l);
    const uint32_t direct = q.row[1 + cy] + q.col[1 + cx];
    if (WALLS && cy != 0 && cz == 0)
      load(rz[1], (cy > 0 ? q.lo : q.hi) ? here + (uint32_t)d3::opp(l) * plane_b : direct + (uint32_t)l * plane_b, 0u,
           f[0][l], f[NS - 1][l]);
    else
      load(rz[1 + cz], direct, uni((uint32_t)l * plane_b), f[0][l], f[NS - 1][l]);
  }
  if constexpr (WALLS) {  // links 15, 17 off the lower wall, 16, 18 off the upper one
    load(rz[1], q.lo ? here + 16 * plane_b : (q.hi ? here + 15 * plane_b : off), 0u, fb[0][0], fb[NS - 1][0]);
    load(rz[1], q.lo ? here + 18 * plane_b : (q.hi ? here + 17 * plane_b : off), 0u, fb[0][1], fb[NS - 1][1]);
  }
}

template <bool WALLS, typename R, int NS>
__device__ __forceinline__ void wall_fix3(const Pull3 &q, const R (&fb)[NS][2], R (&f)[NS][19]) {
  if constexpr (WALLS) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      f[s][15] = q.lo ? fb[s][0] : f[s][15];
      f[s][17] = q.lo ? fb[s][1] : f[s][17];
      f[s][16] = q.hi ? fb[s][0] : f[s][16];
      f[s][18] = q.hi ? fb[s][1] : f[s][18];
    }
  }
}

// Parameters of a lattice in the arithmetic type.
template <typename R, int NS>
struct Site3 {
  R K[NS][7], tau[NS], om[NS], rref[NS], psiw[NS], rhow[NS], T1, T2, gx, gy, gz, psi0, nirho0;
  __device__ explicit Site3(const Lb3Args &a) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
      for (int q = 0; q < 7; ++q) K[s][q] = R(a.K[s][q]);
      tau[s] = R(a.tau[s]);
      om[s] = R(a.omega[s]);
      rref[s] = R(a.rho_ref[s]);
      psiw[s] = R(a.psi_w[s]);
      rhow[s] = R(a.rho_w[s]);
    }
    T1 = R(a.T[0]);
    T2 = R(a.T[1]);
    gx = R(a.body[0]);
    gy = R(a.body[1]);
    gz = R(a.body[2]);
    psi0 = R(a.psi0);
    nirho0 = R(-a.irho0);
  }
};

// Force and outputs of site (x, y, z) from its pulled populations f and its neighbours' psi(dx, dy,
// dz) and xr(dx, dy, dz) (rho or psi): the post-collision populations to lane offset `at` of rd
// (WHAT_STEP) or the moments (WHAT_MOMENTS) where site_ok.
template <class C, int NS, int WHAT, int STP, typename PSI, typename XR>
__device__ __forceinline__ void site3_update(const Lb3Args &a, const Site3<typename C::R, NS> &p,
                                             const typename C::R (&f)[NS][19], const PSI &psi, const XR &xr, int x, int y,
                                             int z, bool site_ok, const Rsrc rd, uint32_t at, uint32_t plane_b) {
  using R = typename C::R;
  using V = Vec<R, NS>;
  R drho[NS], rho[NS], jx[NS], jy[NS], jz[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    R sum = f[s][0];
#pragma unroll
    for (int l = 1; l < 19; ++l) sum += f[s][l];
    drho[s] = sum;
    rho[s] = p.rref[s] + sum;
    jx[s] = ((f[s][1] + f[s][7]) + (f[s][9] + f[s][11]) + f[s][13]) -
            ((f[s][2] + f[s][8]) + (f[s][10] + f[s][12]) + f[s][14]);
    jy[s] = ((f[s][3] + f[s][7]) + (f[s][10] + f[s][15]) + f[s][17]) -
            ((f[s][4] + f[s][8]) + (f[s][9] + f[s][16]) + f[s][18]);
    jz[s] = ((f[s][5] + f[s][11]) + (f[s][14] + f[s][15]) + f[s][18]) -
            ((f[s][6] + f[s][12]) + (f[s][13] + f[s][16]) + f[s][17]);
  }

  const V pc = psi(0, 0, 0);
  R Fx[NS], Fy[NS], Fz[NS];
  {
    R ax[NS], ay[NS], az[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) ax[s] = ay[s] = az[s] = R(0);
    // the scheduler would hoist all 92 neighbours' loads and spill; a few links at a time suffice
    // to cover the LDS latency
    int link = 0;
#define LB3_ACC(q, dx, dy, dz)                                                   \
  {                                                                              \
    const V pp = psi(dx, dy, dz), pm = psi(-(dx), -(dy), -(dz));                 \
    _Pragma("unroll") for (int s = 0; s < NS; ++s) {                             \
      const R kd = p.K[s][q] * (pp.v[s] - pm.v[s]);                              \
      if ((dx) != 0) ax[s] = fmadd(R(dx), kd, ax[s]);                            \
      if ((dy) != 0) ay[s] = fmadd(R(dy), kd, ay[s]);                            \
      if ((dz) != 0) az[s] = fmadd(R(dz), kd, az[s]);                            \
    }                                                                            \
    if (++link % 8 == 0) __builtin_amdgcn_sched_barrier(0);                      \
  }
    LB3_HALF_LINKS(LB3_ACC)
#undef LB3_ACC
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      Fx[s] = fmadd(-pc.v[s], ax[s], rho[s] * p.gx);
      Fy[s] = fmadd(-pc.v[s], ay[s], rho[s] * p.gy);
      Fz[s] = fmadd(-pc.v[s], az[s], rho[s] * p.gz);
    }
  }
  if (NS == 2) {
    // A-B repulsion over the D3Q19 links, between densities (or psi)
    const V c0 = xr(0, 0, 0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int o = 1 - s;
      const R ex = xr(1, 0, 0).v[o] - xr(-1, 0, 0).v[o];
      const R ey = xr(0, 1, 0).v[o] - xr(0, -1, 0).v[o];
      const R ez = xr(0, 0, 1).v[o] - xr(0, 0, -1).v[o];
      const R pxy = xr(1, 1, 0).v[o] - xr(-1, -1, 0).v[o], mxy = xr(1, -1, 0).v[o] - xr(-1, 1, 0).v[o];
      const R pxz = xr(1, 0, 1).v[o] - xr(-1, 0, -1).v[o], mxz = xr(1, 0, -1).v[o] - xr(-1, 0, 1).v[o];
      const R pyz = xr(0, 1, 1).v[o] - xr(0, -1, -1).v[o], myz = xr(0, 1, -1).v[o] - xr(0, -1, 1).v[o];
      const R cxs = fmadd(p.T1, ex, p.T2 * ((pxy + mxy) + (pxz + mxz)));
      const R cys = fmadd(p.T1, ey, p.T2 * ((pxy - mxy) + (pyz + myz)));
      const R czs = fmadd(p.T1, ez, p.T2 * ((pxz - mxz) + (pyz - myz)));
      Fx[s] = fmadd(-c0.v[s], cxs, Fx[s]);
      Fy[s] = fmadd(-c0.v[s], cys, Fy[s]);
      Fz[s] = fmadd(-c0.v[s], czs, Fz[s]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // the force is complete here: without this the compiler sinks it under the outputs' conditions, away
  // from the neighbours' reads, and spills those
#pragma unroll
  for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(Fx[s]), "+v"(Fy[s]), "+v"(Fz[s]));

  // common velocity u' = sum_s (j_s / tau_s) / sum_s (rho_s / tau_s)
  R nux = jx[0] * p.om[0], nuy = jy[0] * p.om[0], nuz = jz[0] * p.om[0], den = rho[0] * p.om[0];
#pragma unroll
  for (int s = 1; s < NS; ++s) {
    nux = fmadd(jx[s], p.om[s], nux);
    nuy = fmadd(jy[s], p.om[s], nuy);
    nuz = fmadd(jz[s], p.om[s], nuz);
    den = fmadd(rho[s], p.om[s], den);
  }
  const R iden = C::rcp(den);
  const R upx = nux * iden, upy = nuy * iden, upz = nuz * iden;

  if (WHAT == WHAT_MOMENTS && site_ok) {
    R srho = rho[0], mx = jx[0] + R(0.5) * Fx[0], my = jy[0] + R(0.5) * Fy[0], mz = jz[0] + R(0.5) * Fz[0];
#pragma unroll
    for (int s = 1; s < NS; ++s) {
      srho += rho[s];
      mx += jx[s] + R(0.5) * Fx[s];
      my += jy[s] + R(0.5) * Fy[s];
      mz += jz[s] + R(0.5) * Fz[s];
    }
    const size_t nsite = (size_t)a.lx * a.ly * a.lz;
    const size_t site = ((size_t)z * a.ly + y) * a.lx + x;
    if (a.out_rho) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (a.out_f32) static_cast<float *>(a.out_rho)[s * nsite + site] = float(rho[s]);
        else static_cast<double *>(a.out_rho)[s * nsite + site] = double(rho[s]);
      }
    }
    if (a.out_u) {
      const R ux = mx / srho, uy = my / srho, uz = mz / srho;
      if (a.out_f32) {
        float *u = static_cast<float *>(a.out_u);
        u[site] = float(ux);
        u[nsite + site] = float(uy);
        u[2 * nsite + site] = float(uz);
      } else {
        double *u = static_cast<double *>(a.out_u);
        u[site] = double(ux);
        u[nsite + site] = double(uy);
        u[2 * nsite + site] = double(uz);
      }
    }
  }

  if (WHAT == WHAT_STEP) {
    R fs[NS][19];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const R ir = C::rcp(rho[s]);
      const R ux = fmadd(p.tau[s] * Fx[s], ir, upx);
      const R uy = fmadd(p.tau[s] * Fy[s], ir, upy);
      const R uz = fmadd(p.tau[s] * Fz[s], ir, upz);
      // f^eq_l - W_l rho_ref = W_l (drho - 3/2 rho u.u) + W_l rho cu (3 + 9/2 cu)
      const R m15 = R(-1.5) * fmadd(ux, ux, fmadd(uy, uy, uz * uz));
      const R r18 = rho[s] * R(1.0 / 18.0), r36 = rho[s] * R(1.0 / 36.0);
      const R b18 = fmadd(r18, m15, drho[s] * R(1.0 / 18.0)), b36 = fmadd(r36, m15, drho[s] * R(1.0 / 36.0));
      const R o = p.om[s];
      auto relax = [o](R fl, R b, R r, R cu) { return fmadd(o, fmadd(r, cu * fmadd(R(4.5), cu, R(3)), b) - fl, fl); };
      fs[s][1] = relax(f[s][1], b18, r18, ux);
      fs[s][2] = relax(f[s][2], b18, r18, -ux);
      fs[s][3] = relax(f[s][3], b18, r18, uy);
      fs[s][4] = relax(f[s][4], b18, r18, -uy);
      fs[s][5] = relax(f[s][5], b18, r18, uz);
      fs[s][6] = relax(f[s][6], b18, r18, -uz);
      fs[s][7] = relax(f[s][7], b36, r36, ux + uy);
      fs[s][8] = relax(f[s][8], b36, r36, -(ux + uy));
      fs[s][9] = relax(f[s][9], b36, r36, ux - uy);
      fs[s][10] = relax(f[s][10], b36, r36, -(ux - uy));
      fs[s][11] = relax(f[s][11], b36, r36, ux + uz);
      fs[s][12] = relax(f[s][12], b36, r36, -(ux + uz));
      fs[s][13] = relax(f[s][13], b36, r36, ux - uz);
      fs[s][14] = relax(f[s][14], b36, r36, -(ux - uz));
      fs[s][15] = relax(f[s][15], b36, r36, uy + uz);
      fs[s][16] = relax(f[s][16], b36, r36, -(uy + uz));
      fs[s][17] = relax(f[s][17], b36, r36, uy - uz);
      fs[s][18] = relax(f[s][18], b36, r36, -(uy - uz));
      R t = fs[s][1];
#pragma unroll
      for (int l = 2; l < 19; ++l) t += fs[s][l];
      fs[s][0] = drho[s] - t;
    }
#pragma unroll
    for (int l = 0; l < 19; ++l) {
      if (NS == 2) C::template bstore2<STP>(rd, at, uni((uint32_t)l * plane_b), fs[0][l], fs[NS - 1][l]);
      else C::template bstore<STP>(rd, at, uni((uint32_t)l * plane_b), fs[0][l]);
    }
  }
}

}  // namespace lb355
