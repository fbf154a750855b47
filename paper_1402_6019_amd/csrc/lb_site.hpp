#pragma once
// The per-site arithmetic of one time step for kernels that hold a site's pulled populations in
// registers and its neighbours' psi and rho somewhere else: the fused step's expressions,
// operation for operation (same expressions, same order), so every kernel built from these gives
// bitwise the populations of the row-marching step.

#include "lb_step.hpp"

namespace lb355 {

// rho and psi of a fluid site from its pulled (decoded) populations.
template <class C, int NS>
__device__ __forceinline__ void site_psi(const SiteConsts<typename C::R> &p, const typename C::R (&f)[NS][9],
                                         Vec<typename C::R, NS> &ps, Vec<typename C::R, NS> &rh) {
  using R = typename C::R;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    rh.v[s] = p.rref[s] + sum9(f[s]);
    ps.v[s] = p.psi0 * (R(1) - C::expo(rh.v[s] * p.nirho0));
  }
}

// Density, momentum and force of a site: f its pulled populations (decoded), ps(dx, dy) the psi of a
// neighbour of the two belts, xr(dx, dy) the rho (or psi) of a neighbour of the first.
template <class C, int NS, typename PS, typename XR>
__device__ __forceinline__ void site_force(const SiteConsts<typename C::R> &p, const typename C::R (&f)[NS][9],
                                           const PS &ps, const XR &xr, typename C::R (&drho)[NS], typename C::R (&rho)[NS],
                                           typename C::R (&jx)[NS], typename C::R (&jy)[NS], typename C::R (&Fx)[NS],
                                           typename C::R (&Fy)[NS]) {
  using R = typename C::R;
  using V = Vec<R, NS>;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    drho[s] = sum9(f[s]);
    rho[s] = p.rref[s] + drho[s];
    jx[s] = (f[s][1] + f[s][5] + f[s][8]) - (f[s][3] + f[s][6] + f[s][7]);
    jy[s] = (f[s][2] + f[s][5] + f[s][6]) - (f[s][4] + f[s][7] + f[s][8]);
  }
  {
    const V pc = ps(0, 0);
    const V e1 = ps(1, 0), w1 = ps(-1, 0), n1 = ps(0, 1), s1 = ps(0, -1);
    const V ne = ps(1, 1), sw = ps(-1, -1), se = ps(1, -1), nw = ps(-1, 1);
    const V e2 = ps(2, 0), w2 = ps(-2, 0), n2 = ps(0, 2), s2 = ps(0, -2);
    const V qa = ps(2, 1), qA = ps(-2, -1), qb = ps(2, -1), qB = ps(-2, 1);
    const V qc = ps(1, 2), qC = ps(-1, -2), qd = ps(1, -2), qD = ps(-1, 2);
    const V d8a = ps(2, 2), d8A = ps(-2, -2), d8b = ps(2, -2), d8B = ps(-2, 2);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const R dE = e1.v[s] - w1.v[s], dN = n1.v[s] - s1.v[s];
      const R dd1 = ne.v[s] - sw.v[s], dd2 = se.v[s] - nw.v[s];
      const R d4x = e2.v[s] - w2.v[s], d4y = n2.v[s] - s2.v[s];
      const R da = qa.v[s] - qA.v[s], db = qb.v[s] - qB.v[s];
      const R dc = qc.v[s] - qC.v[s], dd = qd.v[s] - qD.v[s];
      const R ea = d8a.v[s] - d8A.v[s], eb = d8b.v[s] - d8B.v[s];
      const R sx = fmadd(p.K1[s], dE, fmadd(p.K2[s], dd1 + dd2, fmadd(p.K4[s], d4x,
                   fmadd(p.K5[s], R(2) * (da + db) + (dc + dd), p.K8[s] * (ea + eb)))));
      const R sy = fmadd(p.K1[s], dN, fmadd(p.K2[s], dd1 - dd2, fmadd(p.K4[s], d4y,
                   fmadd(p.K5[s], (da - db) + R(2) * (dc - dd), p.K8[s] * (ea - eb)))));
      Fx[s] = fmadd(-pc.v[s], sx, rho[s] * p.gx);
      Fy[s] = fmadd(-pc.v[s], sy, rho[s] * p.gy);
    }
  }
  if (NS == 2) {
    const V c0 = xr(0, 0);
    const V xe = xr(1, 0), xw = xr(-1, 0), xn = xr(0, 1), xs = xr(0, -1);
    const V xne = xr(1, 1), xsw = xr(-1, -1), xse = xr(1, -1), xnw = xr(-1, 1);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int o = 1 - s;
      const R t1 = xne.v[o] - xsw.v[o], t2 = xse.v[o] - xnw.v[o];
      const R cx = fmadd(p.T1, xe.v[o] - xw.v[o], p.T2 * (t1 + t2));
      const R cy = fmadd(p.T1, xn.v[o] - xs.v[o], p.T2 * (t1 - t2));
      Fx[s] = fmadd(-c0.v[s], cx, Fx[s]);
      Fy[s] = fmadd(-c0.v[s], cy, Fy[s]);
    }
  }
}

// Velocity shift and collision of a site from those: the post-collision deviations, without the
// exchange with a moving wall.
template <class C, int NS>
__device__ __forceinline__ void site_relax(const SiteConsts<typename C::R> &p, const typename C::R (&f)[NS][9],
                                           const typename C::R (&drho)[NS], const typename C::R (&rho)[NS],
                                           const typename C::R (&jx)[NS], const typename C::R (&jy)[NS],
                                           const typename C::R (&Fx)[NS], const typename C::R (&Fy)[NS],
                                           typename C::R (&fsa)[NS][9]) {
  using R = typename C::R;
  R nux = jx[0] * p.om[0], nuy = jy[0] * p.om[0], den = rho[0] * p.om[0];
#pragma unroll
  for (int s = 1; s < NS; ++s) {
    nux = fmadd(jx[s], p.om[s], nux);
    nuy = fmadd(jy[s], p.om[s], nuy);
    den = fmadd(rho[s], p.om[s], den);
  }
  const R iden = C::rcp(den);
  const R upx = nux * iden, upy = nuy * iden;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const R ir = C::rcp(rho[s]);
    const R ux = fmadd(p.tau[s] * Fx[s], ir, upx);
    const R uy = fmadd(p.tau[s] * Fy[s], ir, upy);
    const R m15 = R(-1.5) * fmadd(ux, ux, uy * uy);
    const R r9 = rho[s] * R(1.0 / 9.0), r36 = rho[s] * R(1.0 / 36.0);
    const R b9 = fmadd(r9, m15, drho[s] * R(1.0 / 9.0)), b36 = fmadd(r36, m15, drho[s] * R(1.0 / 36.0));
    const R o = p.om[s];
    auto relax = [o](R fl, R b, R r, R cu) { return fmadd(o, fmadd(r, cu * fmadd(R(4.5), cu, R(3)), b) - fl, fl); };
    R (&fs)[9] = fsa[s];
    fs[1] = relax(f[s][1], b9, r9, ux);
    fs[3] = relax(f[s][3], b9, r9, -ux);
    fs[2] = relax(f[s][2], b9, r9, uy);
    fs[4] = relax(f[s][4], b9, r9, -uy);
    fs[5] = relax(f[s][5], b36, r36, ux + uy);
    fs[7] = relax(f[s][7], b36, r36, -(ux + uy));
    fs[6] = relax(f[s][6], b36, r36, uy - ux);
    fs[8] = relax(f[s][8], b36, r36, -(uy - ux));
    fs[0] = drho[s] - ((((fs[1] + fs[2]) + (fs[3] + fs[4])) + ((fs[5] + fs[6]) + (fs[7] + fs[8]))));
  }
}

// Both.
template <class C, int NS, typename PS, typename XR>
__device__ __forceinline__ void site_update(const SiteConsts<typename C::R> &p, const typename C::R (&f)[NS][9],
                                            const PS &ps, const XR &xr, typename C::R (&rho)[NS],
                                            typename C::R (&fsa)[NS][9]) {
  typename C::R drho[NS], jx[NS], jy[NS], Fx[NS], Fy[NS];
  site_force<C, NS>(p, f, ps, xr, drho, rho, jx, jy, Fx, Fy);
  site_relax<C, NS>(p, f, drho, rho, jx, jy, Fx, Fy, fsa);
}

// The momentum a moving wall hands the populations it reflects, on the rows next to the walls
// (see the fused step's store).
template <typename R, int NS>
__device__ __forceinline__ void moving_walls(const double (&wall_mom)[2][2], int y, int ly, R (&fsa)[NS][9]) {
  if (y == 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      fsa[s][7] += R(wall_mom[0][s]);
      fsa[s][8] -= R(wall_mom[0][s]);
    }
  }
  if (y == ly - 1) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      fsa[s][6] += R(wall_mom[1][s]);
      fsa[s][5] -= R(wall_mom[1][s]);
    }
  }
}

// The value a store of v (species s, plane l) followed by a load returns: the storage's rounding
// of an intermediate step, bit for bit (hs: the site's random seed of the step).
template <int MODE>
__device__ __forceinline__ typename Codec<MODE>::R stored_value(typename Codec<MODE>::R v, int s, int l, uint32_t hs) {
  using C = Codec<MODE>;
  if constexpr (MODE == MODE_BF16SR) {
    const uint32_t rnd = mix32(hs + (uint32_t)l * 0x9e3779b9u);
    return C::decode(C::round_sr(v, s == 0 ? (rnd & 0xffffu) : (rnd >> 16)) & 0xffffu);
  } else if constexpr (MODE == MODE_BF16) {
    return C::decode(C::encode(v));
  } else {
    return v;
  }
}

}  // namespace lb355
