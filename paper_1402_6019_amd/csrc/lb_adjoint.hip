// Hand-written adjoint (reverse-time) step of the two-belt pseudopotential lattice
// Boltzmann map, for gradients of the time-averaged wall stress and flow rate with respect
// to the couplings G_ss,1, G_ss,2, G_AB and the body force g.
//
// Forward map of one step (state x = pre-collision populations f(t), canonical layout):
//   rho_s = sum_l x_l,  j_s = sum_l c_l x_l,  psi_s = psi0 (1 - exp(-rho_s / rho0))
//   F_s   = -psi_s sum_h K_s(q) c (psi_s(x+c) - psi_s(x-c))              (eq. (FORCE))
//           -G_AB r_s sum_{h in belt 1} t(q) c (r_sbar(x+c) - r_sbar(x-c)) (r = rho or psi)
//           +rho_s g
//   u'    = sum_s omega_s j_s / sum_s omega_s rho_s,   u_s = u' + tau_s F_s / rho_s
//   y_l   = (1 - omega_s) x_l + omega_s f^eq_l(rho_s, u_s)                 (eq. (LB))
//   x'_l(x) = y_l(x - c_l), or y_opp(l)(x) when x - c_l is a wall row      (streaming)
// Loss of one step (weights cW = lw0 / T, cQ = lw1 / T):
//   cW (W_bot + W_top) / 2,  W_bot = (1/lx) sum_x sum_s sum_{c_ly = -1} 2 c_lx y_l(x, 0)
//   cQ Q,  Q = (1/lx) sum_x u_x,  u = (sum_s j_s + F_s / 2) / sum_s rho_s
//
// Reverse step, given lambda' = dL/dx(t+1):
//   a_l(x)   = lambda'_l(x + c_l), or lambda'_opp(l)(x) when x + c_l is a wall row (the
//              transpose of streaming), plus the wall-stress source on the wall rows;
//   then the chain rule through the collision, the velocity shift and u' per site gives
//   the local part of lambda(t), the force adjoint Fbar_s and the parameter sensitivities
//   Fbar_s . dF_s/dtheta; finally the force's dependence on the neighbours' psi (and rho)
//   is a gather with the same stencil:
//     psibar_s(y) += sum_h K_s(q) c . (A_s(y+c) - A_s(y-c)),   A_s = psi_s Fbar_s
//     rbar_sbar(y) += G_AB sum_{h in belt 1} t(q) c . (B_s(y+c) - B_s(y-c)),  B_s = r_s Fbar_s
//   and rhobar = psi'(rho) psibar enters every lambda_l(t).
// One kernel does both parts of a reverse step on canonical-layout arrays [..][y][x]: a workgroup
// takes the local part for its tile plus a frame of two sites, keeps A and B of those in LDS and
// gathers for its tile.  As two kernels (the local part of every site to memory, then the gather)
// a step of a 512 x 256 channel in FP64 took 19.5 + 7.3 us, most of it the latency of one wave per
// tile row with nothing to overlap it, and wrote and read A and B (128 bytes per site) between
// them; the local part of the frame, computed by two tiles, costs less.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "lb_internal.hpp"
#include "lb_step.hpp"
#include "lb_tables.hpp"

namespace lb355 {

namespace {

__device__ inline int wrapx(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// Calls f(std::integral_constant<int, i>{}) for i = 0, 1, ..., N - 1 in order, so that the stencil
// constants indexed by i are compile-time values inside f.
template <typename F, int... I>
__device__ inline void each_index(F &f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ inline void each_index(F &&f) {
  each_index(f, std::make_integer_sequence<int, N>{});
}

// C v for a stencil constant C in {-2, ..., 2}, C != 0: +-1 are a copy or a negation.  Terms
// whose constant is zero are left out of the sums below altogether: they only add a signed
// zero, which leaves a sum unchanged.
template <int C, typename R>
__device__ inline R cmul(R v) {
  static_assert(C != 0, "zero terms are left out");
  if constexpr (C == 1) return v;
  else if constexpr (C == -1) return -v;
  else return R(C) * v;
}

// a b + c: fused in FP64, where it only drops a rounding; two operations in FP32, whose sensitivities
// (sums that nearly cancel) would move with any change of their roundings.
__device__ inline double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline float mad(float a, float b, float c) { return a * b + c; }

// The equilibrium polynomial's derivative along one axis, 3 c + 9 (c_l . u) c - 3 u_a for
// c = c_l,a, grouped as ((3 c) + (9 (c_l . u)) c) - 3 u_a.
template <int C, typename R>
__device__ inline R eq_grad(R cu, R ua) {
  if constexpr (C == 0) return -(R(3) * ua);
  else return (R(3 * C) + cmul<C>(R(9) * cu)) - R(3) * ua;
}

// c . d for a half-link c = (CX, CY), zero components left out.
template <int CX, int CY, typename R>
__device__ inline R pair_dot(R dx, R dy) {
  if constexpr (CX != 0 && CY != 0) return cmul<CX>(dx) + cmul<CY>(dy);
  else if constexpr (CX != 0) return cmul<CX>(dx);
  else return cmul<CY>(dy);
}

template <typename T>
__device__ inline T block_sum(T v, T *sm) {
  // wave reduction, then across the waves of the block (sm: one slot per wave)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sm[wv] = v;
  __syncthreads();
  T r = 0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += sm[k];
  return r;
}

}  // namespace

// The term of lambda common to every l at one site: the force's dependence on the
// neighbours' psi (and rho), gathered with the forward stencil from A_s = psi_s Fbar_s and
// B_s = r_s Fbar_s.  ab(which, s, dx, dy, bx, by) gives A_s (which = 0) or B_s (which = 1) at
// the neighbour (dx, dy), zero off the lattice; rho holds the site's densities.
template <typename R, int NS, typename AB>
__device__ inline void gather_corr(const AdjArgs &a, const AB &ab, const R (&rho)[2], R (&corr)[2]) {
  R psib[2] = {0, 0}, rbar[2] = {0, 0};
  for (int s = 0; s < NS; ++s) {
    R Kq[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) Kq[q] = R(a.K[s][q]);
    R acc = 0;
    each_index<NHALF>([&](auto H) {
      constexpr int h = decltype(H)::value, hx = HX[h], hy = HY[h];
      R px, py, mx, my;
      ab(0, s, hx, hy, px, py);
      ab(0, s, -hx, -hy, mx, my);
      acc = mad(Kq[HQ[h]], pair_dot<hx, hy>(px - mx, py - my), acc);
    });
    psib[s] += acc;
  }
  if (NS == 2) {
    for (int s = 0; s < 2; ++s) {  // species s's force depends on species o = 1 - s's field
      const int o = 1 - s;
      R acc = 0;
      each_index<4>([&](auto H) {
        constexpr int h = decltype(H)::value, hx = HX[h], hy = HY[h];
        R px, py, mx, my;
        ab(1, s, hx, hy, px, py);
        ab(1, s, -hx, -hy, mx, my);
        acc = mad(R(a.t[HQ[h]]), pair_dot<hx, hy>(px - mx, py - my), acc);
      });
      // B_s uses species s's own r (r_s Fbar_s); it lands on the other species' field
      if (a.cross_psi) psib[o] += R(a.gab) * acc;
      else rbar[o] += R(a.gab) * acc;
    }
  }
  for (int s = 0; s < NS; ++s) corr[s] = rbar[s] + psib[s] * R(a.psi0) * R(a.irho0) * exp(-rho[s] * R(a.irho0));
}

// An array of planes of n sites as one buffer range, planes in the uniform offset; WIDE (an array past
// 4 GiB) takes a range per plane instead, spanning up to three (a reflected link reads the plane two
// above or below its own).
template <typename R, bool WIDE>
struct Planes {
  Rsrc all;
  const void *base;
  size_t n;
  __device__ Planes(const void *p, int planes, size_t nn)
      : all(make_rsrc(p, WIDE ? 0u : (uint32_t)planes * (uint32_t)(nn * sizeof(R)))), base(p), n(nn) {}
  __device__ __forceinline__ Rsrc range(int pl) const {
    return WIDE ? make_rsrc(static_cast<const R *>(base) + (size_t)pl * n, 3u * (uint32_t)(n * sizeof(R))) : all;
  }
  __device__ __forceinline__ uint32_t plane(int pl) const { return WIDE ? 0u : uni((uint32_t)pl * (uint32_t)(n * sizeof(R))); }
  __device__ __forceinline__ R load(int pl, uint32_t off) const {
    if constexpr (sizeof(R) == 8) return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(range(pl), off, plane(pl), 0));
    else return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(range(pl), off, plane(pl), 0));
  }
  __device__ __forceinline__ void store(int pl, uint32_t off, R v) const {
    if constexpr (sizeof(R) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), range(pl), off, plane(pl), 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), range(pl), off, plane(pl), 0);
  }
};

// Sites of a tile's local region (frame of two) and of the staged psi and rho (frame of four).
template <int BX, int BY>
struct AdjDims {
  static constexpr int LX = BX + 4, LY = BY + 4, SX = BX + 8, SY = BY + 8, NL = LX * LY, NSTG = SX * SY;
};
template <typename R, int NS, int BX, int BY, int NT>
constexpr size_t adj_lds_bytes() {
  using D = AdjDims<BX, BY>;
  return (size_t)NS * (2 * D::NSTG + 4 * D::NL) * sizeof(R) + (size_t)ADJ_N * BX * BY * sizeof(double);
}

// One reverse step: lambda(t) from lambda(t+1) (a.lam_next) and the state of step t (a.fields, a.x), and
// this step's sensitivities and loss terms, added to the tile's row of running sums.
// The gather over A and B reads two sites past the tile, so the local part runs on the tile and a frame
// of two and A and B never leave LDS: FP64 with two species moves 352 B per site (8 planes of fields, 18
// of lambda each way) where a local and a gather pass moved 640.  Bound by FP64 and address
// instructions at two waves per SIMD (244 registers), not by memory: 512 x 256 walled, FP64, two
// species, beside the recompute stream: 23.0 us (2 TB/s) against 19.5 + 7.3 us for the two passes; alone
// 20.3 us, vector units busy 37% of it (the frame's round occupies half of the waves; in 64 x 8 tiles
// 19.9 us, in 16 x 16 26).  One
// buffer range per array, planes in the uniform offset: a range per plane spilled scalar registers (728
// of 2800 vector instructions only moved them; 25.9 us).
template <typename R, int NS, bool WALLS, bool WIDE, int BX, int BY, int NT>
__global__ __launch_bounds__(NT) void adj_step_kernel(AdjArgs a) {
  using D = AdjDims<BX, BY>;
  constexpr int M = (D::NL + NT - 1) / NT, MT = (BX * BY + NT - 1) / NT;  // rounds of the region and of the tile
  constexpr int NU = BX * BY;
  double *const sm = reinterpret_cast<double *>(lb_smem);  // the tile's sites' terms of the sums [ADJ_N][NU]
  R *const sps = reinterpret_cast<R *>(sm + ADJ_N * NU);   // psi of the state [NS][SY][SX]
  R *const srh = sps + NS * D::NSTG;              // rho
  R *const sab = srh + NS * D::NSTG;              // A_s, B_s (x, y each) [NS][4][LY][LX]
  const int tid = threadIdx.x, lx = a.lx, ly = a.ly;
  const size_t n = (size_t)lx * ly;
  const Planes<R, WIDE> fields(a.fields, 8, n), lnext(a.lam_next, NS == 2 ? 18 : 9, n), lout(a.lam, NS == 2 ? 18 : 9, n);
  const int ntx = (lx + BX - 1) / BX;
  const int by = (int)blockIdx.x / ntx, bx = (int)blockIdx.x - by * ntx;
  const int x0 = bx * BX, y0 = by * BY;
  const bool narrow = lx < 2 * D::SX || ly < 2 * D::SY;
  auto wrap = [&](int v, int m) { return narrow ? ((v % m) + m) % m : wrapx(v, m); };
  // Site i of the local region: the tile's sites first, then its frame (two rows below and above, two
  // columns on either side), relative to the tile's first site.
  auto site = [&](int i, int &sx, int &sy) {
    sy = i / BX;
    sx = i - sy * BX;
    if (i >= BX * BY) {
      const int q = i - BX * BY, t = q - 4 * D::LX, r = q / D::LX, c = t & 3;
      sx = t < 0 ? q - r * D::LX - 2 : (c < 2 ? c - 2 : c + BX - 2);
      sy = t < 0 ? (r < 2 ? r - 2 : r + BY - 2) : t >> 2;
    }
  };

  // psi and rho of the tile and a frame of four; past a wall the ghost values
  constexpr int NST = (D::NSTG + NT - 1) / NT;
  R vps[NST][NS], vrh[NST][NS];
  bool solid[NST];
#pragma unroll
  for (int it = 0; it < NST; ++it) {
    const int k = min(tid + it * NT, D::NSTG - 1), hy = k / D::SX, hx = k - hy * D::SX;
    const int y = y0 + hy - 4;
    solid[it] = WALLS && (y < 0 || y >= ly);
    const int yc = WALLS ? min(max(y, 0), ly - 1) : wrap(y, ly);
    const uint32_t off = (uint32_t)(((size_t)yc * lx + wrap(x0 + hx - 4, lx)) * sizeof(R));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      vps[it][s] = fields.load(2 + s, off);
      vrh[it][s] = fields.load(s, off);
    }
  }
#pragma unroll
  for (int it = 0; it < NST; ++it) {
    const int k = tid + it * NT;
    if (k < D::NSTG) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        sps[s * D::NSTG + k] = solid[it] ? R(a.psi_w[s]) : vps[it][s];
        srh[s * D::NSTG + k] = solid[it] ? R(a.rho_w[s]) : vrh[it][s];
      }
    }
  }
  __syncthreads();

  R lam[MT][NS][Q];  // the local part of lambda(t) at the tile's sites
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int i0 = tid + m * NT;
    if ((m + 1) * NT > D::NL && i0 >= D::NL) continue;
    int sx, sy;
    site(i0, sx, sy);
    const bool own = m < MT && i0 < BX * BY;
    const int e = (sy + 2) * D::LX + sx + 2;
    const int yr = y0 + sy;
    if (WALLS && (yr < 0 || yr >= ly)) {  // not a site: nothing of it enters a gather
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) sab[(s * 4 + c) * D::NL + e] = R(0);
      if (own)
#pragma unroll
        for (int k = 0; k < ADJ_N; ++k) sm[k * NU + i0] = 0.0;
      continue;
    }
    const int x = wrap(x0 + sx, lx), y = WALLS ? yr : wrap(yr, ly);
    const bool live = own && x0 + sx < lx && yr < ly;
    const uint32_t pb = (uint32_t)(n * sizeof(R));
    const uint32_t off = (uint32_t)(((size_t)y * lx + x) * sizeof(R));

    // lambda(t+1) where the populations leaving the site arrive: along c_l, or bounced back into
    // opp(l) at the site where x + c_l lies past a wall (the range of each pair of links spans both)
    R lsrc[NS][Q], jx[NS], jy[NS];
    each_index<Q>([&](auto L) {
      constexpr int l = decltype(L)::value, cx = CXS[l], cy = CYS[l], lo = l < OPPS[l] ? l : OPPS[l];
      const int yn = y + cy;
      const bool bounce = WALLS && cy != 0 && (yn < 0 || yn >= ly);
      const uint32_t up = bounce ? (uint32_t)(OPPS[l] - lo) * pb : (uint32_t)(l - lo) * pb;  // walls: planes above lo
      const uint32_t j = bounce ? off : (uint32_t)(((size_t)(WALLS ? yn : wrapx(yn, ly)) * lx + wrapx(x + cx, lx)) * sizeof(R));
#pragma unroll
      for (int s = 0; s < NS; ++s)
        lsrc[s][l] = WALLS && cy != 0 ? lnext.load(s * Q + lo, up + j) : lnext.load(s * Q + l, j);
    });
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      jx[s] = fields.load(4 + s, off);
      jy[s] = fields.load(6 + s, off);
    }
    const R *const pp = sps + (sy + 4) * D::SX + sx + 4, *const rr = srh + (sy + 4) * D::SX + sx + 4;
    auto psi_at = [&](int s, int dx, int dy) -> R { return pp[s * D::NSTG + dy * D::SX + dx]; };
    auto rho_at = [&](int s, int dx, int dy) -> R { return rr[s * D::NSTG + dy * D::SX + dx]; };

    R rho[2], psi[2], Fx[2], Fy[2];
    R s1x[2], s1y[2], s2x[2], s2y[2], xx[2], xy[2], self[2];
    for (int s = 0; s < NS; ++s) {
      rho[s] = rho_at(s, 0, 0);
      psi[s] = psi_at(s, 0, 0);
      // two-belt sums with the attractive (w) and repulsive (p) shell weights
      R ax = 0, ay = 0, bx = 0, by = 0;
      each_index<NHALF>([&](auto H) {
        constexpr int h = decltype(H)::value, hx = HX[h], hy = HY[h];
        const R d = psi_at(s, hx, hy) - psi_at(s, -hx, -hy);
        const R wq = R(a.w[HQ[h]]), pq = R(a.p[HQ[h]]);
        if constexpr (hx != 0) {
          ax = mad(cmul<hx>(wq), d, ax);
          bx = mad(cmul<hx>(pq), d, bx);
        }
        if constexpr (hy != 0) {
          ay = mad(cmul<hy>(wq), d, ay);
          by = mad(cmul<hy>(pq), d, by);
        }
      });
      s1x[s] = ax; s1y[s] = ay; s2x[s] = bx; s2y[s] = by;
      Fx[s] = -psi[s] * (R(a.g1[s]) * ax + R(a.g2[s]) * bx);
      Fy[s] = -psi[s] * (R(a.g1[s]) * ay + R(a.g2[s]) * by);
      xx[s] = 0; xy[s] = 0; self[s] = 0;
      __builtin_amdgcn_sched_barrier(0);
    }
    if (NS == 2) {
      for (int s = 0; s < 2; ++s) {
        const int o = 1 - s;
        R cx = 0, cy = 0;
        each_index<4>([&](auto H) {
          constexpr int h = decltype(H)::value, hx = HX[h], hy = HY[h];
          const R d = a.cross_psi ? psi_at(o, hx, hy) - psi_at(o, -hx, -hy) : rho_at(o, hx, hy) - rho_at(o, -hx, -hy);
          const R tq = R(a.t[HQ[h]]);
          if constexpr (hx != 0) cx = mad(cmul<hx>(tq), d, cx);
          if constexpr (hy != 0) cy = mad(cmul<hy>(tq), d, cy);
        });
        xx[s] = cx;
        xy[s] = cy;
        self[s] = a.cross_psi ? psi[s] : rho[s];
        Fx[s] -= R(a.gab) * self[s] * cx;
        Fy[s] -= R(a.gab) * self[s] * cy;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    for (int s = 0; s < NS; ++s) {
      Fx[s] = mad(rho[s], R(a.body[0]), Fx[s]);
      Fy[s] = mad(rho[s], R(a.body[1]), Fy[s]);
    }

    // common velocity and the shifted equilibrium velocities
    R nx = 0, ny = 0, den = 0, rtot = 0, mx = 0, my = 0;
    for (int s = 0; s < NS; ++s) {
      const R om = R(a.omega[s]);
      nx = mad(om, jx[s], nx);
      ny = mad(om, jy[s], ny);
      den = mad(om, rho[s], den);
      rtot += rho[s];
      mx += mad(R(0.5), Fx[s], jx[s]);
      my += mad(R(0.5), Fy[s], jy[s]);
    }
    // reciprocals taken once per site: the rest of the pass multiplies
    // 1 / lx comes from the host, rounded in R as a division here would round it
    const R iden = R(1) / den, irt = R(1) / rtot, ilx = sizeof(R) == 8 ? R(a.ilx) : R(a.ilxf);
    const R upx = nx * iden, upy = ny * iden;
    const R urx = mx * irt;  // reported (half-force) velocity, x component
    const R ilr = ilx * irt;  // 1 / (lx rho_tot)

    // adjoint sources of this step's loss
    const R cW = R(a.cW), cQ = R(a.cQ);
    double loss_w = 0.0;
    const double loss_q = live ? double(cQ * urx) : 0.0;  // divided by lx with the tile's sum

    R ubx = 0, uby = 0;  // adjoint of u'
    R rbar[2], jbx[2], jby[2], fbx[2], fby[2];
    R lp[2][Q];
    for (int s = 0; s < NS; ++s) {
      const R om = R(a.omega[s]), tau = R(a.tau[s]);
      const R ir = R(1) / rho[s];
      const R ux = upx + tau * Fx[s] * ir, uy = upy + tau * Fy[s] * ir;
      const R uu = ux * ux + uy * uy;
      R rb = 0, bx = 0, by = 0;
      each_index<Q>([&](auto L) {
        constexpr int l = decltype(L)::value, cx = CXS[l], cy = CYS[l];
        R al = lsrc[s][l];
        R cu = R(0);  // c_l . u
        if constexpr (cx != 0 && cy != 0) cu = cmul<cx>(ux) + cmul<cy>(uy);
        else if constexpr (cx != 0) cu = cmul<cx>(ux);
        else if constexpr (cy != 0) cu = cmul<cy>(uy);
        const R wl = R(WD2Q9[l]);
        const R poly = R(1) + R(3) * cu + R(4.5) * cu * cu - R(1.5) * uu;  // f^eq_l / (W_l rho_s)
        const R feq = wl * rho[s] * poly;
        if constexpr (WALLS && cy != 0) {
          if (y == (cy < 0 ? 0 : ly - 1)) {
            // wall stress: d/dy_l of cW (1/2)(1/lx) (2 c_lx y_l - 6 W_l rho_w c_lx^2 U); the
            // moving wall's share is constant
            if constexpr (cx != 0) al += cmul<cx>(cW) * ilx;
            // post-collision population leaving the wall row, from its pre-collision one
            const R xl = R(a.x[((size_t)(s * Q + l) * 2 + (cy < 0 ? 0 : 1)) * lx + x]);
            const R yl = (R(1) - om) * xl + om * feq;
            const R mw = R(3) * wl * R(a.rho_w[s]) * R(cx * cx) * R(cy < 0 ? a.u_wall[0] : a.u_wall[1]);
            if (live) loss_w += double(cW * (R(cx) * yl - mw));
          }
        }
        lp[s][l] = (R(1) - om) * al;
        rb = mad(om * al * wl, poly, rb);  // omega al f^eq / rho
        const R k = om * al * wl * rho[s];
        bx = mad(k, eq_grad<cx>(cu, ux), bx);
        by = mad(k, eq_grad<cy>(cu, uy), by);
      });
      // u_s = u' + tau F_s / rho_s
      ubx += bx;
      uby += by;
      fbx[s] = tau * bx * ir;
      fby[s] = tau * by * ir;
      rb -= tau * (Fx[s] * bx + Fy[s] * by) * (ir * ir);
      rbar[s] = rb;
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int s = 0; s < NS; ++s) {
      const R om = R(a.omega[s]);
      // u' = sum omega j / sum omega rho
      jbx[s] = om * ubx * iden;
      jby[s] = om * uby * iden;
      rbar[s] -= om * (upx * ubx + upy * uby) * iden;
      // flow rate: Q = (1/lx) sum (sum_s j_s + F_s / 2)_x / sum_s rho_s
      jbx[s] += cQ * ilr;
      fbx[s] += R(0.5) * cQ * ilr;
      rbar[s] -= cQ * urx * ilr;
    }
    // force: F_s = -psi_s S_s - G_AB self_s X_s + rho_s g
    double dg1[2] = {0, 0}, dg2[2] = {0, 0}, dgab = 0, dgx = 0, dgy = 0;
    R psib[2] = {0, 0};
    for (int s = 0; s < NS; ++s) {
      const R Sx = R(a.g1[s]) * s1x[s] + R(a.g2[s]) * s2x[s], Sy = R(a.g1[s]) * s1y[s] + R(a.g2[s]) * s2y[s];
      psib[s] -= fbx[s] * Sx + fby[s] * Sy;
      rbar[s] += fbx[s] * R(a.body[0]) + fby[s] * R(a.body[1]);
      if (NS == 2) {
        const R cb = -R(a.gab) * (fbx[s] * xx[s] + fby[s] * xy[s]);
        if (a.cross_psi) psib[s] += cb;
        else rbar[s] += cb;
      }
      if (live) {
        dg1[s] = double(-psi[s] * (fbx[s] * s1x[s] + fby[s] * s1y[s]));
        dg2[s] = double(-psi[s] * (fbx[s] * s2x[s] + fby[s] * s2y[s]));
        dgab += double(-self[s] * (fbx[s] * xx[s] + fby[s] * xy[s]));
        dgx += double(fbx[s] * rho[s]);
        dgy += double(fby[s] * rho[s]);
      }
      // psi'(rho) = (psi0 / rho0) exp(-rho / rho0)
      rbar[s] += psib[s] * R(a.psi0) * R(a.irho0) * exp(-rho[s] * R(a.irho0));
    }
    if (own) {
#pragma unroll
      for (int s = 0; s < NS; ++s)
        each_index<Q>([&](auto L) {
          constexpr int l = decltype(L)::value, cx = CXS[l], cy = CYS[l];
          R lam_l = lp[s][l] + rbar[s];
          if constexpr (cx != 0) lam_l += cmul<cx>(jbx[s]);
          if constexpr (cy != 0) lam_l += cmul<cy>(jby[s]);
          lam[m < MT ? m : 0][s][l] = lam_l;
        });
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      sab[(s * 4 + 0) * D::NL + e] = psi[s] * fbx[s];
      sab[(s * 4 + 1) * D::NL + e] = psi[s] * fby[s];
      sab[(s * 4 + 2) * D::NL + e] = self[s] * fbx[s];
      sab[(s * 4 + 3) * D::NL + e] = self[s] * fby[s];
    }
    if (own) {
      const double v[ADJ_N] = {dg1[0], dg1[1], dg2[0], dg2[1], dgab, dgx, dgy, loss_w, loss_q};
#pragma unroll
      for (int k = 0; k < ADJ_N; ++k) sm[k * NU + i0] = v[k];  // zeros past the lattice's end
    }
  }
  __syncthreads();

  // the term of lambda(t) common to every l, gathered from the tile and its frame
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int i0 = tid + m * NT, sy = i0 / BX, sx = i0 - sy * BX;
    if (i0 >= BX * BY || x0 + sx >= lx || y0 + sy >= ly) continue;
    const R *const q = sab + (sy + 2) * D::LX + sx + 2;
    auto ab = [&](int which, int s, int dx, int dy, R &vx, R &vy) {
      vx = q[(s * 4 + 2 * which + 0) * D::NL + dy * D::LX + dx];
      vy = q[(s * 4 + 2 * which + 1) * D::NL + dy * D::LX + dx];
    };
    R rho[2] = {0, 0}, corr[2];
#pragma unroll
    for (int s = 0; s < NS; ++s) rho[s] = srh[s * D::NSTG + (sy + 4) * D::SX + sx + 4];
    gather_corr<R, NS>(a, ab, rho, corr);
    const uint32_t off = (uint32_t)(((size_t)(y0 + sy) * lx + x0 + sx) * sizeof(R));
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int l = 0; l < Q; ++l)
        lout.store(s * Q + l, off, lam[m][s][l] + corr[s]);
  }

  // the tile's sums: wave w sums the terms w, w + waves, ... over the sites, in a fixed order, and adds
  // them to the tile's row (a shuffle tree of every term in every wave took as many LDS operations as
  // the update)
  const int lane = tid & 63;
  for (int k = tid >> 6; k < ADJ_N; k += NT / 64) {
    double v = sm[k * NU + lane];
#pragma unroll
    for (int w = 1; w < NU / 64; ++w) v += sm[k * NU + w * 64 + lane];
    v = wave_sum(v);
    if (k == ADJ_LW || k == ADJ_LQ) v /= lx;
    if (lane == 0) a.partials[(size_t)blockIdx.x * ADJ_N + k] += v;
  }
}

// acc[k] += sum over blocks of partials[block][k], in block order (deterministic).
__global__ __launch_bounds__(256) void adj_reduce_kernel(const double *partials, int nblocks, double *acc) {
  __shared__ double sm[4];
  for (int k = 0; k < ADJ_N; ++k) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) v += partials[(size_t)b * ADJ_N + k];
    const double t = block_sum(v, sm);
    if (threadIdx.x == 0) acc[k] += t;
  }
}

__global__ void zero_kernel(uint32_t *p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// Tile of the reverse step: the largest that gives every compute unit one, as the frame it adds to
// the local part shrinks with its size.
static int adj_shape(int lx, int ly, int n_cu) {
  auto tiles = [&](int bx, int by) { return (long long)((lx + bx - 1) / bx) * ((ly + by - 1) / by); };
  return tiles(32, 16) >= n_cu ? 2 : (tiles(16, 16) >= n_cu ? 1 : 0);
}

int adj_blocks(int lx, int ly, int n_cu) {
  const int k = adj_shape(lx, ly, n_cu), bx = k == 2 ? 32 : 16, by = k == 0 ? 8 : 16;
  return ((lx + bx - 1) / bx) * ((ly + by - 1) / by);
}

template <typename R, int NS, bool WALLS, bool WIDE, int BX, int BY, int NT>
static hipError_t adj_step_k(const AdjArgs &a, hipStream_t st) {
  const int nb = ((a.lx + BX - 1) / BX) * ((a.ly + BY - 1) / BY);
  hipLaunchKernelGGL((adj_step_kernel<R, NS, WALLS, WIDE, BX, BY, NT>), dim3(nb), dim3(NT),
                     (adj_lds_bytes<R, NS, BX, BY, NT>()), st, a);
  return hipGetLastError();
}

template <typename R, int NS, bool WALLS>
static hipError_t adj_step_t(int n_cu, const AdjArgs &a, hipStream_t st) {
  if ((size_t)a.lx * a.ly * 9 * NS * sizeof(R) >= ((size_t)1 << 32))  // always the widest tile
    return adj_step_k<R, NS, WALLS, true, 32, 16, 512>(a, st);
  switch (adj_shape(a.lx, a.ly, n_cu)) {
    case 0: return adj_step_k<R, NS, WALLS, false, 16, 8, 256>(a, st);
    case 1: return adj_step_k<R, NS, WALLS, false, 16, 16, 448>(a, st);
  }
  return adj_step_k<R, NS, WALLS, false, 32, 16, 512>(a, st);
}

template <typename R>
static hipError_t adj_step_r(int ns, int walls, int n_cu, const AdjArgs &a, hipStream_t st) {
  if (ns == 1) return walls ? adj_step_t<R, 1, true>(n_cu, a, st) : adj_step_t<R, 1, false>(n_cu, a, st);
  return walls ? adj_step_t<R, 2, true>(n_cu, a, st) : adj_step_t<R, 2, false>(n_cu, a, st);
}

hipError_t launch_adjoint_step(int fp64, int ns, int walls, int n_cu, const AdjArgs &a, hipStream_t st) {
  return fp64 ? adj_step_r<double>(ns, walls, n_cu, a, st) : adj_step_r<float>(ns, walls, n_cu, a, st);
}

hipError_t launch_adjoint_reduce(const double *partials, int nblocks, double *acc, hipStream_t st) {
  hipLaunchKernelGGL(adj_reduce_kernel, dim3(1), dim3(256), 0, st, partials, nblocks, acc);
  return hipGetLastError();
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, static_cast<uint32_t *>(p), n);
  return hipGetLastError();
}

}  // namespace lb355
