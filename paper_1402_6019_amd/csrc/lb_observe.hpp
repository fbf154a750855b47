#pragma once
// Passes that read the current state and store no populations: moments, totals, row profiles and the
// stress field, in rectangular tiles.
//
// A workgroup pulls its tile and a frame of two sites, keeps psi and rho of those in LDS and evaluates
// the tile's sites.  Bound by latency up to a few hundred thousand sites and by the read of the
// populations beyond.  As marched rows, one workgroup per strip and segment, the passes lasted as long as
// a step of a small lattice whatever the size, and their sums cost a shuffle tree per term in every row.
// Before and after: profile of a 1040 x 1040 walled FP32 lattice 53 + 11 us (second pass) and 27 + 5;
// moments of 64 x 64 FP64 10.2 and 3.9, of one 350 000 site lattice of a batch 25.0 and 12.9.
// Sums go through LDS instead: every site's terms are laid out, then a few lanes add each row's (profile)
// or a wave each term's (totals), in an order that only depends on the lattice.
// Tiles of 64 x 8 sites; where those leave compute units idle, the passes without sums take 16 x 8.
//
// Per-site arithmetic: site_force (lb_site.hpp), the step's.

#include "lb_tile.hpp"

namespace lb355 {

// Bytes of LDS: psi and rho of tile and frame, or the terms laid out for the sums.
template <int MODE, int NS, int WHAT, int BX, int BY>
constexpr size_t observe_lds_bytes() {
  constexpr size_t v = (size_t)NS * (MODE == MODE_F64 ? 8 : 4) * NS * (BX + 4) * (BY + 4);
  constexpr size_t s = WHAT == WHAT_PROFILE ? sizeof(double) * PROF_N * BY * (BX + 1)
                                            : (WHAT == WHAT_OBSERVE ? sizeof(double) * RED_N * BX * BY : 0);
  return v > s ? v : s;
}

// The tile (bx, by) of the lattice described by a.  out0: densities (moments), sums [tile column][row]
// [PROF_N] (profile) or pressure tensor (stress); out_u: the velocity; part: the tile's row of partial sums.
template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int NT>
__device__ __forceinline__ void observe_tile(const TileArgs<typename Codec<MODE>::R> &a, const void *const src, const int bx,
                                             const int by, void *const out0, void *const out_u, const int out_f32,
                                             double *const part) {
  using C = Codec<MODE>;
  using R = typename C::R;
  using L = typename C::L;
  using V = Vec<R, NS>;
  static_assert(NT >= BX * BY, "one site per thread");
  constexpr int EX = BX + 4, NU = BX * BY, NE = EX * (BY + 4), M = (NE + NT - 1) / NT;
  V *const psi = reinterpret_cast<V *>(lb_smem);
  V *const rhol = psi + (NS == 2 ? NE : 0);

  const int lx = a.lx, ly = a.ly, tid = threadIdx.x, x0 = bx * BX, y0 = by * BY;
  const bool narrow_x = lx < EX + BX, narrow_y = ly < BY + 4 + BY;
  const SiteConsts<R> &p = a.c;
  const Rsrc rs = make_rsrc(src, a.buf_b);
  // the tile's sites first, one per thread, then the frame
  R f[NS][9];
  L fl[M][NS][9];
  int pe[M], yg[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    int sx, sy;
    tile_site<BX, BY, 0, NT>(tid, m, sx, sy);
    pe[m] = (sy + 2) * EX + sx + 2;
    yg[m] = WALLS ? y0 + sy : wrap_any(y0 + sy, ly, narrow_y);
    uint32_t o[9];
    pull_offsets<WALLS>(a, (uint32_t)(NS * sizeof(typename C::S)), wrap_any(x0 + sx, lx, narrow_x), yg[m], o);
#pragma unroll
    for (int l = 0; l < 9; ++l) {
      if (NS == 2) C::bload2(rs, o[l], uni((uint32_t)l * a.pitch_b), fl[m][0][l], fl[m][NS - 1][l]);
      else fl[m][0][l] = C::bload(rs, o[l], uni((uint32_t)l * a.pitch_b));
    }
  }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    if ((m + 1) * NT > NE && tid + m * NT >= NE) continue;
    R g[NS][9];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int l = 0; l < 9; ++l) {
        g[s][l] = C::dec(fl[m][s][l], s);
        if (m == 0) f[s][l] = g[s][l];
      }
    V ps, rh;
    site_psi<C, NS>(p, g, ps, rh);
    if (WALLS && !row_fluid<WALLS>(yg[m], ly)) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        ps.v[s] = p.psiw[s];
        rh.v[s] = p.rhow[s];
      }
    }
    psi[pe[m]] = ps;
    if (NS == 2) rhol[pe[m]] = rh;
  }
  __syncthreads();

  const int sy = tid / BX, sx = tid - sy * BX, x = x0 + sx, y = y0 + sy;
  const bool in = tid < NU && x < lx && y < ly;
  const size_t site = (size_t)y * lx + x, nsite = (size_t)lx * ly;
  const int at = tid < NU ? pe[0] : 2 * EX + 2;
  const V *const pp = psi + at, *const xp = (a.cross_psi ? psi : rhol) + at;
  auto ps = [&](int dx, int dy) { return pp[dy * EX + dx]; };
  auto xr = [&](int dx, int dy) { return xp[dy * EX + dx]; };
  R drho[NS], rho[NS], jx[NS], jy[NS], Fx[NS], Fy[NS];
  site_force<C, NS>(p, f, ps, xr, drho, rho, jx, jy, Fx, Fy);
  R sr = rho[0], mx = jx[0] + R(0.5) * Fx[0], my = jy[0] + R(0.5) * Fy[0];
#pragma unroll
  for (int s = 1; s < NS; ++s) {
    sr += rho[s];
    mx += jx[s] + R(0.5) * Fx[s];
    my += jy[s] + R(0.5) * Fy[s];
  }

  if constexpr (WHAT == WHAT_MOMENTS) {
    auto put = [&](void *out, size_t i, R v) {
      if (out_f32) static_cast<float *>(out)[i] = float(v);
      else static_cast<double *>(out)[i] = double(v);
    };
    if (in) {
      if (out0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) put(out0, s * nsite + site, rho[s]);
      }
      if (out_u) {
        put(out_u, site, mx / sr);
        put(out_u, nsite + site, my / sr);
      }
    }
  }

  if constexpr (WHAT == WHAT_STRESS) {
    // Pressure tensor of the lattice stress section, per site: sum over species of
    // c_s^2 rho_s delta + sigma^(int)_s + (tau_s - 1/2)^2 F_s F_s / rho_s, plus the A-B pair
    // stress.  sigma^(int) follows Appendix A shell by shell (K(q) = G_1 w(q) + G_2 p(q)):
    //   shells 1, 2: K/2 psi(x) sum psi(x + c) c c
    //   shells 4, 8: K/4 sum [psi(x) psi(x + c) + psi(x - c/2) psi(x + c/2)] c c
    //   shell 5:     K/4 psi(x) sum psi(x + c) c c, plus K/4 (psi(x + c_a) psi(x + c_b) + ...) c c
    //                over the first-belt pairs whose difference is c13, c14, c15 or c16
    double sxx = 0.0, sxy = 0.0, syy = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const R k1 = p.K1[s] * R(0.5), k2 = p.K2[s] * R(0.5), k4 = p.K4[s] * R(0.5);  // K4, K8 hold 2 K
      const R k5 = p.K5[s] * R(0.25), k8 = p.K8[s] * R(0.5);
      auto q = [&](int dx, int dy) { return ps(dx, dy).v[s]; };
      const R p0 = q(0, 0);
      const R E = q(1, 0), W = q(-1, 0), N = q(0, 1), S = q(0, -1);
      const R NE_ = q(1, 1), NW = q(-1, 1), SE = q(1, -1), SW = q(-1, -1);
      const R diag = (NE_ + SW) + (NW + SE), dxy = (NE_ + SW) - (NW + SE);
      const R fa = q(2, 2) + q(-2, -2), fb = q(2, -2) + q(-2, 2);
      const R d8 = fa + fb, d8xy = fa - fb;
      const R mid8 = R(2) * (NE_ * SW + NW * SE), mid8xy = R(2) * (NE_ * SW - NW * SE);
      const R qa = q(2, 1) + q(-2, -1), qb = q(2, -1) + q(-2, 1);   // |c_x| = 2
      const R qc = q(1, 2) + q(-1, -2), qd = q(1, -2) + q(-1, 2);   // |c_y| = 2
      const R qx = qa + qb, qy = qc + qd, qxy = (qa + qc) - (qb + qd);
      const R e13 = NE_ * W + E * SW, e14 = NE_ * S + N * SW, e15 = N * SE + NW * S, e16 = NW * E + W * SE;
      R xx = k1 * p0 * (E + W) + k2 * p0 * diag + k4 * (p0 * (q(2, 0) + q(-2, 0)) + R(2) * (E * W)) +
             k8 * (p0 * d8 + mid8) + k5 * (p0 * (R(4) * qx + qy) + (R(4) * (e13 + e16) + (e14 + e15)));
      R yy = k1 * p0 * (N + S) + k2 * p0 * diag + k4 * (p0 * (q(0, 2) + q(0, -2)) + R(2) * (N * S)) +
             k8 * (p0 * d8 + mid8) + k5 * (p0 * (qx + R(4) * qy) + ((e13 + e16) + R(4) * (e14 + e15)));
      R xy = k2 * p0 * dxy + k8 * (p0 * d8xy + mid8xy) + k5 * R(2) * (p0 * qxy + ((e13 + e14) - (e15 + e16)));
      // ideal gas and the discrete forcing correction
      const R cr = (p.tau[s] - R(0.5)) * (p.tau[s] - R(0.5)) / rho[s];
      xx += rho[s] * R(1.0 / 3.0) + cr * Fx[s] * Fx[s];
      yy += rho[s] * R(1.0 / 3.0) + cr * Fy[s] * Fy[s];
      xy += cr * Fx[s] * Fy[s];
      sxx += double(xx);
      sxy += double(xy);
      syy += double(yy);
    }
    if (NS == 2) {
      // A-B repulsion: (G_AB / 2) sum_l t(q) [r_A(x) r_B(x + c) + r_B(x) r_A(x + c)] c c
      const V c0 = xr(0, 0);
      R xx = 0, xy = 0, yy = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int o = 1 - s;
        const R ax = xr(1, 0).v[o] + xr(-1, 0).v[o], ay = xr(0, 1).v[o] + xr(0, -1).v[o];
        const R da = xr(1, 1).v[o] + xr(-1, -1).v[o], db = xr(1, -1).v[o] + xr(-1, 1).v[o];
        xx += c0.v[s] * (p.T1 * ax + p.T2 * (da + db));
        yy += c0.v[s] * (p.T1 * ay + p.T2 * (da + db));
        xy += c0.v[s] * (p.T2 * (da - db));
      }
      sxx += double(R(0.5) * xx);
      sxy += double(R(0.5) * xy);
      syy += double(R(0.5) * yy);
    }
    if (in) {
      auto put = [&](size_t i, double v) {
        if (out_f32) static_cast<float *>(out0)[i] = float(v);
        else static_cast<double *>(out0)[i] = v;
      };
      put(site, sxx);
      put(nsite + site, sxy);
      put(2 * nsite + site, syy);
    }
  }

  if constexpr (WHAT == WHAT_PROFILE) {
    R fsa[NS][9];
    site_relax<C, NS>(p, f, drho, rho, jx, jy, Fx, Fy, fsa);
    // x-momentum crossing the lines above (c_y = +1) and below (c_y = -1) the row when
    // these populations stream, before any wall term
    double kup = 0.0, kdn = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      kup += double(fsa[s][5] - fsa[s][6]);
      kdn += double(fsa[s][8] - fsa[s][7]);
    }
    // pair forces on this site from partners above it, x components: eq. (FORCE) over the
    // links with c_y = 1 (|c|^2 = 2, 5) and c_y = 2 (|c|^2 = 5, 8), and the A-B term over
    // c = (+-1, 1); each +-c_x pair as one difference, as in the force itself
    double i1 = 0.0, i2 = 0.0;
    const V p0 = ps(0, 0), ne = ps(1, 1), nw = ps(-1, 1), qa = ps(2, 1), qB = ps(-2, 1), qc = ps(1, 2), qD = ps(-1, 2),
            d8a = ps(2, 2), d8B = ps(-2, 2);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const R up1 = fmadd(p.K2[s], ne.v[s] - nw.v[s], p.K5[s] * (R(2) * (qa.v[s] - qB.v[s])));
      const R up2 = fmadd(p.K5[s], qc.v[s] - qD.v[s], p.K8[s] * (d8a.v[s] - d8B.v[s]));
      i1 += double(-p0.v[s] * (up1 + up2));
      i2 += double(-p0.v[s] * up2);
    }
    if (NS == 2) {
      const V c0 = xr(0, 0), xne = xr(1, 1), xnw = xr(-1, 1);
#pragma unroll
      for (int s = 0; s < NS; ++s) i1 += double(-c0.v[s] * (p.T2 * (xne.v[1 - s] - xnw.v[1 - s])));
    }
    const double v[PROF_N] = {double(mx / sr), kup, kdn, i1, i2, double(rho[0]), NS == 2 ? double(rho[NS - 1]) : 0.0};
    __syncthreads();
    double *const sm = reinterpret_cast<double *>(lb_smem);  // [PROF_N][BY][BX + 1]
    if (tid < NU) {
#pragma unroll
      for (int k = 0; k < PROF_N; ++k) sm[(k * BY + sy) * (BX + 1) + sx] = in ? v[k] : 0.0;
    }
    __syncthreads();
    constexpr int G = 8;  // lanes per sum
    static_assert(PROF_N * BY * G <= NT, "one pass over the sums");
    if (tid < PROF_N * BY * G) {
      const int row = tid / G, j = tid - row * G, k = row / BY, r = row - k * BY;
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < BX / G; ++i) t += sm[row * (BX + 1) + i * G + j];
#pragma unroll
      for (int o = G / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
      if (j == 0 && y0 + r < ly) static_cast<double *>(out0)[((size_t)bx * ly + y0 + r) * PROF_N + k] = t;
    }
  }

  if constexpr (WHAT == WHAT_OBSERVE) {
    double v[RED_N] = {};
    bool bad = false;
    v[RED_MASS0] = double(rho[0]);
    if (NS == 2) v[RED_MASS1] = double(rho[NS - 1]);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      v[RED_PX] += double(jx[s]);
      v[RED_PY] += double(jy[s]);
      bad = bad || !(rho[s] > R(0) && rho[s] < R(INFINITY));
    }
    v[RED_FLOW] = double(mx / sr);
    v[RED_BAD] = bad ? 1.0 : 0.0;
    __syncthreads();
    double *const sm = reinterpret_cast<double *>(lb_smem);  // [RED_N][NU]
    if (tid < NU) {
#pragma unroll
      for (int k = 0; k < RED_N; ++k) sm[k * NU + tid] = in ? v[k] : 0.0;
    }
    __syncthreads();
    for (int k = tid >> 6; k < RED_N; k += NT / 64) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < NU / 64; ++i) t += sm[k * NU + i * 64 + (tid & 63)];
      t = wave_sum(t);
      if ((tid & 63) == 0) part[k] = t;
    }
  }
}

// One lattice: one workgroup per tile, row by row, in contiguous ranges over the XCDs.
template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int NT>
__global__ __launch_bounds__(NT) void observe_kernel(TileArgs<typename Codec<MODE>::R> a, void *out0, void *out_u, int out_f32,
                                                     double *partials) {
  const uint32_t logical = (uint32_t)xcd_remap(blockIdx.x, gridDim.x), by = logical / a.ntx;
  observe_tile<MODE, NS, WALLS, WHAT, BX, BY, NT>(a, a.src, (int)(logical - by * a.ntx), (int)by, out0, out_u, out_f32,
                                                  partials ? partials + (size_t)blockIdx.x * RED_N : nullptr);
}

// The totals of many lattices: `blocks` workgroups per instance, of which its own number of tiles work.
template <int MODE, int NS, bool WALLS, int BX, int BY, int NT>
__global__ __launch_bounds__(NT) void batch_observe_kernel(const TileArgs<typename Codec<MODE>::R> *inst, const ReduceJob *jobs,
                                                           const char *src, int first, int blocks, double *partials) {
  const int logical = xcd_remap(blockIdx.x, gridDim.x), i = first + logical / blocks, t = logical - (i - first) * blocks;
  const ReduceJob j = jobs[i];
  if (t >= j.n) return;
  const auto &a = inst[i];
  const int ntx = (a.lx + BX - 1) / BX, by = t / ntx;
  observe_tile<MODE, NS, WALLS, WHAT_OBSERVE, BX, BY, NT>(a, src + a.offset, t - by * ntx, by, nullptr, nullptr, 0,
                                                          partials + (size_t)(j.p0 + t) * RED_N);
}

template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int NT>
static hipError_t launch_observe_k(const StepArgs &a, void *out0, hipStream_t st) {
  using C = Codec<MODE>;
  const auto t = make_tile_args<typename C::R>(a, (uint32_t)(NS * sizeof(typename C::S)), BX, BY);
  const int nb = (int)t.ntx * ((a.ly + BY - 1) / BY);
  hipLaunchKernelGGL((observe_kernel<MODE, NS, WALLS, WHAT, BX, BY, NT>), dim3(nb), dim3(NT),
                     (observe_lds_bytes<MODE, NS, WHAT, BX, BY>()), st, t, out0, a.out_u, a.out_f32,
                     WHAT == WHAT_OBSERVE ? a.partials : nullptr);
  return hipGetLastError();
}

template <int MODE, int NS, bool WALLS>
static hipError_t launch_observe_t(int what, bool wide, const StepArgs &a, hipStream_t st) {
  constexpr int X = kObserveX, Y = kObserveY;
  switch (what) {
    case WHAT_MOMENTS:
      return wide ? launch_observe_k<MODE, NS, WALLS, WHAT_MOMENTS, X, Y, X * Y>(a, a.out_rho, st)
                  : launch_observe_k<MODE, NS, WALLS, WHAT_MOMENTS, 16, 8, 256>(a, a.out_rho, st);
    case WHAT_STRESS:
      return wide ? launch_observe_k<MODE, NS, WALLS, WHAT_STRESS, X, Y, X * Y>(a, a.out_sigma, st)
                  : launch_observe_k<MODE, NS, WALLS, WHAT_STRESS, 16, 8, 256>(a, a.out_sigma, st);
    case WHAT_PROFILE: return launch_observe_k<MODE, NS, WALLS, WHAT_PROFILE, X, Y, X * Y>(a, a.prof, st);
    case WHAT_OBSERVE: return launch_observe_k<MODE, NS, WALLS, WHAT_OBSERVE, X, Y, X * Y>(a, nullptr, st);
  }
  return hipErrorInvalidValue;
}

template <int MODE>
static hipError_t launch_observe_m(int ns, int walls, int what, bool wide, const StepArgs &a, hipStream_t st) {
  if (ns == 1) return walls ? launch_observe_t<MODE, 1, true>(what, wide, a, st) : launch_observe_t<MODE, 1, false>(what, wide, a, st);
  return walls ? launch_observe_t<MODE, 2, true>(what, wide, a, st) : launch_observe_t<MODE, 2, false>(what, wide, a, st);
}

template <int MODE, int NS, bool WALLS>
static hipError_t launch_batch_observe_t(int first, int count, int blocks, const BatchTiles &b, const ReduceJob *jobs,
                                         double *partials, hipStream_t st) {
  constexpr int X = kObserveX, Y = kObserveY;
  hipLaunchKernelGGL((batch_observe_kernel<MODE, NS, WALLS, X, Y, X * Y>), dim3(count * blocks), dim3(X * Y),
                     (observe_lds_bytes<MODE, NS, WHAT_OBSERVE, X, Y>()), st,
                     static_cast<const TileArgs<typename Codec<MODE>::R> *>(b.inst), jobs, b.src, first, blocks, partials);
  return hipGetLastError();
}

template <int MODE>
static hipError_t launch_batch_observe_m(int ns, int walls, int first, int count, int blocks, const BatchTiles &b,
                                         const ReduceJob *jobs, double *partials, hipStream_t st) {
  if (ns == 1)
    return walls ? launch_batch_observe_t<MODE, 1, true>(first, count, blocks, b, jobs, partials, st)
                 : launch_batch_observe_t<MODE, 1, false>(first, count, blocks, b, jobs, partials, st);
  return walls ? launch_batch_observe_t<MODE, 2, true>(first, count, blocks, b, jobs, partials, st)
               : launch_batch_observe_t<MODE, 2, false>(first, count, blocks, b, jobs, partials, st);
}

}  // namespace lb355
