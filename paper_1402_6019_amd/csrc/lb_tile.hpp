#pragma once
// Steps in rectangular tiles, N time steps per launch with the states in between in LDS.
//
// The row-marching step needs tall segments to amortise its five lead rows, and a lattice of a
// few hundred rows spread over 256 compute units leaves one or two rows to each: its launches then
// pull six rows for one and last about 10 us whatever the size, almost all of it latency (a
// dependent chain of loads, barrier and update per row).  Here a workgroup owns a tile of BX x BY
// sites.  The region a tile depends on grows by three sites per step (two for psi, one for the
// pull), so a workgroup that starts from its tile plus 3 N - 1 sites on each side takes N steps by
// itself: the overlaps are recomputed by the neighbours, which costs arithmetic that a small
// lattice leaves idle, and N - 1 launches with their memory round trips are saved; a large one
// crosses memory once per N steps.
//
// Per step, marched (pairs where those were the default) and now: 64 x 64 FP64 9.9 and 2.05 us,
// 188 x 168 9.95 and 2.5 (both latency: about 2 us of loads, barrier, stencil and collision);
// 1024 x 1024 FP32, two species, 27.7 and 19, 4096 x 512 with walls 53.9 and 44 (vector issue: units
// busy 75%, three quarters of the instructions in the updates, 1.63 of them per result in the
// first step; 302 MB per launch of two steps at 3.4 TB/s).
//
// Stage k = 1 .. N of a workgroup, with H = 3 (N - k) the margin around the tile that its result
// must reach:
//   pull of the sites of tile + H + 2 (from memory in the first stage, from the LDS copy of f*
//   later) into registers, psi and rho of each into LDS; barrier; force and collision of the sites
//   of tile + H from the registers and LDS; f* into LDS (rounded as a store and a load would round
//   it), or into memory after the last stage; barrier.
// The sites of tile + H come first in the list that the threads share out, row by row, then the
// two-site frame around them, which only needs psi.  Per-site arithmetic: lb_site.hpp, bitwise
// that of the row-marching step.

#include "lb_site.hpp"

namespace lb355 {

template <int BX, int BY, int N>
struct TileDims {
  static constexpr int h(int k) { return 3 * (N - k); }
  static constexpr int ux(int k) { return BX + 2 * h(k); }
  static constexpr int nu(int k) { return ux(k) * (BY + 2 * h(k)); }          // sites updated
  static constexpr int ex(int k) { return ux(k) + 4; }
  static constexpr int ne(int k) { return ex(k) * (BY + 2 * h(k) + 4); }      // sites pulled
  // entries (values of all species) of the psi, rho (two species) and f* (N > 1) copies
  static constexpr int lds_entries(int ns) { return ne(1) * ns + (N > 1 ? 9 * nu(1) : 0); }
};

template <int MODE, int NS, int BX, int BY, int N>
constexpr size_t tile_lds_bytes() {
  return (size_t)TileDims<BX, BY, N>::lds_entries(NS) * NS * (MODE == MODE_F64 ? 8 : 4);
}

// A coordinate wrapped onto [0, n); lattices narrower than a region may wrap more than once.
__device__ __forceinline__ int wrap_any(int v, int n, bool narrow) { return narrow ? ((v % n) + n) % n : wrapi(v, n); }

// Site tid + m NT of the list of a stage that updates a tile and a margin of H: those sites row by row,
// then the two-site frame around them; relative to the tile's first site.
template <int BX, int BY, int H, int NT>
__device__ __forceinline__ void tile_site(int tid, int m, int &sx, int &sy) {
  constexpr int UX = BX + 2 * H, EX = UX + 4, NU = UX * (BY + 2 * H), NE = EX * (BY + 2 * H + 4);
  const int i = min(tid + m * NT, NE - 1);
  const int r = i / UX;
  sx = i - r * UX - H;
  sy = r - H;
  if ((m + 1) * NT > NU) {
    // the frame: two rows below, two above, then two columns on either side
    const int q = max(i - NU, 0), t = q - 4 * EX;
    const int fr = q / EX, fy = fr < 2 ? fr - 2 : fr + (BY + 2 * H) - 2;
    const int c = t & 3, fc = c < 2 ? c - 2 : c + UX - 2;
    const int fx = t < 0 ? q - fr * EX - 2 : fc, fz = t < 0 ? fy : t >> 2;
    const bool frame = m * NT >= NU || i >= NU;
    sx = frame ? fx - H : sx;
    sy = frame ? fz - H : sy;
  }
}

// Byte offsets of the nine pulls of site (x, y): rows past a wall pull the row next to it (their values
// are not used).  The plane goes into the uniform offset; a reflected pull, of the opposite plane two
// planes up (off the lower wall) or down, has that difference in its lane offset.
template <bool WALLS, typename A>
__device__ __forceinline__ void pull_offsets(const A &a, uint32_t site_b, int x, int yg, uint32_t (&o)[9]) {
  const int lx = a.lx, ly = a.ly;
  const uint32_t plane_b = a.pitch_b, row_b = 9u * a.pitch_b;
  const int y = WALLS ? min(max(yg, 0), ly - 1) : yg;
  const bool lo = y == 0, hi = y == ly - 1;
  const uint32_t ro = (uint32_t)y * row_b;
  const uint32_t rm = lo ? (WALLS ? 2 * plane_b : (uint32_t)(ly - 1) * row_b) : ro - row_b;
  const uint32_t rp = hi ? (WALLS ? ro - 2 * plane_b : 0u) : ro + row_b;
  const uint32_t cc = (uint32_t)x * site_b, cm = (x == 0 ? (uint32_t)lx * site_b : cc) - site_b,
                 cp = x == lx - 1 ? 0u : cc + site_b;
  o[0] = ro + cc;
  o[1] = ro + cm;
  o[3] = ro + cp;
  o[2] = rm + cc;
  o[5] = rm + (WALLS && lo ? cc : cm);
  o[6] = rm + (WALLS && lo ? cc : cp);
  o[4] = rp + cc;
  o[7] = rp + (WALLS && hi ? cc : cp);
  o[8] = rp + (WALLS && hi ? cc : cm);
}

// N steps of the tile whose first site is (x0, y0), of the lattice described by a, from src to dst.
// t0: time step of the first (stochastic rounding); red_mask: which steps reduce, into the
// running sums accrow.
template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int N, int NT, int STP>
__device__ __forceinline__ void tile_steps(const TileArgs<typename Codec<MODE>::R> &a, const void *const src,
                                           void *const dst, const int x0, const int y0, const uint32_t t0,
                                           const uint32_t red_mask, double *const accrow) {
  using C = Codec<MODE>;
  using R = typename C::R;
  using S = typename C::S;
  using L = typename C::L;
  using V = Vec<R, NS>;
  using D = TileDims<BX, BY, N>;
  constexpr bool ACCUM = WHAT == WHAT_STEP_ACCUM;
  constexpr bool FIELDS = WHAT == WHAT_STEP_FIELDS || WHAT == WHAT_STEP_FIELDS32;
  V *const psi = reinterpret_cast<V *>(lb_smem);
  V *const rhol = psi + (NS == 2 ? D::ne(1) : 0);
  V *const fst = psi + NS * D::ne(1);  // f*: [9][rows][FX]
  constexpr int FX = D::ux(1), FN = D::nu(1), FO = D::h(1);

  const int lx = a.lx, ly = a.ly;
  constexpr uint32_t site_b = (uint32_t)(NS * sizeof(S));
  const uint32_t plane_b = a.pitch_b, row_b = 9u * a.pitch_b, buf_b = a.buf_b;
  const int tid = threadIdx.x;
  const bool narrow_x = lx < D::ex(1) + BX, narrow_y = ly < D::ex(1) - BX + 2 * BY;
  const SiteConsts<R> &p = a.c;

  double wb = 0.0, wt = 0.0, nbad = 0.0;

  auto stage = [&](auto kc) {
    constexpr int k = decltype(kc)::value;
    constexpr int H = D::h(k), UX = D::ux(k), EX = D::ex(k), NU = D::nu(k), NE = D::ne(k);
    constexpr int M = (NE + NT - 1) / NT, MU = (NU + NT - 1) / NT;
    int pe[M], yg[M];  // the corner (-2, -2) of the site's neighbourhood in psi, and its row
    R f[M][NS][9];
    if constexpr (k == 1) {
      const Rsrc rs = make_rsrc(src, buf_b);
      L fl[M][NS][9];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        // a wave past the list's end (1024^2, FP32: 21.7 -> 21.1 us per step; an 8 x 8 tile, bound by
        // latency, gains nothing from it and loses 1.5% to the branch)
        if (BX * BY > 64 && (m + 1) * NT - NE >= 64 && (int)uni((uint32_t)tid & ~63u) + m * NT >= NE) continue;
        int sx, sy;
        tile_site<BX, BY, H, NT>(tid, m, sx, sy);
        pe[m] = (sy + H) * EX + sx + H;
        const int x = wrap_any(x0 + sx, lx, narrow_x);
        yg[m] = WALLS ? y0 + sy : wrap_any(y0 + sy, ly, narrow_y);
        uint32_t o[9];
        pull_offsets<WALLS>(a, site_b, x, yg[m], o);
#pragma unroll
        for (int l = 0; l < 9; ++l) {
          if (NS == 2) C::bload2(rs, o[l], uni((uint32_t)l * plane_b), fl[m][0][l], fl[m][NS - 1][l]);
          else fl[m][0][l] = C::bload(rs, o[l], uni((uint32_t)l * plane_b));
        }
      }
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int l = 0; l < 9; ++l) f[m][s][l] = C::dec(fl[m][s][l], s);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if ((m + 1) * NT > NE && tid + m * NT >= NE) continue;
      if constexpr (k > 1) {
        int sx, sy;
        tile_site<BX, BY, H, NT>(tid, m, sx, sy);
        pe[m] = (sy + H) * EX + sx + H;
        yg[m] = WALLS ? y0 + sy : 0;
        const bool lo = WALLS && yg[m] == 0, hi = WALLS && yg[m] == ly - 1;
        const V *q = fst + (sy + FO - 1) * FX + sx + FO - 1;  // corner (-1, -1)
        V g[9];
        g[0] = q[FX + 1];
        g[1] = q[FN + FX];
        g[3] = q[3 * FN + FX + 2];
        g[2] = q[lo ? 4 * FN + FX + 1 : 2 * FN + 1];
        g[5] = q[lo ? 7 * FN + FX + 1 : 5 * FN];
        g[6] = q[lo ? 8 * FN + FX + 1 : 6 * FN + 2];
        g[4] = q[hi ? 2 * FN + FX + 1 : 4 * FN + 2 * FX + 1];
        g[7] = q[hi ? 5 * FN + FX + 1 : 7 * FN + 2 * FX + 2];
        g[8] = q[hi ? 6 * FN + FX + 1 : 8 * FN + 2 * FX];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int l = 0; l < 9; ++l) f[m][s][l] = g[l].v[s];
      }
      V ps, rh;
      site_psi<C, NS>(p, f[m], ps, rh);
      if (WALLS && !row_fluid<WALLS>(yg[m], ly)) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          ps.v[s] = p.psiw[s];
          rh.v[s] = p.rhow[s];
        }
      }
      psi[pe[m] + 2 * EX + 2] = ps;
      if (NS == 2) rhol[pe[m] + 2 * EX + 2] = rh;
    }
    __syncthreads();

    uint32_t tseed = 0;
    if constexpr (MODE == MODE_BF16SR) tseed = mix32((t0 + (uint32_t)(k - 1)) * 0x9e3779b9u + 0x632be5abu);
    const V *const xb = a.cross_psi ? psi : rhol;
#pragma unroll
    for (int m = 0; m < MU; ++m) {
      const int i = tid + m * NT;
      if (i >= NU || !row_fluid<WALLS>(yg[m], ly)) continue;  // nothing pulls from a site past a wall
      const int sy = i / UX - H, sx = i - (i / UX) * UX - H;
      // of the tile's own sites, those of a ragged last tile past the lattice's end are not stored
      const bool in = (unsigned)sx < (unsigned)BX && (unsigned)sy < (unsigned)BY && x0 + sx < lx && y0 + sy < ly;
      if (k == N && !in) continue;
      if constexpr (FIELDS) {
        // what the adjoint's reverse step reads of the state stepped from (see the fused step)
        using RA = typename std::conditional<WHAT == WHAT_STEP_FIELDS, double, float>::type;
        if (in) {
          const int x = x0 + sx, y = y0 + sy;
          const size_t at = (size_t)y * lx + x, nsite = (size_t)lx * ly;
          RA *fl = reinterpret_cast<RA *>(static_cast<char *>(a.fields) + (size_t)(k - 1) * a.fields_stride);
          double *xw = reinterpret_cast<double *>(static_cast<char *>(a.xw) + (size_t)(k - 1) * a.xw_stride);
          const bool wall_row = WALLS && (y == 0 || y == ly - 1);
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            RA r = 0, px = 0, py = 0;
#pragma unroll
            for (int l = 0; l < 9; ++l) {
              const double fv = double(f[m][s][l]) + WD2Q9[l] * a.rho_ref[s];
              if (wall_row) xw[((size_t)(s * 9 + l) * 2 + (y == 0 ? 0 : 1)) * lx + x] = fv;
              const RA g = RA(fv);
              r += g;
              px += RA(CXS[l]) * g;
              py += RA(CYS[l]) * g;
            }
            fl[(size_t)(0 * 2 + s) * nsite + at] = r;
            fl[(size_t)(1 * 2 + s) * nsite + at] = RA(a.psi0) * (RA(1) - exp(-r * RA(a.irho0)));
            fl[(size_t)(2 * 2 + s) * nsite + at] = px;
            fl[(size_t)(3 * 2 + s) * nsite + at] = py;
          }
        }
      }
      R fsa[NS][9], rho[NS];
      const V *pp = psi + pe[m], *xp = xb + pe[m];
      site_update<C, NS>(p, f[m], [&](int dx, int dy) { return pp[(dy + 2) * EX + dx + 2]; },
                         [&](int dx, int dy) { return xp[(dy + 2) * EX + dx + 2]; }, rho, fsa);
      if constexpr (ACCUM) {
        if (in && ((red_mask >> (k - 1)) & 1u)) {
          bool bad = false;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            bad = bad || !(rho[s] > R(0) && rho[s] < R(INFINITY));
            if (WALLS && yg[m] == 0) wb += 2.0 * (double(fsa[s][8]) - double(fsa[s][7])) - 2.0 * a.wall_mom[0][s];
            if (WALLS && yg[m] == ly - 1) wt += 2.0 * (double(fsa[s][5]) - double(fsa[s][6])) - 2.0 * a.wall_mom[1][s];
          }
          nbad += bad ? 1.0 : 0.0;
        }
      }
      if (WALLS && a.moving) moving_walls<R, NS>(a.wall_mom, yg[m], ly, fsa);
      uint32_t hs = 0;
      if constexpr (MODE == MODE_BF16SR) {
        const int x = wrap_any(x0 + sx, lx, narrow_x), y = WALLS ? yg[m] : wrap_any(y0 + sy, ly, narrow_y);
        hs = mix32((uint32_t)(y * lx + x) ^ tseed);
      }
      if constexpr (k == N) {
        const Rsrc rd = make_rsrc(dst, buf_b);
        const uint32_t o = (uint32_t)(y0 + sy) * row_b + (uint32_t)(x0 + sx) * site_b;
#pragma unroll
        for (int l = 0; l < 9; ++l) {
          const uint32_t so = uni((uint32_t)l * plane_b);
          if constexpr (MODE == MODE_BF16SR) {
            const uint32_t rnd = mix32(hs + (uint32_t)l * 0x9e3779b9u);
            if (NS == 2) C::template bstore2_sr<STP>(rd, o, so, fsa[0][l], fsa[NS - 1][l], rnd);
            else C::template bstore_sr<STP>(rd, o, so, fsa[0][l], rnd);
          } else {
            if (NS == 2) C::template bstore2<STP>(rd, o, so, fsa[0][l], fsa[NS - 1][l]);
            else C::template bstore<STP>(rd, o, so, fsa[0][l]);
          }
        }
      } else {
        V *q = fst + (sy + FO) * FX + sx + FO;
#pragma unroll
        for (int l = 0; l < 9; ++l) {
          V v;
#pragma unroll
          for (int s = 0; s < NS; ++s) v.v[s] = stored_value<MODE>(fsa[s][l], s, l, hs);
          q[l * FN] = v;
        }
      }
    }
    if constexpr (k < N) __syncthreads();
  };
  stage(std::integral_constant<int, 1>{});
  if constexpr (N >= 2) stage(std::integral_constant<int, 2>{});
  if constexpr (N >= 3) stage(std::integral_constant<int, 3>{});

  if constexpr (ACCUM) {
    // this workgroup's running sums: every wave's, then the waves in order
    constexpr int NW = NT / 64;
    __shared__ double red[NW][ACC_N];
    const double v[ACC_N] = {wave_sum(wb), wave_sum(wt), wave_sum(nbad)};
    if ((tid & 63) == 0) {
#pragma unroll
      for (int k = 0; k < ACC_N; ++k) red[tid >> 6][k] = v[k];
    }
    __syncthreads();
    if (tid < ACC_N) {
      double t = 0.0;
      for (int w = 0; w < NW; ++w) t += red[w][tid];
      accrow[tid] += t;
    }
  }
}

// One lattice: one workgroup per tile, tiles row by row, in contiguous ranges over the XCDs.
template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int N, int NT, int STP>
__global__ __launch_bounds__(NT) void tile_kernel(TileArgs<typename Codec<MODE>::R> a) {
  const uint32_t logical = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t by = a.ntx_mul ? __umulhi(logical, a.ntx_mul) : logical / a.ntx;
  tile_steps<MODE, NS, WALLS, WHAT, BX, BY, N, NT, STP>(
      a, a.src, a.dst, (int)(logical - by * a.ntx) * BX, (int)by * BY, launch_step_index<MODE>(a.t_step, a.t_base),
      a.red_mask, WHAT == WHAT_STEP_ACCUM ? a.accrows + (size_t)blockIdx.x * ACC_N : nullptr);
}

// Many lattices: one workgroup per entry of the host's list of every instance's tiles.
template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int N, int NT, int STP>
__global__ __launch_bounds__(NT) void batch_tile_kernel(BatchTileArgs<typename Codec<MODE>::R> b) {
  const TileDesc td = b.tiles[xcd_remap(blockIdx.x, gridDim.x)];
  const auto &a = b.inst[uni((uint32_t)td.inst)];
  tile_steps<MODE, NS, WALLS, WHAT, BX, BY, N, NT, STP>(
      a, b.src + a.offset, b.dst + a.offset, (int)uni((uint32_t)td.strip) * BX, (int)uni((uint32_t)td.seg) * BY,
      launch_step_index<MODE>(b.t_step, b.t_base), b.red_mask,
      WHAT == WHAT_STEP_ACCUM ? b.accrows + (size_t)td.part * ACC_N : nullptr);
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------

template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int N, int NT, int STP>
static hipError_t launch_tile_k(const StepArgs &a, const TileOpts &o, hipStream_t st) {
  using C = Codec<MODE>;
  TileArgs<typename C::R> t = make_tile_args<typename C::R>(a, (uint32_t)(NS * sizeof(typename C::S)), BX, BY);
  t.red_mask = o.red_mask;
  t.fields_stride = o.fields_stride;
  t.xw_stride = o.xw_stride;
  const int nb = (int)t.ntx * ((a.ly + BY - 1) / BY);
  hipLaunchKernelGGL((tile_kernel<MODE, NS, WALLS, WHAT, BX, BY, N, NT, STP>), dim3(nb), dim3(NT),
                     (tile_lds_bytes<MODE, NS, BX, BY, N>()), st, t);
  return hipGetLastError();
}

template <int MODE, int NS, bool WALLS, int WHAT, int BX, int BY, int N, int NT, int STP>
static hipError_t launch_tile_k(const BatchTiles &b, const TileOpts &o, hipStream_t st) {
  using R = typename Codec<MODE>::R;
  BatchTileArgs<R> t{static_cast<const TileArgs<R> *>(b.inst), b.tiles, b.src, b.dst, b.accrows, o.red_mask, b.t_step, b.t_base};
  hipLaunchKernelGGL((batch_tile_kernel<MODE, NS, WALLS, WHAT, BX, BY, N, NT, STP>), dim3(b.ntiles), dim3(NT),
                     (tile_lds_bytes<MODE, NS, BX, BY, N>()), st, t);
  return hipGetLastError();
}

// n = 1 .. tile_most_steps steps of a lattice (A: StepArgs) or a batch (BatchTiles) in tiles of the
// shape; store policy by a.stream_stores.
template <int MODE, int NS, bool WALLS, int WHAT, typename A>
static hipError_t launch_tile_w(int shape, int n, const A &a, const TileOpts &o, hipStream_t st) {
  constexpr int WT = kStoreWriteThrough, NTS = kStoreStreaming;
  // two species in FP64 leave one workgroup per compute unit (155 KB of LDS), which then takes twelve
  // waves: 2048 x 1024 106 -> 103 us per step, 4096 x 512 walled 110.6 -> 107.6; else two of eight
  constexpr int LAST = MODE == MODE_F64 && NS == 2 ? 768 : 512;
  switch (shape * 4 + n) {
    case 0 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 4, 8, 1, 128, WT>(a, o, st);
    case 0 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 4, 8, 2, 256, WT>(a, o, st);
    case 0 * 4 + 3: return launch_tile_k<MODE, NS, WALLS, WHAT, 4, 8, 3, 448, WT>(a, o, st);
    case 1 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 8, 8, 1, 256, WT>(a, o, st);
    case 1 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 8, 8, 2, 384, WT>(a, o, st);
    case 1 * 4 + 3: return launch_tile_k<MODE, NS, WALLS, WHAT, 8, 8, 3, 512, WT>(a, o, st);
    case 2 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 8, 1, 256, WT>(a, o, st);
    case 2 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 8, 2, 512, WT>(a, o, st);
    case 2 * 4 + 3: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 8, 3, 512, WT>(a, o, st);
    case 3 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 16, 1, 448, WT>(a, o, st);
    case 3 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 16, 2, 512, WT>(a, o, st);
    case 3 * 4 + 3: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 16, 3, 576, WT>(a, o, st);
    case 4 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 1, 512, WT>(a, o, st);
    case 4 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 2, 768, WT>(a, o, st);
    case 4 * 4 + 3:
      if constexpr (tile_lds_bytes<MODE, NS, 32, 16, 3>() <= 160 * 1024) return launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 3, 768, WT>(a, o, st);
      break;
    case 5 * 4 + 1:
      return a.stream_stores ? launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 1, 512, NTS>(a, o, st)
                             : launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 1, 512, WT>(a, o, st);
    case 5 * 4 + 2:
      return a.stream_stores ? launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 2, LAST, NTS>(a, o, st)
                             : launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 2, LAST, WT>(a, o, st);
  }
  return hipErrorInvalidValue;
}

template <int MODE, int WHAT, typename A>
static hipError_t launch_tile_m(int ns, int walls, int shape, int n, const A &a, const TileOpts &o, hipStream_t st) {
  if (ns == 1) return walls ? launch_tile_w<MODE, 1, true, WHAT>(shape, n, a, o, st) : launch_tile_w<MODE, 1, false, WHAT>(shape, n, a, o, st);
  return walls ? launch_tile_w<MODE, 2, true, WHAT>(shape, n, a, o, st) : launch_tile_w<MODE, 2, false, WHAT>(shape, n, a, o, st);
}

// The passes that also write the adjoint's fields: one or two steps, stores written through (the
// recomputed states' buffers are read again at once).
template <int MODE, int NS, bool WALLS, int WHAT>
static hipError_t launch_tile_fields(int shape, int n, const StepArgs &a, const TileOpts &o, hipStream_t st) {
  constexpr int WT = kStoreWriteThrough;
  switch (shape * 4 + n) {
    case 0 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 4, 8, 1, 128, WT>(a, o, st);
    case 0 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 4, 8, 2, 256, WT>(a, o, st);
    case 1 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 8, 8, 1, 256, WT>(a, o, st);
    case 1 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 8, 8, 2, 384, WT>(a, o, st);
    case 2 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 8, 1, 256, WT>(a, o, st);
    case 2 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 8, 2, 512, WT>(a, o, st);
    case 3 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 16, 1, 448, WT>(a, o, st);
    case 3 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 16, 16, 2, 512, WT>(a, o, st);
    case 4 * 4 + 1:
    case 5 * 4 + 1: return launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 1, 512, WT>(a, o, st);
    case 4 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 2, 768, WT>(a, o, st);
    case 5 * 4 + 2: return launch_tile_k<MODE, NS, WALLS, WHAT, 32, 16, 2, 512, WT>(a, o, st);
  }
  return hipErrorInvalidValue;
}

template <int MODE, int WHAT>
static hipError_t launch_tile_fields_m(int ns, int walls, int shape, int n, const StepArgs &a, const TileOpts &o,
                                       hipStream_t st) {
  if (ns == 1) return walls ? launch_tile_fields<MODE, 1, true, WHAT>(shape, n, a, o, st) : launch_tile_fields<MODE, 1, false, WHAT>(shape, n, a, o, st);
  return walls ? launch_tile_fields<MODE, 2, true, WHAT>(shape, n, a, o, st) : launch_tile_fields<MODE, 2, false, WHAT>(shape, n, a, o, st);
}

template <int MODE, typename A>
static hipError_t launch_tile_what(int ns, int walls, int what, int shape, int n, const A &a, const TileOpts &o,
                                   hipStream_t st) {
  switch (what) {
    case WHAT_STEP: return launch_tile_m<MODE, WHAT_STEP>(ns, walls, shape, n, a, o, st);
    case WHAT_STEP_ACCUM: return launch_tile_m<MODE, WHAT_STEP_ACCUM>(ns, walls, shape, n, a, o, st);
  }
  if constexpr (std::is_same<A, StepArgs>::value && MODE != MODE_BF16SR) {  // the adjoint: one lattice, no random rounding
    switch (what) {
      case WHAT_STEP_FIELDS: return launch_tile_fields_m<MODE, WHAT_STEP_FIELDS>(ns, walls, shape, n, a, o, st);
      case WHAT_STEP_FIELDS32: return launch_tile_fields_m<MODE, WHAT_STEP_FIELDS32>(ns, walls, shape, n, a, o, st);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace lb355
