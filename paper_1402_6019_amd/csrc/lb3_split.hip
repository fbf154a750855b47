// The three-dimensional step of a lattice that the caches hold, in two passes: psi and rho of every
// site into a field, then the update of every site from the field and a second pull.
//
// The march of lb3_march.hip reads memory once but walks its segments plane by plane, each plane a
// chain of loads, barrier and update; a lattice of a few hundred thousand sites leaves segments of a
// few planes, of which four more have to be pulled before the first update, and the launch lasts
// as long as that chain.  Where the populations come from the caches a second read of them
// costs less: both passes here are free of such chains, with every tile independent.
// Per-site arithmetic and its order are those of lb3_kernels.hip (bitwise the same populations).

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lb3_site.hpp"

namespace lb355 {

namespace {

// Tile of the update pass and its frames of two sites (psi) and one (rho).
constexpr int SX = 32, SY = 4, SZ = 4;
constexpr int PX = SX + 4, PY = SY + 4, PZ = SZ + 4, QX = SX + 2, QY = SY + 2, QZ = SZ + 2;

__device__ __forceinline__ int wrap3(int v, int n, bool narrow) { return narrow ? ((v % n) + n) % n : d3::wrap(v, n); }

}  // namespace

extern __shared__ __attribute__((aligned(16))) unsigned char split3_smem[];

// psi and rho (two species) of every site, [z][y][x]: tiles of 32 x 8 sites of a plane.
template <int MODE, int NS, bool WALLS>
__global__ __launch_bounds__(256) void psi3_kernel(Lb3Args a) {
  using C = Codec<MODE>;
  using R = typename C::R;
  using S = typename C::S;
  using V = Vec<R, NS>;
  constexpr uint32_t site_b = (uint32_t)(NS * sizeof(S));
  const uint32_t plane_b = (uint32_t)a.pitch * site_b, row_b = 19u * plane_b;
  const uint64_t zplane_b = (uint64_t)row_b * (uint32_t)a.ly;
  const int x = blockIdx.x * 32 + (threadIdx.x & 31), y = blockIdx.y * 8 + (threadIdx.x >> 5), z = blockIdx.z;
  const bool ok = x < a.lx && y < a.ly;
  const Site3<R, NS> p(a);
  const Pull3 q = pull3_at<WALLS>(ok ? x : 0, ok ? y : 0, a.lx, a.ly, row_b, site_b);
  Rsrc rz[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    rz[k] = make_rsrc(static_cast<const char *>(a.src) + (uint64_t)(uint32_t)d3::wrap(z + 1 - k, a.lz) * zplane_b,
                      (uint32_t)zplane_b);
  R f[NS][19], fb[NS][2];
  pull3<C, NS, WALLS>(rz, q, plane_b, (uint32_t)zplane_b, f, fb);
  wall_fix3<WALLS>(q, fb, f);
  V ps, rh;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    R sum = f[s][0];
#pragma unroll
    for (int l = 1; l < 19; ++l) sum += f[s][l];
    rh.v[s] = p.rref[s] + sum;
    ps.v[s] = p.psi0 * (R(1) - C::expo(rh.v[s] * p.nirho0));
  }
  if (!ok) return;
  const size_t nsite = (size_t)a.lx * a.ly * a.lz, i = ((size_t)z * a.ly + y) * a.lx + x;
  V *out = static_cast<V *>(a.psi);
  out[i] = ps;
  if (NS == 2) out[nsite + i] = rh;
}

template <int MODE, int NS, bool WALLS, int WHAT, int STP>
__global__ __launch_bounds__(SX *SY *SZ) void split3_kernel(Lb3Args a) {
  using C = Codec<MODE>;
  using R = typename C::R;
  using S = typename C::S;
  using V = Vec<R, NS>;
  constexpr int NT = SX * SY * SZ;
  V *const psi_t = reinterpret_cast<V *>(split3_smem);  // [PZ][PY][PX]
  V *const rho_t = psi_t + PX * PY * PZ;                // [QZ][QY][QX] (two species)
  constexpr uint32_t site_b = (uint32_t)(NS * sizeof(S));
  const uint32_t plane_b = (uint32_t)a.pitch * site_b, row_b = 19u * plane_b;
  const uint64_t zplane_b = (uint64_t)row_b * (uint32_t)a.ly;
  const int lx = a.lx, ly = a.ly, lz = a.lz;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int bz = logical / (a.nstrip * a.nband), rem = logical - bz * (a.nstrip * a.nband);
  const int by = rem / a.nstrip, bx = rem - by * a.nstrip;
  const int x0 = bx * SX, y0 = by * SY, z0 = bz * SZ;
  const int tid = threadIdx.x, tx = tid % SX, ty = tid / SX % SY, tz = tid / (SX * SY);
  const int x = x0 + tx, y = y0 + ty, z = (int)uni((uint32_t)(z0 + tz));  // a wave is in one plane
  const bool ok = x < lx && y < ly && z < lz;
  const Site3<R, NS> p(a);
  const Pull3 q = pull3_at<WALLS>(ok ? x : 0, ok ? y : 0, lx, ly, row_b, site_b);
  Rsrc rz[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    rz[k] = make_rsrc(static_cast<const char *>(a.src) + (uint64_t)(uint32_t)d3::wrap(min(z, lz - 1) + 1 - k, lz) * zplane_b,
                      (uint32_t)zplane_b);
  R f[NS][19], fb[NS][2];
  pull3<C, NS, WALLS>(rz, q, plane_b, (uint32_t)zplane_b, f, fb);

  // the field of the tile and its frames
  const bool narrow = lx < 2 * PX || ly < 2 * PY || lz < 2 * PZ;
  const V *const field = static_cast<const V *>(a.psi);
  const size_t nsite = (size_t)lx * ly * lz;
  auto at = [&](int i, int nx, int ny, int m, bool &wall) -> size_t {  // entry i of an nx x ny x . frame of margin m
    const int ez = i / (nx * ny), r = i - ez * nx * ny, ey = r / nx, ex = r - ey * nx;
    const int yy = y0 + ey - m;
    wall = WALLS && (yy < 0 || yy >= ly);
    const int xs = wrap3(x0 + ex - m, lx, narrow), zs = wrap3(z0 + ez - m, lz, narrow);
    const int ys = WALLS ? min(max(yy, 0), ly - 1) : wrap3(yy, ly, narrow);
    return ((size_t)zs * ly + ys) * lx + xs;
  };
  V pw, rw;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    pw.v[s] = p.psiw[s];
    rw.v[s] = p.rhow[s];
  }
#pragma unroll
  for (int k = 0; k < (PX * PY * PZ + NT - 1) / NT; ++k) {
    const int i = tid + k * NT;
    if (i < PX * PY * PZ) {
      bool wall;
      const size_t j = at(i, PX, PY, 2, wall);
      const V v = field[j];
      psi_t[i] = wall ? pw : v;
    }
  }
  if (NS == 2 && !a.cross_psi) {
#pragma unroll
    for (int k = 0; k < (QX * QY * QZ + NT - 1) / NT; ++k) {
      const int i = tid + k * NT;
      if (i < QX * QY * QZ) {
        bool wall;
        const size_t j = at(i, QX, QY, 1, wall);
        const V v = field[nsite + j];
        rho_t[i] = wall ? rw : v;
      }
    }
  }
  wall_fix3<WALLS>(q, fb, f);
  __syncthreads();

  const V *const pc = psi_t + ((tz + 2) * PY + ty + 2) * PX + tx + 2;
  // the cross term's field and its strides (uniform but for the lane)
  const int xy = a.cross_psi ? PX : QX, xz = a.cross_psi ? PX * PY : QX * QY;
  const V *const xc = a.cross_psi ? pc : rho_t + ((tz + 1) * QY + ty + 1) * QX + tx + 1;
  site3_update<C, NS, WHAT, STP>(
      a, p, f, [&](int dx, int dy, int dz) { return pc[(dz * PY + dy) * PX + dx]; },
      [&](int dx, int dy, int dz) { return xc[dz * xz + dy * xy + dx]; }, x, y, z, ok,
      make_rsrc(static_cast<char *>(a.dst) + (uint64_t)(uint32_t)min(z, lz - 1) * zplane_b, (uint32_t)zplane_b),
      ok ? q.row[1] + q.col[1] : (uint32_t)zplane_b, plane_b);
}

int split3_tiles(int lx, int ly, int lz, int *nstrip, int *nband) {
  *nstrip = (lx + SX - 1) / SX;
  *nband = (ly + SY - 1) / SY;
  return *nstrip * *nband * ((lz + SZ - 1) / SZ);
}

template <int MODE, int NS, bool WALLS, int WHAT>
static hipError_t launch_split3_k(int nb, const Lb3Args &a, hipStream_t st) {
  const size_t lds = (size_t)(PX * PY * PZ + (NS == 2 ? QX * QY * QZ : 0)) * NS * (MODE == MODE_F64 ? 8 : 4);
  hipLaunchKernelGGL((psi3_kernel<MODE, NS, WALLS>), dim3((a.lx + 31) / 32, (a.ly + 7) / 8, a.lz), dim3(256), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((split3_kernel<MODE, NS, WALLS, WHAT, kStoreWriteThrough>), dim3(nb), dim3(SX * SY * SZ), lds, st, a);
  return hipGetLastError();
}

template <int MODE, int NS, bool WALLS>
static hipError_t launch_split3_t(int what, int nb, const Lb3Args &a, hipStream_t st) {
  switch (what) {
    case WHAT_STEP: return launch_split3_k<MODE, NS, WALLS, WHAT_STEP>(nb, a, st);
    case WHAT_MOMENTS: return launch_split3_k<MODE, NS, WALLS, WHAT_MOMENTS>(nb, a, st);
  }
  return hipErrorInvalidValue;
}

template <int MODE>
static hipError_t launch_split3_m(int ns, int walls, int what, int nb, const Lb3Args &a, hipStream_t st) {
  if (ns == 1) return walls ? launch_split3_t<MODE, 1, true>(what, nb, a, st) : launch_split3_t<MODE, 1, false>(what, nb, a, st);
  return walls ? launch_split3_t<MODE, 2, true>(what, nb, a, st) : launch_split3_t<MODE, 2, false>(what, nb, a, st);
}

hipError_t launch_split3(int mode, int ns, int walls, int what, int nb, const Lb3Args &a, hipStream_t st) {
  switch (mode) {
    case MODE_F64: return launch_split3_m<MODE_F64>(ns, walls, what, nb, a, st);
    case MODE_F32: return launch_split3_m<MODE_F32>(ns, walls, what, nb, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lb355
