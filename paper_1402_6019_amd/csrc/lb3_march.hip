// The three-dimensional step as it runs by default: tiles marched along z with the pulled
// populations of the planes between psi and update kept in registers.
//
// A workgroup owns a tile of 32 columns (x) by kRows3 rows (y), one site per thread, and marches
// +z through a segment of planes.  The update of plane z needs psi at planes z - 2 .. z + 2, so the
// populations of a site are first needed (for psi) two planes before they are updated.  The kernel
// of lb3_kernels.hip pulls them a second time at the update, which in planes of this size is past
// what L2 holds: its reads reached 2.2 to 2.5 times the populations, and they set its time.  Here
// a register FIFO of four planes (z .. z + 2 and the lead plane z + 3 in flight) holds them, so
// memory is read once plus the two-site frame around a tile: (36 x 20) / (32 x 16) = 1.41 times in
// FP32, (36 x 12) / (32 x 8) = 1.69 times in FP64, whose FIFO takes a wave's 512 registers alone.
// Every address of a site but its plane's base stays the same through the march: nine lane offsets
// per thread, the population's plane in the uniform offset and z in the buffer descriptor.
// Per-site arithmetic and its order are those of lb3_kernels.hip (bitwise the same populations).
// Two species, us per step before (two pulls) and now: 256^3 FP32 1540 and 1250 (4.1 TB/s of
// populations; vector units busy 35%, two waves per SIMD in step; the frame's loads, issued after the
// stores, are waited for at the next plane, but spilled wherever they were issued earlier: 1494 and
// more), 192 x 128 x 128 FP64 735 and 535; the moments of 256^3 4040 and 860 (that pass
// spilled, see site3_update).

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lb3_internal.hpp"
#include "lb3_site.hpp"
#include "lb_step.hpp"

namespace lb355 {

namespace {

constexpr int TX3 = 32, W3 = TX3 + 4;
constexpr int RING3 = 6, RHO3 = 5;  // planes of psi and of rho (two species) in LDS

template <int MODE>
constexpr int rows3() { return MODE == MODE_F64 ? 8 : 16; }

}  // namespace

extern __shared__ __attribute__((aligned(16))) unsigned char march3_smem[];

template <int MODE, int NS>
constexpr size_t march3_lds_bytes() {
  return ((size_t)W3 * (rows3<MODE>() + 4) + 1) * (NS == 2 ? RING3 + RHO3 : RING3) * NS * (MODE == MODE_F64 ? 8 : 4);
}

template <int MODE, int NS, bool WALLS, int WHAT, int STP>
__global__ __launch_bounds__(TX3 *rows3<MODE>()) __attribute__((amdgpu_waves_per_eu(MODE == MODE_F64 ? 1 : 2)))
void march3_kernel(Lb3Args a) {
  using C = Codec<MODE>;
  using R = typename C::R;
  using S = typename C::S;
  using V = Vec<R, NS>;
  constexpr bool STORE = WHAT == WHAT_STEP;
  constexpr int TY = rows3<MODE>(), H = TY + 4, SLOT = W3 * H, NT = TX3 * TY, NHALO = SLOT - NT;
  constexpr int SLOTP = SLOT + 1;
  V *const psi_ring = reinterpret_cast<V *>(march3_smem);  // [RING3][H][W3]
  V *const rho_ring = psi_ring + RING3 * SLOTP;             // [RHO3][H][W3] (two species)

  const int lx = a.lx, ly = a.ly, lz = a.lz;
  constexpr uint32_t site_b = (uint32_t)(NS * sizeof(S));
  const uint32_t plane_b = (uint32_t)a.pitch * site_b, row_b = 19u * plane_b;
  const uint64_t zplane_b = (uint64_t)row_b * (uint32_t)ly;
  const uint32_t off = (uint32_t)zplane_b;  // past the range (see pull3)
  auto zrsrc = [&](const void *p, int z, bool on) {
    return make_rsrc(static_cast<const char *>(p) + (uint64_t)(uint32_t)z * zplane_b, on ? (uint32_t)zplane_b : 0u);
  };

  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int per_seg = a.nstrip * a.nband;
  const int seg = logical / per_seg;
  const int rem = logical - seg * per_seg;
  const int band = rem / a.nstrip;
  const int strip = rem - band * a.nstrip;
  const int tid = threadIdx.x, tx = tid & (TX3 - 1), ty = tid / TX3;
  const int x0 = strip * TX3, y0 = band * TY;
  const int x = x0 + tx, y = y0 + ty;
  const bool site_ok = x < lx && y < ly;
  const int zA = seg * a.sz, zB = min(zA + a.sz, lz);

  const Site3<R, NS> p(a);

  // This thread's site; past the end of a ragged strip or band the periodic image, or the wall's
  // ghost (pulling the row next to it), which only feeds the ring.
  const bool solid = WALLS && y >= ly;
  Pull3 own = pull3_at<WALLS>(x % lx, WALLS ? min(y, ly - 1) : y % ly, lx, ly, row_b, site_b);
  const int own_e = (ty + 2) * W3 + tx + 2;
  // Its site of the two-site frame (threads below NHALO): the two rows below and above the tile,
  // then the two columns on either side.
  const bool has_halo = tid < NHALO;
  int hx = 0, hy = 0;
  {
    const int h = has_halo ? tid : 0;
    if (h < 4 * W3) {
      const int r = h / W3;
      hx = h - r * W3 - 2;
      hy = r < 2 ? r - 2 : TY + (r - 2);
    } else {
      const int k = h - 4 * W3, c = k & 3;
      hy = k >> 2;
      hx = c < 2 ? c - 2 : TX3 + (c - 2);
    }
  }
  const int halo_e = has_halo ? (hy + 2) * W3 + hx + 2 : SLOT;
  const bool halo_solid = WALLS && (y0 + hy < 0 || y0 + hy >= ly);
  Pull3 halo = pull3_at<WALLS>(((x0 + hx) % lx + lx) % lx,
                                     WALLS ? min(max(y0 + hy, 0), ly - 1) : ((y0 + hy) % ly + ly) % ly, lx, ly, row_b,
                                     site_b);

  if (!has_halo) {
    halo.lo = halo.hi = false;
    for (int k = 0; k < 3; ++k) {
      halo.row[k] = off;
      halo.col[k] = 0u;
    }
  }

  auto pull = [&](const Pull3 &q, int z, bool on, R (&f)[NS][19], R (&fb)[NS][2]) {
    const Rsrc rz[3] = {zrsrc(a.src, d3::wrap(z + 1, lz), on), zrsrc(a.src, z, on), zrsrc(a.src, d3::wrap(z - 1, lz), on)};
    pull3<C, NS, WALLS>(rz, q, plane_b, off, f, fb);
  };
  // psi and rho of a pulled site into entry e of ring slots sp (psi) and sr (rho)
  auto ring_put = [&](R (&f)[NS][19], const R (&fb)[NS][2], const Pull3 &q, bool wall, int sp, int sr, int e) {
    wall_fix3<WALLS>(q, fb, f);
    V ps, rh;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      R sum = f[s][0];
#pragma unroll
      for (int l = 1; l < 19; ++l) sum += f[s][l];
      rh.v[s] = p.rref[s] + sum;
      ps.v[s] = p.psi0 * (R(1) - C::expo(rh.v[s] * p.nirho0));
      if (WALLS && wall) {
        ps.v[s] = p.psiw[s];
        rh.v[s] = p.rhow[s];
      }
    }
    psi_ring[sp * SLOTP + e] = ps;
    if (NS == 2) rho_ring[sr * SLOTP + e] = rh;
  };
  auto zwrap = [&](int p) { return (int)uni((uint32_t)d3::wrap(d3::wrap(p, lz), lz)); };

  // FIFO: plane z lives in B[(z - zA) mod 4]; psi plane p in slot (p - zA + 2) mod 6, rho plane p
  // in slot (p - zA + 2) mod 5.
  R B[4][NS][19], hf[NS][19], ob[NS][2], hb[NS][2];
  {
    // prologue: psi of zA - 2 .. zA + 1, two planes at a time (the frame of the second in a FIFO
    // plane that is still free); zA, zA + 1 and the lead plane zA + 2 stay in B
    R ob2[NS][2], hb2[NS][2];
    pull(own, zwrap(zA - 2), true, B[2], ob);
    pull(own, zwrap(zA - 1), true, B[3], ob2);
    pull(halo, zwrap(zA - 2), true, hf, hb);
    pull(halo, zwrap(zA - 1), true, B[0], hb2);
    ring_put(B[2], ob, own, solid, 0, 0, own_e);
    ring_put(B[3], ob2, own, solid, 1, 1, own_e);
    ring_put(hf, hb, halo, halo_solid, 0, 0, halo_e);
    ring_put(B[0], hb2, halo, halo_solid, 1, 1, halo_e);
    R ob3[NS][2];
    pull(own, zA, true, B[0], ob3);
    pull(own, zwrap(zA + 1), true, B[1], ob2);
    pull(halo, zA, true, hf, hb);
    pull(halo, zwrap(zA + 1), true, B[3], hb2);
    pull(own, zwrap(zA + 2), true, B[2], ob);
    ring_put(B[0], ob3, own, solid, 2, 2, own_e);
    ring_put(B[1], ob2, own, solid, 3, 3, own_e);
    ring_put(hf, hb, halo, halo_solid, 2, 2, halo_e);
    ring_put(B[3], hb2, halo, halo_solid, 3, 3, halo_e);
    pull(halo, zwrap(zA + 2), true, hf, hb);
  }

  // One plane: f = its populations, fl = those of the lead plane z + 2, fn receives plane z + 3's.
  int s0 = 0, r1 = 1;  // ring slots of psi plane z - 2 and rho plane z - 1
  auto plane = [&](const int z, const R (&f)[NS][19], R (&fl)[NS][19], R (&fn)[NS][19]) {
    const int sp = s0, sr = r1;
    if constexpr (WALLS && NS == 2) {
      // the nineteen offsets of each site are summed anew for every plane: kept, they spilled
      // (periodic lattices need nine, which fit)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        asm volatile("" : "+v"(own.row[k]), "+v"(own.col[k]), "+v"(halo.row[k]), "+v"(halo.col[k]));
    }
    const int sl = s0 >= 2 ? s0 - 2 : s0 + 4, srl = r1 >= 2 ? r1 - 2 : r1 + 3;  // slots of plane z + 2
    ring_put(fl, ob, own, solid, sl, srl, own_e);
    ring_put(hf, hb, halo, halo_solid, sl, srl, halo_e);
    const bool more = z + 1 < zB;  // the lead plane after this one is needed
    pull(own, zwrap(z + 3), more, fn, ob);
    __syncthreads();
    s0 = s0 + 1 >= RING3 ? 0 : s0 + 1;
    r1 = r1 + 1 >= RHO3 ? 0 : r1 + 1;

    const V *pl[5];  // corner (-2, -2) of the site's neighbourhood in psi planes z - 2 .. z + 2
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const int sm = sp + m >= RING3 ? sp + m - RING3 : sp + m;
      pl[m] = psi_ring + sm * SLOTP + ty * W3 + tx;
    }
    uint32_t xo[3];  // first entries of the cross term's planes z - 1 .. z + 1 (uniform)
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const int sm = sp + 1 + m >= RING3 ? sp + 1 + m - RING3 : sp + 1 + m;
      const int rm = sr + m >= RHO3 ? sr + m - RHO3 : sr + m;
      xo[m] = uni((uint32_t)((a.cross_psi ? sm : RING3 + rm) * SLOTP));
    }
    auto xr = [&](int dx, int dy, int dz) { return psi_ring[(int)xo[dz + 1] + (ty + dy + 2) * W3 + tx + dx + 2]; };
    site3_update<C, NS, WHAT, STP>(
        a, p, f, [&](int dx, int dy, int dz) { return pl[dz + 2][(dy + 2) * W3 + dx + 2]; },
        xr, x, y, z, site_ok, zrsrc(a.dst, z, STORE), site_ok ? own.row[1] + own.col[1] : off, plane_b);
    // the frame's loads last: in registers that the updated populations have left
    __builtin_amdgcn_sched_barrier(0);
    pull(halo, zwrap(z + 3), more, hf, hb);
  };

  for (int z = zA; z < zB; z += 4) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (z + k < zB) plane(z + k, B[k], B[(k + 2) & 3], B[(k + 3) & 3]);
  }
}

int march3_rows(int mode) { return mode == MODE_F64 ? rows3<MODE_F64>() : rows3<MODE_F32>(); }

template <int MODE, int NS, bool WALLS, int WHAT, int STP>
static hipError_t launch_march3_k(int nb, const Lb3Args &a, hipStream_t st) {
  hipLaunchKernelGGL((march3_kernel<MODE, NS, WALLS, WHAT, STP>), dim3(nb), dim3(TX3 * rows3<MODE>()),
                     (march3_lds_bytes<MODE, NS>()), st, a);
  return hipGetLastError();
}

template <int MODE, int NS, bool WALLS>
static hipError_t launch_march3_t(int what, int nb, const Lb3Args &a, hipStream_t st) {
  switch (what) {
    case WHAT_STEP:
      return a.stream_stores ? launch_march3_k<MODE, NS, WALLS, WHAT_STEP, kStoreStreaming>(nb, a, st)
                             : launch_march3_k<MODE, NS, WALLS, WHAT_STEP, kStoreWriteThrough>(nb, a, st);
    case WHAT_MOMENTS: return launch_march3_k<MODE, NS, WALLS, WHAT_MOMENTS, 0>(nb, a, st);
  }
  return hipErrorInvalidValue;
}

template <int MODE>
static hipError_t launch_march3_m(int ns, int walls, int what, int nb, const Lb3Args &a, hipStream_t st) {
  if (ns == 1) return walls ? launch_march3_t<MODE, 1, true>(what, nb, a, st) : launch_march3_t<MODE, 1, false>(what, nb, a, st);
  return walls ? launch_march3_t<MODE, 2, true>(what, nb, a, st) : launch_march3_t<MODE, 2, false>(what, nb, a, st);
}

hipError_t launch_march3(int mode, int ns, int walls, int what, int nb, const Lb3Args &a, hipStream_t st) {
  switch (mode) {
    case MODE_F64: return launch_march3_m<MODE_F64>(ns, walls, what, nb, a, st);
    case MODE_F32: return launch_march3_m<MODE_F32>(ns, walls, what, nb, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lb355
