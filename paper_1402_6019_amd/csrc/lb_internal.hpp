// Internal declarations shared by the host runtime (lb_api.cpp) and the device kernels
// (lb_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lb355 {

// MODE_BF16SR: BF16 storage whose population stores round stochastically (the step kernels
// only; every other kernel reads and writes it like MODE_BF16).
enum StoreMode { MODE_F64 = 0, MODE_F32 = 1, MODE_BF16 = 2, MODE_BF16SR = 3 };

// What one launch of the fused step kernel does.
enum StepWhat {
  WHAT_STEP = 0,         // stream + force + collide, store f*
  WHAT_MOMENTS = 2,      // write rho_s and the half-force velocity, store nothing
  WHAT_OBSERVE = 3,      // partial sums of the current state, store nothing
  WHAT_PROFILE = 4,      // per-row sums of the current state (velocity, stress parts), store nothing
  WHAT_STRESS = 5,       // write the site pressure tensor of the current state, store nothing
  WHAT_STEP_ACCUM = 6,   // step, adding wall stress and health counts to per-workgroup FP64 running sums
  // tile step, also writing what the adjoint's reverse step reads of the states it steps from: rho,
  // psi, j of every site (out_rho, [4][2][ly][lx], FP64 / FP32) and the canonical FP64
  // populations of the rows next to the walls (out_u, [s][l][2][lx])
  WHAT_STEP_FIELDS = 7,
  WHAT_STEP_FIELDS32 = 8
};

// Running sums of WHAT_STEP_ACCUM, per workgroup row.
enum AccSlot { ACC_WBOT = 0, ACC_WTOP, ACC_BAD, ACC_N };

// Per-row sums written by a WHAT_PROFILE launch, per tile column (64 columns) of a row:
//   PROF_U   sum of the half-force velocity u_x
//   PROF_KUP sum_s (f*_5 - f*_6): x-momentum the populations with c_y = +1 carry up
//   PROF_KDN sum_s (f*_8 - f*_7): x-momentum the populations with c_y = -1 carry down
//   PROF_I1  x-force on the row's sites from partners at c_y >= 1 (pairs crossing line y + 1/2)
//   PROF_I2  the part of PROF_I1 from partners at c_y = 2 (pairs also crossing line y + 3/2)
//   PROF_RA, PROF_RB  sums of the species densities (B zero for one component)
enum ProfSlot { PROF_U = 0, PROF_KUP, PROF_KDN, PROF_I1, PROF_I2, PROF_RA, PROF_RB, PROF_N };

// Partial-sum slots written per workgroup (and totals after the second pass).
enum RedSlot {
  RED_MASS0 = 0, RED_MASS1, RED_PX, RED_PY, RED_FLOW, RED_BAD, RED_N
};

// Kernel arguments of the fused step (passed by value through the kernarg segment).
struct StepArgs {
  const void *src;      // post-collision populations of the previous step (pull source)
  void *dst;            // post-collision populations of this step
  double *partials;     // [gridDim.x][RED_N] when reducing
  void *out_rho;        // moments: [ns][ly][lx]
  void *out_u;          // moments: [2][ly][lx]
  long long plane;      // elements per (species, l) plane = ly * pitch
  int lx, ly, pitch;    // lattice and row pitch (elements)
  int sy, nseg;         // rows per workgroup, workgroups per strip
  int out_f32;          // moments output type
  int cross_psi;        // A-B term between psi (1) or rho (0)
  double K[2][5];       // folded shell couplings G_ss,1 w(q) + G_ss,2 p(q)
  double T[2];          // G_AB t(1), G_AB t(2)
  double body[2];       // acceleration g
  double tau[2], omega[2];
  double psi0, irho0;
  double rho_w[2], psi_w[2];  // wall ghost rows (channel)
  double rho_ref[2];          // FP32 / BF16 deviation reference
  long long offset;           // batch: byte offset of this instance in each population buffer
  double wall_mom[2][2];      // [bottom, top][species]: rho_w,s U / 6, added on reflection
  int moving;                 // some wall moves (wall_mom != 0)
  double *prof;               // profile: [64-column blocks][ly][PROF_N]
  int stream_stores;          // both population buffers exceed the Infinity Cache: non-temporal stores
  uint32_t t_step;            // MODE_BF16SR: time step of the launch, plus *t_base when t_base is set
  const double *t_base;       // (graph replays: the step at which the replay starts)
  void *out_sigma;            // stress: [3][ly][lx] (xx, xy, yy)
  double *accrows;            // WHAT_STEP_ACCUM: [gridDim.x][ACC_N] running sums
};

// Parameters of a lattice as the per-site arithmetic uses them, in the arithmetic type.
template <typename R>
struct SiteConsts {
  R K1[2], K2[2], K4[2], K5[2], K8[2];  // shell couplings K(q); K4 and K8 twice it (|c| = 2 along an axis)
  R tau[2], om[2], rref[2], psiw[2], rhow[2];
  R T1, T2, gx, gy, psi0, nirho0;
};

// Kernel arguments of the tile step (lb_tile.hpp), passed by value.  The parameters come in the
// arithmetic type: converting them per wave cost as much as a third of a site's update.
template <typename R>
struct TileArgs {
  const void *src;     // post-collision populations of the previous step (pull source)
  void *dst;           // post-collision populations of the launch's last step
  double *accrows;     // reducing launches: [gridDim.x][ACC_N] running sums
  void *fields;        // WHAT_STEP_FIELDS*: fields of the states stepped from and the populations
  void *xw;            // of their rows next to the walls (StepArgs::out_rho, out_u), the bytes from
  size_t fields_stride, xw_stride;  // one state to the next
  uint32_t pitch_b, buf_b;          // bytes of a plane row and of the buffer
  int lx, ly;
  uint32_t ntx, ntx_mul;            // tiles per row; b / ntx = mulhi(b, ntx_mul) for every workgroup b (0: divide)
  int cross_psi, moving;
  uint32_t red_mask;                // which steps of the launch reduce (bit k: step k)
  uint32_t t_step;                  // MODE_BF16SR: as StepArgs
  const double *t_base;
  double wall_mom[2][2];
  double rho_ref[2], psi0, irho0;   // the fields' own (FP64) parameters
  long long offset;                 // batch: byte offset of this instance in each population buffer
  SiteConsts<R> c;
};

// The arguments of a tile launch from those of the row-marching step.
template <typename R>
inline TileArgs<R> make_tile_args(const StepArgs &a, uint32_t site_b, int bx, int by) {
  TileArgs<R> t{};
  t.offset = a.offset;
  t.src = a.src;
  t.dst = a.dst;
  t.accrows = a.accrows;
  t.fields = a.out_rho;
  t.xw = a.out_u;
  t.pitch_b = (uint32_t)a.pitch * site_b;
  t.buf_b = 9u * (uint32_t)a.plane * site_b;
  t.lx = a.lx;
  t.ly = a.ly;
  t.ntx = (uint32_t)((a.lx + bx - 1) / bx);
  // exact while tiles per row times tiles stay below 2^32
  const uint64_t tiles = (uint64_t)t.ntx * (uint32_t)((a.ly + by - 1) / by);
  t.ntx_mul = t.ntx > 1 && tiles * t.ntx < (1ull << 32) ? (uint32_t)(((1ull << 32) + t.ntx - 1) / t.ntx) : 0u;
  t.cross_psi = a.cross_psi;
  t.moving = a.moving;
  t.t_step = a.t_step;
  t.t_base = a.t_base;
  t.psi0 = a.psi0;
  t.irho0 = a.irho0;
  for (int s = 0; s < 2; ++s) {
    t.rho_ref[s] = a.rho_ref[s];
    for (int w = 0; w < 2; ++w) t.wall_mom[w][s] = a.wall_mom[w][s];
    t.c.K1[s] = R(a.K[s][0]);
    t.c.K2[s] = R(a.K[s][1]);
    t.c.K4[s] = R(2.0 * a.K[s][2]);
    t.c.K5[s] = R(a.K[s][3]);
    t.c.K8[s] = R(2.0 * a.K[s][4]);
    t.c.tau[s] = R(a.tau[s]);
    t.c.om[s] = R(a.omega[s]);
    t.c.rref[s] = R(a.rho_ref[s]);
    t.c.psiw[s] = R(a.psi_w[s]);
    t.c.rhow[s] = R(a.rho_w[s]);
  }
  t.c.T1 = R(a.T[0]);
  t.c.T2 = R(a.T[1]);
  t.c.gx = R(a.body[0]);
  t.c.gy = R(a.body[1]);
  t.c.psi0 = R(a.psi0);
  t.c.nirho0 = R(-a.irho0);
  return t;
}

// What a tile launch does beside stepping.
struct TileOpts {
  uint32_t red_mask = 0;                     // WHAT_STEP_ACCUM: which steps of the launch reduce
  size_t fields_stride = 0, xw_stride = 0;   // WHAT_STEP_FIELDS*: bytes from one state's outputs to the next's
};

// Tile shapes of the tile step: sites per tile, and the most steps of one launch.  The last two are the
// same tile, of one workgroup per compute unit (more threads, three steps) and of two.
constexpr int kTileShapes = 6;
constexpr int kTileX[kTileShapes] = {4, 8, 16, 16, 32, 32}, kTileY[kTileShapes] = {8, 8, 8, 16, 16, 16};

// Steps of one launch at most: three, in 32 x 16 tiles with one per compute unit (512 x 256, FP32,
// walled: 4.40 us per step against 4.64 for two; beyond that the overlaps cost more than the launches:
// 4096 x 512 62 and 44) unless the copy of f* outgrows LDS (two species in FP64).
inline int tile_most_steps(int shape, bool fp64, int ns) { return shape == 5 || (shape == 4 && fp64 && ns == 2) ? 2 : 3; }

// Tiles of the observation passes (lb_observe.hpp) with sums, and of those without on large lattices.
constexpr int kObserveX = 64, kObserveY = 8;
inline int observe_blocks(int lx, int ly) { return ((lx + kObserveX - 1) / kObserveX) * ((ly + kObserveY - 1) / kObserveY); }

// Batched launches: one tile of one instance.
struct TileDesc {
  int inst;   // instance index (into BatchArgs::inst)
  int strip;  // strip of blockDim.x columns
  int seg;    // segment of StepArgs::sy rows
  int part;   // row of reduction partials this tile writes
};

// Kernel arguments of the batched step: the ntiles tiles of the table.
struct BatchArgs {
  const StepArgs *inst;  // [n] per-instance arguments (device)
  const TileDesc *tiles; // tile table (device)
  int ntiles;
  const char *src;       // population buffers holding every instance at StepArgs::offset
  char *dst;
  int stream_stores;     // non-temporal population stores (see StepArgs)
  double *accrows;       // WHAT_STEP_ACCUM: [tiles][ACC_N] running sums, row TileDesc::part
  uint32_t t_step;       // MODE_BF16SR: time step of the launch (see StepArgs)
  const double *t_base;
};

// Kernel arguments of the batched tile step, and the same as the host passes them to the launcher
// (inst: device array of TileArgs in the batch's arithmetic type).
template <typename R>
struct BatchTileArgs {
  const TileArgs<R> *inst;
  const TileDesc *tiles;
  const char *src;
  char *dst;
  double *accrows;  // reducing launches: [tiles][ACC_N], row TileDesc::part
  uint32_t red_mask, t_step;
  const double *t_base;
};
struct BatchTiles {
  const void *inst;
  const TileDesc *tiles;
  int ntiles, stream_stores;
  const char *src;
  char *dst;
  double *accrows;
  uint32_t t_step;
  const double *t_base;
};

// Second reduction pass of one batch instance: partial rows [p0, p0 + n).
struct ReduceJob {
  int p0, n;
  double inv_lx;
};

// Arguments of the layout kernels (init / checkpoint / restore).
struct LayoutArgs {
  const void *in;
  void *out;
  long long plane;
  int lx, ly, pitch, ns;
  double rho_ref[2];
};

// Reverse step of the adjoint (lb_adjoint.hip).  Arrays are canonical [..][y][x]; R is
// double for FP64 contexts and float otherwise.
struct AdjArgs {
  const double *x;       // pre-collision populations f(t) of the rows next to the walls, [s][l][2][x]
                         // (bottom row, then top row), FP64; read with walls only
  const void *lam_next;  // lambda(t+1) [s][l][y][x] (R)
  void *lam;             // lambda(t) (R, written)
  const void *fields;    // [4][2][y][x] (R): rho, psi, jx, jy of f(t)
  double *partials;      // [blocks][ADJ_N]
  int lx, ly;
  int cross_psi, pad_;
  double K[2][5];        // G_ss,1 w(q) + G_ss,2 p(q)
  double w[5], p[5], t[2];
  double g1[2], g2[2], gab;
  double body[2], tau[2], omega[2];
  double psi0, irho0;
  double rho_w[2], psi_w[2];
  double cW, cQ;         // per-step loss weights
  double ilx;            // 1 / lx, and the same rounded from a float division
  float ilxf, pad2_;
  double u_wall[2];      // x-velocity of the bottom and top wall
};

// Per-block partial sums of the adjoint: parameter sensitivities and the loss.
enum AdjSlot { ADJ_G1A = 0, ADJ_G1B, ADJ_G2A, ADJ_G2B, ADJ_GAB, ADJ_GX, ADJ_GY, ADJ_LW, ADJ_LQ, ADJ_N };

int adj_blocks(int lx, int ly, int n_cu);  // n_cu: compute units
// One reverse step; adds this step's per-block sensitivities to a.partials.
hipError_t launch_adjoint_step(int fp64, int ns, int walls, int n_cu, const AdjArgs &a, hipStream_t st);
// acc[k] += sum over blocks of partials[block][k] (fixed order).
hipError_t launch_adjoint_reduce(const double *partials, int nblocks, double *acc, hipStream_t st);
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st);

// Host-side launchers (lb_kernels.hip).  Return hipSuccess or the launch error.
hipError_t launch_step2(int mode, int ns, int walls, int nblocks, const StepArgs &a, hipStream_t st);
hipError_t launch_step(int mode, int ns, int walls, int what, int tx, int nblocks, const StepArgs &a,
                       hipStream_t st);
// A pass over the current state (WHAT_MOMENTS, WHAT_OBSERVE, WHAT_PROFILE or WHAT_STRESS; a.src, the pass's
// outputs in a) of one lattice; n_cu: compute units.  WHAT_OBSERVE writes observe_blocks rows of partials.
hipError_t launch_observe(int mode, int ns, int walls, int what, int n_cu, const StepArgs &a, hipStream_t st);
hipError_t launch_reduce(const double *partials, int nblocks, double *totals, double inv_lx, hipStream_t st);
hipError_t launch_init(int mode, int walls, const LayoutArgs &a, hipStream_t st);
hipError_t launch_checkpoint(int mode, int walls, const LayoutArgs &a, hipStream_t st);
hipError_t launch_restore(int mode, int walls, const LayoutArgs &a, hipStream_t st);

hipError_t launch_fill(double *p, double v, int n, hipStream_t st);
// Grid-stride copy of n16 16-byte elements (blocks workgroups of 256), non-temporal if asked.
hipError_t launch_stream_copy(void *dst, const void *src, size_t n16, int nontemporal, int blocks, hipStream_t st);
// acc[0..1] += (column sums of rows' wall stress) * inv_lx, acc[2] += count, acc[3] += bad;
// rows are cleared.
hipError_t launch_flush(double *rows, int nrows, double *acc, double count, double inv_lx, hipStream_t st);
// The same per batch instance: rows of job i into acc[4 i ..].
hipError_t launch_batch_flush(double *rows, const ReduceJob *jobs, int njobs, double *acc, double count,
                              hipStream_t st);

// Profile second pass: out[0..ly) = ubar, out[ly..2ly] = sigma, out[2ly+1..4ly+1) = the
// species densities per row (see lb_profile).  wb0, wt0:
// sum_s rho_w,s U / 3 of the bottom and top wall.
hipError_t launch_profile_finish(const double *prof, int ncb, int lx, int ly, int walls, double wb0, double wt0,
                                 double *out, hipStream_t st);
hipError_t launch_profile_stats(const double *samples, long long n, int ly, int walls, int k0, double u_bot,
                                double u_top, double *out, hipStream_t st);

hipError_t launch_batch_step(int mode, int ns, int walls, int what, int tx, int grid, const BatchArgs &b,
                             hipStream_t st);
// WHAT_OBSERVE over instances [first, first + count) of a batch: b.inst and b.src; instance i's
// observe_blocks rows of partials start at jobs[i].p0 (device).  blocks: the most of any instance.
hipError_t launch_batch_observe(int mode, int ns, int walls, int first, int count, int blocks, const BatchTiles &b,
                                const ReduceJob *jobs, double *partials, hipStream_t st);
hipError_t launch_batch_reduce(const double *partials, const ReduceJob *jobs, int njobs, double *totals, hipStream_t st);

size_t step_lds_bytes(int mode, int ns, int tx);

// Static device scratch of the entry points that allocate nothing (lb_static.hip), in doubles.
constexpr size_t kStaticScratchDoubles = (size_t)1 << 19;
// Looks up the scratch array's address on `device` once (makes it current for the lookup).
hipError_t static_scratch_setup(int device);
// That address (nullptr before static_scratch_setup succeeded on the device).
double *static_scratch(int device);

// n steps (1 .. tile_most_steps) of the tile step of one lattice, or of a batch; what: WHAT_STEP,
// WHAT_STEP_ACCUM or, one lattice and at most two steps, WHAT_STEP_FIELDS*.  Per storage mode in lb_tile_f64.hip, lb_tile_f32.hip, lb_tile_bf16.hip.
#define LB_TILE_LAUNCHERS(A)                                                                                       \
  hipError_t launch_tile(int mode, int ns, int walls, int what, int shape, int n, const A &a, const TileOpts &o,  \
                         hipStream_t st);                                                                          \
  hipError_t launch_tile_f64(int ns, int walls, int what, int shape, int n, const A &a, const TileOpts &o,        \
                             hipStream_t st);                                                                      \
  hipError_t launch_tile_f32(int ns, int walls, int what, int shape, int n, const A &a, const TileOpts &o,        \
                             hipStream_t st);                                                                      \
  hipError_t launch_tile_bf16(int ns, int walls, int what, int shape, int n, const A &a, const TileOpts &o,       \
                              hipStream_t st);                                                                     \
  hipError_t launch_tile_bf16sr(int ns, int walls, int what, int shape, int n, const A &a, const TileOpts &o,     \
                                hipStream_t st);
LB_TILE_LAUNCHERS(StepArgs)
LB_TILE_LAUNCHERS(BatchTiles)
#undef LB_TILE_LAUNCHERS

// Per storage mode (lb_step_f64.hip, lb_step_f32.hip, lb_step_bf16.hip): the launchers that
// launch_step / launch_batch_step / step_blocks_per_cu dispatch to.
hipError_t launch_step_f64(int ns, int walls, int what, int tx, int nb, const StepArgs &a, hipStream_t st);
hipError_t launch_step_f32(int ns, int walls, int what, int tx, int nb, const StepArgs &a, hipStream_t st);
hipError_t launch_step_bf16(bool stochastic, int ns, int walls, int what, int tx, int nb, const StepArgs &a,
                            hipStream_t st);
hipError_t launch_batch_f64(int ns, int walls, int what, int tx, int grid, const BatchArgs &b, hipStream_t st);
hipError_t launch_batch_f32(int ns, int walls, int what, int tx, int grid, const BatchArgs &b, hipStream_t st);
hipError_t launch_batch_bf16(bool stochastic, int ns, int walls, int what, int tx, int grid, const BatchArgs &b,
                             hipStream_t st);
hipError_t launch_observe_f64(int ns, int walls, int what, bool wide, const StepArgs &a, hipStream_t st);
hipError_t launch_observe_f32(int ns, int walls, int what, bool wide, const StepArgs &a, hipStream_t st);
hipError_t launch_observe_bf16(int ns, int walls, int what, bool wide, const StepArgs &a, hipStream_t st);
hipError_t launch_batch_observe_f64(int ns, int walls, int first, int count, int blocks, const BatchTiles &b,
                                    const ReduceJob *jobs, double *partials, hipStream_t st);
hipError_t launch_batch_observe_f32(int ns, int walls, int first, int count, int blocks, const BatchTiles &b,
                                    const ReduceJob *jobs, double *partials, hipStream_t st);
hipError_t launch_batch_observe_bf16(int ns, int walls, int first, int count, int blocks, const BatchTiles &b,
                                     const ReduceJob *jobs, double *partials, hipStream_t st);
int blocks_per_cu_f64(int ns, int walls, int tx);
// Two time steps per launch (lb_step2.hpp): one wave per workgroup, strips of 54 columns,
// nb = strips x segments workgroups, a.sy rows per segment.
hipError_t launch_step2_f64(int ns, int walls, int nb, const StepArgs &a, hipStream_t st);
hipError_t launch_step2_f32(int ns, int walls, int nb, const StepArgs &a, hipStream_t st);
hipError_t launch_step2_bf16(bool stochastic, int ns, int walls, int nb, const StepArgs &a, hipStream_t st);
int blocks2_per_cu_f32(int ns, int walls);  // also BF16 (the same registers and LDS)
int blocks2_per_cu_f64(int ns, int walls);
int blocks_per_cu_f32(int ns, int walls, int tx);
int blocks_per_cu_bf16(int ns, int walls, int tx);
// Workgroups of tx threads of the plain step kernel that one compute unit holds at once.
int step_blocks_per_cu(int mode, int ns, int walls, int tx);

}  // namespace lb355
