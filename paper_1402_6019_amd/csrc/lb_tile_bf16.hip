// Tile step of the BF16-deviation storage mode, rounding to nearest or stochastically: the
// instantiations of the tile kernel for this mode.

#include "lb_tile.hpp"

namespace lb355 {

template <int MODE>
static hipError_t launch_bf16(int ns, int walls, int what, int shape, int n, const StepArgs &a, const TileOpts &o,
                              hipStream_t st) {
  switch (what) {
    case WHAT_STEP: return launch_tile_m<MODE, WHAT_STEP>(ns, walls, shape, n, a, o, st);
    case WHAT_STEP_ACCUM: return launch_tile_m<MODE, WHAT_STEP_ACCUM>(ns, walls, shape, n, a, o, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_tile_bf16(bool stochastic, int ns, int walls, int what, int shape, int n, const StepArgs &a,
                            const TileOpts &o, hipStream_t st) {
  return stochastic ? launch_bf16<MODE_BF16SR>(ns, walls, what, shape, n, a, o, st)
                    : launch_bf16<MODE_BF16>(ns, walls, what, shape, n, a, o, st);
}

}  // namespace lb355
