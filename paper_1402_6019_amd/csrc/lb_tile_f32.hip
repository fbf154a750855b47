// Tile step of the F32 storage mode: the instantiations of the tile kernel for this mode.

#include "lb_tile.hpp"

namespace lb355 {

hipError_t launch_tile_f32(int ns, int walls, int what, int shape, int n, const StepArgs &a, const TileOpts &o,
                           hipStream_t st) {
  switch (what) {
    case WHAT_STEP: return launch_tile_m<MODE_F32, WHAT_STEP>(ns, walls, shape, n, a, o, st);
    case WHAT_STEP_ACCUM: return launch_tile_m<MODE_F32, WHAT_STEP_ACCUM>(ns, walls, shape, n, a, o, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lb355
