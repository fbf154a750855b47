// Tile step of the FP32 storage mode: the instantiations of the tile kernels for this mode.

#include "lb_tile.hpp"

namespace lb355 {

hipError_t launch_tile_f32(int ns, int walls, int what, int shape, int n, const StepArgs &a, const TileOpts &o,
                           hipStream_t st) {
  return launch_tile_what<MODE_F32>(ns, walls, what, shape, n, a, o, st);
}

hipError_t launch_tile_f32(int ns, int walls, int what, int shape, int n, const BatchTiles &b, const TileOpts &o,
                           hipStream_t st) {
  return launch_tile_what<MODE_F32>(ns, walls, what, shape, n, b, o, st);
}

}  // namespace lb355
