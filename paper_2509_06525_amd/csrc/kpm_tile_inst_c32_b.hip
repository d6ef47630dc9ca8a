// Instances of the tiled recurrence for complex-float vectors, rows of up to 4 and 6 entries (kpm_tile.hpp).
#include "kpm_tile_inst.hpp"

namespace tbk {
template void launch_tile_steps<float, 4>(const TilePlan &, bool, int, unsigned, hipStream_t,
                                        const TileArgs<float> &);
template void launch_tile_steps<float, 6>(const TilePlan &, bool, int, unsigned, hipStream_t,
                                        const TileArgs<float> &);
}  // namespace tbk
