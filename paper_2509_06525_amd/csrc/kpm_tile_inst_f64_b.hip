// Instances of the tiled recurrence for complex-double vectors, rows of up to 4 and 6 entries (kpm_tile.hpp).
#include "kpm_tile_inst.hpp"

namespace tbk {
template void launch_tile_steps<double, 4>(const TilePlan &, bool, int, unsigned, hipStream_t,
                                        const TileArgs<double> &);
template void launch_tile_steps<double, 6>(const TilePlan &, bool, int, unsigned, hipStream_t,
                                        const TileArgs<double> &);
}  // namespace tbk
