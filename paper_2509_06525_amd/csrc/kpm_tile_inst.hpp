// Launch of the tiled recurrence kernels; included by the kpm_tile_inst_*.hip
// translation units, each of which instantiates some (vector type, width).
#pragma once

#include "kpm_tile.hpp"

namespace tbk {
namespace {

template <class VT, int W, int SHAPE, bool DIAG, int FORM>
void launch(unsigned grid, hipStream_t s, const TileArgs<VT> &a) {
    constexpr int NT = tile_threads(SHAPE), K = tile_slots(SHAPE, W, sizeof(VT) == 8);
    // Every entry one value: 12 of the 74 bytes a row takes per pass of one vector, and a
    // third of its registers (100 M rows, one vector, the call: 119 ms, 106 so).  For large
    // pristine sheets without onsite energies alone; in the doubling form the zero behind
    // the rows is 16 bytes too many for two workgroups in LDS.
    if constexpr (SHAPE == kTileLarge && W == 3 && !DIAG && FORM != kTileDoubling) {
        if (a.hop) {
            k_tile_steps<VT, NT, K, W, DIAG, FORM, true><<<grid, NT, 0, s>>>(a);
            return;
        }
    }
    k_tile_steps<VT, NT, K, W, DIAG, FORM, false><<<grid, NT, 0, s>>>(a);
}

template <class VT, int W, int SHAPE, int FORM>
void launch_diag(bool diag, unsigned grid, hipStream_t s, const TileArgs<VT> &a) {
    if (diag) launch<VT, W, SHAPE, true, FORM>(grid, s, a);
    else launch<VT, W, SHAPE, false, FORM>(grid, s, a);
}

template <class VT, int W, int SHAPE>
void launch_shape(bool diag, int form, unsigned grid, hipStream_t s, const TileArgs<VT> &a) {
    if (form == kTileDoubling) launch_diag<VT, W, SHAPE, kTileDoubling>(diag, grid, s, a);
    else if (form == kTilePropagate) launch_diag<VT, W, SHAPE, kTilePropagate>(diag, grid, s, a);
    else launch_diag<VT, W, SHAPE, kTileDirect>(diag, grid, s, a);
}

}  // namespace

template <class VT, int W>
void launch_tile_steps(const TilePlan &tp, bool diag, int form, unsigned grid, hipStream_t s,
                       const TileArgs<VT> &a) {
    // large_diag differs from large where its rows per thread do
    constexpr bool own = tile_slots(kTileLargeDiag, W, sizeof(VT) == 8) != tile_slots(kTileLarge, W, sizeof(VT) == 8);
    if (tp.shape == kTileWhole) launch_shape<VT, W, kTileWhole>(diag, form, grid, s, a);
    else if (tp.shape == kTileLargeDiag && own) launch_shape<VT, W, kTileLargeDiag>(diag, form, grid, s, a);
    else if (sizeof(VT) == 4 && tp.shape == kTileSmall) launch_shape<VT, W, sizeof(VT) == 4 ? kTileSmall : kTileLarge>(diag, form, grid, s, a);
    else launch_shape<VT, W, kTileLarge>(diag, form, grid, s, a);
}

}  // namespace tbk
