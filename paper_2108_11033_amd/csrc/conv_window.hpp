// Where the windows of a convolution tile lie in a feature map: the arithmetic that decides whether a tile's loads need
// range checks, shared by the convolution kernels and by the host check that walks every load of every tile.
#pragma once
#include "xcd_map.hpp"

namespace grim {

// Element (inside a channel) under the centre tap for the first of the 8 positions from nb on.  Stride 2: positions of the
// output grid with rows padded to Wp, a multiple of 8; pieces behind the last one (of a map of less than a tile, never
// stored) take its place, so that windows never start later than those of the tile's last piece.
// wp_inverse: divide_inverse(Wp)
template <bool S2>
GRIM_HOST_DEVICE int conv_piece_start(int nb, int W, int Ho, int Wp, uint32_t wp_inverse) {
    if (!S2) return nb;
    const int last = Ho * Wp - 8;
    nb = nb < last ? nb : last;
    const int h = divide_by(nb, Wp, wp_inverse);
    return 2 * (h * W + (nb - h * Wp));
}
template <bool S2>
GRIM_HOST_DEVICE int conv_piece_start(int nb, int W, int Ho, int Wp) {
    return conv_piece_start<S2>(nb, W, Ho, Wp, S2 ? 0xffffffffu / (uint32_t)Wp : 0u);
}

// Can a window of a tile whose first and last piece start at `first` and `last` begin before the feature map or end behind
// it (in the first or last channel)?  centre: offset of the centre tap, by which window starts move either way.
template <bool S2>
GRIM_HOST_DEVICE bool conv_tile_at_edge(int first, int last, int centre, int HW) {
    return first < centre || last + (S2 ? 16 : 8) + centre > HW;
}

}  // namespace grim
