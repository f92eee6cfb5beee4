// Which pixels of a channel a tile of bcr_conv_patch holds: the arithmetic of the kernel and its launcher, shared with the host
// check that walks every tap of every position.
#pragma once
#include <cstdint>

#include "host_device.hpp"
#include "xcd_map.hpp"

namespace grim {

// Pixel (of a channel) under the centre tap of output position n, and its row and column; wo_inverse: divide_inverse(Wo)
GRIM_HOST_DEVICE int patch_pixel_of(int n, int W, int Wo, uint32_t wo_inverse, bool s2, int *h, int *w) {
    const int ho = divide_by(n, Wo, wo_inverse);
    *h = ho << (s2 ? 1 : 0);
    *w = (n - ho * Wo) << (s2 ? 1 : 0);
    return *h * W + *w;
}
GRIM_HOST_DEVICE int patch_pixel_of(int n, int W, int Wo, bool s2, int *h, int *w) {
    return patch_pixel_of(n, W, Wo, 0xffffffffu / (uint32_t)Wo, s2, h, w);
}

// The first and last pixel that a tap of positions [n0, n0 + 64) can meet; `odd`: the map starts at an odd element (the
// first pixel is moved to an even one where there is one, and there are eight from it on)
GRIM_HOST_DEVICE int patch_first(int n0, int W, int Wo, uint32_t wo_inverse, bool s2, int centre, int HW, int odd) {
    int h, w;
    int lo = patch_pixel_of(n0, W, Wo, wo_inverse, s2, &h, &w) - centre;
    lo = lo < 0 ? 0 : lo > HW - 8 ? HW - 8 : lo;
    return lo - (lo > 0 ? (odd + lo) & 1 : 0);
}
GRIM_HOST_DEVICE int patch_last(int n0, int Nv, int W, int Wo, uint32_t wo_inverse, bool s2, int centre, int HW) {
    int h, w;
    const int hi = patch_pixel_of(n0 + 64 < Nv ? n0 + 63 : Nv - 1, W, Wo, wo_inverse, s2, &h, &w) + centre;
    return hi < HW - 1 ? hi : HW - 1;
}
GRIM_HOST_DEVICE int patch_first(int n0, int W, int Wo, bool s2, int centre, int HW, int odd) {
    return patch_first(n0, W, Wo, 0xffffffffu / (uint32_t)Wo, s2, centre, HW, odd);
}
GRIM_HOST_DEVICE int patch_last(int n0, int Nv, int W, int Wo, bool s2, int centre, int HW) {
    return patch_last(n0, Nv, W, Wo, 0xffffffffu / (uint32_t)Wo, s2, centre, HW);
}

// The most pixels any tile spans, in whole eights
inline int64_t patch_pixels(int32_t H, int32_t W, int32_t kh, int32_t kw, int32_t stride) {
    const int64_t Wo = (W + stride - 1) / stride, turns = (63 + Wo - 1) / Wo;
    const int64_t span = (stride == 2 ? 126 + 2 * (W - Wo) * turns : 63) + 2 * ((int64_t)(kh / 2) * W + kw / 2) + 1;
    return ((span < (int64_t)H * W - 1 ? span : (int64_t)H * W - 1) / 8 + 1) * 8;
}

// Waves of a workgroup: eight while every workgroup has a compute unit of its own, four, two of them to a compute unit, beyond.  What
// counts is the launch, with the workgroups that xcd_map adds where tiles are no multiple of eight: 117 tiles of 2 runs make a
// launch of 264, 33 to an XCD of 32 compute units (128 -> 96 channels, 3 x 3, on 13 maps of 23 x 23 16.2 us with eight waves, 12.5 with
// four; 12.7 on 16-row runs).
inline int patch_waves(int32_t tiles, int64_t runs) {
    int64_t workgroups = 0;
    xcd_map(tiles, runs, &workgroups);
    return workgroups <= 256 ? 8 : 4;
}

}  // namespace grim
