// Host walk over the taps of a patch convolution's tiles, with the kernel's arithmetic (csrc/conv_patch.hpp): how many pixels
// that a tap meets are not among those the tile loads, or lie outside the room for them, and how many loads leave the channel.
#include <cstdint>
#include <vector>

#include "conv_patch.hpp"

extern "C" int64_t conv_patch_faults(int H, int W, int kh, int kw, int stride, int odd) {
    const int s = stride, Ho = (H + s - 1) / s, Wo = (W + s - 1) / s, HW = H * W, Nv = Ho * Wo, ph = kh / 2, pw = kw / 2, centre = ph * W + pw;
    const int64_t room = grim::patch_pixels(H, W, kh, kw, s);
    int64_t bad = 0;
    for (int tile = 0; tile * 64 < Nv; ++tile) {
        int n0 = tile * 64 + 64 > Nv ? Nv - 64 : tile * 64;
        n0 = n0 < 0 ? 0 : n0;
        const int lo = grim::patch_first(n0, W, Wo, s == 2, centre, HW, odd), hi = grim::patch_last(n0, Nv, W, Wo, s == 2, centre, HW);
        std::vector<char> held(room, 0);
        for (int q = 0; q < (hi - lo) / 8 + 1; ++q) {
            const int at = lo + 8 * q < HW - 8 ? lo + 8 * q : HW - 8;
            for (int j = 0; j < 8; ++j) {
                const int slot = at - lo + j;
                if (at + j < 0 || at + j >= HW || slot < 0 || slot >= room) ++bad;
                else held[slot] = 1;
            }
        }
        for (int n = n0; n < n0 + 64 && n < Nv; ++n) {
            int h, w;
            const int pix = grim::patch_pixel_of(n, W, Wo, s == 2, &h, &w);
            if (h != n / Wo * s || w != n % Wo * s) ++bad;
            for (int tap = 0; tap < kh * kw; ++tap) {
                const int y = h + tap / kw - ph, x = w + tap % kw - pw;
                if (y < 0 || y >= H || x < 0 || x >= W) continue;
                const int slot = pix + (tap / kw - ph) * W + tap % kw - pw - lo;
                if (slot < 0 || slot >= room || !held[slot]) ++bad;
            }
        }
    }
    return bad;
}

// The most workgroups of a launch that one XCD is dealt, and the waves each has
extern "C" int conv_patch_per_xcd(int tiles, int runs, int *waves) {
    int64_t workgroups = 0;
    grim::xcd_map(tiles, runs, &workgroups);
    *waves = grim::patch_waves(tiles, runs);
    return (int)((workgroups + 7) / 8);
}
