// Host walk over the loads of a planned convolution's tiles, with the arithmetic of the kernels (csrc/conv_window.hpp): how
// many loads of the form without range checks would touch an element outside the feature map.
#include <cstdint>

#include "conv_window.hpp"

namespace {

// one image of Cin channels of H x W; tiles of `tn` positions
template <bool S2>
int64_t outside(int Cin, int H, int W, int kh, int kw, int tn) {
    const int Ho = S2 ? (H + 1) / 2 : H, Wo = S2 ? (W + 1) / 2 : W, Wp = (Wo + 7) / 8 * 8;
    const int HW = H * W, total = Cin * HW, Nv = S2 ? Ho * Wp : HW, ph = kh / 2, pw = kw / 2, centre = ph * W + pw, pieces = tn / 8;
    int64_t bad = 0;
    for (int tile = 0; tile * tn < Nv; ++tile) {
        int n0 = tile * tn + tn > Nv ? Nv - tn : tile * tn;
        n0 = n0 < 0 ? 0 : n0;
        auto start = [&](int c) { return grim::conv_piece_start<S2>(n0 + c * 8, W, Ho, Wp); };
        if (grim::conv_tile_at_edge<S2>(start(0), start(pieces - 1), centre, HW)) continue;       // every load is range-checked
        for (int ch = 0; ch < Cin; ++ch)
            for (int tap = 0; tap < kh * kw; ++tap)
                for (int c = 0; c < pieces; ++c) {
                    const int e0 = ch * HW + (tap / kw - ph) * W + (tap % kw - pw) + start(c), ea = e0 - (e0 & 1);
                    int end = ea + (S2 ? 16 : 8);
                    if (!S2 && c == pieces - 1 && (e0 & 1)) end = e0 + 8;                         // the boundary element
                    if (ea < 0 || end > total) ++bad;
                }
    }
    return bad;
}

}  // namespace

extern "C" int64_t conv_loads_outside(int Cin, int H, int W, int kh, int kw, int stride, int tn) {
    return stride == 2 ? outside<true>(Cin, H, W, kh, kw, tn) : outside<false>(Cin, H, W, kh, kw, tn);
}
