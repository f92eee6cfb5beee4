// Which form a convolution runs in: the rules of its launchers, on the host, where the tests of the dispatch use them too.
#pragma once
#include "bcr_matrix.hpp"
#include "conv_patch.hpp"

namespace grim {

constexpr int kConvLongWaves = 12;
constexpr int kConvMaxTaps = 31;   // 5 bits of the packed (tap, window start) word, one value left for padding slots
constexpr int kPatchTasks = 192;                           // tasks of a chunk that octets are chosen for
constexpr int kPatchWaveBytes = 20480;                     // eight waves, or two workgroups of four, fill a compute unit's LDS
constexpr int patch_pixel_bytes(int octets) { return octets == 1 ? 16 : octets * 16 + 16; }      // (padded: spreads reads and writes over the banks)

// Wave per (tile, strip) instead of four waves splitting a strip's steps: strips of at most 8 steps (two batches of a
// wave) with enough pairs to fill the GPU, and longer strips once there are half as many pairs again (measured: 9 steps
// x 1568 pairs 11.3 -> 10.4 us, 18 steps x 12544 pairs 144 -> 129 us; 18 steps x 784 pairs 11.1 -> 12.9 us)
// (the convolution kernel, with more work per step: 9 x 1568 15.4 -> 16.3 us, 18 x 12544 138 -> 113 us; it asks for 4096)
inline bool gather_strip_to_a_wave(const grim_bcr_matrix *A, int64_t pairs, int64_t pairs_for_long_strips) {
    return (A->gather.max_steps <= 8 && pairs >= 1024) || (A->gather.max_steps <= 40 && pairs >= pairs_for_long_strips);
}

// a wave's share of the steps of the longest strip when twelve waves split it
inline int conv_share(const grim_bcr_matrix *A) { return (A->gather.max_steps + kConvLongWaves - 1) / kConvLongWaves; }

// 32-position tiles (two sub-tiles of 16) for maps of 14 x 14 and less, where 64-position tiles leave compute units without a
// workgroup.  Stride 1: if a wave's share of a strip's steps is one batch of six where 64-position tiles would take two (72 steps
// at 14 x 14: 12.0 -> 9.4 us).  Stride 2, whose 64-position tiles have two steps in flight against three: once four waves of
// those need a second batch (36 steps onto 7 x 7: 11.9 -> 7.5 us, 12 steps onto 7 x 7 8.0 -> 6.8, 54 steps 15.3 -> 11.7).
inline int conv_subtiles(const grim_bcr_matrix *A, int64_t positions, int32_t batch, int32_t stride, bool planned) {
    const bool long_enough = stride == 2 ? A->gather.max_steps > 8 : A->gather.max_steps >= 16 && conv_share(A) <= 6;
    return planned && long_enough && (positions + 31) / 32 * batch * (int64_t)A->gather.nstrips <= 256 ? 2 : 4;
}

// Waves that split a strip's steps, by the number of (tile, strip) pairs: the launch forms of the row-gathering kernel (one
// wave: a pair per wave); few pairs and strips of more than a batch of four waves: twelve up to 256 pairs (one workgroup per
// compute unit), eight up to 512 (two per compute unit; 28 x 28 layers: 11.0 -> 9.4 us with 18 steps, 14.1 -> 13.3 us with 36;
// 13 steps on three 9 x 9 maps 12.3 -> 10.4).  At stride 2 four waves are as quick up to 15 steps.
inline int conv_strip_waves(const grim_bcr_matrix *A, int nt, int64_t pairs, int32_t stride) {
    if (gather_strip_to_a_wave(A, pairs, 4096)) return 1;
    if (nt == 2) return kConvLongWaves;
    return A->gather.max_steps <= (stride == 2 ? 15 : 12) ? 4 : pairs <= 256 ? kConvLongWaves : pairs <= 512 ? 8 : 4;
}

// At stride 1, does a batch split a strip's sum over as many waves as one image does?  (Its sums then have the same bits.)
inline bool conv_batch_sums_as_one(const grim_bcr_matrix *A, int64_t positions, int32_t batch) {
    const int64_t tiles = (positions + 63) / 64 * (int64_t)A->gather.nstrips;
    const int nt = conv_subtiles(A, positions, batch, 1, true), nt_one = conv_subtiles(A, positions, 1, 1, true);
    return conv_strip_waves(A, nt, tiles * batch, 1) == conv_strip_waves(A, nt_one, tiles, 1);
}

// Octets of channels to a chunk: the most that leave eight waves a chunk each, fit their share of LDS and are asked for in one
// go (what is not is waited for once per 64 tasks: 416 -> 96 channels, 3 x 3, from 20 x 30 at stride 2 18.1 us with 4 octets);
// 0: the layer is not for this kernel
inline int32_t patch_octets(int64_t Cin, int32_t H, int32_t W, int32_t kh, int32_t kw, int32_t stride) {
    if (kh * kw < 2 || kh * kw > kConvMaxTaps || (int64_t)H * W < 8 || Cin < 8 || Cin % 4 != 0) return 0;
    const int64_t pixels = patch_pixels(H, W, kh, kw, stride);
    for (int32_t co = 4; co >= 1; co /= 2)
        if ((co == 1 || (Cin >= 64 * co && pixels / 8 * 2 * co <= kPatchTasks)) && (pixels + 1) * patch_pixel_bytes(co) <= kPatchWaveBytes)
            return co;
    return 0;
}

}  // namespace grim
