// What room a staged matrix-core kernel has for a chunk's rows of X and step records, in LDS and in its fetching waves' registers: the
// launchers choose among their compiled forms by it, the packer cuts the records so that they fit.
#pragma once
#include <algorithm>

#include "bcr_matrix.hpp"
#include "conv_taps.hpp"

namespace grim {

constexpr int64_t kStagedLds = 160 * 1024;

// ---- wide-tile kernel
constexpr int kWideMulWaves = 8;     // multiplying waves, two strips each
constexpr int kWideThreads = (kWideMulWaves + kWideFetchWaves) * 64;
constexpr int kWideStrips = 2 * kWideMulWaves;   // strips per workgroup
// 16-byte record units per fetching thread and chunk: 8 = 32 KB per (chunk, group), the layout's limit; the
// 192-column shape, whose rows of X take more registers, has room for 4 (16 KB)
constexpr int wide_sru(int tn) { return tn == 192 ? 4 : 8; }
static_assert(wide_sru(128) * kWideFetchThreads * 16 == kWideMaxRecordBytes, "record staging registers cover the layout's limit");

// Rows of a stage are padded by 32 bytes: consecutive rows then start 32 bytes apart modulo the 256-byte bank line
// (pitches 224, 288 and 416 give eight distinct offsets), so the four rows one transpose read gathers -- 32 bytes
// of each -- spread over the banks without a swizzle, and the addresses of a row's sub-tiles differ by constants.
constexpr int kWidePad = 32;

__host__ __device__ inline int wide_stage_bytes(int chunk_rows, int tn, int amax) {
    return (chunk_rows + 1) * (tn * 2 + kWidePad) + amax * 16;
}

// Bytes between the rows of a strip's 16-bit outputs where they pass through LDS (32-row strips), and LDS for all of them: 16
// bytes of padding put the two rows a write names on different banks.
constexpr int wide_out_pitch(int tn) { return tn * 2 + 16; }
constexpr int wide_out_bytes(int tn) { return kWideMulWaves * 32 * wide_out_pitch(tn); }

// compiled tile widths: BR = 16: 128 and 192 columns, BR = 32: 96 columns (its accumulators leave no room for more)
constexpr bool wide_tile_ok(int BR, int tn) { return BR == 16 ? (tn == 128 || tn == 192) : BR == 32 ? tn == 96 : false; }

// do the records of a chunk fit the fetching waves' registers, and two stages LDS?
inline int64_t wide_lds_bytes(const MmaLayout &L, int tn) { return 2 * (int64_t)wide_stage_bytes(L.chunk_rows, tn, L.amax[2]); }
inline bool wide_records_fit(const MmaLayout &L, int tn) { return (int64_t)L.amax[2] <= (int64_t)wide_sru(tn) * kWideFetchThreads; }
inline bool wide_fits(const MmaLayout &L, int BR, int tn) {
    return wide_tile_ok(BR, tn) && wide_records_fit(L, tn) && wide_lds_bytes(L, tn) <= kStagedLds;
}
// LDS of a convolution with KK kernel taps
inline int64_t conv_wide_lds(const MmaLayout &L, int BR, int tn, int KK) {
    // two stages; kConvAnyTap: the (tap, piece) mask table, four per-chunk row tables
    const int64_t out = BR == 32 ? wide_out_bytes(tn) : 0;      // the outputs' way through LDS, when the stages are done with
    const int64_t stages = std::max(wide_lds_bytes(L, tn), out);
    if (conv_tap_ways(tn, KK, L.chunk_rows)) return stages;
    return stages + (int64_t)(KK + 1) * (tn / 8) * 16 + 4 * (int64_t)wide_max_chunk_rows(BR) * 8;
}
inline bool conv_wide_fits(const MmaLayout &L, int BR, int tn, int KK) {
    return wide_tile_ok(BR, tn) && wide_records_fit(L, tn) && conv_wide_lds(L, BR, tn, KK) <= kStagedLds;
}

// ---- staged kernel
// LDS bytes of one stage: staged X rows + zero row, then room for amax 16-byte units of
// records rounded up to whole 1 KB slots
__host__ __device__ inline int mma_stage_bytes(int chunk_rows, int pitch, int amax) {
    return (chunk_rows + 1) * pitch + ((amax * 16 + 1023) / 1024 + 1) * 1024;
}

// Compiled launch shapes.  Groups of 4 strips use 4 consumer waves, larger groups 8 (LDS reads
// per MFMA are high, so a second consumer wave per SIMD hides their latency); always 8
// producer waves (two teams of 4), each holding SX slots of X and SR slots of records.
struct MmaShape { int tn, strips, nw, sx, sr; };
inline bool mma_shape(int BR, int tn, int strips, MmaShape *out) {
    const int sx = tn == 32 ? 4 : tn == 64 ? 8 : tn == 128 ? 16 : 0;      // 256 staged rows
    const int sr = strips == 4 ? 4 : strips == 8 ? 8 : strips == 16 ? 12 : 0;
    if (!sx || !sr) return false;
    if (tn == 128 && strips != 4) return false;
    const int nw = strips == 4 ? 4 : 8;
    if (BR == 32 && (strips / nw) * (tn / 32) > 4) return false;           // accumulator registers
    *out = MmaShape{tn, strips, nw, sx, sr};
    return true;
}
inline int mma_amax(const MmaLayout &L, int strips) { return L.amax[strips <= 4 ? 0 : strips <= 8 ? 1 : strips <= 16 ? 2 : 3]; }
inline bool mma_shape_fits(const MmaLayout &L, int BR, int tn, int strips) {
    MmaShape sh;
    if (!mma_shape(BR, tn, strips, &sh)) return false;
    const int rps = 1024 / (tn * 2), amax = mma_amax(L, strips);
    if ((L.chunk_rows + rps - 1) / rps > 4 * sh.sx) return false;
    if ((amax * 16 + 1023) / 1024 > 4 * sh.sr) return false;
    return 2 * (int64_t)mma_stage_bytes(L.chunk_rows, tn * 2, amax) + (int64_t)L.nchunks * (strips + 1) * 8 <= kStagedLds;
}

// Has `L` room in every compiled form that `other`, of the same matrix with K columns, has room in?  (wide: the wide-tile kernel's forms,
// products and convolutions of every number of taps that divides K -- kernels are odd both ways; otherwise the staged kernel's)
inline bool fits_wherever(const MmaLayout &L, const MmaLayout &other, int BR, int64_t K, bool wide) {
    if (wide) {
        for (int tn : {96, 128, 192}) {
            if (wide_fits(other, BR, tn) && !wide_fits(L, BR, tn)) return false;
            for (int KK = 1; KK <= 255; KK += 2)
                if (K % KK == 0 && conv_wide_fits(other, BR, tn, KK) && !conv_wide_fits(L, BR, tn, KK)) return false;
        }
        return true;
    }
    for (int tn : {32, 64, 128})
        for (int strips : {4, 8, 16})
            if (mma_shape_fits(other, BR, tn, strips) && !mma_shape_fits(L, BR, tn, strips)) return false;
    return true;
}

}  // namespace grim
