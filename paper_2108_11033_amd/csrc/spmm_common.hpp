// Definitions shared by the SpMM kernel files: vector types, the matrix-core and LDS transpose-read
// wrappers, the LDS swizzle of staged rows and the XCD-aware workgroup id map.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "bcr_matrix.hpp"
#include "xcd_map.hpp"

namespace grim {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int DT> struct Elem;
template <> struct Elem<GRIM_F32> { using type = float; };
template <> struct Elem<GRIM_F16> { using type = _Float16; };
template <> struct Elem<GRIM_BF16> { using type = unsigned short; };

template <int DT> __device__ __forceinline__ float to_f32(typename Elem<DT>::type v);
template <> __device__ __forceinline__ float to_f32<GRIM_F32>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<GRIM_F16>(_Float16 v) { return (float)v; }
template <> __device__ __forceinline__ float to_f32<GRIM_BF16>(unsigned short v) {
    return __builtin_bit_cast(float, (unsigned int)v << 16);
}

template <bool BF16>
__device__ __forceinline__ f32x4 mfma16(i16x8 a, i16x8 b, f32x4 c) {
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <bool BF16>
__device__ __forceinline__ f32x16 mfma32(i16x8 a, i16x8 b, f32x16 c) {
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// LDS transpose read: the 16 lanes of a block each name 8 bytes (4 values along n of one
// staged row); lane i of the block receives value (i % 4) of the chunks named by lanes
// i / 4, 4 + i / 4, 8 + i / 4 and 12 + i / 4 -- four rows at one column, the MFMA k order.
__device__ __forceinline__ i16x4 lds_tr_read_at(unsigned int lds_byte_address) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(uintptr_t)lds_byte_address);
}
__device__ __forceinline__ i16x4 lds_tr_read(const char *lds_addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(lds_addr));
}

// Staged rows have no padding; the 16-byte chunks of a row are XOR-swizzled by the row
// number so that the four rows one transpose read touches fall into different bank groups
// whenever their numbers differ mod 4 (mod 8 for 128-byte rows, where consecutive rows
// already sit in opposite halves of the 256-byte bank line; measured 3-7 % faster).
template <int CPR>   // 16-byte chunks per staged row
__device__ __forceinline__ int swizzle(int row) {
    return CPR == 8 ? (((row >> 1) & 3) << 1) : CPR > 8 ? ((row & 3) << 1) : (((row >> 1) & 1) << 1);
}

// first of the `nst` steps of a strip (below 2^28) that wave `wave` of `waves` takes
__device__ __forceinline__ int wave_share(int nst, int wave, int waves) { return (int)((unsigned int)nst * (unsigned int)wave / (unsigned int)waves); }

// 16 bytes of X at any 2-byte alignment: a single access on this GPU
__device__ __forceinline__ u32x4 load_piece_any(const unsigned short *src) {
    struct __attribute__((packed, aligned(2))) { unsigned int d[4]; } v;
    __builtin_memcpy(&v, src, 16);
    return u32x4{v.d[0], v.d[1], v.d[2], v.d[3]};
}
// A piece that would reach past the end of X is fetched `n` < 8 elements early; this moves it into place.
__device__ __forceinline__ u32x4 drop_elements(u32x4 v, unsigned int n) {
    unsigned __int128 x = (unsigned __int128)v[0] | (unsigned __int128)v[1] << 32 | (unsigned __int128)v[2] << 64 | (unsigned __int128)v[3] << 96;
    x >>= 16 * n;
    return u32x4{(unsigned int)x, (unsigned int)(x >> 32), (unsigned int)(x >> 64), (unsigned int)(x >> 96)};
}

// Waves that split a long strip's steps in the few-workgroups form of the row-gathering kernels.  A 36-step strip of a
// 14 x 14 layer: 8 waves of the product kernel (4 steps per batch) 7.66 us, 12 waves 7.63, 16 waves 8.56; the convolution
// kernel (3 steps per batch) 11.0 us with 8, 8.6 us with 12 -- every wave then needs one batch only --, 9.7 us with 16.
constexpr int kGatherLongWaves = 8, kGatherSmallTileWaves = 12;


}  // namespace grim
