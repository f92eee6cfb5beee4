// What the two planned convolutions on 64-row runs share.
#pragma once
#include "conv_gather_kernel.hpp"

namespace grim {

struct ConvTallParams : ConvParams {
    // the matrix's 16-row runs, `own_plan` their window-start words
    const int32_t *own_sptr;
    const uint32_t *own_plan, *own_desc;
    const unsigned char *own_payload;
    int32_t own_usteps;
};

// output row r of 16-row run `run` at position n: the run's k slots in order, zero weights where row r does not keep one
template <bool BF16, bool S2>
__device__ __forceinline__ float conv_own_run(const ConvTallParams &p, const unsigned short *Fimg, int run, int r, int n) {
    constexpr int DT = BF16 ? GRIM_BF16 : GRIM_F16;
    using T = typename Elem<DT>::type;
    const int rowlen = S2 ? p.Wp : p.W, ho = n / rowlen, wo = n - ho * rowlen;
    const int h = S2 ? 2 * ho : ho, w = S2 ? 2 * wo : wo, start = h * p.W + w - (1 << 25);
    const int s0 = p.own_usteps ? run * p.own_usteps : p.own_sptr[run], s1 = p.own_usteps ? s0 + p.own_usteps : p.own_sptr[run + 1];
    float sum = 0.f;
#pragma unroll 1
    for (int s = s0; s < s1; ++s) {
#pragma unroll 1
        for (int g = 0; g < 4; ++g) {
            const uint2 d = reinterpret_cast<const uint2 *>(p.own_desc)[(int64_t)s * 4 + g];
            const bool kept = (d.x >> r) & 1u;
            const T *wt = reinterpret_cast<const T *>(p.own_payload) + ((int64_t)d.y + (kept ? __builtin_popcount(d.x & ((1u << r) - 1u)) : 0)) * 8;
#pragma unroll 1
            for (int j = 0; j < 8; ++j) {
                const unsigned int word = p.own_plan[(int64_t)s * 32 + j * 4 + g];
                const int tap = (int)(word >> 27);
                if (tap == p.KK) continue;       // padding
                const int hh = h + tap / p.kw - (p.kh >> 1), ww = w + tap % p.kw - (p.kw >> 1);
                const bool inside = hh >= 0 && hh < p.H && ww >= 0 && ww < p.W;
                const unsigned short x = inside ? Fimg[(int)(word & 0x7ffffffu) + start] : (unsigned short)0;
                sum = __builtin_fmaf(kept ? to_f32<DT>(wt[j]) : 0.f, to_f32<DT>(__builtin_bit_cast(T, x)), sum);
            }
        }
    }
    return sum;
}

}  // namespace grim
