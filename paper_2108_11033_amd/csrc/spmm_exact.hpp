// Products with non-finite values of X on the kernels that multiply whole 16-row runs on the matrix cores: there a row of
// the run that does not keep a column multiplies that row of X by zero, which an infinity or NaN turns into NaN.  The
// kernels that include this look for such values in what they fetch, or for sums that are not finite (every row of the run
// has one then); the outputs concerned are formed from the canonical arrays instead, kept weights only, as on the vector ALUs.
#pragma once
#include "spmm_common.hpp"

namespace grim {

struct ExactArrays {
    const int32_t *row_ptr, *col_ptr;
    const uint16_t *row_idx, *col_idx;
    const int64_t *blk_ptr;
    const void *weights;
    int32_t BR, BC, nbc;
};
inline ExactArrays exact_arrays(const grim_bcr_matrix *A) {
    return ExactArrays{A->dev.row_ptr, A->dev.col_ptr, A->dev.row_idx, A->dev.col_idx, A->dev.blk_ptr, A->dev.weights,
                       A->BR, A->BC, (int32_t)A->nbc};
}

// sums[e] = the kept weights of stored row `sr` times column n + e of X, for n + e < N (others: column N - 1, not used)
template <int DT, int E>
__device__ __forceinline__ void exact_row(const ExactArrays &a, const void *Xv, int64_t N, int64_t ldx, int64_t sr, int64_t n, float (&sums)[E]) {
    using T = typename Elem<DT>::type;
    const T *X = static_cast<const T *>(Xv), *W = static_cast<const T *>(a.weights);
    const int64_t strip = sr / a.BR;
    const int local = (int)(sr - strip * a.BR);
#pragma unroll
    for (int e = 0; e < E; ++e) sums[e] = 0.f;
    for (int32_t c = 0; c < a.nbc; ++c) {
        const int64_t b = strip * a.nbc + c;
        const int32_t q0 = a.row_ptr[b], q1 = a.row_ptr[b + 1], c0 = a.col_ptr[b], kc = a.col_ptr[b + 1] - c0;
        int32_t q = q0;
        while (q < q1 && a.row_idx[q] != local) ++q;
        if (q == q1) continue;
        const T *w = W + a.blk_ptr[b] + (int64_t)(q - q0) * kc;
        for (int32_t j = 0; j < kc; ++j) {
            const T *x = X + ((int64_t)c * a.BC + a.col_idx[c0 + j]) * ldx;
#pragma unroll
            for (int e = 0; e < E; ++e) sums[e] = __builtin_fmaf(to_f32<DT>(w[j]), to_f32<DT>(x[n + e < N ? n + e : N - 1]), sums[e]);
        }
    }
}

}  // namespace grim
