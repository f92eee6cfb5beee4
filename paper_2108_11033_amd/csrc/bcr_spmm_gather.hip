#include <algorithm>

#include "conv_rules.hpp"
#include "group_rules.hpp"
#include "spmm_gather_kernel.hpp"

namespace grim {

bool gather_wave_per_strip(const grim_bcr_matrix *A, int64_t pairs, int64_t pairs_for_long_strips) { return gather_strip_to_a_wave(A, pairs, pairs_for_long_strips); }

bool gather_applies(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx) {
    return A->gather.present && N >= 4 && N % 4 == 0 && ldx % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 8 == 0;
}
// (Below 64 columns the kernel reads the last 16 bytes of X as a whole: there have to be that many.  Blocks of more than 64
// rows are taken with the aligned rows of gather_applies only.)
bool gather_any_applies(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx) {
    return A->gather.present && reinterpret_cast<uintptr_t>(X) % 2 == 0 && (N >= 64 || (A->K - 1) * ldx + N >= 8) &&
           (A->BR <= 64 || gather_applies(A, X, N, ldx));
}

// Bytes through one compute unit, the quantity both matrix-core kernels are bound by at these
// sizes: a workgroup fetches the rows of X its strip keeps (128 bytes each) and the strip's
// records, pays a start-up, and 256 compute units share the workgroups.
double gather_cost(const grim_bcr_matrix *A, int64_t N) {
    const GatherLayout &L = A->gather;
    const double nbr = (double)L.nstrips;
    const double per_wg = (double)L.xrows / nbr * 128.0 + ((double)L.nsteps * 160.0 + (double)L.payload.size()) / nbr;
    const double nwg = (double)((N + 63) / 64) * nbr;
    // the bytes go through the compute units one after the other; the start-up of a workgroup overlaps with the
    // three others a compute unit holds
    return (nwg > 256.0 ? nwg / 256.0 : 1.0) * per_wg + (nwg > 1024.0 ? nwg / 1024.0 : 1.0) * 30e3;
}

// Two products Y = A X and Y2 = A2 X2 of fewer than 64 columns in one launch (the two gate products of a GRU step):
// same element type, number of 16-row runs, N and leading dimensions; K may differ.
bool gather_pair_applies(const grim_bcr_matrix *A, const void *X, const grim_bcr_matrix *A2, const void *X2, int64_t N,
                         int64_t ldx) {
    return N < 64 && gather_any_applies(A, X, N, ldx) && gather_any_applies(A2, X2, N, ldx) && A->dtype == A2->dtype &&
           A->gather.nstrips == A2->gather.nstrips;
}

// Parameters, grid and kernel form of a launch (see launch_spmm_gather); GRIM_ERR_UNSUPPORTED when the kernel does not apply.
grim_status gather_setup(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, float *Y, int64_t ldy,
                         const grim_bcr_matrix *A2, const void *X2, float *Y2, GatherParams *out, GatherForm *form, bool alone) {
    if (!gather_any_applies(A, X, N, ldx)) return GRIM_ERR_UNSUPPORTED;
    if (A2 && !gather_pair_applies(A, X, A2, X2, N, ldx)) return GRIM_ERR_UNSUPPORTED;
    GatherParams p;
    p.sptr = A->gather.d_sptr;
    p.rows = A->gather.d_rows;
    p.desc = A->gather.d_desc;
    p.payload = A->gather.d_payload;
    p.out_row = A->gather.d_out_row;
    p.X = static_cast<const unsigned short *>(X);
    p.Y = Y;
    p.N = N; p.ldx = ldx; p.ldy = ldy;
    p.nbr = (int32_t)A->gather.nstrips;
    p.K = (int32_t)A->K;
    p.usteps = A->gather.usteps;
    p.exact = exact_arrays(A);
    // fewer than 64 columns: one tile of the narrowest width that holds them
    // Long strips and few tiles (14 x 14 maps and less): 32-column tiles, whose twice as many workgroups have twelve waves
    // with three steps in flight -- 512 x 4608 at 147 columns 8.0 -> 5.0 us, at 64 / 196 / 256 columns 6.0 / 6.4 / 6.2 ->
    // 4.0 / 5.1 / 4.6, 256 x 4608 in 16 x 16 blocks at 392 columns 8.5 -> 6.6 -- while every workgroup has a compute unit: with
    // 288 or 384 (tile, run) pairs 512 x 1152, 512 x 2304 and 1024 x 2304 take 4.5 to 4.9 us in 64-column tiles, 5.3 to 5.7 in
    // these.  Strips below 16 steps stay (256 x 1152 at 256 columns 3.8 us either way).
    const bool small_tiles = alone && N >= 64 && A->gather.max_steps >= 16 && (N + 31) / 32 * p.nbr <= 256;
    const int nt = small_tiles ? 2 : N > 32 ? 4 : N > 16 ? 2 : 1;
    p.ntiles = (int32_t)((N + nt * 16 - 1) / (nt * 16));
    p.second = GatherSecond{p.sptr, p.out_row, p.rows, p.desc, p.payload, p.X, p.Y, p.usteps, p.K, exact_arrays(A)};
    if (A2)
        p.second = GatherSecond{A2->gather.d_sptr, A2->gather.d_out_row, A2->gather.d_rows, A2->gather.d_desc,
                                A2->gather.d_payload, static_cast<const unsigned short *>(X2), Y2, A2->gather.usteps, (int32_t)A2->K,
                                exact_arrays(A2)};
    // strips of at most 8 steps (two batches of a wave) with enough (tile, strip) pairs to fill the GPU: wave per pair;
    // long strips and fewer workgroups than compute units: eight waves per strip
    const bool narrow = N < 64;
    // Beside the wide-tile kernel and for long strips only: with 512 x 4608 and 512 to 1024 columns left over, products of 24 576
    // columns and those 1 to 2 % faster; strips of 18 steps took 12.4 us for 12.0 on a 2304-row product.
    p.touch = !alone && A->gather.max_steps >= 40 ? 1 : 0;
    const bool solo = !narrow && !small_tiles && gather_wave_per_strip(A, (int64_t)p.ntiles * p.nbr, 1536);
    // Narrow tiles: eight waves only where four need more than a batch of steps and every workgroup has a compute unit --
    // 4608 x 2048 at four columns, 288 workgroups: 6.5 us with eight, 4.65 with four; 2048 x 2048 at nine, 20 steps: 5.7, 4.3.
    const int64_t pairs = (int64_t)p.ntiles * p.nbr * (A2 ? 2 : 1);
    const int longest = std::max(A->gather.max_steps, A2 ? A2->gather.max_steps : 0);
    const bool eight = !solo && (narrow ? longest > 4 * gather_narrow_steps(nt) && pairs <= 256 : longest >= 16 && (small_tiles || pairs <= 256));
    const int64_t per_tile = solo ? (p.nbr + 3) / 4 : p.nbr;
    if (((int64_t)p.ntiles + 7) / 8 * 8 * per_tile > 0x7fffffff) return GRIM_ERR_SHAPE;
    int64_t nwg = 0;
    p.map = xcd_map(p.ntiles, per_tile, &nwg);
    if (nwg > 0x7fffffff) return GRIM_ERR_SHAPE;
    form->narrow = narrow;
    form->solo = solo;
    form->eight = eight;
    form->nt = nt;
    // (steps past a wave's share are fetched too: no more than a short strip has)
    form->steps = longest <= 8 ? 2 : longest <= 16 ? 4 : 8;
    form->aligned = N % 8 == 0 && ldx % 8 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 &&
                    (!A2 || reinterpret_cast<uintptr_t>(X2) % 16 == 0);
    form->nwg = nwg;
    *out = p;
    return GRIM_OK;
}

// X of fewer than the eight elements that make up a 16-byte load (one row of four columns): an output per thread
template <int DT>
__global__ void __launch_bounds__(256) bcr_spmm_few_elements(ExactArrays a, const int32_t *out_row, const void *X, int64_t N, int64_t ldx, float *Y,
                                                             int64_t ldy, int64_t rows) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, sr = i / N, n = i - sr * N;
    if (sr >= rows || out_row[sr] < 0) return;
    float v[1];
    exact_row<DT, 1>(a, X, N, ldx, sr, n, v);
    Y[out_row[sr] * ldy + n] = v[0];
}

grim_status launch_spmm_gather(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, float *Y, int64_t ldy,
                               hipStream_t stream, const grim_bcr_matrix *A2, const void *X2, float *Y2) {
    if (!A2 && gather_applies(A, X, N, ldx) && !gather_any_applies(A, X, N, ldx)) {
        const int64_t rows = A->gather.nstrips * 16;
        if (rows * N / 256 > 0x7ffffffe) return GRIM_ERR_SHAPE;
        const dim3 few((unsigned)((rows * N + 255) / 256));
        if (A->dtype == GRIM_BF16) hipLaunchKernelGGL(bcr_spmm_few_elements<GRIM_BF16>, few, dim3(256), 0, stream, exact_arrays(A), A->gather.d_out_row, X, N, ldx, Y, ldy, rows);
        else hipLaunchKernelGGL(bcr_spmm_few_elements<GRIM_F16>, few, dim3(256), 0, stream, exact_arrays(A), A->gather.d_out_row, X, N, ldx, Y, ldy, rows);
        return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
    }
    GatherParams p;
    GatherForm form;
    const grim_status st = gather_setup(A, X, N, ldx, Y, ldy, A2, X2, Y2, &p, &form);
    if (st != GRIM_OK) return st;
    const bool narrow = form.narrow, solo = form.solo, eight = form.eight, aligned = form.aligned;
    const int64_t nwg = form.nwg;
    const int waves = gather_waves(narrow, eight, form.nt);
    const int in_flight = gather_steps(aligned, narrow, eight, form.nt, 0);      // (of the forms that park a batch as a whole)
    const size_t lds = (size_t)waves * gather_wave_lds(form.nt, gather_buffers(narrow, form.nt, in_flight));
    const dim3 grid((unsigned)nwg, A2 ? 2u : 1u), block(waves * 64);
#define GRIM_GATHER(BF, AL, NR, SO, EI, ...)                                                                              \
    do {                                                                                                             \
        auto kern = bcr_spmm_gather<BF, AL, NR, SO, EI, __VA_ARGS__>;                                                          \
        static std::atomic<bool> attr_done{false};   /* raising a kernel's LDS limit is needed once per process */  \
        if (lds > 64 * 1024 && !attr_done) {                                                                         \
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, \
                                    160 * 1024) != hipSuccess) {                                                     \
                (void)hipGetLastError();                                                                             \
                return GRIM_ERR_DEVICE;                                                                              \
            }                                                                                                        \
            attr_done = true;                                                                                        \
        }                                                                                                            \
        hipLaunchKernelGGL(kern, grid, block, lds, stream, p);                                                       \
    } while (0)
#define GRIM_GATHER_AL(BF, AL)                                                                                       \
    if (narrow && form.nt == 1) {                                                                                    \
        if (eight) GRIM_GATHER(BF, AL, true, false, true, 1);                                                        \
        else if (form.steps == 2) GRIM_GATHER(BF, AL, true, false, false, 1, 2);                                     \
        else if (form.steps == 4) GRIM_GATHER(BF, AL, true, false, false, 1, 4);                                     \
        else GRIM_GATHER(BF, AL, true, false, false, 1);                                                             \
    }                                                                                                                \
    else if (narrow && form.nt == 2) { if (eight) GRIM_GATHER(BF, AL, true, false, true, 2); else GRIM_GATHER(BF, AL, true, false, false, 2); } \
    else if (narrow) { if (eight) GRIM_GATHER(BF, AL, true, false, true, 4); else GRIM_GATHER(BF, AL, true, false, false, 4); } \
    else if (form.nt == 2) GRIM_GATHER(BF, AL, false, false, true, 2);                                               \
    else if (solo) GRIM_GATHER(BF, AL, false, true, false, 4);                                                       \
    else if (eight) GRIM_GATHER(BF, AL, false, false, true, 4);                                                      \
    else GRIM_GATHER(BF, AL, false, false, false, 4);
#define GRIM_GATHER_DT(BF)                                                                                           \
    if (aligned) { GRIM_GATHER_AL(BF, true) } else { GRIM_GATHER_AL(BF, false) }
    if (A->dtype == GRIM_BF16) { GRIM_GATHER_DT(true) } else { GRIM_GATHER_DT(false) }
#undef GRIM_GATHER_DT
#undef GRIM_GATHER_AL
#undef GRIM_GATHER
    return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
}


// One 16-column tile for each of the matrices of a group (grid.y), whose layouts come out of a table.  Bound by latency (row
// numbers, then rows of x and weights, then the sums) and hence by waves in flight: two steps per wave and 54 registers, eight waves
// to a SIMD; up to four columns just their bytes of a row of x are fetched, since 16 bytes at an odd element cost the vector L1 about three
// times what they cost at an even one (64 of 2048 x 2048 of mixed rates at 1 / 2 / 3 / 4 columns 35.3 / 27.3 / 35.6 / 27.7 -> 24.4 /
// 24.7 / 30.3 / 26.3 us, 43 of 3872 x 1248 at one 31.4 -> 21.2).  (Four steps, 74 registers: 64 of 2048 x 2048 at 8 columns 29.3 -> 33.2 us, 30 of 1856 x 992 at one 11.6 -> 14.1).
template <bool BF16, bool SOLO, int COLS>
__global__ void __launch_bounds__(256, 4) bcr_spmm_gather_many(GatherParams p, const GatherSecond *table, int64_t x_stride, int64_t y_stride) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    using Entry = const __attribute__((address_space(4))) GatherSecond *;       // (read once per wave, through the scalar cache)
    const Entry m = (Entry)table + blockIdx.y;
    p.sptr = m->sptr; p.out_row = m->out_row; p.rows = m->rows; p.desc = m->desc; p.payload = m->payload;
    p.usteps = m->usteps;
    p.exact.row_ptr = m->exact.row_ptr; p.exact.col_ptr = m->exact.col_ptr;
    p.exact.row_idx = m->exact.row_idx; p.exact.col_idx = m->exact.col_idx;
    p.exact.blk_ptr = m->exact.blk_ptr; p.exact.weights = m->exact.weights;
    p.X += (int64_t)blockIdx.y * x_stride;
    p.Y += (int64_t)blockIdx.y * y_stride;
    gather_body<BF16, false, true, SOLO, false, 1, kGatherLongWaves, 2, COLS>(p, lds, blockIdx.x, 0);
}

size_t gather_entry_bytes() { return sizeof(GatherSecond); }
void gather_fill_entry(const grim_bcr_matrix *A, void *entry) {
    *static_cast<GatherSecond *>(entry) = GatherSecond{A->gather.d_sptr, A->gather.d_out_row, A->gather.d_rows, A->gather.d_desc, A->gather.d_payload,
                                                       nullptr, nullptr, A->gather.usteps, (int32_t)A->K, exact_arrays(A)};
}

grim_status launch_spmm_gather_many(const grim_bcr_group *G, const void *X, int64_t x_stride, int64_t N, int64_t ldx, float *Y, int64_t y_stride,
                                    int64_t ldy, hipStream_t stream) {
    if (!G->d_gather || N > 16 || reinterpret_cast<uintptr_t>(X) % 2 != 0 || (G->K - 1) * ldx + N < 8) return GRIM_ERR_UNSUPPORTED;
    GatherParams p = {};
    p.X = static_cast<const unsigned short *>(X);
    p.Y = Y;
    p.N = N; p.ldx = ldx; p.ldy = ldy;
    p.nbr = (int32_t)G->gather_runs;
    p.ntiles = 1;
    p.K = (int32_t)G->K;
    p.exact.BR = G->BR; p.exact.BC = G->BC; p.exact.nbc = (int32_t)G->nbc;
    const bool solo = group_run_to_a_wave((int64_t)G->count * G->gather_runs, G->gather_steps);
    int64_t nwg = 0;
    p.map = xcd_map_one_tile(solo ? (G->gather_runs + 3) / 4 : G->gather_runs, &nwg);
    if (nwg > 0x7fffffff) return GRIM_ERR_SHAPE;
    const dim3 grid((unsigned)nwg, (unsigned)G->count);
    const size_t lds = 4 * gather_wave_lds(1);
    const GatherSecond *table = static_cast<const GatherSecond *>(G->d_gather);
#define GRIM_MANY(BF, SO, CO) hipLaunchKernelGGL((bcr_spmm_gather_many<BF, SO, CO>), grid, dim3(256), lds, stream, p, table, x_stride, y_stride)
#define GRIM_MANY_SO(BF, CO) if (solo) GRIM_MANY(BF, true, CO); else GRIM_MANY(BF, false, CO)
#define GRIM_MANY_DT(BF) if (N == 1) { GRIM_MANY_SO(BF, 1); } else if (N == 2) { GRIM_MANY_SO(BF, 2); } else if (N == 3) { GRIM_MANY_SO(BF, 3); } else if (N == 4) { GRIM_MANY_SO(BF, 4); } else { GRIM_MANY_SO(BF, 0); }
    if (G->dtype == GRIM_BF16) { GRIM_MANY_DT(true) } else { GRIM_MANY_DT(false) }
#undef GRIM_MANY_DT
#undef GRIM_MANY_SO
#undef GRIM_MANY
    return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
}


}  // namespace grim
