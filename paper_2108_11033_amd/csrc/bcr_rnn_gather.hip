// One step of a recurrent layer for a batch of columns in one launch on the matrix cores: the gate product(s) with the
// cell in the epilogue (Section 3.1: an RNN layer is one product per time step; Section 6.3 times the GRU step by step).
#include <algorithm>

#include "rnn_cell.hpp"
#include "spmm_exact.hpp"

namespace grim {

// Workgroup = (16 hidden units, 16 columns).  The gate rows of the units are 16-row runs of the row-gathering layout
// (LSTM: four of [W_ih | W_hh]; GRU: three of W_i and three of W_h); WPR waves split the steps of each run as in
// bcr_spmm_gather's 16-column tile, the partial tiles meet in LDS, and one thread per (unit, column) adds them in wave
// order, stores the pre-activations and applies the cell.  Against the products as a launch of their own and the cell as
// another this saves the second dispatch and the pre-activations' way through memory; the workgroup cannot be smaller,
// since the cell needs all gates of a unit.
// Bound: two dependent fetches (row numbers, then rows of X and weights) and the launch.  1024 units and inputs in 8 x 12 of
// 32 x 32: LSTM 32 columns 8.8 -> 7.2 us per step, 9 columns 29.9 -> 8.3; GRU 32 columns 7.8 -> 6.4, 64 columns 12.2 -> 7.3;
// LSTM of mixed rates, one column 11.6 -> 8.4.
// With all steps of a batch parked in LDS before the first is multiplied 6.8 us for the LSTM's 32 columns, 6.1 for the GRU's, 8.2 at mixed rates.
struct RnnGatherMatrix {
    const int32_t *sptr;
    const uint32_t *rows, *desc;
    const unsigned char *payload;
    const int32_t *strip_pos;    // stored position of every original strip; null: stored in original order
    const unsigned short *X;     // K x N, leading dimension ldx
    float *G;                    // pre-activations, leading dimension ldg
    int64_t ldx, ldg;
    int32_t usteps, K, BR;
    ExactArrays exact;
};
struct RnnGatherParams {
    RnnGatherMatrix m[2];        // LSTM: the gate matrix; GRU: W_i, W_h
    const float *bias, *bias2;
    float *state, *h32;          // LSTM: c and an optional fp32 copy of h; GRU: the state in fp32, null
    void *h;
    int64_t lds, ldh, ldh32;
    int32_t H, N, hdt;
};

// SB: steps a wave has in flight (steps past its last are fetched too: few where a run has few)
template <bool BF16, int CELL, int SB>
__global__ void __launch_bounds__(CELL == 1 ? 1024 : 768) bcr_rnn_gather(RnnGatherParams p) {
    constexpr int GATES = CELL == 1 ? 4 : 3, NRUN = CELL == 1 ? 4 : 6, WPR = CELL == 1 ? 4 : 2, NWV = NRUN * WPR;
    constexpr int DT = BF16 ? GRIM_BF16 : GRIM_F16;
    constexpr int PITCH = 32;                    // bytes of a staged row
    constexpr int WLDS = SB * 1024;              // a step buffer of 32 rows x 16 columns for every step in flight
    __shared__ __attribute__((aligned(16))) char lds[NWV * WLDS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int run = wave / WPR, share = wave % WPR, mi = CELL == 2 ? run / 3 : 0, gate = CELL == 2 ? run % 3 : run;
    const RnnGatherMatrix &A = p.m[mi];
    // (the arguments in one trip through the scalar cache, as in bcr_spmm_gather)
    asm volatile("" ::"s"(A.sptr), "s"(A.rows), "s"(A.desc), "s"(A.payload), "s"(A.strip_pos), "s"(A.X), "s"(A.ldx), "s"(A.usteps), "s"(A.K),
                 "s"(A.BR), "s"(p.H), "s"(p.N), "s"(p.state), "s"(p.lds), "s"(p.bias), "s"(p.bias2));
    const int unit0 = blockIdx.x * 16, n0 = blockIdx.y * 16, N = p.N;
    // stored run of the 16 gate rows from original row `row` on (in one strip, or strips stored in original order)
    auto stored_run = [&](const RnnGatherMatrix &M, int row) {
        if (!M.strip_pos) return row / 16;
        return (M.strip_pos[row / M.BR] * M.BR + row % M.BR) / 16;
    };
    const int t = stored_run(A, gate * p.H + unit0);
    const int g0 = A.usteps ? t * A.usteps : A.sptr[t], nst = A.usteps ? A.usteps : A.sptr[t + 1] - g0;
    const int s_beg = g0 + nst * share / WPR, s_end = g0 + nst * (share + 1) / WPR;

    // the cell's threads: (unit, column); their state and biases are asked for now
    const int cu = tid >> 4, cn = n0 + (tid & 15);
    const bool cell_thread = tid < 256 && cn < N;
    const int64_t unit = unit0 + cu;
    float st = 0.f, bb[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (cell_thread) {
        st = p.state[unit * p.lds + cn];
#pragma unroll
        for (int k = 0; k < GATES; ++k) {
            if (p.bias) bb[k] = p.bias[k * (int64_t)p.H + unit];
            if (CELL == 2 && p.bias2) bb[3 + k] = p.bias2[k * (int64_t)p.H + unit];
        }
    }

    // fetch side: lane = (k slot rs, 16-byte piece c of its row), at any alignment; a piece behind the last element of X
    // is fetched from the last 16 bytes and shifted, one of a column past N from the tile's first (never stored)
    const int rs = lane >> 1, c = lane & 1, col = n0 + c * 8;
    const unsigned short *xcol = A.X + (col < N ? col : n0);
    const unsigned short *x_last = A.X + ((int64_t)(A.K - 1) * A.ldx + N - 8);
    char *buf = lds + wave * WLDS;
    const int i16 = lane & 15, kgroup = lane >> 4, qd = i16 >> 2;
    const unsigned int below = (1u << i16) - 1u;
    const char *tr = buf + (kgroup * 8 + qd) * PITCH + (i16 & 3) * 8;
    const uint2 *desc2 = reinterpret_cast<const uint2 *>(A.desc);
    const i16x8 *pay = reinterpret_cast<const i16x8 *>(A.payload);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s = s_beg; s < s_end; s += SB) {
        const int nb = s_end - s < SB ? s_end - s : SB;
        unsigned int row[SB], flags[SB];         // flags: bit 31: padding slot; below: elements fetched early
        uint2 dsc[SB];
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const int at = s + (u < nb ? u : nb - 1);
            row[u] = A.rows[(int64_t)at * 32 + (rs & 7) * 4 + (rs >> 3)];
            dsc[u] = desc2[(int64_t)at * 4 + kgroup];
        }
        u32x4 rx[SB];
        i16x8 w[SB];
        f32x4 part = {0.f, 0.f, 0.f, 0.f};       // (half a batch is summed apart: see bcr_spmm_gather)
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const bool pad = row[u] == 0xffffffffu;
            const unsigned short *src = xcol + (int64_t)(pad ? 0u : row[u]) * A.ldx;
            const int over = src > x_last ? (int)(src - x_last) : 0;
            flags[u] = (unsigned int)over | (pad ? 0x80000000u : 0u);
            rx[u] = load_piece_any(src - over);
            const bool kept = (dsc[u].x >> i16) & 1u;
            const i16x8 wv = pay[dsc[u].y + (kept ? __builtin_popcount(dsc[u].x & below) : 0)];
            w[u] = kept ? wv : i16x8{0, 0, 0, 0, 0, 0, 0, 0};
        }
        // All steps are parked before the first is multiplied (steps past the last again, and not multiplied): one trip through LDS
        // for all of them, not one after the other
        i16x8 x[SB];
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            u32x4 v = rx[u];
            if (__builtin_amdgcn_ballot_w64((flags[u] & 15u) != 0)) v = drop_elements(v, flags[u] & 15u);    // (the last rows of X only)
            if (flags[u] >> 31) v = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4 *>(buf + u * 1024 + rs * PITCH + c * 16) = v;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const i16x4 lo = lds_tr_read(tr + u * 1024), hi = lds_tr_read(tr + 4 * PITCH + u * 1024);
            x[u] = i16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (u < nb) part = mfma16<BF16>(x[u], w[u], part);
            if (u == SB - 1 || (SB > 4 && u == SB / 2 - 1)) {
                acc[0] += part[0]; acc[1] += part[1]; acc[2] += part[2]; acc[3] += part[3];
                part = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    // lane: gate row lane % 16, columns 4 (lane / 16) .. + 3; the partial tile goes into the wave's own idle buffers
    *reinterpret_cast<f32x4 *>(buf + lane * 16) = acc;
    __syncthreads();
    if (!cell_thread) return;
    const int at = (cu + 16 * ((tid & 15) >> 2)) * 16 + (tid & 3) * 4;
    float sum[6];
#pragma unroll
    for (int j = 0; j < NRUN; ++j) {
        float s = *reinterpret_cast<const float *>(lds + j * WPR * WLDS + at);
#pragma unroll
        for (int w = 1; w < WPR; ++w) s += *reinterpret_cast<const float *>(lds + (j * WPR + w) * WLDS + at);
        const RnnGatherMatrix &M = p.m[CELL == 2 ? j / 3 : 0];
        const int64_t grow = (int64_t)(CELL == 2 ? j % 3 : j) * p.H + unit;
        if (__builtin_fmaf(s, 0.f, 0.f) != 0.f) {      // not finite: is there an infinity or NaN that the row keeps?
            float e[1];
            exact_row<DT, 1>(M.exact, M.X, N, M.ldx, (int64_t)stored_run(M, (int)(grow - cu)) * 16 + cu, cn, e);
            s = e[0];
        }
        M.G[grow * M.ldg + cn] = s;
        sum[j] = s;
    }
    float h;
    if constexpr (CELL == 1) {
        h = lstm_cell_apply(sum[0] + bb[0], sum[1] + bb[1], sum[2] + bb[2], sum[3] + bb[3], st);
        p.state[unit * p.lds + cn] = st;
        if (p.h32) p.h32[unit * p.ldh32 + cn] = h;
    } else {
        h = gru_cell_apply(sum[0] + bb[0], sum[1] + bb[1], sum[2] + bb[2], sum[3] + bb[3], sum[4] + bb[4], sum[5] + bb[5], st);
        p.state[unit * p.lds + cn] = h;
    }
    if (p.h) rnn_store_h(p.h, p.hdt, unit * p.ldh + cn, h);
}

static bool rnn_gather_matrix_ok(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, int64_t H) {
    // the 16 gate rows of 16 units are one run: inside a strip, or across strips that are stored in original order
    return gather_any_applies(A, X, N, ldx) && (A->K - 1) * ldx + N >= 8 && H % 16 == 0 &&
           (A->BR % 16 == 0 ? H % A->BR == 0 : A->order_identity);
}

// A workgroup per compute unit at most: beyond that the products as a launch of their own are quicker (LSTM, 2048 units, 512
// inputs, 64 columns, 512 workgroups: 13.2 us as two launches, 21.1 here).
bool rnn_gather_applies(const grim_bcr_matrix *A, const void *X, int64_t ldx, const grim_bcr_matrix *A2, const void *X2, int64_t ldx2,
                        int64_t H, int32_t batch) {
    if (batch < 1 || batch > 64 || H / 16 * ((batch + 15) / 16) > 256) return false;
    // (an LSTM's long runs on 56 and 64 aligned columns, which the products take as one tile: 1024 units and inputs in 8 x 32
    // blocks, 56 columns 9.7 us as two launches, 10.4 here; 256 units, 1024 inputs, 64 columns 7.1 and 7.5)
    if (!A2 && batch >= 56 && batch % 8 == 0 && ldx % 8 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 &&
        (batch == 64 ? A->K >= 1024 : A->gather.max_steps > 24))
        return false;
    return rnn_gather_matrix_ok(A, X, batch, ldx, H) && (!A2 || (A->dtype == A2->dtype && rnn_gather_matrix_ok(A2, X2, batch, ldx2, H)));
}

// The output vectors must not overlap the inputs (workgroups finish at different times).
grim_status launch_rnn_gather(const grim_bcr_matrix *A, const void *X, int64_t ldx, float *G, int64_t ldg, const grim_bcr_matrix *A2,
                              const void *X2, int64_t ldx2, float *G2, int64_t ldg2, int32_t batch, const RnnCell &cell, hipStream_t stream) {
    auto fill = [](const grim_bcr_matrix *M, const void *x, int64_t ldx_, float *g, int64_t ldg_) {
        return RnnGatherMatrix{M->gather.d_sptr, M->gather.d_rows, M->gather.d_desc, M->gather.d_payload,
                               M->order_identity ? nullptr : M->dev.strip_pos, static_cast<const unsigned short *>(x), g, ldx_, ldg_,
                               M->gather.usteps, (int32_t)M->K, M->BR, exact_arrays(M)};
    };
    RnnGatherParams p;
    p.m[0] = fill(A, X, ldx, G, ldg);
    p.m[1] = A2 ? fill(A2, X2, ldx2, G2, ldg2) : p.m[0];
    p.bias = cell.bias; p.bias2 = cell.bias2;
    p.state = cell.c; p.lds = cell.ldc;
    p.h32 = cell.h32; p.ldh32 = cell.ldh32;
    p.h = cell.h; p.ldh = cell.ldh;
    p.H = cell.H; p.N = batch; p.hdt = cell.hdt;
    const dim3 grid((unsigned)(cell.H / 16), (unsigned)((batch + 15) / 16));
    const int share = (std::max(A->gather.max_steps, A2 ? A2->gather.max_steps : 0) + (A2 ? 1 : 3)) / (A2 ? 2 : 4);     // steps of a wave
#define GRIM_RNN(BF, CE, TH)                                                                                              \
    do {                                                                                                                  \
        if (share <= 2) hipLaunchKernelGGL((bcr_rnn_gather<BF, CE, 2>), grid, dim3(TH), 0, stream, p);                    \
        else if (share <= 3) hipLaunchKernelGGL((bcr_rnn_gather<BF, CE, 3>), grid, dim3(TH), 0, stream, p);               \
        else if (share > 6 && share <= 8) hipLaunchKernelGGL((bcr_rnn_gather<BF, CE, 8>), grid, dim3(TH), 0, stream, p);  \
        else hipLaunchKernelGGL((bcr_rnn_gather<BF, CE, 6>), grid, dim3(TH), 0, stream, p);                               \
    } while (0)
    if (A2) { if (A->dtype == GRIM_BF16) GRIM_RNN(true, 2, 768); else GRIM_RNN(false, 2, 768); }
    else { if (A->dtype == GRIM_BF16) GRIM_RNN(true, 1, 1024); else GRIM_RNN(false, 1, 1024); }
#undef GRIM_RNN
    return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
}

}  // namespace grim
