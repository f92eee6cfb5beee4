// Row-gathering SpMM kernel for fp32: Y = W_bcr * X (Section 3.1; Section 4.4: the rows of X a block keeps are loaded once
// and reused by all of its kept rows) on v_mfma_f32_16x16x4_f32, whose products and sums are fp32 multiply-adds.
#include <algorithm>

#include "spmm_exact.hpp"

namespace grim {

// Workgroup = (tile of 16 NT columns of X, one 16-row run of the stored row order); its waves split the run's steps (K)
// and add their partial tiles in wave order at the end.  SOLO: a (tile, run) per wave, four consecutive runs per
// workgroup, no split and no barrier.
//
// A step is 16 k slots, four groups of four.  Lane (i = lane % 16, kg = lane / 16) fetches the NT consecutive columns
// n0 + NT i .. of the four rows of X behind group kg, and output row i's four weights of that group.  Multiply s of the step
// takes element s of every group: its operands are then whole registers as loaded -- sub-tile q is component q of the
// lanes' pieces, the columns NT i + q -- so X passes neither through LDS nor through a shuffle, and a row piece is one
// 16-byte load per lane, 256 contiguous bytes per row.  Columns being the rows of the MFMA result, a lane ends with the
// columns 4 NT kg + NT r + q (r, q < 4, NT) of one output row: contiguous.
//
// Bound: rows of X through L2 and the vector L1 (each run fetches the rows it keeps: 58 MB where X is 14 MB, 256 x 1152 in
// 16 x 32 blocks at 3136 columns), then MFMA, 32 cycles each, 16 a step: 2.9 us there.  That product takes 11.6 us, on the
// vector ALUs 46.9; 512 x 4608 of mixed rates at 777 columns 25.6 against 130, 64 x 288 in 4 x 16 blocks at 20000 columns
// 17.6 against 106, 256 x 256 at 64 columns 3.3 against 4.8.
struct Gather32Params {
    const int32_t *sptr;
    const int32_t *out_row;
    const uint32_t *rows;     // per step 16 rows of X, group by group (0xffffffff: padding)
    const uint32_t *desc;     // per step and group (row mask, place of its weights in 16-byte units)
    const float *payload;
    const float *X;
    float *Y;
    int64_t N, ldx, ldy;
    int32_t nbr, ntiles, usteps, K;
    XcdMap map;
    ExactArrays exact;
};

template <int NT> struct Piece32;
template <> struct Piece32<4> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Piece32<2> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Piece32<1> { typedef float type __attribute__((ext_vector_type(1), aligned(4))); };

template <int NT, bool NARROW, bool SOLO, int NWV>
__global__ void __launch_bounds__(NWV * 64, 4) bcr_spmm_gather32(Gather32Params p) {
    constexpr int TN = 16 * NT;
    constexpr int SB = NT == 4 ? 3 : 4;          // steps a wave has in flight (four of 16 X registers each spill)
    using Piece = typename Piece32<NT>::type;
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ f32x4 red[SOLO ? 1 : NWV * NT * 64];
    __shared__ int odd_values[NWV];              // per wave: it met an infinity or NaN
    // (the arguments in one trip through the scalar cache, as in bcr_spmm_gather)
    asm volatile("" ::"s"(p.map.per_tile), "s"(p.map.tail_slot0), "s"(p.map.tail_tile0), "s"(p.map.shift), "s"(p.map.per_part),
                 "s"(p.map.per_tile_inv), "s"(p.map.per_part_inv), "s"(p.ntiles), "s"(p.nbr), "s"(p.usteps), "s"(p.sptr), "s"(p.out_row),
                 "s"(p.rows), "s"(p.desc), "s"(p.payload), "s"(p.X), "s"(p.N), "s"(p.ldx), "s"(p.K));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile, unit;
    if (!xcd_map_at(p.map, blockIdx.x, p.ntiles, &tile, &unit)) return;
    const int t = SOLO ? unit * NWV + wave : unit;
    if (t >= p.nbr) return;                      // (SOLO has no barrier a wave could be missed at)
    int64_t n0 = (int64_t)tile * TN;
    if (!NARROW && n0 + TN > p.N) n0 = p.N - TN;   // ragged last tile: overlap the neighbour (same sums, same bits)
    const int g0 = p.usteps ? t * p.usteps : p.sptr[t], nst = p.usteps ? p.usteps : p.sptr[t + 1] - g0;
    const int s_beg = SOLO ? g0 : g0 + wave_share(nst, wave, NWV);
    const int s_end = SOLO ? g0 + nst : g0 + wave_share(nst, wave + 1, NWV);

    const int i16 = lane & 15, kg = lane >> 4;
    const unsigned int below = (1u << i16) - 1u;
    const int orow = p.out_row[(int64_t)t * 16 + i16];
    // NARROW: a lane whose piece lies past column N takes column 0 (never stored); columns past N inside a piece belong
    // to the next row of X, except behind its last element
    const int col = i16 * NT, valid = NARROW ? (col < p.N ? (int)p.N - col : NT) : NT;
    const float *x_last = p.X + (int64_t)(p.K - 1) * p.ldx + p.N - NT;
    const float *xcol = p.X + n0 + (NARROW && col >= p.N ? 0 : col);
    const uint2 *desc2 = reinterpret_cast<const uint2 *>(p.desc);
    const u32x4 *rows4 = reinterpret_cast<const u32x4 *>(p.rows);
    const f32x4 *pay = reinterpret_cast<const f32x4 *>(p.payload);

    f32x4 acc[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bad = 0.f;                             // NaN once a fetched value was infinite or NaN
    u32x4 hdr[SB];
    uint2 dsc[SB];
    auto ask_headers = [&](int s) {              // (past the last step: the last one again, not multiplied)
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const int st = s + u < s_end ? s + u : s_end - 1;
            hdr[u] = rows4[(int64_t)st * 4 + kg];
            dsc[u] = desc2[(int64_t)st * 4 + kg];
        }
    };
    // Long runs: every eight batches the sums so far are added to the wave's part of `red`, for no longer chain of additions than
    // the vector ALUs' (64 x 16384, 1024 steps over eight waves: 2.1e-7 in one chain, 1.45e-7 there).
    int batches = 0;
    bool folded = false;
    auto fold = [&]() {
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            f32x4 &r = red[(wave * NT + q) * 64 + lane];
            if (folded) { acc[q][0] += r[0]; acc[q][1] += r[1]; acc[q][2] += r[2]; acc[q][3] += r[3]; }
            r = acc[q];
            acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        folded = true;
    };
    if (s_beg < s_end) ask_headers(s_beg);
    for (int s = s_beg; s < s_end; s += SB) {
        if constexpr (!SOLO)
            if (batches++ == 8) { fold(); batches = 1; }
        Piece rx[SB][4];
        f32x4 w[SB];
        unsigned int shifts = 0u;                // 2 bits per piece
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (u == 0 || s + u < s_end) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // (a padding slot has zero weights in every row: any row of X will do)
                    const unsigned int row = hdr[u][j] == 0xffffffffu ? 0u : hdr[u][j];
                    const float *src = xcol + (int64_t)row * p.ldx;
                    // (a piece that reaches past the last element of X is fetched from there back and shifted below)
                    const int over = NARROW && NT > 1 && src > x_last ? (int)(src - x_last) : 0;
                    if constexpr (NARROW && NT > 1) shifts |= (unsigned int)over << (2 * (u * 4 + j));
                    rx[u][j] = *reinterpret_cast<const Piece *>(src - over);
                }
                const bool kept = (dsc[u].x >> i16) & 1u;
                const f32x4 wv = pay[dsc[u].y + (kept ? __builtin_popcount(dsc[u].x & below) : 0)];
                w[u] = kept ? wv : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        if (s + SB < s_end) ask_headers(s + SB);
        if constexpr (NARROW && NT > 1) {
            if (__builtin_amdgcn_ballot_w64(shifts != 0u)) {                 // (the last row of X only)
#pragma unroll
                for (int u = 0; u < SB; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int over = (shifts >> (2 * (u * 4 + j))) & 3u;
                        const Piece f = rx[u][j];
#pragma unroll
                        for (int e = 0; e < NT; ++e) {
                            float v = f[e];
#pragma unroll
                            for (int o = 1; o < NT; ++o) v = over == o ? (e + o < NT ? f[e + o < NT ? e + o : e] : 0.f) : v;
                            rx[u][j][e] = v;
                        }
                    }
            }
        }
        // A step's sixteen terms are summed from zero and then added: a run of hundreds of terms in one chain of fp32
        // additions would be less exact than the vector-ALU kernel's sixteen partial sums (512 x 4608 in 16 x 32 blocks, a
        // wave per run: relative error 3.1e-7 in one chain).
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (u == 0 || s + u < s_end) {
                f32x4 part[NT];
#pragma unroll
                for (int q = 0; q < NT; ++q) part[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
#pragma unroll
                    for (int q = 0; q < NT; ++q) {
                        bad = __builtin_fmaf(NARROW && q >= valid ? 0.f : rx[u][j][q], 0.f, bad);
                        part[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(rx[u][j][q], w[u][j], part[q], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int q = 0; q < NT; ++q) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[q][r] += part[q][r];
                }
            }
        }
    }

    // piece r of the lane: columns 4 NT kg + NT r + 0 .. NT - 1 of output row i16
    auto put = [&](int r, const float (&v)[NT]) {
        const int64_t n = n0 + 4 * NT * kg + NT * r;
        if (orow < 0 || (NARROW && n >= p.N)) return;
        float *dst = p.Y + (int64_t)orow * p.ldy + n;
        if (!NARROW || n + NT <= p.N) {
            Piece o;
#pragma unroll
            for (int q = 0; q < NT; ++q) o[q] = v[q];
            *reinterpret_cast<Piece *>(dst) = o;
        } else {
#pragma unroll
            for (int q = 0; q < NT; ++q)
                if (n + q < p.N) dst[q] = v[q];
        }
    };
    auto put_exact = [&](int r) {
        const int64_t n = n0 + 4 * NT * kg + NT * r;
        if (orow < 0 || (NARROW && n >= p.N)) return;
        float v[NT];
        exact_row<GRIM_F32, NT>(p.exact, p.X, p.N, p.ldx, (int64_t)t * 16 + i16, n, v);
        put(r, v);
    };
    const bool met = __builtin_amdgcn_ballot_w64(bad != bad) != 0;
    if constexpr (SOLO) {
        if (met) {
#pragma unroll 1
            for (int r = 0; r < 4; ++r) put_exact(r);
            return;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float v[NT];
#pragma unroll
            for (int q = 0; q < NT; ++q) v[q] = acc[q][r];
            put(r, v);
        }
        return;
    }
    fold();
    if (lane == 0) odd_values[wave] = met;
    __syncthreads();
    if (wave >= 4) return;                       // wave r finishes piece r of every lane
    int any = 0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) any |= odd_values[w];
    if (__builtin_amdgcn_readfirstlane(any)) {
        put_exact(wave);
        return;
    }
    const float *redf = reinterpret_cast<const float *>(red);
    float v[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) v[q] = redf[(q * 64 + lane) * 4 + wave];
#pragma unroll
    for (int w = 1; w < NWV; ++w)
#pragma unroll
        for (int q = 0; q < NT; ++q) v[q] += redf[((w * NT + q) * 64 + lane) * 4 + wave];
    put(wave, v);
}

bool gather32_applies(const grim_bcr_matrix *A, const void *X) {
    return A->gather32.present && reinterpret_cast<uintptr_t>(X) % 4 == 0;
}

// Is this kernel the quicker one for N > 8 columns?  A run of blocks of a few rows has a group of four k slots per strip and
// block, of whose sixteen rows few hold anything: its workgroup then takes longer than the workgroups of its strips on the
// vector ALUs do side by side, until there are enough of those to fill the GPU.  Both times in us, by what they grew with
// over 280 products of 1 to 64 rows to a block, 32 x 65536 to 4096 x 512 at 9 to 25088 columns: here a run's steps, one after
// the other (0.05, 0.075 and 0.105 each at up to 16, 32 and 64 columns, 0.128 on unaligned rows of less than 64); there the
// blocks of a strip that a wave walks, each a chain of fetches that eight kept columns share.  (256 x 1152 in 2 x 32 blocks
// keeping 1 x 8, 64 columns: 10.5 us there, 19.5 here; 1024 x 1024 in 2 x 16 blocks at 64: 27.7, 18.3.)
bool gather32_quicker(const grim_bcr_matrix *A, int64_t N) {
    const GatherLayout &L = A->gather32;
    const int nt = N > 32 ? 4 : N > 16 ? 2 : 1, waves = A->BR <= 16 ? 16 : A->BR <= 32 ? 8 : 4;
    const double tiles = (double)((N + nt * 16 - 1) / (nt * 16)), rounds = std::max(1.0, (double)A->nbr * ((N + 63) / 64) / 256);
    const double step = nt == 4 ? (N < 64 ? 0.128 : 0.105) : nt == 2 ? 0.075 : 0.05;
    const double here = 4 + step * std::max((double)L.max_steps, (double)L.nsteps * tiles / 256);
    const double kept = (double)A->col_idx.size() / (double)A->nb, block = kept < 8 ? 1.6 + 0.16 * kept : 2.9 * kept / 8;
    const double there = 3 + block * (double)((A->nbc + waves - 1) / waves) * rounds;
    return here * 1.05 <= there;
}

grim_status launch_spmm_gather32(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, float *Y, int64_t ldy, hipStream_t stream) {
    const GatherLayout &L = A->gather32;
    if (!gather32_applies(A, X)) return GRIM_ERR_UNSUPPORTED;
    Gather32Params p{L.d_sptr, L.d_out_row, L.d_rows, L.d_desc, reinterpret_cast<const float *>(L.d_payload),
                     static_cast<const float *>(X), Y, N, ldx, ldy, (int32_t)L.nstrips, 0, L.usteps, (int32_t)A->K, {}, exact_arrays(A)};
    const int nt = N > 32 ? 4 : N > 16 ? 2 : 1;
    const bool narrow = N < 64;
    p.ntiles = (int32_t)((N + nt * 16 - 1) / (nt * 16));
    const int64_t pairs = (int64_t)p.ntiles * p.nbr;
    // A run per wave: no exchange of partial tiles, but one chain of additions a step long each, so only for runs of few
    // steps (512 x 4608 at 25088 columns, 72 steps: relative error 1.5e-7 in one chain, 1.0e-7 on the vector ALUs).  Eight
    // waves: few runs, or steps in plenty.
    const bool solo = !narrow && L.max_steps <= 18 && pairs >= (L.max_steps <= 8 ? 1024 : 4096);
    const bool eight = !solo && ((L.max_steps >= 16 && pairs <= 512) || L.max_steps > 72);
    const int64_t per_tile = solo ? (p.nbr + 3) / 4 : p.nbr;
    if (((int64_t)p.ntiles + 7) / 8 * 8 * per_tile > 0x7fffffff) return GRIM_ERR_SHAPE;
    int64_t nwg = 0;
    p.map = xcd_map(p.ntiles, per_tile, &nwg);
    if (nwg > 0x7fffffff) return GRIM_ERR_SHAPE;
#define GRIM_G32(NT, NA, SO, NW) hipLaunchKernelGGL((bcr_spmm_gather32<NT, NA, SO, NW>), dim3((unsigned)nwg), dim3(NW * 64), 0, stream, p)
    if (nt == 1) { if (eight) GRIM_G32(1, true, false, 8); else GRIM_G32(1, true, false, 4); }
    else if (nt == 2) { if (eight) GRIM_G32(2, true, false, 8); else GRIM_G32(2, true, false, 4); }
    else if (narrow) { if (eight) GRIM_G32(4, true, false, 8); else GRIM_G32(4, true, false, 4); }
    else if (solo) GRIM_G32(4, false, true, 4);
    else if (eight) GRIM_G32(4, false, false, 8);
    else GRIM_G32(4, false, false, 4);
#undef GRIM_G32
    return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
}

}  // namespace grim
