// Kernel of bcr_spmm_gather.hip as a header: the wide-tile kernel's launcher builds a kernel that runs both.
#pragma once
#include <type_traits>

#include "spmm_exact.hpp"

namespace grim {

// Row-gathering matrix-core SpMM kernel for Y = W_bcr * X (Section 3.1; Section 4.4: the rows of X a block
// keeps are loaded once and reused by all of its kept rows).
// ------------------------------------------------------------------------------------------
// row-gathering matrix-core kernel (fp16 / bf16; block heights that divide 16 or are multiples of
// 16: the rows of the matrix in stored order are cut into runs of 16, "strips" below)
//
// Workgroup = (tile of 64 columns of X, one 16-row strip); its 4 waves split the strip's steps
// (i.e. K) between them and add their partial tiles in a fixed order at the end -- the only
// barrier.  A wave works on its own: it reads the row numbers and block descriptors of a batch
// of steps, then fetches exactly the rows of X those steps multiply (8 lanes per 128-byte row
// piece) and the kept rows of the blocks' weights straight into registers, parks the X rows of
// one step in a private 4 KB LDS buffer in k-slot order, and reads them back with transpose
// reads as MFMA operands.  No producer/consumer hand-over: latency is covered by the four
// workgroups a compute unit holds and by the batch of loads a wave has in flight.
// Unlike the staged kernel a row of X is fetched once per strip that keeps it (not once per
// group of strips), but only kept rows are fetched, and every compute unit has work even when
// the tiles are few.
// ------------------------------------------------------------------------------------------
struct GatherSecond {
    const int32_t *sptr;
    const int32_t *out_row;
    const uint32_t *rows;
    const uint32_t *desc;
    const unsigned char *payload;
    const unsigned short *X;
    float *Y;
    int32_t usteps;
    int32_t K;
    ExactArrays exact;
};

struct GatherParams {
    const int32_t *sptr;
    const int32_t *out_row;   // original row of stored row t * 16 + m, -1 past the matrix
    const uint32_t *rows;
    const uint32_t *desc;
    const unsigned char *payload;
    const unsigned short *X;
    float *Y;
    int64_t N, ldx, ldy;
    int32_t nbr, ntiles;      // nbr: 16-row runs of the stored row order
    int32_t usteps;           // > 0: steps of every run (sptr is not read)
    int32_t K;                // rows of X
    int32_t touch;            // beside the wide-tile kernel: start the tile's rows of X on their way from HBM when the workgroup starts
    XcdMap map;
    ExactArrays exact;
    GatherSecond second;
};


// which form of the kernel a launch takes, and its workgroups
struct GatherForm {
    bool aligned, narrow, solo, eight;
    int nt;                   // sub-tiles of 16 columns per tile
    int steps;                // steps in flight of a 16-column tile on four waves
    int64_t nwg;
};
grim_status gather_setup(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, float *Y, int64_t ldy,
                         const grim_bcr_matrix *A2, const void *X2, float *Y2, GatherParams *out, GatherForm *form,
                         bool alone = true);      // false: workgroups beside the wide-tile kernel's

// four results at any 4-byte alignment (a single access on this GPU)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// What the way to the first row numbers needs of the arguments in one trip through the scalar cache: asked for where each is first
// used, the trips follow one another.  (What narrow tiles need for infinities, and the second of a pair, comes later.)  Not for the
// groups of bcr_spmm_gather_many, whose pointers come out of a table behind the first trip: the whole entry would be waited for where the
// steps are all that is wanted (20 of 2400 x 1664 of mixed rates, one vector each: 9.36 us before, 9.60 so, 9.25 without).
__device__ __forceinline__ void gather_arguments(const GatherParams &p) {
    asm volatile("" ::"s"(p.map.per_tile), "s"(p.map.tail_slot0), "s"(p.map.tail_tile0), "s"(p.map.shift), "s"(p.map.per_part),
                 "s"(p.map.per_tile_inv), "s"(p.map.per_part_inv), "s"(p.ntiles), "s"(p.nbr), "s"(p.usteps), "s"(p.sptr), "s"(p.out_row),
                 "s"(p.rows), "s"(p.desc), "s"(p.payload), "s"(p.X), "s"(p.N), "s"(p.ldx), "s"(p.K));
}

// ALIGNED: rows of X are 16-byte aligned and N a multiple of 8.  Otherwise a piece is still one 16-byte load, at
// whatever alignment its row has: from an 8-byte-aligned row it costs the vector L1 next to nothing more, from a row that
// starts at an odd element about three aligned ones -- against the staged and vector-ALU kernels, which took such
// products element by element before (512 x 4608 in 4 x 16 blocks at 785 columns: 414 -> 25.6 us; in 16 x 32 blocks at 147,
// with small tiles, 66 -> 5.0).
// NARROW: N below the tile's width: one tile, whose pieces past N are fetched from column 0 and never stored.
// NT: 16-column sub-tiles of a tile (4; 2 and 1 for products of at most 32 and 16 columns, whose pieces then take a half
// or a quarter of the load instructions and LDS traffic of a padded 64-column tile; 2 also for long strips and few tiles).
// SOLO: strips of a few steps only (a 3 x 3 layer of 64 channels has 5, a dense first layer 1) -- every wave takes a
// (tile, strip) of its own, four consecutive strips per workgroup: no split of K, no partial tiles, no barrier
// EIGHT: eight waves split a strip's steps instead of four (few workgroups, long strips: the 14 x 14 layers)
// The body of the kernel as a function of the workgroup's number (block_x; block_y: second product of a pair), so that
// another kernel can run such workgroups next to its own (the wide-tile kernel does, for the columns it leaves over).
// Its first NWV waves must call it together; `lds` = NWV * gather_wave_lds(..) bytes of workgroup memory.
// LONGW: the waves that split a strip in the EIGHT form (eight in the kernel of its own; a caller with more waves to
// spare may pass more: fewer steps per wave, fewer dependent batches).
constexpr int gather_narrow_steps(int nt) { return nt == 1 ? 8 : 4; }
constexpr int gather_steps(bool aligned, bool narrow, bool eight, int nt, int steps) {
    return steps ? steps : narrow ? gather_narrow_steps(nt) : nt == 2 || (!aligned && !eight) ? 3 : 4;
}
// Step buffers of a wave, 32 rows x 16 nt columns each: two, or one for every step in flight on small tiles (NT = 2, twelve
// waves), which are all latency: three steps through LDS in one trip, 512 x 4608 at 64 / 147 / 196 / 256 columns 4.14 / 4.85 / 5.04 / 4.27
// -> 4.09 / 4.70 / 4.80 / 4.11 us.  (Below 64 columns 4.25 -> 4.1 at 32 and 9.0 -> 9.2 at 17: not there.)
constexpr int gather_buffers(bool narrow, int nt, int steps) { return nt == 2 && !narrow ? steps : 2; }
constexpr int gather_wave_lds(int nt, int buffers = 2) { return buffers * nt * 1024; }
// STEPS: steps a wave has in flight, where the form has a choice (0: as its registers allow).
// COLS: 0, or the columns there are (1 .. 4; NARROW, NT = 1): of a row of X just their bytes are fetched then.
template <bool BF16, bool ALIGNED, bool NARROW, bool SOLO, bool EIGHT, int NT = 4, int LONGW = kGatherLongWaves, int STEPS = 0, int COLS = 0>
__device__ __forceinline__ void gather_body(const GatherParams &p, char *lds, int block_x, int block_y) {
    constexpr int NWV = EIGHT ? LONGW : 4;                     // waves of the workgroup
    constexpr int TN = NT * 16, PITCH = TN * 2, CPR = 2 * NT;  // columns, bytes and 16-byte pieces of a staged row
    constexpr int RPI = 64 / CPR, LI = 32 / RPI;               // rows per load instruction, load instructions per step
    // forms of operands that other kernels used to take, which multiply kept weights only: an infinity or NaN in X must
    // not reach the rows of the run that do not keep its column
    constexpr bool WATCH = NARROW || !ALIGNED;
    constexpr int SB = gather_steps(ALIGNED, NARROW, EIGHT, NT, STEPS);
    constexpr int WLDS = gather_wave_lds(NT, gather_buffers(NARROW, NT, SB));
    constexpr bool kTouch = !NARROW && NT == 4 && EIGHT && LONGW > kGatherLongWaves;      // (the wide-tile kernel's)
    constexpr bool ALL = gather_buffers(NARROW, NT, SB) > 2;           // a batch is parked as a whole
    static_assert(NT == 1 || NT == 2 || NT == 4, "pieces of a row are dealt to 2, 4 or 8 lanes");
    // workgroup -> (tile, stored strip, or four of them for SOLO)
    const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, unit;
    if (!xcd_map_at(p.map, block_x, p.ntiles, &tile, &unit)) return;
    const int t = SOLO ? unit * 4 + wave0 : unit;
    if (t >= p.nbr) return;                                           // (SOLO has no barrier a wave could be missed at)
    // the matrix and operands of this workgroup: grid.y = 1 selects the second product of a two-product launch
    const int32_t *sptr = p.sptr, *out_row = p.out_row;
    const uint32_t *rows = p.rows, *desc = p.desc;
    const unsigned char *payload = p.payload;
    const unsigned short *X = p.X;
    float *Y = p.Y;
    int usteps = p.usteps;
    int K = p.K;
    const ExactArrays *exact = &p.exact;
    if constexpr (NARROW) {
        if (block_y) {
            exact = &p.second.exact;
            sptr = p.second.sptr; out_row = p.second.out_row; rows = p.second.rows; desc = p.second.desc;
            payload = p.second.payload; X = p.second.X; Y = p.second.Y; usteps = p.second.usteps; K = p.second.K;
        }
    }
    int64_t n0 = (int64_t)tile * TN;
    if (!NARROW && n0 + TN > p.N) n0 = p.N - TN;     // ragged last tile: overlap the neighbour

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Beside the wide-tile kernel, whose stream of X and Y keeps pushing lines out of L2: a wave learns which rows of X it needs
    // only after a first round trip (row numbers), and fetches them in one or two batches: up to three dependent trips to
    // memory.  The strips of a tile run at the same time on one XCD and together keep nearly every row of the tile (16 strips
    // keeping a quarter each leave 1 % out), so each workgroup starts its share of ALL the tile's rows on their way into that
    // XCD's L2 right now -- one byte from the first and the last 128-byte line of every row piece, values never used -- and the
    // fetches proper find them there or on their way.  Alone on the GPU the same requests are only in the way of the first
    // fetches: few strips to a tile make many requests of each workgroup (bf16 / f16, 4608 rows of X: 512 x 784 / 785 columns
    // 18.0 / 20.2 with -> 16.7 / 19.0 us, 128 x 784 9.15 -> 7.68, 64 x 6272 / 12 543 21.9 / 73.2 -> 14.9 / 40.1; 16 384 rows,
    // 256 x 784 20.6 -> 15.9; nothing was faster with them).
    if constexpr (kTouch) {
        if (p.touch) {
            const int units = p.map.per_tile;                          // workgroups of this tile
            const int per = (K + units - 1) / units;
            const int r_end = (unit + 1) * per < K ? (unit + 1) * per : K;
            const char *base = reinterpret_cast<const char *>(X + n0) + (tid & 1) * (TN * 2 - 1);
            for (int r = unit * per + (tid >> 1); r < r_end; r += NWV * 32)
                (void)*reinterpret_cast<const volatile unsigned char *>(base + (int64_t)r * p.ldx * 2);
        }
    }
    // one dependent memory round trip less at the start when every run has the same number of steps
    const int g0 = usteps ? t * usteps : sptr[t], nst = usteps ? usteps : sptr[t + 1] - g0;
    const int s_beg = SOLO ? g0 : g0 + wave_share(nst, wave, NWV);
    const int s_end = SOLO ? g0 + nst : g0 + wave_share(nst, wave + 1, NWV);
    char *buf = lds + wave * WLDS;

    // fetch side: lane = (row slot rs, 16-byte piece c); its i-th load is k slot i * RPI + rs
    const int rs = lane / CPR, c = lane % CPR;
    const bool in_n = !NARROW || c * 8 < p.N;
    const unsigned short *xcol = X + n0 + (in_n ? c * 8 : 0);
    // NARROW: pieces may reach past the last element of X (row K - 1, columns from N on): such a piece is fetched from
    // `x_last`, the last 16 bytes of X, and shifted into place when it is parked -- a branch around the load instead cost
    // the other loads their overlap (4096 x 4096 at 5 columns: 7.9 us)
    const unsigned short *x_last = X + ((int64_t)(K - 1) * p.ldx + p.N - 8);
    // (the swizzle is the same for the rows of all load instructions: RPI is a multiple of its period)
    const int wr_off = rs * PITCH + ((c ^ (CPR == 2 ? 0 : swizzle<CPR>(rs))) << 4);
    // multiply side: lane = (output row m_row, k group); the two transpose reads of a sub-tile
    // name k slots kgroup * 8 + qd and + 4
    const int i16 = lane & 15, kgroup = lane >> 4, qd = i16 >> 2, m_row = i16;
    const unsigned int below = (1u << m_row) - 1u;
    const int ncolb = (4 * (i16 & 3)) * 2, cl = ncolb >> 4, within = ncolb & 15;
    // The first read of sub-tile q: row r0, 16-byte chunk (2 q + cl) ^ swizzle.  The second is row r0 + 4, whose swizzle
    // differs from row r0's by 4 (8 chunks per row) or not at all: the address of the first read of sub-tile q ^ 2 or
    // of q itself, plus four rows -- a constant, so that the reads take NT address registers and no arithmetic.
    const int r0 = kgroup * 8 + qd;
    const int sw0 = CPR == 2 ? 0 : swizzle<CPR>(r0);
    const char *tr[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) tr[q] = buf + r0 * PITCH + within + (((q * 2 + cl) ^ sw0) << 4);

    f32x4 acc[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int orow = out_row[(int64_t)t * 16 + (lane & 15)];     // asked for now, needed at the very end

    const uint2 *desc2 = reinterpret_cast<const uint2 *>(desc);
    const i16x8 *pay = reinterpret_cast<const i16x8 *>(payload);
    // the row numbers of the lane's k slots of a step: slot s sits at position (s % 8) * 4 + s / 8
    typedef unsigned int Hdr __attribute__((ext_vector_type(LI)));
    auto ask_hdr = [&](int st) {
        Hdr h;
        if constexpr (NT == 4) {
            h = reinterpret_cast<const Hdr *>(rows)[(int64_t)st * 8 + rs];
        } else {
#pragma unroll
            for (int i = 0; i < LI; ++i) h[i] = rows[(int64_t)st * 32 + (rs & 7) * 4 + (rs >> 3) + 2 * i];
        }
        return h;
    };
    // Row numbers and descriptor of the first step of the next batch are asked for together with
    // the current batch's, so that a wave whose steps do not fit one batch (18 steps over 4 waves:
    // 4 + 1) starts the rows of X of the next batch without another dependent round trip.
    Hdr nhdr = 0u;
    uint2 ndsc = {0u, 0u};
    if (s_beg < s_end) {
        nhdr = ask_hdr(s_beg);
        ndsc = desc2[(int64_t)s_beg * 4 + kgroup];
    }
    // The rows of X of a step (pad: bit i set = the lane's i-th k slot is padding and multiplies zeros; kept instead of
    // the row numbers; bits 8 + 4 i: elements its piece was fetched early) and its weights, asked for into a register set
    struct StepRows { u32x4 rx[LI]; unsigned int pad; };
    auto ask_rows = [&](StepRows &r, const Hdr &h) {
        r.pad = 0u;
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            r.pad |= h[i] == 0xffffffffu ? 1u << i : 0u;
            const unsigned int row = h[i] == 0xffffffffu ? 0u : h[i];
            const unsigned short *src = xcol + (int64_t)row * p.ldx;
            if constexpr (ALIGNED) {
                r.rx[i] = *reinterpret_cast<const u32x4 *>(src);
            } else if constexpr (COLS > 0) {     // (n0 = 0; both lanes of a row fetch it, columns from COLS on are never stored)
                static_assert(NARROW && NT == 1 && COLS <= 4, "whole rows of a 16-column tile");
                struct __attribute__((packed, aligned(2))) { unsigned short e[COLS]; } v;
                unsigned int d[2] = {0u, 0u};
                __builtin_memcpy(&v, X + (int64_t)row * p.ldx, sizeof(v));
                __builtin_memcpy(d, &v, sizeof(v));
                r.rx[i] = u32x4{d[0], d[1], 0u, 0u};
            } else if constexpr (NARROW) {
                const int over = src > x_last ? (int)(src - x_last) : 0;      // elements, below 8
                r.pad |= (unsigned int)over << (8 + 4 * i);
                r.rx[i] = load_piece_any(src - over);
            } else {
                r.rx[i] = load_piece_any(src);
            }
        }
    };
    auto ask_weights = [&](const uint2 &d) {
        const bool kept = (d.x >> m_row) & 1u;
        const unsigned int idx = d.y + (kept ? __builtin_popcount(d.x & below) : 0);
        const i16x8 wv = pay[idx];               // a group's first row if it does not have this lane's (zeroed below)
        return kept ? wv : i16x8{0, 0, 0, 0, 0, 0, 0, 0};
    };
    // A batch: SB steps in flight.  The rows of the first step of the NEXT batch are asked for as soon as this batch's
    // first step has left its registers -- its row numbers came with this batch's -- so that a wave with one step more
    // than a batch holds (18 steps over 4 waves: 4 + 1) does not pay a whole further round trip for it: the request
    // travels while the rest of this batch arrives (FIRST: the batch that finds nothing asked for yet).  (With the
    // request made unconditional in a copy of the batch for "another batch follows", so that every wait counts exactly
    // the younger loads, the compiler needs 158 registers for what takes 128 here: not done.)
    StepRows early;
    auto batch = [&](int s, auto first_tag) {
        constexpr bool FIRST = decltype(first_tag)::value;
        const int nb = s_end - s < SB ? s_end - s : SB;
        Hdr hdr[SB];
        uint2 dsc[SB];
        hdr[0] = nhdr;
        dsc[0] = ndsc;
#pragma unroll
        for (int u = 1; u < SB; ++u) {
            const int st = s + (u < nb ? u : nb - 1);
            hdr[u] = ask_hdr(st);
            dsc[u] = desc2[(int64_t)st * 4 + kgroup];
        }
        {
            const int st = s + SB < s_end ? s + SB : s_end - 1;
            nhdr = ask_hdr(st);
            ndsc = desc2[(int64_t)st * 4 + kgroup];
        }
        // WATCH forms took over from kernels with sixteen partial sums: a batch's steps (half of eight) are summed from
        // zero and then added, which keeps their errors (512 x 4608 in 4 x 16 blocks, 25 steps to a wave: 1.26e-7 in one chain, 0.98e-7 before)
        f32x4 part[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) part[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        StepRows R[SB];
        i16x8 PW[SB];
        if constexpr (!FIRST) R[0] = early;      // asked for during the batch before
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (FIRST || u > 0) ask_rows(R[u], hdr[u]);
            PW[u] = ask_weights(dsc[u]);
        }
        auto park = [&](int u) {
            char *b = buf + (ALL ? u : u & 1) * (32 * PITCH);
            if constexpr (NARROW && !ALIGNED && COLS == 0) {
                if (__builtin_amdgcn_ballot_w64(R[u].pad >> 8 != 0)) {       // (the last rows of X only)
#pragma unroll
                    for (int i = 0; i < LI; ++i) R[u].rx[i] = drop_elements(R[u].rx[i], (R[u].pad >> (8 + 4 * i)) & 15u);
                }
            }
#pragma unroll
            for (int i = 0; i < LI; ++i) {
                const u32x4 v = (R[u].pad >> i) & 1u ? u32x4{0u, 0u, 0u, 0u} : R[u].rx[i];
                *reinterpret_cast<u32x4 *>(b + wr_off + i * (RPI * PITCH)) = v;
            }
        };
        auto gathered = [&](int u, i16x8 (&x)[NT]) {
            const int at = (ALL ? u : u & 1) * (32 * PITCH);
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                const i16x4 lo = lds_tr_read(tr[q] + at);
                const i16x4 hi = lds_tr_read(tr[NT == 4 ? q ^ 2 : q] + 4 * PITCH + at);
                x[q] = i16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
        };
        auto multiply = [&](int u, const i16x8 (&x)[NT]) {
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                if constexpr (WATCH) part[q] = mfma16<BF16>(x[q], PW[u], part[q]);
                else acc[q] = mfma16<BF16>(x[q], PW[u], acc[q]);
            }
        };
        i16x8 xs[ALL ? SB : 1][NT];
        if constexpr (ALL) {
            // (steps past the wave's last are parked and read again and not multiplied)
#pragma unroll
            for (int u = 0; u < SB; ++u) park(u);
            __builtin_amdgcn_wave_barrier();
            if (s + SB < s_end) ask_rows(early, nhdr);
#pragma unroll
            for (int u = 0; u < SB; ++u) gathered(u, xs[u]);
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (u < nb) {
                if constexpr (ALL) {
                    multiply(u, xs[u]);
                } else {
                    park(u);
                    __builtin_amdgcn_wave_barrier();
                    if (u == 0 && s + SB < s_end) ask_rows(early, nhdr);   // set 0's rows are out of their registers
                    gathered(u, xs[0]);
                    multiply(u, xs[0]);
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (WATCH && (u == SB - 1 || (SB > 4 && u == SB / 2 - 1))) {
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    acc[q][0] += part[q][0]; acc[q][1] += part[q][1]; acc[q][2] += part[q][2]; acc[q][3] += part[q][3];
                    part[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
    };
    if (s_beg < s_end) batch(s_beg, std::true_type{});
    for (int s = s_beg + SB; s < s_end; s += SB) batch(s, std::false_type{});

    // D[n][m] of sub-tile q: lane holds m = lane % 16, n = 4 * (lane / 16) + 0..3
    auto put = [&](int q, const f32x4 &v) {
        const int64_t row = orow;
        const int64_t n = n0 + q * 16 + 4 * (lane >> 4);
        if (row < 0 || (NARROW && n >= p.N)) return;
        float *dst = Y + row * p.ldy + n;
        if (!NARROW || n + 4 <= p.N) {
            *reinterpret_cast<f32x4_any *>(dst) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (n + e < p.N) dst[e] = v[e];
        }
    };
    auto put_exact = [&](int q) {
        const int64_t n = n0 + q * 16 + 4 * (lane >> 4);
        if (orow < 0 || n >= p.N) return;
        float v[4];
        exact_row<BF16 ? GRIM_BF16 : GRIM_F16, 4>(*exact, X, p.N, p.ldx, (int64_t)t * 16 + (lane & 15), n, v);
        put(q, f32x4{v[0], v[1], v[2], v[3]});
    };
    // WATCH: has the lane a sum that is not finite in a column below N?  (An infinity or NaN among the rows of X a run keeps
    // makes the sums of all 16 rows so, whether they keep it or not: no other lane needs a look.)
    auto odd = [&](int q, const f32x4 &v) {
        const int64_t n = n0 + q * 16 + 4 * (lane >> 4);
        float z = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) z = __builtin_fmaf(!NARROW || n + e < p.N ? v[e] : 0.f, 0.f, z);
        return z != z;
    };
    if constexpr (SOLO) {
        // the wave owns the whole 16-row tile
        unsigned int again = 0u;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            put(q, acc[q]);
            if (WATCH && odd(q, acc[q])) again |= 1u << q;
        }
        if (WATCH && __builtin_amdgcn_ballot_w64(again != 0u)) {
#pragma unroll 1
            for (int q = 0; q < NT; ++q)
                if ((again >> q) & 1u) put_exact(q);
        }
        return;
    }
    // add the waves' partial tiles in wave order; wave q finishes sub-tile q.  A wave parks its
    // partial tile in its own (now idle) step buffers.
    constexpr int RPW = WLDS / 16;
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
    for (int q = 0; q < NT; ++q) red[wave * RPW + q * 64 + lane] = acc[q];
    __syncthreads();
    if (wave >= NT) return;                      // the first waves finish the sub-tiles
    const int q = wave;
    // (the small-tile form's twelve: three sums of four, so that more partial tiles do not mean a longer chain of roundings)
    constexpr int CHAIN = NT == 2 && !NARROW ? 4 : NWV;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < NWV; g += CHAIN) {
        f32x4 s = red[g * RPW + q * 64 + lane];
#pragma unroll
        for (int w = g + 1; w < g + CHAIN; ++w) {
            const f32x4 v = red[w * RPW + q * 64 + lane];
            s[0] += v[0]; s[1] += v[1]; s[2] += v[2]; s[3] += v[3];
        }
        if (g == 0) sum = s;
        else { sum[0] += s[0]; sum[1] += s[1]; sum[2] += s[2]; sum[3] += s[3]; }
    }
    put(q, sum);
    if (WATCH && odd(q, sum)) put_exact(q);
}

constexpr int gather_waves(bool narrow, bool eight, int nt) { return !eight ? 4 : nt == 2 && !narrow ? kGatherSmallTileWaves : kGatherLongWaves; }
template <bool BF16, bool ALIGNED, bool NARROW, bool SOLO, bool EIGHT, int NT, int STEPS = 0>
__global__ void __launch_bounds__((gather_waves(NARROW, EIGHT, NT) * 64), (EIGHT ? 2 : NARROW ? 2 : 4)) bcr_spmm_gather(GatherParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    gather_arguments(p);
    gather_body<BF16, ALIGNED, NARROW, SOLO, EIGHT, NT, gather_waves(NARROW, EIGHT, NT), STEPS>(p, lds, blockIdx.x, blockIdx.y);
}

}  // namespace grim
