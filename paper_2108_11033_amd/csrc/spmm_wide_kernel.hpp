// The wide-tile staged kernel (see bcr_spmm_wide.hip for the design): one template for the product on a matrix X in
// memory and for the convolution whose im2col matrix is never formed (CONV: the fetching waves build the rows of
// that matrix in LDS straight from the feature maps; everything after the fetch is the same; two ways of dealing the
// rows to the fetching threads, kConvAnyTap and kConvByTap).
#pragma once
#include <algorithm>

#include "spmm_common.hpp"
#include "staged_room.hpp"

namespace grim {

struct WideParams {
    const unsigned char *recs;
    const int32_t *cptr;
    const int32_t *bptr;
    const int32_t *strip_order;
    const unsigned short *X;
    float *Y;
    int64_t N, ldx, ldy;
    int32_t K, nbr, nchunks, chunk_rows;
    int32_t ntiles, ngroups;
    int32_t amax;   // 16-byte units of records one LDS stage must hold
    // ---- convolution (CONV): X is null; column n of the product is output position n % HW of image n / HW, row
    // k = cin * KK + r * kw + q of the never-formed matrix is feature map F[img][cin] shifted by kernel tap (r, q)
    const unsigned short *F;     // batch x [Cin][H][W], images f_img_stride elements apart
    int32_t H, W, HW, kh, kw, KK;
    int32_t kk_magic;            // ceil(2^31 / KK): k / KK = umulhi(2 k, magic) (k * KK < 2^31: checked at launch)
    int32_t kw_magic;            // ceil(256 / kw): tap / kw = tap * magic >> 8 (checked for every tap at launch)
    int32_t f_img_stride;        // elements
    int32_t f_total;             // elements from F to the end of the last image (f_total * 2 < 2^31)
    int32_t tap_ways;            // kConvByTap: fetching threads that share the rows of one (tap, piece)
    int64_t n_begin;             // first column of this launch (N is its end)
    int64_t y_img_stride;        // elements between the [M][ldy] outputs of two images
    const float *bias;           // M values added to every position of a row, or null
    int32_t relu, odt;           // max(., 0) after the bias; element type of Y
    int32_t y_vec4, y_vec8;      // four, eight consecutive 16-bit outputs of a row can be stored at once
};

// fp32 -> bf16, round to nearest even; NaN stays NaN
__device__ __forceinline__ unsigned short wide_f32_to_bf16(float f) {
    unsigned int u = __builtin_bit_cast(unsigned int, f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// two values rounded to a 16-bit type, nearest even, NaN stays NaN: one instruction on this GPU
template <int ODT>
__device__ __forceinline__ unsigned int wide_pair(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    if constexpr (ODT == GRIM_BF16) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(unsigned int, __builtin_convertvector((f32x2{a, b}), bf16x2));
    } else {
        typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(unsigned int, __builtin_convertvector((f32x2{a, b}), f16x2));
    }
}

// 16 bytes of a feature map at any 2-byte alignment
struct __attribute__((packed, aligned(2))) WideWindow {
    unsigned int d[4];
};

constexpr int wide_gcd(int a, int b) { return b == 0 ? a : wide_gcd(b, a % b); }

// How the convolution's rows of a chunk are dealt to the fetching threads.
//   kConvAnyTap: 16-byte units in order; the row's channel and tap and the unit's validity mask come out of tables in LDS.
//   kConvByTap:  a thread keeps one (tap, piece of the tile) and takes every tap_ways-th channel: the mask is four registers,
//                a row's address one addition.  Taken where there is a thread for every (tap, piece) and the rows of a chunk
//                are at most wide_tap_units per thread (conv_tap_ways, conv_taps.hpp); 5 x 5 kernels have more of them than there are
//                threads.
// 512 channels, 3 x 3, eight 56 x 56 maps, 32-row blocks of mixed rates 88 -> 74 us; 256 channels, 3 x 3, four 112 x 112 maps, 16-row
// blocks 80 -> 67.5; 1 x 1, 512 -> 256 channels on three 112 x 112 maps 35.6 -> 30.6 (graphs of one call): two dependent LDS reads
// and a table-driven address per unit are gone, a fetching wave's instructions per unit from about 35 to 12.
constexpr int kConvNone = 0, kConvAnyTap = 1, kConvByTap = 2;

// third dword of a raw buffer descriptor on this GPU family (32-bit data format); only the range check matters here
constexpr unsigned int kBufferFlags = 0x00020000u;

// BR = 16: v_mfma_f32_16x16x32, product taken as (X^T tile) x (W^T fragment): a lane ends with 4 consecutive
//          columns of one output row.  BR = 32: v_mfma_f32_32x32x16, weights first: a lane holds one column, 16 rows.
// (the body as a function of the workgroup's number, so that a kernel can run other workgroups next to these)
template <bool BF16, int BR, int NT, int CONV>
__device__ __forceinline__ void wide_body(const WideParams &p, char *lds, int block_x) {
    constexpr int NSUB = BR == 16 ? 16 : 32;
    constexpr int TN = NT * NSUB;
    constexpr int PITCH = TN * 2 + kWidePad;     // LDS row pitch in bytes
    constexpr int CPR = TN / 8;                  // 16-byte units per staged row
    constexpr int NTB = NT == 12 ? 3 : NT % 4 == 0 ? 4 : NT;  // sub-tiles per pipeline item (NT <= 3: all of them)
    constexpr int NB = NT / NTB;                 // items per step
    constexpr int KS = BR == 16 ? 32 : 16;       // k slots per step
    constexpr int HDR = KS * 2 + (KS / 8) * 8;   // header bytes per step
    constexpr int SXU = (wide_max_chunk_rows(BR) * CPR + kWideFetchThreads - 1) / kWideFetchThreads;   // X units per fetching thread and chunk
    constexpr int NW = kWideMulWaves;
    constexpr int SRU = wide_sru(TN);
    static_assert(NT % NTB == 0, "sub-tiles come in whole batches");
    using Acc = typename std::conditional<BR == 16, f32x4, f32x16>::type;

    // (most of what the prologue needs of the arguments in one trip through the scalar cache; the tables of steps follow)
    asm volatile("" ::"s"(p.recs), "s"(p.cptr), "s"(p.bptr), "s"(p.nbr), "s"(p.nchunks), "s"(p.chunk_rows), "s"(p.ntiles), "s"(p.ngroups), "s"(p.amax),
                 "s"(p.N), "s"(p.K));
    if constexpr (CONV != kConvNone)
        asm volatile("" ::"s"(p.F), "s"(p.H), "s"(p.W), "s"(p.HW), "s"(p.kh), "s"(p.kw), "s"(p.KK), "s"(p.kk_magic), "s"(p.f_img_stride), "s"(p.f_total),
                     "s"(p.tap_ways), "s"(p.n_begin));
    else asm volatile("" ::"s"(p.X), "s"(p.ldx));
    const int xbytes = (p.chunk_rows + 1) * PITCH;            // X rows + zero row
    const int stage_bytes = xbytes + p.amax * 16;

    // workgroup -> (tile, strip group).  Workgroup ids are dealt to the 8 XCDs round-robin and each XCD has its own L2:
    // all groups of a tile run on the same XCD, and so do tiles 2 k and 2 k + 1 -- a 96-column tile is one and a half
    // 128-byte lines wide, so these two share a line of every row, which the pair then takes from HBM once.
    const int id = block_x;
    const int xcd = id & 7, slot = id >> 3;
    const int tslot = slot / p.ngroups;
    const int tile = (tslot >> 1) * 16 + xcd * 2 + (tslot & 1);
    const int group = slot % p.ngroups;
    if (tile >= p.ntiles) return;
    // a ragged last tile is shifted left to end at N (N >= TN, N a multiple of 8: checked at launch); it overlaps
    // its neighbour and both write the same bits to the shared columns
    int64_t n0 = (CONV ? p.n_begin : 0) + (int64_t)tile * TN;
    if (n0 + TN > p.N) n0 = p.N - TN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The two step tables are read with wave-uniform indices only; named in the constant address space they are
    // fetched through the scalar cache into scalar registers (they are never written while a kernel runs).
    using Table = const __attribute__((address_space(4))) int32_t *;
    const Table cptr = (Table)p.cptr, bptr = (Table)p.bptr;
    const int t0 = group * kWideStrips;
    const int t1 = t0 + kWideStrips < p.nbr ? t0 + kWideStrips : p.nbr;

    if (wave >= NW) {
        // ------------------------------------------------------------------ fetching waves
        const int ft = tid - NW * 64;            // 0 .. 255
        // A convolution of 16-row blocks waits for its windows and not for its multiplies: its fetching waves go first where
        // a SIMD has the choice (256 channels, 3 x 3, four 112 x 112 maps 64.1 -> 54.2 us, mixed rates 68.0 -> 64.8).  The
        // 32-row form, which multiplies twice as much per window, loses by it (76.8 -> 80.9), products gain nothing.
        if constexpr (CONV == kConvByTap && BR == 16) __builtin_amdgcn_s_setprio(1);
        // zero rows (gather target of padded k slots), one per stage
        static_assert(2 * (PITCH / 4) <= kWideFetchThreads, "one thread per dword of the two zero rows");
        if (ft < 2 * (PITCH / 4)) {
            const int st = ft / (PITCH / 4), w = ft % (PITCH / 4);
            *reinterpret_cast<unsigned int *>(lds + st * stage_bytes + p.chunk_rows * PITCH + w * 4) = 0u;
        }
        // Where the records of the group's strips in a chunk start and how many 16-byte units they are: two table
        // reads through the scalar cache, asked for at the top of a chunk period and used at its end, so that their
        // latency runs under the period's stores
        struct RecRange { int b0, units; };
        auto rec_range = [&](int chunk) {
            chunk = chunk < p.nchunks ? chunk : p.nchunks - 1;
            const Table bp = bptr + (int64_t)chunk * (p.nbr + 1);
            RecRange r;
            r.b0 = __builtin_amdgcn_readfirstlane(bp[t0]);
            r.units = __builtin_amdgcn_readfirstlane(bp[t1]) - r.b0;
            return r;
        };
        // A chunk's records go from global memory straight into the stage's record area (no registers, no LDS store
        // instructions): a wave's load puts lane l's 16 bytes at the wave's base (in M0) + 16 l; lanes past the range's
        // end are masked off and write nothing.  The stage must be free when the load is ISSUED (see the loop below).
        // Written as assembly so that the compiler's own wait insertion does not see these loads: it would otherwise
        // drain every load of the wave before the next LDS store and before every barrier, which ends the rows'
        // two-chunk prefetch.  The waits it computes for the rows stay valid -- loads it does not know of only make a
        // wait for an older load stricter -- and the wait for the records themselves is explicit (landed_but_rows).
        const int fwave = __builtin_amdgcn_readfirstlane(ft >> 6);
        auto direct_records = [&](int chunk, const RecRange &r) {
            const int sbase = (int)(uintptr_t)(__attribute__((address_space(3))) char *)lds + (chunk & 1) * stage_bytes + xbytes;
            const unsigned char *src = p.recs + (int64_t)r.b0 * 16;
#pragma unroll
            for (int i = 0; i < SRU; ++i) {
                if (i * kWideFetchThreads < r.units) {
                    const int u = i * kWideFetchThreads + ft;
                    if (u < r.units)
                        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                                     :: "s"(sbase + (i * kWideFetchThreads + fwave * 64) * 16), "v"(src + (int64_t)u * 16)
                                     : "memory", "m0");
                }
            }
        };
        if constexpr (CONV == kConvByTap) {
            // Thread = (tap, 16-byte piece c of the tile, way): its unit i of a chunk is the row of its tap of the (way +
            // tap_ways i)-th channel that begins its tap in the chunk.  Rows a thread has none of and rows past the chunk
            // go into the padding bytes of row 0, which nobody reads; rows past K are never multiplied.
            constexpr int U = wide_tap_units(TN);
            const int pairs = p.KK * CPR;
            const int way = ft / pairs, pair = ft - way * pairs;
            const int tap = pair / CPR, c = pair - tap * CPR;
            const int tr = tap / p.kw, tq = tap - tr * p.kw;
            const int dr = tr - (p.kh >> 1), dq = tq - (p.kw >> 1);
            // (fewer than 2^30 positions: checked at launch; a 64-bit division is 150 instructions)
            const unsigned int n = (unsigned int)n0 + c * 8;
            const int img = (int)(n / (unsigned int)p.HW);
            const int pos = (int)(n - (unsigned int)img * (unsigned int)p.HW);
            unsigned int mask[4] = {0u, 0u, 0u, 0u};     // the positions whose shifted pixel lies inside the image
            {
                int h = pos / p.W, w = pos - h * p.W;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool ok = h + dr >= 0 && h + dr < p.H && w + dq >= 0 && w + dq < p.W;
                    mask[j >> 1] |= ok ? (j & 1 ? 0xffff0000u : 0x0000ffffu) : 0u;
                    if (++w == p.W) { w = 0; ++h; }
                }
            }
            const bool idle = way >= p.tap_ways;
            const int ebase = idle ? 0 : img * p.f_img_stride + pos + dr * p.W + dq + way * p.HW;
            const int rbase = idle ? 1 << 20 : way * p.KK;             // (idle: every row is past the chunk)
            const int estep = p.tap_ways * p.HW, rstep = p.tap_ways * p.KK;
            const int spare = TN * 2 + (c & 1) * 16;
            // first channel of a chunk and the tap its first row is
            auto first_of = [&](int chunk, int &cin, int &t) {
                const unsigned int k0 = (unsigned int)(chunk * p.chunk_rows);
                cin = (int)__umulhi(k0 << 1, (unsigned int)p.kk_magic);
                t = (int)k0 - cin * p.KK;
            };
            auto element = [&](int cin, int t) {                       // of the thread's unit 0 (its channel begins one later
                return (int)((unsigned int)ebase + (unsigned int)(cin + (tap < t ? 1 : 0)) * (unsigned int)p.HW);   // if its tap of the first is past)
            };
            const int emax = p.f_total - 8;
            auto load_taps = [&](int chunk, u32x4 (&rx)[U]) {
                int cin, t;
                first_of(chunk < p.nchunks ? chunk : p.nchunks - 1, cin, t);
                unsigned int e = (unsigned int)element(cin, t);
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    const int ec = (int)e < 0 ? 0 : (int)e > emax ? emax : (int)e;      // (windows at the ends of the batch: see below)
                    WideWindow wv;
                    __builtin_memcpy(&wv, reinterpret_cast<const char *>(p.F) + (unsigned int)(ec * 2), 16);
                    rx[i] = u32x4{wv.d[0], wv.d[1], wv.d[2], wv.d[3]};
                    e += (unsigned int)estep;
                }
            };
            // can a window of the chunk reach before the first or behind the last element of the batch?  (the same for the
            // whole workgroup; windows of rows past K do not count)
            const int img0 = (int)((unsigned int)n0 / (unsigned int)p.HW), img1 = (int)((unsigned int)(n0 + TN - 8) / (unsigned int)p.HW);
            const int64_t elo = (int64_t)img0 * p.f_img_stride + (n0 - (int64_t)img0 * p.HW) - ((p.kh >> 1) * p.W + (p.kw >> 1));
            const int64_t ehi = (int64_t)img1 * p.f_img_stride + (n0 + TN - (int64_t)img1 * p.HW) +
                                (p.kh - 1 - (p.kh >> 1)) * p.W + (p.kw - 1 - (p.kw >> 1));
            const int last_cin = p.K / p.KK - 1;
            auto store_taps = [&](int chunk, u32x4 (&rx)[U]) {
                int cin, t;
                first_of(chunk, cin, t);
                const int cend = cin + (p.chunk_rows + p.KK - 1) / p.KK < last_cin ? cin + (p.chunk_rows + p.KK - 1) / p.KK : last_cin;
                if (elo + (int64_t)cin * p.HW < 0 || ehi + (int64_t)cend * p.HW > p.f_total) {
                    unsigned int e = (unsigned int)element(cin, t);
#pragma unroll
                    for (int i = 0; i < U; ++i) {
                        const int ec = (int)e < 0 ? 0 : (int)e > emax ? emax : (int)e;
                        const int d = (int)e - ec;    // the pixels wanted start d elements behind (before: d < 0) the ones loaded
                        if (d != 0) {
                            unsigned __int128 x = (unsigned __int128)rx[i][0] | (unsigned __int128)rx[i][1] << 32 |
                                                  (unsigned __int128)rx[i][2] << 64 | (unsigned __int128)rx[i][3] << 96;
                            x = d >= 8 || d <= -8 ? (unsigned __int128)0 : d > 0 ? x >> (16 * d) : x << (16 * -d);
                            rx[i] = u32x4{(unsigned int)x, (unsigned int)(x >> 32), (unsigned int)(x >> 64), (unsigned int)(x >> 96)};
                        }
                        e += (unsigned int)estep;
                    }
                }
                char *sbase = lds + (chunk & 1) * stage_bytes;
                int row = rbase + tap - t + (tap < t ? p.KK : 0);
                int at = row * PITCH + c * 16;
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    const u32x4 v = u32x4{rx[i][0] & mask[0], rx[i][1] & mask[1], rx[i][2] & mask[2], rx[i][3] & mask[3]};
                    *reinterpret_cast<u32x4 *>(sbase + (row < p.chunk_rows ? at : spare)) = v;
                    row += rstep;
                    at += rstep * PITCH;
                }
            };
            // A chunk's windows come out of the caches: asked for one period before they are written to LDS.  They have
            // arrived when that period begins; waiting for them before the records are asked for keeps the wait from
            // covering those too (loads return in order).
            u32x4 RX[U];
            RecRange rcur = rec_range(0), rnxt = rec_range(1);
            load_taps(0, RX);
            direct_records(0, rcur);
            store_taps(0, RX);
            rcur = rnxt;
            load_taps(1, RX);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(U) : "memory");
            __syncthreads();
            for (int ch = 0; ch < p.nchunks; ++ch) {
                rnxt = rec_range(ch + 2);
                __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0)
                if (ch + 1 < p.nchunks) { direct_records(ch + 1, rcur); store_taps(ch + 1, RX); }
                rcur = rnxt;
                load_taps(ch + 2, RX);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(U) : "memory");   // the records are in LDS
                __syncthreads();
            }
            return;
        }
        // The thread's i-th unit of a chunk is unit i * 256 + ft = (row of the chunk, 16-byte piece of the row).
        // The loads of the rows are buffer loads, always issued: a row past the end of K is out of the buffer's range
        // and reads zeros without a fetch -- no conditional load among them, so a wait for an older set of rows never
        // has to assume that the younger set is missing.
        // SpMM: byte offset of the unit inside the tile's columns of X.  CONV: element of F at which the unit's 8
        // positions start (image and position of the piece), to which a row of the matrix adds its channel and tap.
        // (CONV: a thread's units i, i + XP, i + 2 XP, ... are the same piece of different rows, so XP offsets do)
        constexpr int XSTEP = kWideFetchThreads % CPR;
        constexpr int XP = !CONV ? SXU : XSTEP == 0 ? 1 : (CPR / wide_gcd(CPR, XSTEP) < SXU ? CPR / wide_gcd(CPR, XSTEP) : SXU);
        int xoff[XP];
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            const int u = i * kWideFetchThreads + ft;
            const int row = u / CPR, c = u - row * CPR;
            if constexpr (CONV) {
                const unsigned int n = (unsigned int)n0 + c * 8;
                const unsigned int img = n / (unsigned int)p.HW;
                xoff[i] = (int)img * p.f_img_stride + (int)(n - img * (unsigned int)p.HW);
            } else {
                xoff[i] = (int)(row * p.ldx * 2 + c * 16);      // below 2^31: checked at launch
            }
        }
        // CONV: per (kernel tap, piece of the tile) the 16-byte mask of the positions whose shifted pixel lies inside
        // the image (a piece never straddles two images: HW is a multiple of 8); entry KK is all zero (rows past K).
        // It sits behind the two stages.
        u32x4 *vtab = reinterpret_cast<u32x4 *>(lds + 2 * stage_bytes);
        const int centre = CONV ? (p.kh >> 1) * p.W + (p.kw >> 1) : 0;
        if constexpr (CONV) {
            for (int e = ft; e < (p.KK + 1) * CPR; e += kWideFetchThreads) {
                const int tap = e / CPR, c = e - tap * CPR;
                const int r = tap / p.kw, q = tap - r * p.kw;
                const int dr = r - (p.kh >> 1), dq = q - (p.kw >> 1);
                const int pos = (int)(((unsigned int)n0 + c * 8) % (unsigned int)p.HW);
                int h = pos / p.W, w = pos - h * p.W;
                unsigned int m[4] = {0u, 0u, 0u, 0u};
                if (tap < p.KK) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const bool ok = h + dr >= 0 && h + dr < p.H && w + dq >= 0 && w + dq < p.W;
                        m[j >> 1] |= ok ? (j & 1 ? 0xffff0000u : 0x0000ffffu) : 0u;
                        if (++w == p.W) { w = 0; ++h; }
                    }
                }
                vtab[e] = u32x4{m[0], m[1], m[2], m[3]};
            }
        }
        // (channel-and-tap offset, tap) of row k of the never-formed matrix; rows past K: tap KK (masked to zero)
        auto conv_row = [&](int k, int &tap) {
            const bool past = k >= p.K;
            const unsigned int kk = past ? 0u : (unsigned int)k;
            const unsigned int cin = __umulhi(kk << 1, (unsigned int)p.kk_magic);
            const int t_ = (int)(kk - cin * (unsigned int)p.KK);
            const int r = (t_ * p.kw_magic) >> 8;
            tap = past ? p.KK : t_;
            return (int)cin * p.HW + r * p.W + (t_ - r * p.kw) - centre;
        };
        // That split is made once per row and chunk, not once per 16-byte unit: a ring of four per-chunk tables in LDS
        // (behind the mask table) holds it for the chunks whose rows are being asked for or written; one thread per row
        // fills the table of chunk c + 4 during the period of chunk c, a barrier before anyone reads it.
        constexpr int RTP = wide_max_chunk_rows(BR);
        int2 *rowtab = reinterpret_cast<int2 *>(lds + 2 * stage_bytes + (CONV ? (p.KK + 1) * CPR * 16 : 0));
        auto fill_rows = [&](int chunk) {
            if (ft < RTP) {
                int tap;
                const int eb = conv_row(chunk * p.chunk_rows + ft, tap);
                rowtab[(chunk & 3) * RTP + ft] = int2{eb, tap};
            }
        };
        if constexpr (CONV) {
            for (int ch = 0; ch < 4; ++ch) fill_rows(ch);
            __syncthreads();                     // both tables are complete before the first chunk is asked for
        }
        // rows 0 .. K - 1 of the tile's columns: the last valid byte is the end of row K - 1's piece
        const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned short *>(CONV ? p.F : p.X + n0), 0, CONV ? 16 : (int)(((int64_t)(p.K - 1) * p.ldx + TN) * 2), kBufferFlags);
        u32x4 RX0[SXU], RX1[SXU];
        // (past the last chunk the last one is fetched again and never stored)
        // every load of this wave has arrived (the direct ones: is in LDS) except the youngest SXU: loads return in
        // order, and a chunk's rows are at least SXU load instructions, always issued
        auto landed_but_rows = [&]() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(SXU) : "memory"); };
        auto load_rows = [&](int chunk, u32x4 (&rx)[SXU]) {
            const int chunk_u = chunk;           // (CONV: rows past the last chunk are past K: any address, never stored)
            chunk = chunk < p.nchunks ? chunk : p.nchunks - 1;
            if constexpr (CONV) {
                // the unit's 8 pixels: one 16-byte load at a 2-byte alignment, always issued, at an address clamped
                // into the batch (a window that starts before it or ends behind it is shifted into place when stored)
                // (the rows' table entries are read together, so that their LDS round trips overlap)
                int eb[SXU];
#pragma unroll
                for (int i = 0; i < SXU; ++i) eb[i] = rowtab[(chunk_u & 3) * RTP + (i * kWideFetchThreads + ft) / CPR].x;
#pragma unroll
                for (int i = 0; i < SXU; ++i) {
                    int e = xoff[i % XP] + eb[i];
                    e = e < 0 ? 0 : e > p.f_total - 8 ? p.f_total - 8 : e;
                    WideWindow wv;
                    __builtin_memcpy(&wv, reinterpret_cast<const char *>(p.F) + (unsigned int)(e * 2), 16);
                    rx[i] = u32x4{wv.d[0], wv.d[1], wv.d[2], wv.d[3]};
                }
            } else {
                const int soff = __builtin_amdgcn_readfirstlane((int)((int64_t)chunk * p.chunk_rows * p.ldx * 2));
#pragma unroll
                for (int i = 0; i < SXU; ++i) rx[i] = __builtin_amdgcn_raw_buffer_load_b128(xres, xoff[i], soff, 0);
            }
        };
        // SpMM: where in a stage the thread's units go, held in registers (a store is then one instruction); a unit of
        // a row past the chunk's last goes into the 32 padding bytes of row 0, which nobody reads -- no branch
        int saddr[CONV ? 1 : SXU];
        if constexpr (!CONV) {
#pragma unroll
            for (int i = 0; i < SXU; ++i) {
                const int u = i * kWideFetchThreads + ft;
                const int row = u / CPR, c = u - row * CPR;
                saddr[i] = row < p.chunk_rows ? row * PITCH + c * 16 : TN * 2 + (u & 1) * 16;
            }
        }
        auto store_rows = [&](int chunk, const u32x4 (&rx)[SXU]) {
            char *sbase = lds + (chunk & 1) * stage_bytes;
            int fo = ft;
            if constexpr (CONV) asm volatile("" : "+v"(fo));   // the unit addresses are recomputed here, not held in registers across the loop
            if constexpr (CONV) {
                // three units at a time: their table entries, then their masks, are read together (two dependent LDS
                // round trips per group instead of per unit)
                constexpr int G = 3;
#pragma unroll
                for (int g = 0; g < SXU; g += G) {
                    int2 ri[G];
                    u32x4 vm[G];
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        const int i = g + j < SXU ? g + j : SXU - 1;
                        ri[j] = rowtab[(chunk & 3) * RTP + (i * kWideFetchThreads + fo) / CPR];
                    }
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        const int i = g + j < SXU ? g + j : SXU - 1;
                        const int u = i * kWideFetchThreads + fo;
                        vm[j] = vtab[ri[j].y * CPR + (u - u / CPR * CPR)];
                    }
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        if (g + j < SXU) {
                            const int i = g + j;
                            const int u = i * kWideFetchThreads + fo;
                            const int row = u / CPR, c = u - row * CPR;
                            u32x4 v = rx[i];
                            const int e = xoff[i % XP] + ri[j].x;
                            const int ec = e < 0 ? 0 : e > p.f_total - 8 ? p.f_total - 8 : e;
                            const int d = e - ec;    // the pixels wanted start d elements behind (before: d < 0) the ones loaded
                            if (__builtin_amdgcn_ballot_w64(d != 0) != 0 && d != 0) {      // (rare: the first and last pixels of the batch)
                                unsigned __int128 x = (unsigned __int128)v[0] | (unsigned __int128)v[1] << 32 |
                                                      (unsigned __int128)v[2] << 64 | (unsigned __int128)v[3] << 96;
                                x = d >= 8 || d <= -8 ? (unsigned __int128)0 : d > 0 ? x >> (16 * d) : x << (16 * -d);
                                v = u32x4{(unsigned int)x, (unsigned int)(x >> 32), (unsigned int)(x >> 64), (unsigned int)(x >> 96)};
                            }
                            v = u32x4{v[0] & vm[j][0], v[1] & vm[j][1], v[2] & vm[j][2], v[3] & vm[j][3]};
                            if (row < p.chunk_rows) *reinterpret_cast<u32x4 *>(sbase + row * PITCH + c * 16) = v;
                        }
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < SXU; ++i) *reinterpret_cast<u32x4 *>(sbase + saddr[i]) = rx[i];
            }
        };
        // Chunk c is multiplied from stage c % 2 while chunk c + 1 is written to the other stage (read last in chunk
        // c - 1, so free from the barrier that ends period c - 1).  Rows of X come from HBM: two register sets, a chunk's
        // rows are asked for two chunks before they are written.  Records come from L2 and go straight into the stage:
        // asked for at the top of the period that fills the stage, before the rows are written, and waited for (with
        // everything older, i.e. the rows asked for in the period before) ahead of the period's new row requests,
        // which therefore stay in flight across the barrier.
        RecRange rcur = rec_range(0), rnxt = rec_range(1);     // rcur: the range of the next chunk to be filled
        load_rows(0, RX0);
        direct_records(0, rcur);
        load_rows(1, RX1);
        store_rows(0, RX0);
        rcur = rnxt;
        load_rows(2, RX0);
        landed_but_rows();
        __syncthreads();
        for (int c = 0; c < p.nchunks; c += 2) {
            rnxt = rec_range(c + 2);
            if constexpr (CONV) fill_rows(c + 4);
            if (c + 1 < p.nchunks) { direct_records(c + 1, rcur); store_rows(c + 1, RX1); }
            rcur = rnxt;
            load_rows(c + 3, RX1);
            landed_but_rows();
            __syncthreads();
            // (no way out of the loop here: with one, the waits the compiler computes for the first half assume that the
            // second half's loads may not have been issued, and drain the rows asked for one period earlier; an odd
            // number of chunks ends with one idle period, for which the multiplying waves have a barrier of their own)
            rnxt = rec_range(c + 3);
            if constexpr (CONV) fill_rows(c + 5);
            if (c + 2 < p.nchunks) { direct_records(c + 2, rcur); store_rows(c + 2, RX0); }
            rcur = rnxt;
            load_rows(c + 4, RX0);
            landed_but_rows();
            __syncthreads();
        }
        return;
    }

    // ---------------------------------------------------------------------- multiplying waves
    Acc acc[2][NT];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < NT; ++q)
#pragma unroll
            for (int e = 0; e < (BR == 16 ? 4 : 16); ++e) acc[s][q][e] = 0.f;

    // per-lane constants of the gather: byte column inside a sub-tile
    const int i16 = lane & 15;
    const int ncolb = ((BR == 16 ? 0 : 16 * ((lane >> 4) & 1)) + 4 * (i16 & 3)) * 2;
    // per-lane constants of the weight fragment: output row inside the strip and k group
    const int m_row = BR == 16 ? (lane & 15) : (lane & 31);
    const int kgroup = BR == 16 ? (lane >> 4) : (lane >> 5);
    const unsigned int below = (1u << m_row) - 1u, mybit = 1u << m_row;
    const int hdr_rows = (kgroup * 4 + (i16 >> 2)) * 4;        // this lane's pair of staged-row numbers
    const int hdr_desc = KS * 2 + kgroup * 8;                  // its group's (row mask, payload offset)
    // stored strips of this wave: strips are stored by decreasing work, so the wave with the k-th heaviest strip of the
    // group's first half takes the k-th lightest of the second half
    const int tA = t0 + wave, tB = t0 + 2 * NW - 1 - wave;

    auto lds_address = [](const char *at) { return (unsigned int)(uintptr_t)(__attribute__((address_space(3))) const char *)at; };
    struct Hdr { unsigned int rr; uint2 dsc; };
    auto load_hdr = [&](const char *h) {
        Hdr f;
        f.rr = *reinterpret_cast<const unsigned int *>(h + hdr_rows);
        f.dsc = *reinterpret_cast<const uint2 *>(h + hdr_desc);
        return f;
    };
    auto load_x = [&](const char *stage, const Hdr &f, int b, i16x8 (&x)[NTB]) {
        const int r0 = f.rr & 0xffff, r1 = f.rr >> 16;
        const char *x0 = stage + r0 * PITCH + ncolb;
        const char *x1 = stage + r1 * PITCH + ncolb;
#pragma unroll
        for (int j = 0; j < NTB; ++j) {
            const int qoff = (b * NTB + j) * NSUB * 2;            // a constant: folded into the read's offset field
            const i16x4 lo = lds_tr_read(x0 + qoff);
            const i16x4 hi = lds_tr_read(x1 + qoff);
            x[j] = i16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    };

    // (steps, region offset) of the wave's two strips in a chunk -- wave-uniform, read through the scalar cache
    struct Entry { int nA, nB, offA, offB; };
    auto entry_of = [&](int ch) {
        const Table cp = cptr + (int64_t)ch * (p.nbr + 1), bp = bptr + (int64_t)ch * (p.nbr + 1);
        const int a0 = tA < p.nbr ? tA : p.nbr, a1 = tA + 1 < p.nbr ? tA + 1 : p.nbr;
        const int b0 = tB < p.nbr ? tB : p.nbr, b1 = tB + 1 < p.nbr ? tB + 1 : p.nbr;
        const int base = bp[t0];
        Entry e;
        e.nA = cp[a1] - cp[a0];
        e.nB = cp[b1] - cp[b0];
        e.offA = (bp[a0] - base) * 16;
        e.offB = (bp[b0] - base) * 16;
        return e;
    };

    // A pipeline item is (step, batch of NTB sub-tiles).  The loads of the next item -- for a new step its weights, its
    // gathered rows and the header of the step after it -- are issued BEFORE the current item is multiplied and land in
    // a second set of registers; items are taken in pairs so that the two sets swap roles without a copy (a copy
    // would wait for the load it copies).  The scheduling barriers keep the compiler from moving the multiplies ahead
    // of the loads: the LDS round trip of one item has to run under the multiplies of the item before it.  A lane whose
    // row the block does not keep reads its weights from the stage's zero row (zeroed in registers instead, four more
    // instructions a step: 512 x 4608 of mixed rates in 32-row blocks at 25 088 columns 79.4 us, 76.6 so).
    struct Frag { i16x8 x[NTB]; i16x8 w; };
    auto compute = [&](int ch, const Entry &en) {
        const int n = en.nA + en.nB;
        if (n <= 0) return;
        const char *stage = lds + (ch & 1) * stage_bytes;
        const unsigned int zero_row = lds_address(stage) + p.chunk_rows * PITCH;
        const char *regA = stage + xbytes + en.offA, *regB = stage + xbytes + en.offB;
        // virtual step v of the wave's list: strip A's steps, then strip B's (clamped to the last one)
        auto region_of = [&](int v) { return v < en.nA ? regA : regB; };
        auto hdr_of = [&](int v) {
            v = v < n ? v : n - 1;
            return v < en.nA ? regA + v * HDR : regB + (v - en.nA) * HDR;
        };
        // item it = v * NB + b
        auto issue = [&](int it, const Hdr &h, const Frag &prev, Frag &f) {
            const int b = it % NB;
            if (b == 0) {
                int v = it / NB;
                v = v < n ? v : n - 1;                    // (a step past the list is loaded and not multiplied)
                const unsigned int at = lds_address(region_of(v)) + (__builtin_popcount(h.dsc.x & below) + h.dsc.y) * 16;
                f.w = *(__attribute__((address_space(3))) const i16x8 *)(uintptr_t)(h.dsc.x & mybit ? at : zero_row);
            } else {
                f.w = prev.w;
            }
            load_x(stage, h, b, f.x);
        };
        auto multiply = [&](Acc (&a)[NT], int b, const Frag &f) {
#pragma unroll
            for (int j = 0; j < NTB; ++j) {
                if constexpr (BR == 16) a[b * NTB + j] = mfma16<BF16>(f.x[j], f.w, a[b * NTB + j]);
                else a[b * NTB + j] = mfma32<BF16>(f.w, f.x[j], a[b * NTB + j]);
            }
        };
        Frag fa, fb;
        Hdr hc, hn;    // headers of the step of the item in flight and of the step after it
        // One step (NB items, NB even or 1) or a pair of steps (NB = 1) per block, so that every block starts with
        // fa holding the loads of its first item, hc that item's header and hn the header of the next step.
        if constexpr (NB == 1) {
            auto pair = [&](int v, Acc (&a0)[NT], Acc (&a1)[NT]) {
                hc = load_hdr(hdr_of(v + 2));
                issue(v + 1, hn, fa, fb);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a0, 0, fa);
                __builtin_amdgcn_sched_barrier(0);
                hn = load_hdr(hdr_of(v + 3));
                issue(v + 2, hc, fb, fa);
                __builtin_amdgcn_sched_barrier(0);
                if (v + 1 < n) multiply(a1, 0, fb);       // (a pair may reach one step past the list)
                __builtin_amdgcn_sched_barrier(0);
            };
            hc = load_hdr(hdr_of(0));
            hn = load_hdr(hdr_of(1));
            issue(0, hc, fb, fa);
            // Steps go in pairs on every path (a separate single-step tail that updates the accumulators on one path
            // only makes the compiler keep a second copy of them); a pair that reaches one step past the list skips
            // its second multiply.
            int v = 0;
            for (; v + 1 < en.nA; v += 2) pair(v, acc[0], acc[0]);
            if (v < en.nA) {
                pair(v, acc[0], acc[1]);
                v += 2;
            }
            for (; v < n; v += 2) pair(v, acc[1], acc[1]);
        } else {
            static_assert(NB == 1 || NB % 2 == 0, "a step's items come in pairs");
            auto step = [&](int v, Acc (&a)[NT]) {
#pragma unroll
                for (int b = 0; b < NB; b += 2) {
                    issue(v * NB + b + 1, hc, fa, fb);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(a, b, fa);
                    __builtin_amdgcn_sched_barrier(0);
                    if (b + 2 < NB) {
                        issue(v * NB + b + 2, hc, fb, fa);
                    } else {
                        issue((v + 1) * NB, hn, fb, fa);          // the next step's first item
                        hc = hn;
                        hn = load_hdr(hdr_of(v + 2));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(a, b + 1, fb);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            hc = load_hdr(hdr_of(0));
            hn = load_hdr(hdr_of(1));
            issue(0, hc, fb, fa);
            for (int v = 0; v < en.nA; ++v) step(v, acc[0]);
            for (int v = en.nA; v < n; ++v) step(v, acc[1]);
        }
    };

    if constexpr (CONV == kConvAnyTap) __syncthreads();         // (the fetching waves' tables)
    Entry en = entry_of(0);
    __syncthreads();
    for (int c = 0; c < p.nchunks; ++c) {
        const Entry en1 = entry_of(c + 1 < p.nchunks ? c + 1 : c);
        compute(c, en);
        en = en1;
        __syncthreads();
    }
    if (CONV != kConvByTap && (p.nchunks & 1)) __syncthreads();  // (the fetching waves' periods come in pairs)

    // ---- write the strip tiles of Y (original row order); streaming stores: Y is written once and not read here ----
    // CONV: the layer's epilogue (bias, rectifier, rounding to the next layer's element type); column n is position
    // n % HW of image n / HW, whose [M][ldy] output starts y_img_stride elements after the previous image's.  The output
    // type is chosen once and a strip's biases are fetched before its first store: stores and loads share a counter, so a
    // bias fetched between two stores is waited for behind the stores (512 channels, 3 x 3, eight 56 x 56 maps: 107 -> 88 us; 1 x 1, 512 -> 256
    // channels on five 112 x 112 maps in 16-row blocks, whose four 16-bit outputs of a row are one store: 69 -> 44).
    //
    // 16-bit outputs of 32-row strips: a lane's 16 sums of a sub-tile are one column of 16 rows.  Stored as they stand they are
    // 96 stores of 64 bytes a row with as many addresses, and the rounding to bf16 six instructions a value: 5 of the 74 us
    // of the layer above, all of it instructions.  A strip goes through LDS, idle by now, and leaves in 16-byte pieces.
    auto finish_through_lds = [&](auto out_type) {
        constexpr int ODT = decltype(out_type)::value;
        constexpr int OP = wide_out_pitch(TN), PIECES = TN / 8, RPP = 64 / PIECES;        // pieces of a row, rows per pass
        char *const mine = lds + wave * (32 * OP);
        const int c = lane % PIECES, r = lane / PIECES;
        const unsigned int n = (unsigned int)n0 + c * 8, img = n / (unsigned int)p.HW;     // (a piece lies in one image)
        unsigned short *const Y = reinterpret_cast<unsigned short *>(p.Y) + img * p.y_img_stride + (n - img * (unsigned int)p.HW);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int t = s == 0 ? tA : tB;
            if (t >= p.nbr) continue;
            const int64_t row0 = (int64_t)p.strip_order[t] * BR;
            float bias[16] = {};
            if (p.bias) {
#pragma unroll
                for (int e = 0; e < 16; ++e) bias[e] = p.bias[row0 + 4 * (lane >> 5) + 8 * (e >> 2) + (e & 3)];
            }
            char *const at = mine + 4 * (lane >> 5) * OP + (lane & 31) * 2;
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    float v[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        v[k] = acc[s][q][e + k] + bias[e + k];
                        if (p.relu) v[k] = __builtin_elementwise_maximum(v[k], 0.f);       // NaN stays NaN
                    }
                    const unsigned int two = wide_pair<ODT>(v[0], v[1]);
                    char *const to = at + 8 * (e >> 2) * OP + (e & 3) * OP + q * 64;
                    *reinterpret_cast<unsigned short *>(to) = (unsigned short)two;
                    *reinterpret_cast<unsigned short *>(to + OP) = (unsigned short)(two >> 16);
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k * RPP < 32; ++k) {
                const int row = r + k * RPP;
                if (row < 32 && r < RPP)
                    *reinterpret_cast<u32x4 *>(Y + (row0 + row) * p.ldy) = *reinterpret_cast<const u32x4 *>(mine + row * OP + c * 16);
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
    auto finish = [&](auto out_type) {
        constexpr int ODT = decltype(out_type)::value;
        using Out = typename Elem<ODT>::type;
        Out *const Y = reinterpret_cast<Out *>(p.Y);
        auto rounded = [](float v) {
            if constexpr (ODT == GRIM_BF16) return wide_f32_to_bf16(v);
            else return (Out)v;
        };
        int64_t col[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int64_t n = n0 + q * NSUB + (BR == 16 ? 4 * (lane >> 4) : lane & 31);
            col[q] = n;
            if constexpr (CONV) {
                const unsigned int img = (unsigned int)n / (unsigned int)p.HW;       // (fewer than 2^30 positions: checked at launch)
                col[q] = img * p.y_img_stride + ((unsigned int)n - img * (unsigned int)p.HW);
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int t = s == 0 ? tA : tB;
            if (t >= p.nbr) continue;
            const int64_t row0 = (int64_t)p.strip_order[t] * BR;
            constexpr int NBIAS = BR == 16 ? 1 : 16;
            // BR = 16: D[n][m]: lane holds m = lane % 16, n = 4 * (lane / 16) + 0..3
            // BR = 32: D[m][n]: lane holds n = lane % 32, m = 8 * (e / 4) + 4 * (lane / 32) + e % 4
            const int64_t lane_row = row0 + (BR == 16 ? lane & 15 : 4 * (lane >> 5));
            float bias[NBIAS] = {};
            if constexpr (CONV) {
                if (p.bias) {
#pragma unroll
                    for (int e = 0; e < NBIAS; ++e) bias[e] = p.bias[lane_row + 8 * (e >> 2) + (e & 3)];
                }
            }
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                Out *const at = Y + lane_row * p.ldy + col[q];
                auto value = [&](int e) {
                    float v = acc[s][q][e];
                    if constexpr (CONV) {
                        v += bias[BR == 16 ? 0 : e];
                        if (p.relu) v = __builtin_elementwise_maximum(v, 0.f);       // NaN stays NaN
                    }
                    return v;
                };
                if constexpr (BR == 16) {
                    if constexpr (ODT == GRIM_F32) {       // (16-byte aligned: checked at launch)
                        __builtin_nontemporal_store(f32x4{value(0), value(1), value(2), value(3)}, reinterpret_cast<f32x4 *>(at));
                    } else {
                        Out v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = rounded(value(e));
                        if (p.y_vec4) {
                            uint2 w;
                            __builtin_memcpy(&w, v, 8);
                            *reinterpret_cast<uint2 *>(at) = w;
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) at[e] = v[e];
                        }
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        Out *const to = at + (8 * (e >> 2) + (e & 3)) * p.ldy;
                        if constexpr (ODT == GRIM_F32) __builtin_nontemporal_store(value(e), to);
                        else *to = rounded(value(e));
                    }
                }
            }
        }
    };
    if (!CONV || p.odt == GRIM_F32) finish(std::integral_constant<int, GRIM_F32>{});
    else if constexpr (CONV) {
        if constexpr (BR == 32) {
            if (p.y_vec8) {
                if (p.odt == GRIM_F16) finish_through_lds(std::integral_constant<int, GRIM_F16>{});
                else finish_through_lds(std::integral_constant<int, GRIM_BF16>{});
                return;
            }
        }
        if (p.odt == GRIM_F16) finish(std::integral_constant<int, GRIM_F16>{});
        else finish(std::integral_constant<int, GRIM_BF16>{});
    }
}

template <bool BF16, int BR, int NT, int CONV = kConvNone>
__global__ void __launch_bounds__(kWideThreads) bcr_spmm_wide(WideParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    wide_body<BF16, BR, NT, CONV>(p, lds, blockIdx.x);
}

}  // namespace grim
