// Kernel of bcr_conv.hip as a header: the wide-tile convolution's launcher builds a kernel that runs both.
#pragma once
#include "conv_rules.hpp"
#include "conv_window.hpp"
#include "spmm_common.hpp"

namespace grim {

// ------------------------------------------------------------------------------------------
// convolution with the im2col matrix never formed (Section 3.1: CONV = filter matrix x im2col
// matrix; Section 4.5: rows of that matrix whose weights are all pruned are skipped)
//
// Same scheme and layout as the row-gathering kernel; only the fetch differs.  Row k of the
// im2col matrix is (input channel cin, kernel row r, kernel column q) with k = cin * kh * kw +
// r * kw + q, and its entry at output position n = h * W + w is F[cin][h + r - kh/2][w + q - kw/2]
// (zero outside the image).  For 8 consecutive positions these are 8 consecutive elements of the
// feature map starting at cin * H * W + n + (r - kh/2) * W + (q - kw/2) -- at any 2-byte alignment
// -- with some of them invalid at the image border.  A lane loads its window with one 16-byte
// load at that address, and when the step is multiplied zeroes the invalid elements with a
// 16-byte mask that depends on (kernel tap, piece of the tile) only and is read from a table the
// workgroup builds in LDS when it starts.  A window that would reach outside the feature map
// (the first and last few positions of the first and last channel) is put together from single
// guarded element loads instead.  Only rows kept by the strip are ever touched, and the feature
// map is read instead of a matrix kh * kw times its size.
// ------------------------------------------------------------------------------------------
struct ConvParams {
    const int32_t *sptr;
    const int32_t *out_row;
    const uint32_t *rows;
    const uint32_t *desc;
    const unsigned char *payload;
    const unsigned short *F;     // [Cin][H][W]
    void *Y;                     // [M][ldy] of fp32, fp16 or bf16 (odt), position n = h * W + w
    const float *bias;           // [M] added to every position of a row, or null
    int64_t ldy;
    int32_t odt, relu;           // element type of Y; max(., 0) after the bias
    int32_t N, H, W, kh, kw;     // N = H * W
    int32_t KK, kk_magic;        // kh * kw and ceil(2^31 / KK): k / KK = umulhi(2 k, magic) while k * KK < 2^31 (checked at launch)
    int32_t kw_magic;            // ceil(256 / kw): tap / kw = tap * magic >> 8 (checked for every tap at launch)
    int32_t total;               // elements of the feature map
    int32_t nbr, ntiles;
    int32_t usteps;              // > 0: steps of every run (sptr is not read)
    int32_t yvec;
    // a convolution plan: per k slot of `rows` the tap and the window start for output position 0, already split
    // (tap << 27 | start + 2^25; tap = KK for padding slots); null: the kernel splits the row numbers itself
    const uint32_t *plan;
    int32_t batch, tiles_per_img;        // images; ntiles = batch * tiles_per_img
    uint32_t tiles_inv, row_inv;         // divide_by: tiles_per_img; positions of a row as the tiles walk it (W, or Wp at stride 2)
    int64_t f_img_stride, y_img_stride;  // elements between images of F and of Y
    // The 64 positions of a tile are output positions; stride 2: of output rows padded to Wp, a multiple of 8, so that a
    // lane's 8 positions never straddle two rows (Ho x Wo outputs; stride 1: Wp is not used)
    int32_t stride, Ho, Wo, Wp;
    int32_t Nv;                  // positions the tiles of one image walk: H * W, the end of a range, or Ho * Wp
    int32_t img0, pos_begin;     // first image of the launch; first position the tiles walk (a range of one image)
    XcdMap map;
};

// fp32 -> bf16, round to nearest even; NaN stays NaN
__device__ __forceinline__ unsigned short conv_f32_to_bf16(float f) {
    unsigned int u = __builtin_bit_cast(unsigned int, f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// which of two positions, nb and nb + 1 (a row of positions has `rowlen` of them), see a pixel of the image under a kernel tap: a
// dword of the 16-byte mask of 8 positions; tap KK: none
template <bool S2>
__device__ __forceinline__ unsigned int conv_pair_mask(const ConvParams &p, int tap, int nb, int rowlen) {
    const int r = (tap * p.kw_magic) >> 8, q = tap - r * p.kw;
    const int dr = r - (p.kh >> 1), dq = q - (p.kw >> 1);
    const int h0 = divide_by(nb, rowlen, p.row_inv), w0 = nb - h0 * rowlen;
    unsigned int m = 0u;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        int h = h0, w = w0 + j;
        if (!S2 && w >= rowlen) { w -= rowlen; ++h; }          // (positions past the last, of a small map: h >= H, never stored)
        if constexpr (S2) { h *= 2; w *= 2; }
        const bool ok = tap < p.KK && h + dr >= 0 && h + dr < p.H && w + dq >= 0 && w + dq < p.W;
        m |= ok ? (j ? 0xffff0000u : 0x0000ffffu) : 0u;
    }
    return m;
}

// epilogue of a layer for four consecutive positions n .. n + 3 of output channel `row`: bias `b`, rectifier,
// rounding to the next layer's element type
template <bool S2>
__device__ __forceinline__ void conv_finish(const ConvParams &p, int img, int64_t row, float b, int64_t n, f32x4 sum) {
    char *Yimg = static_cast<char *>(p.Y) + (int64_t)img * p.y_img_stride * (p.odt == GRIM_F32 ? 4 : 2);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sum[e] += b;
        if (p.relu) sum[e] = __builtin_elementwise_maximum(sum[e], 0.f);    // NaN stays NaN
    }
    // how many of the four are outputs, and where the first goes
    int left = (int)(p.Nv - n);                  // below 4 only in the one tile of a map of fewer than 64 positions
    if constexpr (S2) {
        const int h = (int)n / p.Wp, w = (int)n - h * p.Wp;
        left = h < p.Ho ? p.Wo - w : 0;
        n = (int64_t)h * p.Wo + w;
    }
    const bool vec = p.yvec == 4 && (n & 3) == 0;
    if (p.odt == GRIM_F32) {
        float *dst = reinterpret_cast<float *>(Yimg) + row * p.ldy + n;
        if (vec && left >= 4) {
            *reinterpret_cast<f32x4 *>(dst) = sum;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < left) dst[e] = sum[e];
        }
    } else {
        unsigned short h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (p.odt == GRIM_F16) {
                const _Float16 v = (_Float16)sum[e];
                __builtin_memcpy(&h[e], &v, 2);
            } else {
                h[e] = conv_f32_to_bf16(sum[e]);
            }
        }
        unsigned short *dst = reinterpret_cast<unsigned short *>(Yimg) + row * p.ldy + n;
        if (vec && left >= 4) {
            *reinterpret_cast<uint2 *>(dst) = uint2{(unsigned int)h[0] | ((unsigned int)h[1] << 16), (unsigned int)h[2] | ((unsigned int)h[3] << 16)};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < left) dst[e] = h[e];
        }
    }
}

struct __attribute__((packed, aligned(4))) ConvWindow {
    unsigned int d[4];
};

// Sixteen bytes fetched d elements before (d > 0) or behind the place they are wanted from, moved there: eight dwords, four of
// them zero, shifted down by 0 .. 7 elements.
__device__ __forceinline__ u32x4 conv_shift(const u32x4 &f, int d) {
    const bool none = d >= 8 || d <= -8, up = d < 0;
    const int e = up ? d + 8 : d;
    const u32x4 zero = {0u, 0u, 0u, 0u}, lo = none || up ? zero : f, hi = !none && up ? f : zero;
    const unsigned int a0 = e & 4 ? lo[2] : lo[0], a1 = e & 4 ? lo[3] : lo[1], a2 = e & 4 ? hi[0] : lo[2], a3 = e & 4 ? hi[1] : lo[3],
                       a4 = e & 4 ? hi[2] : hi[0], a5 = e & 4 ? hi[3] : hi[1];
    const unsigned int b0 = e & 2 ? a1 : a0, b1 = e & 2 ? a2 : a1, b2 = e & 2 ? a3 : a2, b3 = e & 2 ? a4 : a3, b4 = e & 2 ? a5 : a4;
    const unsigned int sh = (e & 1) * 16u;
    return u32x4{__builtin_amdgcn_alignbit(b1, b0, sh), __builtin_amdgcn_alignbit(b2, b1, sh), __builtin_amdgcn_alignbit(b3, b2, sh),
                 __builtin_amdgcn_alignbit(b4, b3, sh)};
}

constexpr int kConvTableBytes = (kConvMaxTaps + 1) * 8 * 16;   // validity masks, behind the waves' step buffers

// SOLO, EIGHT: as in the row-gathering kernel -- a (tile, strip) pair per wave for strips of a few steps, eight
// waves per strip for long strips with few workgroups
// MODE: 0 = row numbers split in the kernel, stride 1; 1 = a plan's words, stride 1; 2 = a plan's words, stride 2.
// Compile-time, so that the plain form carries none of the others' state in registers.
// The body as a function of the workgroup's number, so that another kernel can run such workgroups behind its own (the
// wide-tile convolution does, for the positions it leaves over).  All (LONGW ? LONGW : 4) waves call it together; `lds`:
// 8 KB per wave plus the validity table.
// LONGW: 0, or the waves that split a long strip's steps (8 or 12).  NT: 16-column sub-tiles of a tile, 4 or 2.
// SB: steps a wave has in flight (steps past its last are fetched too: no more than its share)
constexpr int conv_batch(int stride) { return stride == 2 ? 2 : 3; }      // of a 64-position tile, as the registers allow
constexpr int conv_wave_lds(int nt) { return nt * 2048; }      // two step buffers of 32 rows x 16 nt columns
template <bool BF16, bool SOLO, int LONGW, int MODE, int NT = 4, int SB = conv_batch(MODE == 2 ? 2 : 1)>
__device__ __forceinline__ void conv_gather_body(const ConvParams &p, char *lds, int block_x) {
    constexpr bool EIGHT = LONGW > 0;
    constexpr bool PLAN = MODE != 0, S2 = MODE == 2;
    constexpr int TN = NT * 16, PITCH = TN * 2, CPR = 2 * NT;  // columns, bytes and 16-byte pieces of a staged row
    constexpr int RPI = 64 / CPR, LI = 32 / RPI;               // rows per load instruction, windows per lane and step
    constexpr int LW = S2 ? 2 : 1;               // 16-byte loads per window (stride 2: 16 elements, of which every second one counts)
    constexpr int NWV = EIGHT ? LONGW : 4;       // waves of the workgroup
    // (what the way to the first slot words needs of the arguments in one trip through the scalar cache: where each is asked for
    // when it is first used, the trips follow one another.  The map's sizes, the taps and the payload come a trip later, beside those words)
    asm volatile("" ::"s"(p.map.per_tile), "s"(p.map.tail_slot0), "s"(p.map.tail_tile0), "s"(p.map.shift), "s"(p.map.per_part),
                 "s"(p.map.per_tile_inv), "s"(p.map.per_part_inv), "s"(p.ntiles), "s"(p.tiles_per_img), "s"(p.tiles_inv), "s"(p.nbr),
                 "s"(p.usteps), "s"(p.plan), "s"(p.rows), "s"(p.desc), "s"(p.out_row), "s"(p.F), "s"(p.f_img_stride), "s"(p.Nv));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile, unit;
    if (!xcd_map_at(p.map, block_x, p.ntiles, &tile, &unit)) return;
    const int img_l = divide_by(tile, p.tiles_per_img, p.tiles_inv);
    tile -= img_l * p.tiles_per_img;
    const int img = img_l + p.img0;
    const unsigned short *Fimg = p.F + (int64_t)img * p.f_img_stride;
    const int t_raw = SOLO ? unit * 4 + wave : unit;
    const bool active = t_raw < p.nbr;           // SOLO: the last workgroup of a tile may have idle waves
    const int t = active ? t_raw : p.nbr - 1;
    int n0 = p.pos_begin + tile * TN;
    if (n0 + TN > p.Nv) n0 = p.Nv - TN;          // ragged last tile: overlap the neighbour
    n0 = n0 < 0 ? 0 : n0;                        // a map of fewer than 64 positions: one tile, its columns past N never stored

    // one dependent memory round trip less at the start when every run has the same number of steps
    const int g0 = p.usteps ? t * p.usteps : p.sptr[t], nst = p.usteps ? p.usteps : p.sptr[t + 1] - g0;
    const int s_beg = SOLO ? g0 : g0 + wave_share(nst, wave, NWV);
    const int s_end = SOLO ? g0 + nst : g0 + wave_share(nst, wave + 1, NWV);
    char *buf = lds + wave * conv_wave_lds(NT);
    const int row = p.out_row[(int64_t)t * 16 + (lane & 15)];     // output channel and bias: asked for now, needed at the very end
    const uint2 *desc2 = reinterpret_cast<const uint2 *>(p.desc);
    const uint32_t *slots = PLAN ? p.plan : p.rows;
    u32x4 *vtab = reinterpret_cast<u32x4 *>(lds + NWV * conv_wave_lds(NT));
    const int ph = p.kh >> 1, pw = p.kw >> 1;

    // fetch side: lane = (row slot rs, piece c): positions n0 + 8 c .. n0 + 8 c + 7 of the tile
    const int rs = lane / CPR, c = lane % CPR;
    const int wr_off0 = rs * PITCH + ((c ^ swizzle<CPR>(rs)) << 4);     // the swizzle does not depend on i (row i * RPI + rs: RPI is a multiple of its period)
    // multiply side (as in the row-gathering kernel)
    const int i16 = lane & 15, kgroup = lane >> 4, qd = i16 >> 2, m_row = i16;
    const unsigned int below = (1u << m_row) - 1u;
    const int ncolb = (4 * (i16 & 3)) * 2, cl = ncolb >> 4, within = ncolb & 15;
    const int r0 = kgroup * 8 + qd, r1 = r0 + 4;
    const int sw0 = swizzle<CPR>(r0), sw1 = swizzle<CPR>(r1);
    const int x0 = r0 * PITCH + within, x1 = r1 * PITCH + within;
    // the lane's two transpose reads of sub-tile 0
    const unsigned int buf_lds = (unsigned int)(uintptr_t)(__attribute__((address_space(3))) char *)buf;
    const unsigned int tr0 = x0 + ((cl ^ sw0) << 4), tr1 = x1 + ((cl ^ sw1) << 4);           // offsets in a step buffer

    const i16x8 *pay = reinterpret_cast<const i16x8 *>(p.payload);
    const char *Fb = reinterpret_cast<const char *>(Fimg);
    const int HW = p.N, wstep = p.W - p.kw, emax = p.total - 8;
    const int centre = ph * p.W + pw;            // offset of the centre tap: window starts are relative to it
    // element (inside a channel) under the centre tap for the first of the 8 positions of piece cc
    auto pos_off = [&](int cc) { return conv_piece_start<S2>(n0 + cc * 8, p.W, p.Ho, p.Wp, p.row_inv); };
    // Stride 1: the tile's first position goes into the (uniform) window start of a k slot and a lane adds only its
    // piece's 8 c -- this split, not the sum formed per lane, is what keeps the fetch loop within its registers.
    const int tile_pos = S2 ? __builtin_amdgcn_readfirstlane(pos_off(0)) : n0;
    const int cofs = (S2 ? pos_off(c) - tile_pos : c * 8) - (1 << 25);     // this lane's piece, and the bias of the packed form
    // can a window of this tile start before the feature map or end behind it?  (only in the first / last channel)
    bool tile_edge = conv_tile_at_edge<S2>(pos_off(0), pos_off(CPR - 1), centre, HW);
    if constexpr (S2) tile_edge = __builtin_amdgcn_readfirstlane(tile_edge) != 0;
    // A batch: the slot words and block descriptors of SB steps (past the wave's last: the last again), then their windows
    // and weights, all in registers at once.
    //   Where twelve waves split a strip (few workgroups, a batch or two per wave: the form is all latency) a lane reads the
    // plan's words of its own LI windows.  Handed on by lane permutes as below, each window is asked for behind a trip through
    // LDS (512 channels, 3 x 3, 14 x 14: 6.9 us; 6.3 so, with the windows ahead of the validity table).  With fewer waves and
    // more workgroups the loads are what is short and the words' cost 1 to 4 % (192 channels, 5 x 5, six 56 x 56 maps 112 us, 115
    // so; eight waves: 64 -> 96 channels, 3 x 3, 72 x 72 9.4, 9.8 so).
    //   Otherwise lane j takes k slot j % 32 of every step -- without a plan it splits the slot's row number into (window
    // start for the tile's first column, tap) -- and the lanes that fetch the slot's row pieces pick that pair up with a
    // lane permute: one integer division per lane and step instead of four.
    // Packed as tap (or KK for padding) << 27 | window start + 2^25.
    constexpr bool ALONE = LONGW == kConvLongWaves;           // twelve waves: a workgroup has its compute unit to itself
    constexpr bool OWN = PLAN && ALONE;          // a lane has the words of its windows
    constexpr bool NEED_PK = !OWN || (!S2 && NT == 4);        // ... or the word of k slot lane % 32
    constexpr bool OWN_EXT = OWN && !S2 && NT == 2;          // the last lane of a row piece asks for the element behind its window itself
    unsigned int pk[SB], words[SB][LI];
    uint2 dsc[SB];
    u32x4 RX[SB][LI][LW];
    unsigned int vsel[SB];                   // per step, 8 bits per window: validity mask (the tap; KK: padding) | odd start << 7
    i16x8 PW[SB];
    unsigned int ext[SB][OWN_EXT ? LI : 1];
    auto ask_words = [&](int st, unsigned int (&w)[LI]) {
        if constexpr (NT == 4) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(slots + (int64_t)st * 32 + rs * 4);
#pragma unroll
            for (int i = 0; i < LI; ++i) w[i] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < LI; ++i) w[i] = slots[(int64_t)st * 32 + (rs & 7) * 4 + (rs >> 3) + 2 * i];
        }
    };
    auto step = [&](int s) { return s < s_end ? s : s_end - 1 < 0 ? 0 : s_end - 1; };     // (a wave without steps: any valid step, never used)
    auto ask_headers = [&](int s) {
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const int st = step(s + u);
            if constexpr (OWN) ask_words(st, words[u]);
            if constexpr (NEED_PK) pk[u] = slots[(int64_t)st * 32 + (lane & 7) * 4 + ((lane >> 3) & 3)];
            dsc[u] = desc2[(int64_t)st * 4 + kgroup];
        }
    };
    auto ask_windows = [&](int s) {
        // window start of piece (u, i) for this lane, and the selector of its validity mask
        const int own = cofs + tile_pos;
        auto piece = [&](int u, int i, unsigned int &sel) {
            const unsigned int v = OWN ? words[u][i] : (unsigned int)__shfl((int)pk[u], i * RPI + rs);
            sel = v >> 27;
            return (int)(v & 0x7ffffffu) + (OWN ? own : cofs);
        };
        // SAFE: the tile touches the first or last positions of the feature map, where a window can reach
        // outside it (first / last channel only); every other tile skips those checks altogether.
        auto fetch = [&](auto safe_tag) {
            constexpr bool SAFE = decltype(safe_tag)::value;
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                bool is_pad = false;
                int eb = 0;                      // window start for the tile's first position
                if constexpr (PLAN && NEED_PK) { // already split when the plan was made
                    is_pad = (int)(pk[u] >> 27) == p.KK;
                    eb = (int)(pk[u] & 0x7ffffffu) - (1 << 25) + tile_pos;
                    if constexpr (!OWN) pk[u] = (pk[u] & 0xf8000000u) | (unsigned int)(eb + (1 << 25));
                } else if constexpr (!PLAN) {
                    is_pad = pk[u] == 0xffffffffu;
                    const unsigned int kk = is_pad ? 0u : pk[u];
                    // (24-bit multiplies: Cin, H * W, W and the tap numbers are all below 2^24)
                    const unsigned int cin = __umulhi(kk << 1, (unsigned int)p.kk_magic);
                    const int tap = (int)(kk - __umul24(cin, (unsigned int)p.KK));
                    const unsigned int r = __umul24((unsigned int)tap, (unsigned int)p.kw_magic) >> 8;   // tap / kw
                    // r * W + (tap - r * kw), less the centre tap's offset
                    eb = (int)__umul24(cin, (unsigned int)HW) + __mul24((int)r, wstep) + tap - centre + tile_pos;   // (W < kw: wstep < 0)
                    pk[u] = (unsigned int)(is_pad ? p.KK : tap) << 27 | (unsigned int)(eb + (1 << 25));
                }
                // A 16-byte load at an odd element (2 bytes off a dword) costs about three aligned ones in the
                // vector L1, a load that is only dword-aligned next to nothing.  A window that starts at an odd
                // element is therefore fetched one element early; when the step is written the lane shifts it
                // by 16 bits and takes its last element from the next lane's first dword.  The last lane of a
                // row piece has no such neighbour: lanes 0..31 fetch the boundary element of their k slot with
                // one extra 2-byte load per step, handed over by a lane permute (on 32-position tiles, whose form is all
                // latency, the last lane asks for it itself).  (Stride 2: the window's 16 elements
                // start at the even element below, and the even or the odd eight of them are the window.)
                if constexpr (!S2 && !OWN_EXT) {
                    const int e7 = eb + (CPR - 1) * 8;
                    bool need = lane < 32 && !is_pad && (e7 & 1);
                    if constexpr (SAFE) need = need && e7 + 7 >= 0 && e7 + 7 < p.total;
                    ext[u][0] = need ? (unsigned int)Fimg[e7 + 7] : 0u;
                }
            }
            bool edge_any = false;
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                vsel[u] = 0u;
#pragma unroll
                for (int i = 0; i < LI; ++i) {
                    unsigned int sel;
                    const int e0 = piece(u, i, sel);
                    const int odd = e0 & 1;
                    vsel[u] |= (sel | (unsigned int)odd << 7) << (8 * i);
                    int ea = e0 - odd;
                    if constexpr (OWN_EXT) {
                        bool need = c == CPR - 1 && odd != 0 && (int)sel != p.KK;
                        if constexpr (SAFE) need = need && e0 + 7 >= 0 && e0 + 7 < p.total;
                        ext[u][i] = need ? (unsigned int)Fimg[e0 + 7] : 0u;
                    }
                    if constexpr (SAFE && !S2) {
                        const bool edge = e0 < 0 || e0 > emax;
                        edge_any |= edge;
                        ea = edge ? 0 : ea;
                    }
#pragma unroll
                    for (int l = 0; l < LW; ++l) {
                        int el = ea + 8 * l;                             // (byte offset below 2^31)
                        if constexpr (SAFE && S2) {
                            const int ec = el < 0 ? 0 : el > emax ? emax : el;
                            edge_any |= ec != el;
                            el = ec;
                        }
                        ConvWindow wv;
                        __builtin_memcpy(&wv, Fb + (unsigned int)(el * 2), 16);
                        RX[u][i][l] = u32x4{wv.d[0], wv.d[1], wv.d[2], wv.d[3]};
                    }
                }
            }
            if constexpr (SAFE) {
                if (__builtin_amdgcn_ballot_w64(edge_any)) {
                    // (the words are read again: kept for this rare branch, they would not fit beside the windows)
                    if constexpr (OWN) {
#pragma unroll
                        for (int u = 0; u < SB; ++u) ask_words(step(s + u), words[u]);
                    }
#pragma unroll
                    for (int u = 0; u < SB; ++u) {
#pragma unroll
                        for (int i = 0; i < LI; ++i) {
                            unsigned int sel;
                            const int e0 = piece(u, i, sel);
                            if constexpr (S2) {
                                // moved loads are shifted back into place (element by element the loads of a map's edge cost
                                // a call with few steps a microsecond); what lies outside the map is masked
#pragma unroll
                                for (int l = 0; l < LW; ++l) {
                                    const int el = (e0 & ~1) + 8 * l, d = el - (el < 0 ? 0 : el > emax ? emax : el);
                                    RX[u][i][l] = conv_shift(RX[u][i][l], d);
                                }
                            } else if (e0 < 0 || e0 > emax) {
                                // the same elements the common path fetches (one early for an odd start), so
                                // that the lane's neighbours find what they expect in its first dword
                                unsigned int d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                                for (int j = 0; j < 8; ++j) {
                                    const int e = (e0 & ~1) + j;
                                    const unsigned int v = e >= 0 && e < p.total ? Fimg[e] : 0u;
                                    d[j >> 1] |= v << ((j & 1) * 16);
                                }
                                RX[u][i][0] = u32x4{d[0], d[1], d[2], d[3]};
                            }
                        }
                    }
                }
            }
        };
        if (tile_edge) fetch(std::true_type{}); else fetch(std::false_type{});
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const bool kept = (dsc[u].x >> m_row) & 1u;
            const unsigned int idx = dsc[u].y + (kept ? __builtin_popcount(dsc[u].x & below) : 0);
            const i16x8 wv = pay[idx];
            PW[u] = kept ? wv : i16x8{0, 0, 0, 0, 0, 0, 0, 0};
        }
    };
    // The first batch's headers, and where twelve waves split a strip its windows too, travel while the validity table is
    // built: per (tap, piece of the tile) the 16-byte mask of the piece's 8 positions, a dword per thread; entry KK is all
    // zero (padding slots).  (With fewer a second copy of the windows' code costs as much as their latency, which
    // other workgroups hide: 1 x 1, 160 channels on eight 42 x 65 maps 15.8 us, 16.4 so.)
    ask_headers(s_beg);
    if (ALONE && s_beg < s_end) ask_windows(s_beg);
    for (int z = tid; z < (p.KK + 1) * CPR * 4; z += NWV * 64) {
        const int e = z >> 2, tap = e / CPR, cc = e % CPR;
        reinterpret_cast<unsigned int *>(vtab)[z] = conv_pair_mask<S2>(p, tap, n0 + cc * 8 + (z & 3) * 2, S2 ? p.Wp : p.W);
    }
    const float bias = p.bias && row >= 0 ? p.bias[row] : 0.f;
    __syncthreads();
    if (SOLO && !active) return;                 // (no barrier follows in that form)

    f32x4 acc[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int s = s_beg; s < s_end; s += SB) {
        const int nb = s_end - s < SB ? s_end - s : SB;
        if (s != s_beg) ask_headers(s);
        if (!ALONE || s != s_beg) ask_windows(s);
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (u < nb) {
                char *b = buf + (u & 1) * (32 * PITCH);
#pragma unroll
                for (int i = 0; i < LI; ++i) {
                    const unsigned int sel = (vsel[u] >> (8 * i)) & 0xffu;
                    const u32x4 vm = vtab[(sel & 0x7fu) * CPR + c];
                    u32x4 v;
                    if constexpr (S2) {
                        const unsigned int pick = sel >> 7 ? 0x07060302u : 0x05040100u;       // odd or even halves of two dwords
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const u32x4 &f = RX[u][i][d >> 1];
                            v[d] = __builtin_amdgcn_perm(f[2 * d % 4 + 1], f[2 * d % 4], pick) & vm[d];
                        }
                    } else {
                        const u32x4 &f = RX[u][i][0];
                        const unsigned int sh = (sel >> 7) * 16u;         // 16: the window starts one element into the fetch
                        // the dword after the lane's four: the next lane's first one, or the boundary element
                        const unsigned int w0 = f[0];
                        const unsigned int nxt = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)w0, 0x101 /* row_shl:1 */, 0xf, 0xf, true);
                        const unsigned int bnd = OWN_EXT ? ext[u][OWN_EXT ? i : 0] : (unsigned int)__shfl((int)ext[u][0], i * RPI + rs);
                        const unsigned int w4 = c == CPR - 1 ? bnd : nxt;
                        v = u32x4{__builtin_amdgcn_alignbit(f[1], w0, sh) & vm[0], __builtin_amdgcn_alignbit(f[2], f[1], sh) & vm[1],
                                  __builtin_amdgcn_alignbit(f[3], f[2], sh) & vm[2], __builtin_amdgcn_alignbit(w4, f[3], sh) & vm[3]};
                    }
                    *reinterpret_cast<u32x4 *>(b + wr_off0 + i * RPI * PITCH) = v;
                }
                __builtin_amdgcn_wave_barrier();
                // The 16-byte chunk of sub-tile q is (2 q + cl) ^ swizzle = (cl ^ swizzle) ^ 2 q: the eight
                // read addresses are two bases with q << 5 XOR-ed in.  The empty asm keeps the compiler from
                // holding all eight in registers across the loop (they would not fit and spill).
                unsigned int a0 = tr0, a1 = tr1;
                asm volatile("" : "+v"(a0), "+v"(a1));
                const unsigned int sb = buf_lds + (u & 1) * (32 * PITCH);
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const i16x4 lo = lds_tr_read_at(sb + (a0 ^ (unsigned int)(q << 5)));
                    const i16x4 hi = lds_tr_read_at(sb + (a1 ^ (unsigned int)(q << 5)));
                    const i16x8 x = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    acc[q] = mfma16<BF16>(x, PW[u], acc[q]);
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }

    if constexpr (SOLO) {
        if (row >= 0) {
#pragma unroll
            for (int q = 0; q < NT; ++q) conv_finish<S2>(p, img, row, bias, n0 + q * 16 + 4 * (lane >> 4), acc[q]);
        }
        return;
    }
    // the waves' partial tiles go through their step buffers; the tables behind them stay intact
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
    for (int q = 0; q < NT; ++q) red[wave * (conv_wave_lds(NT) / 16) + q * 64 + lane] = acc[q];
    __syncthreads();
    if (wave >= NT) return;                      // the first waves finish the sub-tiles
    const int q = wave;
    f32x4 sum = red[q * 64 + lane];
#pragma unroll
    for (int w = 1; w < NWV; ++w) {
        const f32x4 v = red[w * (conv_wave_lds(NT) / 16) + q * 64 + lane];
        sum[0] += v[0]; sum[1] += v[1]; sum[2] += v[2]; sum[3] += v[3];
    }
    if (row >= 0) conv_finish<S2>(p, img, row, bias, n0 + q * 16 + 4 * (lane >> 4), sum);
}

template <bool BF16, bool SOLO, int LONGW, int MODE, int NT, int SB>
__global__ void __launch_bounds__(LONGW ? LONGW * 64 : 256, LONGW ? 1024 / (LONGW * 64) : MODE == 2 ? 3 : 4) bcr_conv_gather(ConvParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    conv_gather_body<BF16, SOLO, LONGW, MODE, NT, SB>(p, lds, blockIdx.x);
}

// which form of the kernel a launch takes, its workgroups and workgroup memory
struct ConvForm {
    bool solo;
    int longw, mode, nt, batch;      // batch: steps in flight
    int64_t nwg;
    size_t lds;
};
grim_status conv_gather_setup(const grim_bcr_matrix *A, const void *F, int32_t Cin, int32_t H, int32_t W, int32_t kh, int32_t kw,
                              const float *bias, int32_t relu, void *Y, int32_t odt, int64_t ldy, int32_t batch, int32_t stride,
                              int64_t f_img_stride, int64_t y_img_stride, const uint32_t *plan, int32_t img0, int64_t pos_begin,
                              int64_t pos_end, ConvParams *out, ConvForm *form);

}  // namespace grim
