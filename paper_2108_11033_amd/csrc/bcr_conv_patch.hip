// Planned convolution of kernels larger than 1 x 1 with 64 rows of the matrix to a workgroup, the im2col matrix never formed
// (Section 3.1: CONV = filter matrix x im2col matrix).
#include "conv_patch.hpp"
#include "conv_tall.hpp"

namespace grim {

// A 64-row run of a matrix in small blocks keeps nearly every row of the im2col matrix, and forming those rows -- kh * kw
// shifted copies of each channel, masked and parked in LDS -- is most of what bcr_conv_tall does.  Here a channel's pixels
// under a tile go to LDS once, eight channels of a pixel side by side (turned around in registers on the way), and a kernel
// tap is an address: a lane's eight k values of a multiply are the eight channels of one pixel, always 16 aligned bytes, and a
// position whose tap lies outside the image reads a pixel of zeros.  The weights are the plan's dense copy in the order the
// multiplies take them: zeros are multiplied, but nothing is looked up, expanded or masked.
//
// Workgroup = (tile of 64 positions, 64-row run).  Its waves split the channels, each with pixels of its own in LDS: no
// barrier until the partial tiles are added.  A step is 32 k values = four (tap, channel octet) pairs: 16 multiplies for 4 KB
// of weights out of L2 and 4 KB of pixels out of LDS.
//
// 256 channels, 3 x 3, four 28 x 28 maps in 4 x 16 blocks 16.5 -> 11.1 us (1.9 of them multiplies at the matrix cores' rate,
// 4 the launch), 448 on seven 52 x 12 maps 40 -> 25.7, the same from 103 x 24 at stride 2 118 -> 36.  Bound by what a compute unit takes
// in (295 KB of weights and 65 KB of pixels at some 30 bytes a cycle, from its first cycles on) and the multiplies of its waves; more pixels per task (eight channels) take registers that
// spill, two steps of weights in flight instead of three cost 4 %.
//
// Sums: the steps are all of K, not what a run keeps, so a plain fp32 chain over a wave's steps would be up to four times as long
// as the one it takes the place of, and its error with it.  A chain ends after up to kPatchChain steps: its sum moves into a total,
// what that addition rounds off begins the next chain, and the waves' totals are added in 64 bits.  Error of fp32 outputs (2-norm,
// 1e-8) of the compact runs / one chain per wave / this: 448 channels on seven 52 x 12 maps in 16 x 32 blocks 9.1 / 13.0 / 8.7, 512
// on 32 of 14 x 14 in 4 x 16 blocks 13.1 / 13.5 / 8.8, 192 channels, 5 x 5, on four 18 x 18 in 32 x 32 blocks 8.5 / 11.2 / 7.7; of 126
// layers of 32 to 512 channels 0.51 to 1.01 times the compact runs'.  It costs 0.2 us per layer for the 64 bits and 0.6 us per settled
// chain of a compute unit's waves: 11.0 -> 11.1, 25.2 -> 25.8, 47.0 -> 48.5, 16.6 -> 18.9 us.  (Waves' totals as a tree in fp32: an
// error of 9.1 -> 8.6 where the compact runs have 7.8.)
//
// Infinities and NaNs: as in bcr_conv_tall, sums that are not finite are formed again from the 16-row runs.
struct ConvPatchParams : ConvTallParams {
    const unsigned char *dense;      // [run][channel chunk][step][16-row run][lane] 16 bytes
    int32_t cin, chunks, steps;      // channels, chunks of 8 CO of them, steps per chunk
    int32_t zero_at;                 // byte offset of the pixel of zeros
    int32_t wave_lds;                // bytes per wave
    int32_t chain, settlings;        // LONG: steps to a chain, chains of the longest wave but for its last
    uint32_t wo_inv;                 // divide_by: Wo
    uint32_t row_ones;               // bit r * kw of every kernel row r
};

// steps of weights in flight (five: 11.5 where this takes 11.2; a compute unit's weights, 295 KB for 256 channels, 3 x 3, come at
// some 30 bytes a cycle however early they are asked for)
constexpr int kPatchDepth = 3;
constexpr int kPatchChain = 12;                            // steps whose sums follow one another in fp32, to the group that ends them

// LONG: a wave has more than kPatchChain steps (its totals take the registers of a third task asked for ahead)
template <bool BF16, int CO, int NWV, bool LONG>
__global__ void __launch_bounds__(NWV * 64, 2) bcr_conv_patch(ConvPatchParams p) {
    constexpr int R = kConvTallRuns, NT = 4, TN = 64, SB = patch_pixel_bytes(CO);
    constexpr int D = kPatchDepth, AHEAD = LONG ? 2 : 3;    // tasks of a chunk asked for ahead, in 64s: as the registers allow
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // (what the way to the first pixels needs of the arguments in one trip through the scalar cache, as in bcr_conv_gather)
    asm volatile("" ::"s"(p.map.per_tile), "s"(p.map.tail_slot0), "s"(p.map.tail_tile0), "s"(p.map.shift), "s"(p.map.per_part),
                 "s"(p.map.per_tile_inv), "s"(p.map.per_part_inv), "s"(p.ntiles), "s"(p.tiles_per_img), "s"(p.tiles_inv), "s"(p.nbr),
                 "s"(p.F), "s"(p.f_img_stride), "s"(p.Nv), "s"(p.W), "s"(p.Wo), "s"(p.wo_inv), "s"(p.N), "s"(p.stride), "s"(p.kh), "s"(p.kw),
                 "s"(p.cin), "s"(p.chunks), "s"(p.steps), "s"(p.dense), "s"(p.wave_lds), "s"(p.out_row));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile, t;
    if (!xcd_map_at(p.map, blockIdx.x, p.ntiles, &tile, &t) || t >= p.nbr) return;
    const int img = divide_by(tile, p.tiles_per_img, p.tiles_inv);
    tile -= img * p.tiles_per_img;
    const unsigned short *Fimg = p.F + (int64_t)img * p.f_img_stride;
    int n0 = tile * TN;
    if (n0 + TN > p.Nv) n0 = p.Nv - TN;                    // ragged last tile: overlap the neighbour
    n0 = n0 < 0 ? 0 : n0;                                  // fewer than 64 positions: one tile, its columns past them never stored
    char *patch = lds + wave * p.wave_lds;

    const int kgroup = lane >> 4, i16 = lane & 15;
    const int c_beg = p.chunks * wave / NWV, c_end = p.chunks * (wave + 1) / NWV;
    const i16x8 *wt = reinterpret_cast<const i16x8 *>(p.dense) + (int64_t)t * p.chunks * p.steps * (R * 64);
    i16x8 PW[D][R];
    // (a group of D steps past a chunk's last, or a chunk past the wave's last: any valid step, never used)
    auto fetch_weights = [&](i16x8 (&w)[R], int chunk, int st) {
        st = st < p.steps ? st : p.steps - 1;
        const i16x8 *src = wt + (int64_t)(chunk * p.steps + st) * (R * 64);
#pragma unroll
        for (int m = 0; m < R; ++m) w[m] = src[m * 64 + lane];
    };
    // the pixels (of a channel) that a tap of the tile's positions can meet: [plo, phi]
    const int HW = p.N, centre = (p.kh >> 1) * p.W + (p.kw >> 1), fodd = (int)(reinterpret_cast<uintptr_t>(Fimg) >> 1) & 1;
    const bool s2 = p.stride == 2;
    const int plo = patch_first(n0, p.W, p.Wo, p.wo_inv, s2, centre, HW, fodd);
    const int phi = patch_last(n0, p.Nv, p.W, p.Wo, p.wo_inv, s2, centre, HW);
    const int tasks = ((phi - plo) / 8 + 1) * CO * 2;      // (eight pixels of four channels) to turn around per chunk

    f32x4 acc[R][NT], tot[R][NT];
#pragma unroll
    for (int m = 0; m < R; ++m)
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[m][q] = tot[m][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    // moves the sums into the totals; what an addition rounds off stays behind and is added with the steps that follow
    auto settle = [&]() {
#pragma unroll
        for (int m = 0; m < R; ++m)
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float s = tot[m][q][e] + acc[m][q][e];
                    acc[m][q][e] -= s - tot[m][q][e];
                    tot[m][q][e] = s;
                }
    };

    // A chunk's pixels: task = four channels of eight pixels, loaded along the pixels, written along the channels (the last
    // pixels of a channel are met by moving the eight back, onto pixels that are written twice with the same values).  The
    // first AHEAD * 64 tasks of a chunk are asked for while the chunk before it is multiplied.
    // 16 bytes at an odd element cost the vector L1 about three times what they cost at an even one: such a row is loaded one
    // element early and shifted into place before it is written, its last element fetched then, out of lines just read (maps of an
    // odd number of pixels: 288 channels, 3 x 3, seven 95 x 27 maps at stride 2 32.3 -> 27.5 us)
    const bool any_odd = ((HW | (plo + fodd) | fodd) & 1) != 0;       // (pieces start at plo + 8 q or at HW - 8, HW apart)
    struct Task { u32x4 row[4]; };
    struct Last { unsigned int row[4]; };
    auto load_task = [&](Task &in, int chunk, int id) {
        const int o = id % (CO * 2), p8 = plo + id / (CO * 2) * 8, ch = (chunk * CO * 2 + o) * 4;
        const int e = (ch < p.cin ? ch : p.cin - 4) * HW + (p8 < HW - 8 ? p8 : HW - 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ei = e + i * HW, odd = ei > 0 ? (ei + fodd) & 1 : 0;
            in.row[i] = load_piece_any(Fimg + (unsigned int)(ei - odd));
        }
    };
    auto load_last = [&](Last &in, int chunk, int id) {
        const int o = id % (CO * 2), p8 = plo + id / (CO * 2) * 8, ch = (chunk * CO * 2 + o) * 4;
        const int e = (ch < p.cin ? ch : p.cin - 4) * HW + (p8 < HW - 8 ? p8 : HW - 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) in.row[i] = (unsigned int)Fimg[(unsigned int)(e + i * HW + 7)];
    };
    auto store_task = [&](Task &task, const Last &tail, int chunk, int id) {
        const int o = id % (CO * 2), p8 = plo + id / (CO * 2) * 8, st = p8 < HW - 8 ? p8 : HW - 8, ch = (chunk * CO * 2 + o) * 4;
        u32x4 (&in)[4] = task.row;
        if (any_odd) {
            const int e = (ch < p.cin ? ch : p.cin - 4) * HW + st;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ei = e + i * HW;
                const unsigned int sh = ei > 0 && (ei + fodd) & 1 ? 16u : 0u;
                in[i] = u32x4{__builtin_amdgcn_alignbit(in[i][1], in[i][0], sh), __builtin_amdgcn_alignbit(in[i][2], in[i][1], sh),
                              __builtin_amdgcn_alignbit(in[i][3], in[i][2], sh), __builtin_amdgcn_alignbit(tail.row[i], in[i][3], sh)};
            }
        }
        if (ch >= p.cin) {                                 // (the last chunk's channels past the last)
#pragma unroll
            for (int i = 0; i < 4; ++i) in[i] = u32x4{0u, 0u, 0u, 0u};
        }
        char *dst = patch + (st - plo) * SB + o * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const unsigned int pick = j & 1 ? 0x07060302u : 0x05040100u;
            *reinterpret_cast<uint2 *>(dst + j * SB) = uint2{__builtin_amdgcn_perm(in[1][j >> 1], in[0][j >> 1], pick),
                                                             __builtin_amdgcn_perm(in[3][j >> 1], in[2][j >> 1], pick)};
        }
    };
    Task ahead[AHEAD];
    // (what is derived from the lane is formed anew for every chunk: held over the loop it would not fit the registers)
    auto ask_patch = [&](int chunk) {
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
            if (a * 64 + lane < tasks) load_task(ahead[a], chunk, a * 64 + lane);
    };
    auto take_patch = [&](int chunk) {
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
            if (a * 64 + lane < tasks) {
                Last tail = {};
                if (any_odd) load_last(tail, chunk, a * 64 + lane);
                store_task(ahead[a], tail, chunk, a * 64 + lane);
            }
        for (int id = AHEAD * 64 + lane; id < tasks; id += 64) {
            Task in;
            Last end = {};
            load_task(in, chunk, id);
            if (any_odd) load_last(end, chunk, id);
            store_task(in, end, chunk, id);
        }
        __builtin_amdgcn_wave_barrier();
    };
    // the first pixels, and the weights behind them (loads return in order, and the pixels are wanted first)
    if (c_beg < c_end) {
        ask_patch(c_beg);
#pragma unroll
        for (int u = 0; u < D; ++u) fetch_weights(PW[u], c_beg, u);
    }

    // per sub-tile: where the lane's position lies in the patch (centre tap, the lane's octet) and which taps see the image
    const int octet = kgroup % CO;
    int at[NT];
    unsigned int sees[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const int n = n0 + q * 16 + i16;
        int hh, ww;
        const int pix = patch_pixel_of(n < p.Nv ? n : p.Nv - 1, p.W, p.Wo, p.wo_inv, s2, &hh, &ww);
        at[q] = (pix - plo) * SB + octet * 16;
        const int wlo = (p.kw >> 1) - ww, whi = p.W - ww + (p.kw >> 1);            // taps of a kernel row: [wlo, whi)
        const unsigned int cols = ((1u << (whi < p.kw ? whi : p.kw)) - 1u) & ~((1u << (wlo > 0 ? wlo : 0)) - 1u);
        const int rlo = (p.kh >> 1) - hh, rhi = p.H - hh + (p.kh >> 1);            // kernel rows: [rlo, rhi)
        const unsigned int rows = p.row_ones & ((1u << (rhi < p.kh ? rhi : p.kh) * p.kw) - 1u) & ~((1u << (rlo > 0 ? rlo : 0) * p.kw) - 1u);
        sees[q] = cols * rows;                             // (cols has kw bits: its copies do not meet)
    }
    const int zero_at = p.zero_at + octet * 16;
    if (lane < CO) *reinterpret_cast<u32x4 *>(patch + p.zero_at + lane * 16) = u32x4{0u, 0u, 0u, 0u};

    auto multiply = [&](int st, const i16x8 (&w)[R]) {
        const int tap = (st * 4 + kgroup) / CO;            // (past the last tap: no position sees it)
        const int tr = (int)(__umul24((unsigned int)tap, (unsigned int)p.kw_magic) >> 8), tq = tap - tr * p.kw;
        const int toff = ((tr - (p.kh >> 1)) * p.W + tq - (p.kw >> 1)) * SB;
        i16x8 x[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int a = (sees[q] >> tap) & 1u ? at[q] + toff : zero_at;
            x[q] = *reinterpret_cast<const i16x8 *>(patch + a);
        }
#pragma unroll
        for (int q = 0; q < NT; ++q)
#pragma unroll
            for (int m = 0; m < R; ++m) acc[m][q] = mfma16<BF16>(x[q], w[m], acc[m][q]);
    };
    int since = 0, settled = 0;                            // steps since the last settling, settlings
    // (Leaving out the last group's requests, which nobody waits for, in a copy of the group behind the loop costs more than they do:
    // 448 channels on seven 52 x 12 maps 25.7 us, 26.9 so.)
    for (int chunk = c_beg; chunk < c_end; ++chunk) {
        take_patch(chunk);
        if (chunk + 1 < c_end) ask_patch(chunk + 1);
#pragma unroll 1
        for (int st = 0; st < p.steps; st += D) {
            const bool last = st + D >= p.steps;           // (the next group is the next chunk's first)
            const int nchunk = last && chunk + 1 < c_end ? chunk + 1 : chunk, nst = last ? 0 : st + D;
#pragma unroll
            for (int u = 0; u < D; ++u) {
                if (st + u < p.steps) multiply(st + u, PW[u]);
                fetch_weights(PW[u], nchunk, nst + u);
            }
            if constexpr (LONG) {
                since += p.steps - st < D ? p.steps - st : D;
                if (since >= p.chain && settled < p.settlings) { settle(); since = 0; ++settled; }
            }
        }
    }

    // the waves' partial tiles, added in 64 bits; the waves finish the (16-row run, sub-tile) pairs in turn (as in bcr_conv_tall)
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
    const int wave_red = p.wave_lds / 16;
    constexpr int PAIRS = R * NT / NWV;
    static_assert(R * NT % NWV == 0, "pairs are dealt evenly");
    int row[PAIRS];
    float bias[PAIRS];
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) row[j] = p.out_row[((int64_t)t * R + (wave + j * NWV) / NT) * 16 + i16];
#pragma unroll
    for (int m = 0; m < R; ++m)
#pragma unroll
        for (int q = 0; q < NT; ++q) red[wave * wave_red + (m * NT + q) * 64 + lane] = LONG ? tot[m][q] + acc[m][q] : acc[m][q];
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) bias[j] = p.bias && row[j] >= 0 ? p.bias[row[j]] : 0.f;
    __syncthreads();
    unsigned int again = 0u;                               // bit per pair: one of the lane's four sums is not finite
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        const int i = wave + j * NWV;
        double part[NWV][4];                               // (as a tree: the conversions' latencies side by side)
#pragma unroll
        for (int w = 0; w < NWV; ++w) {
            const f32x4 v = red[w * wave_red + i * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) part[w][e] = (double)v[e];
        }
#pragma unroll
        for (int half = NWV / 2; half > 0; half /= 2)
#pragma unroll
            for (int w = 0; w < half; ++w)
#pragma unroll
                for (int e = 0; e < 4; ++e) part[w][e] += part[w + half][e];
        const f32x4 sum = {(float)part[0][0], (float)part[0][1], (float)part[0][2], (float)part[0][3]};
        float nan = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) nan = __builtin_fmaf(sum[e], 0.f, nan);
        again |= nan != nan ? 1u << i : 0u;
        if (row[j] >= 0) conv_finish<false>(p, img, row[j], bias[j], n0 + i % NT * 16 + 4 * kgroup, sum);
    }
    if (__builtin_amdgcn_ballot_w64(again != 0u)) {
#pragma unroll 1
        for (int i = wave; i < R * NT; i += NWV) {
            const int run = t * R + i / NT, n = n0 + i % NT * 16 + 4 * kgroup;
            const int64_t row = p.out_row[(int64_t)run * 16 + i16];
            if (row < 0 || !((again >> i) & 1u)) continue;
            f32x4 sum;
#pragma unroll 1
            for (int e = 0; e < 4; ++e) {
                float v = 0.f;
                if (n + e < p.Nv) v = s2 ? conv_own_run<BF16, true>(p, Fimg, run, i16, n + e) : conv_own_run<BF16, false>(p, Fimg, run, i16, n + e);
                sum[0] = e == 0 ? v : sum[0]; sum[1] = e == 1 ? v : sum[1]; sum[2] = e == 2 ? v : sum[2]; sum[3] = e == 3 ? v : sum[3];
            }
            conv_finish<false>(p, img, row, p.bias ? p.bias[row] : 0.f, n, sum);
        }
    }
}

int32_t conv_patch_octets(int64_t Cin, int32_t H, int32_t W, int32_t kh, int32_t kw, int32_t stride) { return patch_octets(Cin, H, W, kh, kw, stride); }

grim_status launch_conv_patch(const grim_bcr_matrix *A, const ConvDense &L, const uint32_t *own_words, const void *F, int32_t Cin, int32_t H, int32_t W,
                              int32_t kh, int32_t kw, const float *bias, int32_t relu, void *Y, int32_t odt, int64_t ldy, hipStream_t stream,
                              int32_t batch, int32_t stride, int64_t f_img_stride, int64_t y_img_stride) {
    ConvPatchParams p;
    ConvForm form;
    const grim_status st = conv_gather_setup(A, F, Cin, H, W, kh, kw, bias, relu, Y, odt, ldy, batch, stride, f_img_stride,
                                             y_img_stride, own_words, 0, 0, 0, &p, &form);
    if (st != GRIM_OK) return st;
    p.own_sptr = p.sptr; p.own_plan = own_words; p.own_desc = p.desc; p.own_payload = p.payload; p.own_usteps = p.usteps;
    p.out_row = L.d_out_row;
    p.dense = L.d_weights;
    p.nbr = (int32_t)L.runs;
    p.cin = Cin;
    p.chunks = L.chunks;
    p.steps = L.steps;
    const int64_t pixels = patch_pixels(H, W, kh, kw, stride);
    p.zero_at = (int32_t)(pixels * patch_pixel_bytes(L.octets));
    // positions are walked without padding of their rows: four of them are stored at once wherever their address allows it
    p.Wp = p.Wo;
    p.Nv = p.Ho * p.Wo;
    const int wide = odt == GRIM_F32 ? 16 : 8, esz_out = odt == GRIM_F32 ? 4 : 2;
    p.yvec = reinterpret_cast<uintptr_t>(Y) % wide == 0 && ldy % 4 == 0 && (batch == 1 || (y_img_stride * esz_out) % wide == 0) ? 4 : 1;
    p.tiles_per_img = (p.Nv + 63) / 64;
    if ((int64_t)p.tiles_per_img * batch > 0x7fffffff / 16) return GRIM_ERR_SHAPE;
    p.ntiles = p.tiles_per_img * batch;
    if (((int64_t)p.ntiles + 7) / 8 * 8 * p.nbr > 0x7fffffff) return GRIM_ERR_SHAPE;
    int64_t nwg = 0;
    p.map = xcd_map(p.ntiles, p.nbr, &nwg);
    if (nwg > 0x7fffffff) return GRIM_ERR_SHAPE;
    const int waves = patch_waves(p.ntiles, p.nbr);
    p.wo_inv = divide_inverse(p.Wo);
    p.tiles_inv = divide_inverse(p.tiles_per_img);
    p.row_ones = 0;
    for (int r = 0; r < kh; ++r) p.row_ones |= 1u << (r * kw);
    p.wave_lds = p.zero_at + patch_pixel_bytes(L.octets);
    p.wave_lds = p.wave_lds < kConvTallRuns * 4096 ? kConvTallRuns * 4096 : p.wave_lds;       // the partial tiles go there later
    const size_t lds = (size_t)waves * p.wave_lds;
    // (the longest wave's steps in as few chains as may be, as long as one another)
    const int wave_steps = (L.chunks + waves - 1) / waves * L.steps, chains = (wave_steps + kPatchChain - 1) / kPatchChain;
    const bool longer = chains > 1;
    p.chain = (wave_steps + chains - 1) / chains - kPatchDepth / 2;          // (ends with the group whose end is nearest)
    p.settlings = chains - 1;
#define GRIM_PATCH(BF, CO, NW, LO)                                                                                   \
    do {                                                                                                             \
        auto kern = bcr_conv_patch<BF, CO, NW, LO>;                                                                     \
        static std::atomic<bool> attr_done{false};   /* raising a kernel's LDS limit is needed once per process */  \
        if (lds > 64 * 1024 && !attr_done) {                                                                         \
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, \
                                    160 * 1024) != hipSuccess) {                                                     \
                (void)hipGetLastError();                                                                             \
                return GRIM_ERR_DEVICE;                                                                              \
            }                                                                                                        \
            attr_done = true;                                                                                        \
        }                                                                                                            \
        hipLaunchKernelGGL(kern, dim3((unsigned)nwg), dim3(NW * 64), lds, stream, p);                                \
    } while (0)
#define GRIM_PATCH_CO(BF, CO)                                                                                        \
    if (waves == 8) { if (longer) GRIM_PATCH(BF, CO, 8, true); else GRIM_PATCH(BF, CO, 8, false); }                  \
    else { if (longer) GRIM_PATCH(BF, CO, 4, true); else GRIM_PATCH(BF, CO, 4, false); }
#define GRIM_PATCH_DT(BF) if (L.octets == 4) { GRIM_PATCH_CO(BF, 4); } else if (L.octets == 2) { GRIM_PATCH_CO(BF, 2); } else { GRIM_PATCH_CO(BF, 1); }
    if (A->dtype == GRIM_BF16) { GRIM_PATCH_DT(true) } else { GRIM_PATCH_DT(false) }
#undef GRIM_PATCH_DT
#undef GRIM_PATCH_CO
#undef GRIM_PATCH
    return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
}

}  // namespace grim
