// Planned convolution with 64 rows of the matrix to a workgroup (Section 3.1: CONV = filter matrix x im2col matrix;
// Section 4.5: rows of that matrix whose weights are all pruned are skipped; Section 4.4: a formed row is reused by all
// kept rows).
#include "conv_tall.hpp"

namespace grim {

// The fetch of bcr_conv_gather -- windows of the feature map at any alignment, shifted, masked and parked in LDS -- costs a
// wave far more than the multiplies that follow, and the 16-row runs of a matrix cut into small blocks fetch nearly the same
// rows over and over: four runs of 4 x 16 blocks that keep 4 of 16 columns name 2.7 rows for every distinct one, four of
// 8 x 16 or 16 x 16 blocks about 1.9.  Here the steps belong to runs of 64 rows (a layout the plan holds) and feed four
// 16-row multiplies each.  Bound by the latency of a step's fetch over the two waves a SIMD holds (three steps in flight
// spill; two asked for as a batch, without the rolling requests below, take 18.4 us where this takes 15.7: 256 channels,
// 3 x 3, four 28 x 28 maps in 4 x 16 blocks, 26.1 on 16-row runs).
//
// Workgroup = (tile of 64 positions, 64-row run), its waves split the run's steps.  64 accumulators and two steps in
// flight leave two waves per SIMD, so a wave covers its own latencies: a step's windows are asked for D steps ahead, into
// the registers of the step that was just parked, its weights likewise after that step's multiplies, and its slot words and
// descriptors D steps before that.
//
// A formed row meets all 64 rows of the run, with zero weights in those that do not keep it, so an infinity or NaN in the map
// would reach 64 output channels; on 16-row runs it reaches the 16 of the runs that name it.  Every sum of such a position is
// then not finite, whichever rows keep it: where a sum is not, the output is formed again from the matrix's own 16-row runs
// (conv_own_run), which costs the tiles that meet no such value nothing but the look at their sums.
template <bool BF16, bool S2, int NWV>
__global__ void __launch_bounds__(NWV * 64, 2) bcr_conv_tall(ConvTallParams p) {
    constexpr int R = kConvTallRuns, NT = 4, TN = 64, PITCH = 128, CPR = 8, LI = 4;
    constexpr int LW = S2 ? 2 : 1;               // 16-byte loads per window
    constexpr int D = 2;                         // steps in flight
    constexpr int WAVE_LDS = R * NT * 1024;      // D step buffers of 4 KB, later the partial tiles
    static_assert(D * 32 * PITCH <= WAVE_LDS, "step buffers fit");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // (most of the arguments in one trip through the scalar cache, as in bcr_conv_gather; with the table of masks made a dword per thread, without
    // divisions by run-time values: 1 x 1 at stride 2, 128 -> 256 channels on four 56 x 56 maps in 4 x 16 blocks 6.82 -> 6.67 us, 96 -> 128 on
    // three 112 x 112 7.46 -> 7.29.  Asking for the first windows ahead of that table's barrier makes the walk wait for everything: 11.0.)
    asm volatile("" ::"s"(p.map.per_tile), "s"(p.map.tail_slot0), "s"(p.map.tail_tile0), "s"(p.map.shift), "s"(p.map.per_part),
                 "s"(p.map.per_tile_inv), "s"(p.map.per_part_inv), "s"(p.ntiles), "s"(p.tiles_per_img), "s"(p.tiles_inv), "s"(p.nbr),
                 "s"(p.usteps), "s"(p.plan), "s"(p.desc), "s"(p.payload), "s"(p.F), "s"(p.f_img_stride), "s"(p.Nv), "s"(p.W), "s"(p.kw), "s"(p.KK));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile, t;
    if (!xcd_map_at(p.map, blockIdx.x, p.ntiles, &tile, &t) || t >= p.nbr) return;
    const int img = divide_by(tile, p.tiles_per_img, p.tiles_inv);
    tile -= img * p.tiles_per_img;
    const unsigned short *Fimg = p.F + (int64_t)img * p.f_img_stride;
    int n0 = tile * TN;
    if (n0 + TN > p.Nv) n0 = p.Nv - TN;          // ragged last tile: overlap the neighbour
    n0 = n0 < 0 ? 0 : n0;                        // fewer than 64 positions: one tile, its columns past them never stored
    const int g0 = p.usteps ? t * p.usteps : p.sptr[t], nst = p.usteps ? p.usteps : p.sptr[t + 1] - g0;
    const int s_beg = g0 + wave_share(nst, wave, NWV), s_end = g0 + wave_share(nst, wave + 1, NWV);
    char *buf = lds + wave * WAVE_LDS;

    const int kgroup = lane >> 4, i16 = lane & 15;
    const uint2 *desc2 = reinterpret_cast<const uint2 *>(p.desc);
    const i16x8 *pay = reinterpret_cast<const i16x8 *>(p.payload);
    // a step's slot word for k slot lane % 32 and the descriptors of this lane's group (past the last step: the last)
    struct Header { unsigned int pk; uint2 d[R]; };
    auto ask_header = [&](Header &h, int st) {
        st = st < s_end ? st : s_end - 1;
        st = st < 0 ? 0 : st;
        h.pk = p.plan[(int64_t)st * 32 + (lane & 7) * 4 + ((lane >> 3) & 3)];
#pragma unroll
        for (int m = 0; m < R; ++m) h.d[m] = desc2[((int64_t)st * R + m) * 4 + kgroup];
    };
    Header hd[D];
#pragma unroll
    for (int u = 0; u < D; ++u) ask_header(hd[u], s_beg + u);
    u32x4 *vtab = reinterpret_cast<u32x4 *>(lds + NWV * WAVE_LDS);
    const int rowlen = S2 ? p.Wp : p.W;
    for (int e = tid; e < (p.KK + 1) * CPR * 4; e += NWV * 64)
        reinterpret_cast<unsigned int *>(vtab)[e] = conv_pair_mask<S2>(p, e / (CPR * 4), n0 + e % (CPR * 4) * 2, rowlen);
    __syncthreads();

    const int rs = lane >> 3, c = lane & 7;
    const int wr_off = rs * PITCH + ((c ^ swizzle<CPR>(rs)) << 4);
    const unsigned int below = (1u << i16) - 1u;
    const int qd = i16 >> 2, ncolb = (4 * (i16 & 3)) * 2, cl = ncolb >> 4, within = ncolb & 15;
    const int r0 = kgroup * 8 + qd, r1 = r0 + 4;
    const unsigned int buf_lds = (unsigned int)(uintptr_t)(__attribute__((address_space(3))) char *)buf;
    const unsigned int tr0 = buf_lds + r0 * PITCH + within + ((cl ^ swizzle<CPR>(r0)) << 4);
    const unsigned int tr1 = buf_lds + r1 * PITCH + within + ((cl ^ swizzle<CPR>(r1)) << 4);

    const char *Fb = reinterpret_cast<const char *>(Fimg);
    const int emax = p.total - 8, centre = (p.kh >> 1) * p.W + (p.kw >> 1);
    auto pos_off = [&](int cc) { return conv_piece_start<S2>(n0 + cc * 8, p.W, p.Ho, p.Wp, p.row_inv); };       // as in bcr_conv_gather
    const int tile_pos = S2 ? __builtin_amdgcn_readfirstlane(pos_off(0)) : n0;
    const int cofs = (S2 ? pos_off(c) - tile_pos : c * 8) - (1 << 25);
    bool tile_edge = conv_tile_at_edge<S2>(pos_off(0), pos_off(CPR - 1), centre, p.N);
    if constexpr (S2) tile_edge = __builtin_amdgcn_readfirstlane(tile_edge) != 0;

    f32x4 acc[R][NT];
#pragma unroll
    for (int m = 0; m < R; ++m)
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[m][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 XW[D][LI * LW];
    unsigned int xsel[D], xext[D];               // xsel: 8 bits per window: tap (KK: padding) | odd start << 7
    i16x8 PW[D][R];

    // the windows of a step (see bcr_conv_gather: an odd start is fetched one element early, and the element behind a row
    // piece's last window comes with one extra load; SAFE: for tiles at the map's edge)
    auto fetch_rows = [&](int u, unsigned int word, auto safe_tag) {
        constexpr bool SAFE = decltype(safe_tag)::value;
        const unsigned int pk = word + (unsigned int)tile_pos;               // (the start has 27 bits, never reached)
        if constexpr (!S2) {
            const int e7 = (int)(pk & 0x7ffffffu) - (1 << 25) + (CPR - 1) * 8;
            bool need = lane < 32 && (int)(word >> 27) != p.KK && (e7 & 1);
            if constexpr (SAFE) need = need && e7 + 7 >= 0 && e7 + 7 < p.total;
            xext[u] = need ? (unsigned int)Fimg[e7 + 7] : 0u;
        }
        xsel[u] = 0u;
        int off[LI * LW];                        // SAFE: elements the load was moved by to stay inside the map
        bool moved = false;
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            const unsigned int v = (unsigned int)__shfl((int)pk, i * 8 + rs);
            const int e0 = (int)(v & 0x7ffffffu) + cofs, odd = e0 & 1;
            xsel[u] |= (v >> 27 | (unsigned int)odd << 7) << (8 * i);
#pragma unroll
            for (int l = 0; l < LW; ++l) {
                int ea = e0 - odd + 8 * l;
                if constexpr (SAFE) {
                    const int ec = ea < 0 ? 0 : ea > emax ? emax : ea;
                    off[i * LW + l] = ea - ec;
                    moved |= ea != ec;
                    ea = ec;
                }
                ConvWindow wv;
                __builtin_memcpy(&wv, Fb + (unsigned int)(ea * 2), 16);
                XW[u][i * LW + l] = u32x4{wv.d[0], wv.d[1], wv.d[2], wv.d[3]};
            }
        }
        if constexpr (SAFE) {
            if (__builtin_amdgcn_ballot_w64(moved)) {        // (first or last channel; what lies outside the map is masked)
#pragma unroll
                for (int i = 0; i < LI * LW; ++i) {
                    XW[u][i] = conv_shift(XW[u][i], off[i]);
                }
            }
        }
    };
    auto fetch_weights = [&](i16x8 (&w)[R], const Header &h) {
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const bool kept = (h.d[m].x >> i16) & 1u;
            const i16x8 wv = pay[h.d[m].y + (kept ? __builtin_popcount(h.d[m].x & below) : 0)];
            w[m] = kept ? wv : i16x8{0, 0, 0, 0, 0, 0, 0, 0};
        }
    };
    auto park = [&](int u) {
        char *b = buf + u * (32 * PITCH);
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            const unsigned int sel = (xsel[u] >> (8 * i)) & 0xffu;
            const u32x4 vm = vtab[(sel & 0x7fu) * CPR + c];
            u32x4 v;
            if constexpr (S2) {
                const unsigned int pick = sel >> 7 ? 0x07060302u : 0x05040100u;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const u32x4 f = d < 2 ? XW[u][i * LW] : XW[u][i * LW + LW - 1];
                    v[d] = __builtin_amdgcn_perm(d % 2 ? f[3] : f[1], d % 2 ? f[2] : f[0], pick) & vm[d];
                }
            } else {
                const u32x4 &f = XW[u][i * LW];
                const unsigned int sh = (sel >> 7) * 16u, w0 = f[0];
                const unsigned int nxt = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)w0, 0x101 /* row_shl:1 */, 0xf, 0xf, true);
                const unsigned int bnd = (unsigned int)__shfl((int)xext[u], i * 8 + rs);
                const unsigned int w4 = c == CPR - 1 ? bnd : nxt;
                v = u32x4{__builtin_amdgcn_alignbit(f[1], w0, sh) & vm[0], __builtin_amdgcn_alignbit(f[2], f[1], sh) & vm[1],
                          __builtin_amdgcn_alignbit(f[3], f[2], sh) & vm[2], __builtin_amdgcn_alignbit(w4, f[3], sh) & vm[3]};
            }
            *reinterpret_cast<u32x4 *>(b + wr_off + i * 8 * PITCH) = v;
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto multiply = [&](int u, const i16x8 (&w)[R]) {
        unsigned int a0 = tr0 + u * (32 * PITCH), a1 = tr1 + u * (32 * PITCH);
        asm volatile("" : "+v"(a0), "+v"(a1));
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const i16x4 lo = lds_tr_read_at(a0 ^ (unsigned int)(q << 5)), hi = lds_tr_read_at(a1 ^ (unsigned int)(q << 5));
            const i16x8 x = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
            for (int m = 0; m < R; ++m) acc[m][q] = mfma16<BF16>(x, w[m], acc[m][q]);
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto walk = [&](auto safe_tag) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            fetch_rows(u, hd[u].pk, safe_tag);
            fetch_weights(PW[u], hd[u]);
            ask_header(hd[u], s_beg + D + u);
        }
        int s = s_beg;
        for (; s + 2 * D <= s_end; s += D) {     // no condition on any load in here: a wait then counts the younger ones
#pragma unroll
            for (int u = 0; u < D; ++u) {
                park(u);
                fetch_rows(u, hd[u].pk, safe_tag);
                multiply(u, PW[u]);
                fetch_weights(PW[u], hd[u]);
                ask_header(hd[u], s + 2 * D + u);
            }
        }
        const int left = s_end - s;              // below 2 D
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (u < left) {
                park(u);
                if (D + u < left) fetch_rows(u, hd[u].pk, safe_tag);
                multiply(u, PW[u]);
                if (D + u < left) fetch_weights(PW[u], hd[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < D - 1; ++u) {
            if (D + u < left) {
                park(u);
                multiply(u, PW[u]);
            }
        }
    };
    if (s_beg < s_end) {
        if (tile_edge) walk(std::true_type{}); else walk(std::false_type{});
    }

    // the waves' partial tiles, added in wave order; the waves finish the (16-row run, sub-tile) pairs in turn (their output
    // channels and biases are asked for ahead of the barrier; at the start of the kernel they would not fit the registers)
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
    constexpr int PAIRS = R * NT / NWV;
    static_assert(R * NT % NWV == 0, "pairs are dealt evenly");
    int row[PAIRS];
    float bias[PAIRS];
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) row[j] = p.out_row[((int64_t)t * R + (wave + j * NWV) / NT) * 16 + i16];
#pragma unroll
    for (int m = 0; m < R; ++m)
#pragma unroll
        for (int q = 0; q < NT; ++q) red[wave * (WAVE_LDS / 16) + (m * NT + q) * 64 + lane] = acc[m][q];
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) bias[j] = p.bias && row[j] >= 0 ? p.bias[row[j]] : 0.f;
    __syncthreads();
    unsigned int again = 0u;                     // bit per pair: one of the lane's four sums is not finite
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        const int i = wave + j * NWV;
        f32x4 sum = red[i * 64 + lane];
#pragma unroll
        for (int w = 1; w < NWV; ++w) {
            const f32x4 v = red[w * (WAVE_LDS / 16) + i * 64 + lane];
            sum[0] += v[0]; sum[1] += v[1]; sum[2] += v[2]; sum[3] += v[3];
        }
        float nan = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) nan = __builtin_fmaf(sum[e], 0.f, nan);
        again |= nan != nan ? 1u << i : 0u;
        if (row[j] >= 0) conv_finish<S2>(p, img, row[j], bias[j], n0 + i % NT * 16 + 4 * kgroup, sum);
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
                const float v = n + e < p.Nv ? conv_own_run<BF16, S2>(p, Fimg, run, i16, n + e) : 0.f;
                sum[0] = e == 0 ? v : sum[0]; sum[1] = e == 1 ? v : sum[1]; sum[2] = e == 2 ? v : sum[2]; sum[3] = e == 3 ? v : sum[3];
            }
            conv_finish<S2>(p, img, row, p.bias ? p.bias[row] : 0.f, n, sum);
        }
    }
}

grim_status launch_conv_tall(const grim_bcr_matrix *A, const GatherLayout &L, const uint32_t *own_words, const void *F, int32_t Cin, int32_t H, int32_t W, int32_t kh,
                             int32_t kw, const float *bias, int32_t relu, void *Y, int32_t odt, int64_t ldy, hipStream_t stream,
                             int32_t batch, int32_t stride, int64_t f_img_stride, int64_t y_img_stride) {
    ConvTallParams p;
    ConvForm form;
    const grim_status st = conv_gather_setup(A, F, Cin, H, W, kh, kw, bias, relu, Y, odt, ldy, batch, stride, f_img_stride,
                                             y_img_stride, L.d_rows, 0, 0, 0, &p, &form);
    if (st != GRIM_OK) return st;
    p.own_sptr = p.sptr; p.own_plan = own_words; p.own_desc = p.desc; p.own_payload = p.payload; p.own_usteps = p.usteps;
    p.sptr = L.d_sptr;
    p.out_row = L.d_out_row;
    p.desc = L.d_desc;
    p.payload = L.d_payload;
    p.nbr = (int32_t)L.nstrips;
    p.usteps = L.usteps;
    p.tiles_per_img = (p.Nv + 63) / 64;
    p.tiles_inv = divide_inverse(p.tiles_per_img);
    p.ntiles = p.tiles_per_img * batch;
    int64_t nwg = 0;
    p.map = xcd_map(p.ntiles, p.nbr, &nwg);
    if (nwg > 0x7fffffff) return GRIM_ERR_SHAPE;
    const int waves = (int64_t)p.ntiles * p.nbr <= 256 ? 8 : 4;
    const size_t lds = (size_t)waves * kConvTallRuns * 4096 + kConvTableBytes;
#define GRIM_TALL(BF, S2, NW)                                                                                        \
    do {                                                                                                             \
        auto kern = bcr_conv_tall<BF, S2, NW>;                                                                       \
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
#define GRIM_TALL_DT(BF)                                                                                             \
    if (stride == 2) { if (waves == 8) GRIM_TALL(BF, true, 8); else GRIM_TALL(BF, true, 4); }                        \
    else { if (waves == 8) GRIM_TALL(BF, false, 8); else GRIM_TALL(BF, false, 4); }
    if (A->dtype == GRIM_BF16) { GRIM_TALL_DT(true) } else { GRIM_TALL_DT(false) }
#undef GRIM_TALL_DT
#undef GRIM_TALL
    return hipGetLastError() == hipSuccess ? GRIM_OK : GRIM_ERR_DEVICE;
}

}  // namespace grim
