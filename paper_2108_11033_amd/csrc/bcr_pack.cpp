// Host side of the library: validation, compaction of the dense matrix into the
// canonical block-compact arrays, the derived device layouts, upload, and the
// extern "C" entry points.
#include <algorithm>
#include <cstring>
#include <future>
#include <map>
#include <memory>
#include <new>
#include <numeric>
#include <system_error>

#include "bcr_matrix.hpp"
#include "conv_rules.hpp"
#include "group_rules.hpp"
#include "staged_room.hpp"

using namespace grim;

namespace {

struct Slab {
    // one device allocation holding every array of a matrix, each 256-byte aligned
    size_t total = 0;
    size_t add(size_t bytes) {
        size_t off = total;
        total += (bytes + 255) & ~size_t(255);
        return off;
    }
};

grim_status validate_sets(int64_t nb, int32_t B, const int32_t *ptr, const uint16_t *idx) {
    if (ptr[0] != 0) return GRIM_ERR_INDEX;
    for (int64_t b = 0; b < nb; ++b) {
        int64_t lo = ptr[b], hi = ptr[b + 1];
        if (hi < lo || hi - lo > B) return GRIM_ERR_INDEX;
        if (hi > lo && idx == nullptr) return GRIM_ERR_NULL;
        for (int64_t t = lo; t < hi; ++t) {
            if (idx[t] >= B) return GRIM_ERR_INDEX;
            if (t > lo && idx[t] <= idx[t - 1]) return GRIM_ERR_INDEX;
        }
    }
    return GRIM_OK;
}

// ---- derived layout: matrix-core SpMM ---------------------------------------------------

// most units any (group of strips, chunk) holds
void staged_amax(const grim_bcr_matrix *A, MmaLayout &L) {
    for (int gi = 0; gi < 4; ++gi) {
        const int64_t Gs = 4 << gi;
        int32_t amax = 0;
        for (int32_t ch = 0; ch < L.nchunks; ++ch) {
            const int32_t *bp = &L.bptr[(size_t)ch * (A->nbr + 1)];
            for (int64_t t0 = 0; t0 < A->nbr; t0 += Gs)
                amax = std::max(amax, bp[std::min<int64_t>(A->nbr, t0 + Gs)] - bp[t0]);
        }
        L.amax[gi] = amax;
    }
}

// Where the regions of a layout with groups of one block each lie (no records): false where they are too many
bool size_one_block_groups(const grim_bcr_matrix *A, MmaLayout &L, int32_t chunk_blocks) {
    L.chunk_blocks = chunk_blocks;
    L.chunk_rows = chunk_blocks * A->BC;
    L.nchunks = (int32_t)((A->nbc + chunk_blocks - 1) / chunk_blocks);
    L.ks = A->BR == 16 ? 32 : 16;
    const int32_t ng = L.ks / 8, hdr = L.ks * 2 + ng * 8;
    L.bptr.assign((size_t)L.nchunks * (A->nbr + 1), 0);
    int64_t units = 0;
    for (int32_t ch = 0; ch < L.nchunks; ++ch) {
        const int64_t c0 = (int64_t)ch * chunk_blocks, c1 = std::min<int64_t>(A->nbc, c0 + chunk_blocks);
        for (int64_t st = 0; st <= A->nbr; ++st) {
            L.bptr[(size_t)ch * (A->nbr + 1) + st] = (int32_t)units;
            if (st == A->nbr) break;
            int64_t groups = 0;
            for (int64_t t = st * A->nbc + c0; t < st * A->nbc + c1; ++t) {
                const int32_t kr = A->row_ptr[t + 1] - A->row_ptr[t], kc = A->col_ptr[t + 1] - A->col_ptr[t];
                if (kr == 0) continue;
                groups += (kc + 7) / 8;
                units += (int64_t)((kc + 7) / 8) * kr;
            }
            units += (groups + ng - 1) / ng * hdr / 16;
        }
        if (units >= int64_t(1) << 31) return false;
    }
    staged_amax(A, L);
    return true;
}

// packed: the kept columns of a (chunk, strip) one after the other, eight to a group whichever blocks they belong to; otherwise a
// block's columns begin a group
bool build_mma_layout_for(grim_bcr_matrix *A, MmaLayout &L, int32_t chunk_blocks, bool packed) {
    L.chunk_blocks = chunk_blocks;
    L.chunk_rows = L.chunk_blocks * A->BC;
    L.nchunks = (int32_t)((A->nbc + L.chunk_blocks - 1) / L.chunk_blocks);
    L.ks = A->BR == 16 ? 32 : 16;
    const int32_t ng = L.ks / 8;                       // groups of 8 k slots per step
    const int32_t hdr = L.ks * 2 + ng * 8;             // header bytes per step (a multiple of 16)
    L.cptr.assign((size_t)L.nchunks * (A->nbr + 1), 0);
    L.bptr.assign((size_t)L.nchunks * (A->nbr + 1), 0);
    L.recs.clear();
    L.recs.reserve(A->weights.size() * 5 / 4 + A->col_idx.size() * 3);
    const uint16_t *w = reinterpret_cast<const uint16_t *>(A->weights.data());
    const uint16_t zero_row = (uint16_t)L.chunk_rows;
    int64_t step = 0;
    uint16_t dense[32][8] = {};                        // weights of the group being filled
    uint16_t rows[8];                                  // its staged rows
    uint32_t rowmask = 0;
    int32_t slots = 0;
    size_t region0 = 0, group = 0;
    auto flush_group = [&]() {
        if (slots == 0) return;
        const size_t q = group++, p0 = L.recs.size();
        L.recs.resize(p0 + (size_t)__builtin_popcount(rowmask) * 16);
        unsigned char *h = L.recs.data() + region0 + q / ng * hdr, *dst = L.recs.data() + p0;
        // slot rows: quad qd of the group pairs slot qd with slot qd + 4
        uint16_t *hs = reinterpret_cast<uint16_t *>(h) + q % ng * 8;
        for (int32_t e = 0; e < slots; ++e) hs[e < 4 ? 2 * e : 2 * (e - 4) + 1] = rows[e];
        uint32_t *hd = reinterpret_cast<uint32_t *>(h + L.ks * 2) + q % ng * 2;
        hd[0] = rowmask;
        hd[1] = (uint32_t)((p0 - region0) / 16);
        for (uint32_t m = rowmask; m; m &= m - 1, dst += 16) {
            uint16_t *r = dense[__builtin_ctz(m)];
            std::memcpy(dst, r, 16);
            std::memset(r, 0, 16);
        }
        rowmask = 0;
        slots = 0;
    };
    for (int32_t ch = 0; ch < L.nchunks; ++ch) {
        const int64_t c0 = (int64_t)ch * L.chunk_blocks, c1 = std::min<int64_t>(A->nbc, c0 + L.chunk_blocks);
        for (int64_t st = 0; st < A->nbr; ++st) {
            L.cptr[(size_t)ch * (A->nbr + 1) + st] = (int32_t)step;
            L.bptr[(size_t)ch * (A->nbr + 1) + st] = (int32_t)(L.recs.size() / 16);
            int64_t cols = 0, groups = 0;
            for (int64_t t = st * A->nbc + c0; t < st * A->nbc + c1; ++t) {
                if (A->row_ptr[t + 1] == A->row_ptr[t]) continue;       // nothing to multiply
                const int32_t kc = A->col_ptr[t + 1] - A->col_ptr[t];
                cols += kc;
                groups += (kc + 7) / 8;
            }
            if (packed) groups = (cols + 7) / 8;
            const size_t nst = (size_t)((groups + ng - 1) / ng);
            region0 = L.recs.size();
            group = 0;
            L.recs.resize(region0 + nst * hdr, 0);
            for (size_t s = 0; s < nst; ++s) {
                uint16_t *hs = reinterpret_cast<uint16_t *>(L.recs.data() + region0 + s * hdr);
                std::fill(hs, hs + L.ks, zero_row);
            }
            for (int64_t c = c0; c < c1; ++c) {
                const int64_t t = st * A->nbc + c;
                const int32_t r0 = A->row_ptr[t], r1 = A->row_ptr[t + 1], k0 = A->col_ptr[t], kc = A->col_ptr[t + 1] - k0;
                if (r0 == r1) continue;
                for (int32_t j = 0; j < kc;) {
                    const int32_t n = std::min<int32_t>(kc - j, 8 - slots);
                    for (int32_t e = 0; e < n; ++e) rows[slots + e] = (uint16_t)((c - c0) * A->BC + A->col_idx[k0 + j + e]);
                    const uint16_t *src = w + A->blk_ptr[t] + j;
                    for (int32_t q = r0; q < r1; ++q, src += kc) {
                        rowmask |= 1u << A->row_idx[q];
                        std::memcpy(&dense[A->row_idx[q]][slots], src, (size_t)n * 2);
                    }
                    slots += n;
                    j += n;
                    if (slots == 8) flush_group();
                }
                if (!packed) flush_group();
            }
            flush_group();
            step += (int64_t)nst;
        }
        L.cptr[(size_t)ch * (A->nbr + 1) + A->nbr] = (int32_t)step;
        L.bptr[(size_t)ch * (A->nbr + 1) + A->nbr] = (int32_t)(L.recs.size() / 16);
    }
    L.nsteps = step;
    staged_amax(A, L);
    return L.recs.size() < (size_t(1) << 31) * 16;
}

// max_rows: most rows of X per chunk; gsel / max_group_bytes: the records of a group of 4 << gsel strips must fit
// max_group_bytes per chunk (the kernel's LDS room for them)
void build_mma_layout(grim_bcr_matrix *A, MmaLayout &L, int32_t chunk_rows_opt, int32_t max_rows, int gsel,
                      int64_t max_group_bytes, bool wide) {
    L.present = false;
    if (A->dtype == GRIM_F32) return;
    if (A->BR != 16 && A->BR != 32) return;
    if (A->BC > max_rows) return;
    const int32_t want = chunk_rows_opt > 0 ? std::min<int32_t>(chunk_rows_opt, max_rows) : max_rows;
    const auto fits = [&](const MmaLayout &R) { return R.chunk_rows <= max_rows && (int64_t)R.amax[gsel] * 16 <= max_group_bytes; };
    // largest chunk whose weight records still leave room in LDS; denser matrices get smaller chunks.  Groups that several blocks
    // share store the rows of all of them, so they take fewer steps and, at some kept counts, more room (512 x 4608 of mixed rates in 32 x 32
    // blocks: 7 % more): they are taken where they have room in every launch form that groups of one block each would have room in.
    const int32_t most = std::max<int32_t>(1, want / A->BC);
    MmaLayout one;
    int32_t blocks = most;
    bool any = size_one_block_groups(A, one, blocks) && fits(one);
    while (!any && blocks > 1) {
        blocks = (blocks + 1) / 2;
        any = size_one_block_groups(A, one, blocks) && fits(one);
    }
    bool done = false;
    for (int32_t b = most; !done && b >= blocks; b = (b + 1) / 2) {
        done = build_mma_layout_for(A, L, b, true) && fits(L) && (!any || fits_wherever(L, one, A->BR, A->K, wide));
        if (b == 1) break;
    }
    if (!done && any) done = build_mma_layout_for(A, L, blocks, false);
    if (!done) {   // even one column block per chunk overflows LDS: leave this matrix to the FMA kernel
        L.cptr.clear(); L.bptr.clear(); L.recs.clear();
        return;
    }
    L.present = true;
}

// ---- derived layout: row-gathering SpMM ----------------------------------------------------
// The steps of the runs u0 .. u1 - 1 of 16 R rows, numbered from zero.
struct GatherChunk {
    std::vector<int64_t> steps;           // per run
    std::vector<uint32_t> rows, desc;
    std::vector<unsigned char> payload;
    int64_t nsteps = 0, xrows = 0;
};
template <int R>
bool build_gather_runs(const grim_bcr_matrix *A, int64_t u0, int64_t u1, GatherChunk &C) {
    constexpr int HEIGHT = 16 * R;
    const uint16_t *w = reinterpret_cast<const uint16_t *>(A->weights.data());
    // A group is the next eight distinct columns that any row of the run keeps, whichever strip and block they belong to:
    // the strips of a run of small blocks meet in shared columns, and a block that keeps a number of columns that is not
    // a multiple of eight leaves no padding behind.
    const int64_t most_strips = std::max<int64_t>(1, HEIGHT / A->BR);        // strips that reach into a run
    struct Part {                                                        // a strip's block in the current column block
        int64_t base;                                                    // its first row, from the run's first
        const uint16_t *q0, *q1, *col, *end, *w;                         // kept rows; next and last kept column; its weights
        int32_t kc;
    };
    std::vector<Part> parts((size_t)most_strips);
    uint16_t dense[HEIGHT][8];                                            // weights of the group being filled
    uint64_t rowmask = 0;
    uint32_t slots = 0, cols[8];
    int64_t ngroups = 0;
    auto flush_group = [&]() {
        if (slots == 0) return true;
        const size_t gi = (size_t)ngroups++, step = gi / 4, g = gi % 4;
        if (g == 0) {
            if ((uint64_t)C.nsteps >= 0x7fffffffu) return false;
            ++C.nsteps;
            C.rows.resize((step + 1) * 32, 0xffffffffu);
            C.desc.resize((step + 1) * 8 * R, 0u);
        }
        const size_t pl0 = C.payload.size();
        if (pl0 / 16 + HEIGHT > 0xffffffffu) return false;
        for (uint32_t j = 0; j < slots; ++j) C.rows[step * 32 + (size_t)j * 4 + g] = cols[j];
        C.payload.resize(pl0 + (size_t)__builtin_popcountll(rowmask) * 16);
        unsigned char *dst = C.payload.data() + pl0;
        for (int32_t m = 0; m < R; ++m) {
            const uint32_t mask = (uint32_t)(rowmask >> (16 * m)) & 0xffffu;
            C.desc[(step * R + m) * 8 + g * 2] = mask;
            C.desc[(step * R + m) * 8 + g * 2 + 1] = mask ? (uint32_t)((dst - C.payload.data()) / 16) : 0u;
            for (int32_t r = 0; r < 16; ++r)
                if ((mask >> r) & 1u) { std::memcpy(dst, dense[16 * m + r], 16); dst += 16; }
        }
        C.xrows += slots;
        std::memset(dense, 0, sizeof(dense));
        rowmask = 0;
        slots = 0;
        return true;
    };
    std::memset(dense, 0, sizeof(dense));
    // (an estimate, so that the arrays grow once: every group full)
    const int64_t nss = (A->M + HEIGHT - 1) / HEIGHT;
    const size_t share = (size_t)((nss + u1 - u0 - 1) / (u1 - u0));
    const size_t steps_about = (A->BR >= 16 ? A->col_idx.size() * (size_t)std::max(1, A->BR / HEIGHT) : A->col_idx.size()) / 32 / share + (size_t)(u1 - u0);
    C.rows.reserve(steps_about * 32);
    C.desc.reserve(steps_about * 8 * R);
    C.payload.reserve(A->weights.size() / share * 5 / 4);
    for (int64_t u = u0; u < u1; ++u) {
        C.steps.push_back(-C.nsteps);
        ngroups = C.nsteps * 4;                                              // a run starts with a step of its own
        const int64_t row0 = u * HEIGHT, row1 = std::min<int64_t>(A->M, row0 + HEIGHT);
        const int64_t p0 = row0 / A->BR, np = (row1 - 1) / A->BR - p0 + 1;   // stored strips that overlap this run
        if (np == 1) {
            // one strip: a block's columns in turn, as many at a time as the group has room for
            for (int64_t c = 0; c < A->nbc; ++c) {
                const int64_t t = p0 * A->nbc + c, base = p0 * A->BR;
                int32_t q0 = A->row_ptr[t], q1 = A->row_ptr[t + 1];
                while (q0 < q1 && base + A->row_idx[q0] < row0) ++q0;
                while (q0 < q1 && base + A->row_idx[q1 - 1] >= row1) --q1;
                if (q0 == q1) continue;
                const int32_t c0 = A->col_ptr[t], kc = A->col_ptr[t + 1] - c0;
                for (int32_t j = 0; j < kc;) {
                    const int32_t n = std::min<int32_t>(kc - j, 8 - (int32_t)slots);
                    for (int32_t e = 0; e < n; ++e) cols[slots + e] = (uint32_t)(c * A->BC + A->col_idx[c0 + j + e]);
                    for (int32_t q = q0; q < q1; ++q) {
                        const int64_t r = base + A->row_idx[q] - row0;
                        rowmask |= uint64_t(1) << r;
                        std::memcpy(&dense[r][slots], w + A->blk_ptr[t] + (int64_t)(q - A->row_ptr[t]) * kc + j, (size_t)n * 2);
                    }
                    slots += (uint32_t)n;
                    j += n;
                    if (slots == 8 && !flush_group()) return false;
                }
            }
            if (!flush_group()) return false;
            C.steps.back() += C.nsteps;
            continue;
        }
        for (int64_t c = 0; c < A->nbc; ++c) {
            for (int64_t i = 0; i < np; ++i) {
                const int64_t t = (p0 + i) * A->nbc + c;
                Part &pt = parts[(size_t)i];
                pt.base = (p0 + i) * A->BR - row0;
                pt.q0 = A->row_idx.data() + A->row_ptr[t];
                pt.q1 = A->row_idx.data() + A->row_ptr[t + 1];
                pt.kc = A->col_ptr[t + 1] - A->col_ptr[t];
                pt.col = A->col_idx.data() + A->col_ptr[t];
                pt.end = pt.q0 == pt.q1 ? pt.col : pt.col + pt.kc;           // (no kept row: its columns do not count)
                pt.w = w + A->blk_ptr[t];
            }
            for (;;) {
                int32_t col = 0x7fffffff;
                for (int64_t i = 0; i < np; ++i)
                    if (parts[(size_t)i].col < parts[(size_t)i].end) col = std::min<int32_t>(col, *parts[(size_t)i].col);
                if (col == 0x7fffffff) break;
                for (int64_t i = 0; i < np; ++i) {
                    Part &pt = parts[(size_t)i];
                    if (pt.col >= pt.end || *pt.col != col) continue;
                    const uint16_t *pw = pt.w++;                             // the column's weights, kc apart
                    ++pt.col;
                    for (const uint16_t *q = pt.q0; q < pt.q1; ++q, pw += pt.kc) {
                        rowmask |= uint64_t(1) << (pt.base + *q);
                        dense[pt.base + *q][slots] = *pw;
                    }
                }
                cols[slots++] = (uint32_t)(c * A->BC + col);
                if (slots == 8 && !flush_group()) return false;
            }
        }
        if (!flush_group()) return false;
        C.steps.back() += C.nsteps;
    }
    return true;
}

// The layout of runs of 16 R rows (R = 1: the matrix's own; R = 4: a convolution plan's, desc and masks per 16 rows).
// L is left empty where the matrix does not have it.
template <int R>
void build_gather_layout(const grim_bcr_matrix *A, GatherLayout &L) {
    constexpr int HEIGHT = 16 * R;
    L = GatherLayout();
    // Block heights that divide 16 or are multiples of 16 map onto 16-row MFMA tiles: stored rows
    // (stored strip p, local row r) are numbered p * BR + r and cut into runs of 16.
    if (A->dtype == GRIM_F32 || A->K > 0x7fffffff || A->M > 0x7fffffff) return;
    if (!(HEIGHT % A->BR == 0 || A->BR % HEIGHT == 0)) return;
    const int64_t nss = (A->M + HEIGHT - 1) / HEIGHT;     // runs of the stored order
    L.nstrips = nss;
    L.sptr.assign((size_t)nss + 1, 0);
    L.out_row.assign((size_t)nss * HEIGHT, -1);
    for (int64_t p = 0; p < A->nbr; ++p)
        for (int32_t r = 0; r < A->BR; ++r)
            L.out_row[(size_t)(p * A->BR + r)] = (int32_t)((int64_t)A->strip_order[p] * A->BR + r);
    // Runs are independent of one another: with enough to write, in four parts side by side (4096 x 4096 of mixed rates:
    // the whole pack 20 -> 12 ms)
    const int64_t parts = A->nnz >= 32 * 1024 && nss >= 8 ? 4 : 1;
    std::vector<GatherChunk> chunk((size_t)parts);
    std::vector<std::future<bool>> done((size_t)parts);
    auto build = [&](int64_t i) { return build_gather_runs<R>(A, nss * i / parts, nss * (i + 1) / parts, chunk[(size_t)i]); };
    for (int64_t i = 1; i < parts; ++i) {
        try {
            done[(size_t)i] = std::async(std::launch::async, build, i);
        } catch (const std::system_error &) {           // no thread to be had
        }
    }
    bool ok = true;
    std::exception_ptr failed;
    for (int64_t i = 0; i < parts; ++i) {               // (every thread is waited for before anything it writes goes away)
        try {
            ok = (done[(size_t)i].valid() ? done[(size_t)i].get() : build(i)) && ok;
        } catch (...) {
            failed = std::current_exception();
        }
    }
    if (failed) std::rethrow_exception(failed);
    int64_t nsteps = 0;
    size_t payload = 0;
    for (const GatherChunk &C : chunk) { nsteps += C.nsteps; payload += C.payload.size(); L.xrows += C.xrows; }
    if (!ok || nsteps > 0x7fffffff || payload / 16 > 0xffffffffu) { L = GatherLayout(); return; }
    L.nsteps = nsteps;
    if (parts == 1) {
        L.rows = std::move(chunk[0].rows); L.desc = std::move(chunk[0].desc); L.payload = std::move(chunk[0].payload);
    } else {
        L.rows.reserve((size_t)nsteps * 32);
        L.desc.reserve((size_t)nsteps * 8 * R);
        L.payload.reserve(payload);
        for (GatherChunk &C : chunk) {
            const uint32_t at = (uint32_t)(L.payload.size() / 16);
            for (size_t i = 1; i < C.desc.size(); i += 2) C.desc[i] += at;
            L.rows.insert(L.rows.end(), C.rows.begin(), C.rows.end());
            L.desc.insert(L.desc.end(), C.desc.begin(), C.desc.end());
            L.payload.insert(L.payload.end(), C.payload.begin(), C.payload.end());
        }
    }
    int64_t at = 0, u = 0;
    for (const GatherChunk &C : chunk)
        for (int64_t n : C.steps) { L.sptr[(size_t)u++] = (int32_t)at; at += n; }
    L.sptr[(size_t)nss] = (int32_t)L.nsteps;
    L.usteps = nss > 0 ? L.sptr[1] - L.sptr[0] : 0;
    for (u = 0; u < nss && L.usteps > 0; ++u)
        if (L.sptr[(size_t)u + 1] - L.sptr[(size_t)u] != L.usteps) L.usteps = 0;
    L.max_steps = 0;
    for (u = 0; u < nss; ++u) L.max_steps = std::max<int32_t>(L.max_steps, L.sptr[(size_t)u + 1] - L.sptr[(size_t)u]);
    L.present = true;
}

// The steps the layout of R-run strips would have, without writing it.
struct RunSteps {
    int64_t total = 0;
    int32_t longest = 0;
    int64_t runs = 0;
};
template <int R>
RunSteps count_run_steps(const grim_bcr_matrix *A) {
    constexpr int HEIGHT = 16 * R;
    RunSteps n;
    if (!(HEIGHT % A->BR == 0 || A->BR % HEIGHT == 0)) return n;
    n.runs = (A->M + HEIGHT - 1) / HEIGHT;
    std::vector<uint64_t> met((size_t)(A->BC + 63) / 64);                    // columns of a block that a strip of the run keeps
    for (int64_t u = 0; u < n.runs; ++u) {
        const int64_t row0 = u * HEIGHT, row1 = std::min<int64_t>(A->M, row0 + HEIGHT);
        const int64_t p0 = row0 / A->BR, p1 = (row1 - 1) / A->BR;
        int64_t columns = 0;
        for (int64_t c = 0; c < A->nbc; ++c) {
            std::fill(met.begin(), met.end(), uint64_t(0));
            for (int64_t p = p0; p <= p1; ++p) {
                const int64_t t = p * A->nbc + c;
                int32_t q0 = A->row_ptr[t], q1 = A->row_ptr[t + 1];
                while (q0 < q1 && p * A->BR + A->row_idx[q0] < row0) ++q0;
                while (q0 < q1 && p * A->BR + A->row_idx[q1 - 1] >= row1) --q1;
                if (q0 == q1) continue;
                for (int32_t j = A->col_ptr[t]; j < A->col_ptr[t + 1]; ++j) met[(size_t)A->col_idx[j] / 64] |= uint64_t(1) << (A->col_idx[j] % 64);
            }
            for (uint64_t w : met) columns += __builtin_popcountll(w);
        }
        const int64_t steps = (columns + 31) / 32;
        n.total += steps;
        n.longest = (int32_t)std::max<int64_t>(n.longest, steps);
    }
    return n;
}

// ---- derived layout: row-gathering SpMM, fp32 ------------------------------------------------
// A block's kept columns in groups of four (a group never holds columns of two blocks: the row mask then says exactly
// which rows keep its columns).
void build_gather32_layout(grim_bcr_matrix *A) {
    GatherLayout &L = A->gather32;
    L = GatherLayout();
    if (A->dtype != GRIM_F32 || A->K > 0x7fffffff || A->M > 0x7fffffff) return;
    if (!(16 % A->BR == 0 || A->BR % 16 == 0) || A->BR > 64) return;         // (taller blocks: no fp32 kernel takes them)
    const float *w = reinterpret_cast<const float *>(A->weights.data());
    const int64_t nss = (A->M + 15) / 16;
    L.nstrips = nss;
    L.sptr.assign((size_t)nss + 1, 0);
    L.out_row.assign((size_t)nss * 16, -1);
    for (int64_t p = 0; p < A->nbr; ++p)
        for (int32_t r = 0; r < A->BR; ++r)
            L.out_row[(size_t)(p * A->BR + r)] = (int32_t)((int64_t)A->strip_order[p] * A->BR + r);
    size_t units = 0;                                                        // 16-byte units of payload written
    L.payload.reserve(A->weights.size() + A->weights.size() / 8);
    for (int64_t u = 0; u < nss; ++u) {
        L.sptr[(size_t)u] = (int32_t)L.nsteps;
        int g = 4;                                                           // next group of the last step
        const int64_t row0 = u * 16, row1 = std::min<int64_t>(A->M, row0 + 16);
        const int64_t p0 = row0 / A->BR, p1 = (row1 - 1) / A->BR;            // stored strips that overlap this run
        for (int64_t c = 0; c < A->nbc; ++c) {
            for (int64_t p = p0; p <= p1; ++p) {
                const int64_t t = p * A->nbc + c, base = p * A->BR;
                int32_t q0 = A->row_ptr[t], q1 = A->row_ptr[t + 1];
                while (q0 < q1 && base + A->row_idx[q0] < row0) ++q0;
                while (q0 < q1 && base + A->row_idx[q1 - 1] >= row1) --q1;
                if (q0 == q1) continue;
                const int32_t c0 = A->col_ptr[t], kc = A->col_ptr[t + 1] - c0;
                uint32_t rowmask = 0;
                for (int32_t q = q0; q < q1; ++q) rowmask |= 1u << (base + A->row_idx[q] - row0);
                for (int32_t j = 0; j < kc; j += 4) {
                    if (g == 4) {
                        if (L.nsteps >= 0x7fffffff) { L = GatherLayout(); return; }
                        ++L.nsteps;
                        L.rows.resize((size_t)L.nsteps * 16, 0xffffffffu);
                        L.desc.resize((size_t)L.nsteps * 8, 0u);
                        g = 0;
                    }
                    const int32_t n = std::min<int32_t>(4, kc - j);
                    const size_t step = (size_t)L.nsteps - 1;
                    for (int32_t e = 0; e < n; ++e) L.rows[step * 16 + (size_t)g * 4 + e] = (uint32_t)(c * A->BC + A->col_idx[c0 + j + e]);
                    if (units + 16 > 0xffffffffu) { L = GatherLayout(); return; }
                    L.desc[step * 8 + (size_t)g * 2] = rowmask;
                    L.desc[step * 8 + (size_t)g * 2 + 1] = (uint32_t)units;
                    L.payload.resize((units + (size_t)(q1 - q0)) * 16);
                    for (int32_t q = q0; q < q1; ++q, ++units)
                        std::memcpy(L.payload.data() + units * 16, w + A->blk_ptr[t] + (int64_t)(q - A->row_ptr[t]) * kc + j, (size_t)n * 4);
                    L.xrows += n;
                    ++g;
                }
            }
        }
    }
    L.sptr[(size_t)nss] = (int32_t)L.nsteps;
    L.usteps = L.sptr[1];
    for (int64_t u = 0; u < nss; ++u) {
        const int32_t n = L.sptr[(size_t)u + 1] - L.sptr[(size_t)u];
        if (n != L.usteps) L.usteps = 0;
        L.max_steps = std::max<int32_t>(L.max_steps, n);
    }
    L.present = true;
}

// ---- derived layout: SpMV --------------------------------------------------------------
void build_gemv_layout(grim_bcr_matrix *A) {
    GemvLayout &G = A->gemv;
    G.present = false;
    G.krmax = G.kcmax = 0;
    if (A->BR > 32 || A->BC > 32) return;
    if (A->nnz >= (int64_t(1) << 31)) return;
    G.masks.assign((size_t)A->nb * 2, 0);
    G.woff.resize((size_t)A->nb + 1);
    int32_t ukr = -2, ukc = -2;
    int32_t vec = 8;
    for (int64_t t = 0; t < A->nb; ++t) {
        uint32_t rm = 0, cm = 0;
        for (int32_t q = A->row_ptr[t]; q < A->row_ptr[t + 1]; ++q) rm |= 1u << A->row_idx[q];
        for (int32_t q = A->col_ptr[t]; q < A->col_ptr[t + 1]; ++q) cm |= 1u << A->col_idx[q];
        int32_t kr = A->row_ptr[t + 1] - A->row_ptr[t], kc = A->col_ptr[t + 1] - A->col_ptr[t];
        if (kr == 0 || kc == 0) { rm = 0; cm = 0; kr = 0; kc = 0; }   // stores nothing
        G.masks[2 * t] = rm;
        G.masks[2 * t + 1] = cm;
        G.woff[t] = (uint32_t)A->blk_ptr[t];
        ukr = ukr == -2 ? kr : (ukr == kr ? ukr : -1);
        ukc = ukc == -2 ? kc : (ukc == kc ? ukc : -1);
        if (kr > 0) while (vec > 1 && kc % vec) vec >>= 1;
        G.krmax = std::max(G.krmax, kr);
        G.kcmax = std::max(G.kcmax, kc);
    }
    G.woff[A->nb] = (uint32_t)A->blk_ptr[A->nb];
    G.uniform_kr = ukr < 0 ? -1 : ukr;
    G.uniform_kc = ukc < 0 ? -1 : ukc;
    if (G.uniform_kr < 0 || G.uniform_kc < 0) G.uniform_kr = G.uniform_kc = -1;
    G.vec = std::min<int32_t>(vec, 16 / dtype_size(A->dtype));
    G.present = true;
}

grim_status upload(grim_bcr_matrix *A) {
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) { (void)hipGetLastError(); return GRIM_ERR_DEVICE; }
    if (hipGetDevice(&A->device) != hipSuccess) return GRIM_ERR_DEVICE;
    Slab s;
    auto bytes = [](const auto &v) { return v.size() * sizeof(v[0]); };
    std::vector<int32_t> strip_pos((size_t)A->nbr);
    for (int64_t q = 0; q < A->nbr; ++q) strip_pos[(size_t)A->strip_order[q]] = (int32_t)q;
    A->order_identity = true;
    for (int64_t q = 0; q < A->nbr; ++q) A->order_identity = A->order_identity && A->strip_order[q] == q;
    size_t o_so = s.add(bytes(A->strip_order));
    size_t o_sp = s.add(bytes(strip_pos));
    size_t o_rp = s.add(bytes(A->row_ptr));
    size_t o_ri = s.add(bytes(A->row_idx));
    size_t o_cp = s.add(bytes(A->col_ptr));
    size_t o_ci = s.add(bytes(A->col_idx));
    size_t o_bp = s.add(bytes(A->blk_ptr));
    size_t o_w = s.add(A->weights.size() + 64);   // slack: vector loads may overrun a row's end
    size_t o_rm = s.add(bytes(A->rowmask64));
    size_t canon_end = s.total;
    size_t o_kp = 0, o_bp2 = 0, o_af = 0, o_gm = 0, o_go = 0;
    if (A->mma.present) {
        o_kp = s.add(bytes(A->mma.cptr));
        o_bp2 = s.add(bytes(A->mma.bptr));
        o_af = s.add(bytes(A->mma.recs) + 2048);   // slack: records are fetched in 1 KB slots
    }
    size_t o_wkp = 0, o_wbp = 0, o_waf = 0;
    if (A->mmaw.present) {
        o_wkp = s.add(bytes(A->mmaw.cptr));
        o_wbp = s.add(bytes(A->mmaw.bptr));
        o_waf = s.add(bytes(A->mmaw.recs) + 2048);
    }
    size_t o_gs = 0, o_gq = 0, o_gr = 0, o_gd = 0, o_gp = 0;
    if (A->gather.present) {
        o_gs = s.add(bytes(A->gather.sptr));
        o_gq = s.add(bytes(A->gather.out_row));
        o_gr = s.add(bytes(A->gather.rows) + 16);
        o_gd = s.add(bytes(A->gather.desc) + 16);
        o_gp = s.add(bytes(A->gather.payload) + 16);
    }
    size_t o_hs = 0, o_hq = 0, o_hr = 0, o_hd = 0, o_hp = 0;
    if (A->gather32.present) {
        o_hs = s.add(bytes(A->gather32.sptr));
        o_hq = s.add(bytes(A->gather32.out_row));
        o_hr = s.add(bytes(A->gather32.rows));
        o_hd = s.add(bytes(A->gather32.desc));
        o_hp = s.add(bytes(A->gather32.payload) + 16);
    }
    size_t mma_end = s.total;
    if (A->gemv.present) {
        o_gm = s.add(bytes(A->gemv.masks));
        o_go = s.add(bytes(A->gemv.woff));
    }
    char *base = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&base), s.total + 256) != hipSuccess) { (void)hipGetLastError(); return GRIM_ERR_ALLOC; }
    if (hipMemset(base, 0, s.total + 256) != hipSuccess) { (void)hipFree(base); return GRIM_ERR_DEVICE; }
    auto put = [&](size_t off, const void *src, size_t n) -> bool {
        return n == 0 || hipMemcpy(base + off, src, n, hipMemcpyHostToDevice) == hipSuccess;
    };
    bool ok = put(o_so, A->strip_order.data(), bytes(A->strip_order)) && put(o_sp, strip_pos.data(), bytes(strip_pos)) && put(o_rp, A->row_ptr.data(), bytes(A->row_ptr)) &&
              put(o_ri, A->row_idx.data(), bytes(A->row_idx)) && put(o_cp, A->col_ptr.data(), bytes(A->col_ptr)) &&
              put(o_ci, A->col_idx.data(), bytes(A->col_idx)) && put(o_bp, A->blk_ptr.data(), bytes(A->blk_ptr)) &&
              put(o_w, A->weights.data(), A->weights.size()) && put(o_rm, A->rowmask64.data(), bytes(A->rowmask64));
    if (ok && A->mma.present)
        ok = put(o_kp, A->mma.cptr.data(), bytes(A->mma.cptr)) && put(o_bp2, A->mma.bptr.data(), bytes(A->mma.bptr)) &&
             put(o_af, A->mma.recs.data(), bytes(A->mma.recs));
    if (ok && A->mmaw.present)
        ok = put(o_wkp, A->mmaw.cptr.data(), bytes(A->mmaw.cptr)) && put(o_wbp, A->mmaw.bptr.data(), bytes(A->mmaw.bptr)) &&
             put(o_waf, A->mmaw.recs.data(), bytes(A->mmaw.recs));
    if (ok && A->gather.present)
        ok = put(o_gs, A->gather.sptr.data(), bytes(A->gather.sptr)) && put(o_gq, A->gather.out_row.data(), bytes(A->gather.out_row)) && put(o_gr, A->gather.rows.data(), bytes(A->gather.rows)) &&
             put(o_gd, A->gather.desc.data(), bytes(A->gather.desc)) && put(o_gp, A->gather.payload.data(), bytes(A->gather.payload));
    if (ok && A->gather32.present)
        ok = put(o_hs, A->gather32.sptr.data(), bytes(A->gather32.sptr)) && put(o_hq, A->gather32.out_row.data(), bytes(A->gather32.out_row)) && put(o_hr, A->gather32.rows.data(), bytes(A->gather32.rows)) &&
             put(o_hd, A->gather32.desc.data(), bytes(A->gather32.desc)) && put(o_hp, A->gather32.payload.data(), bytes(A->gather32.payload));
    if (ok && A->gemv.present)
        ok = put(o_gm, A->gemv.masks.data(), bytes(A->gemv.masks)) && put(o_go, A->gemv.woff.data(), bytes(A->gemv.woff));
    if (!ok) { (void)hipGetLastError(); (void)hipFree(base); return GRIM_ERR_DEVICE; }
    A->dev.strip_order = reinterpret_cast<int32_t *>(base + o_so);
    A->dev.strip_pos = reinterpret_cast<int32_t *>(base + o_sp);
    A->dev.row_ptr = reinterpret_cast<int32_t *>(base + o_rp);
    A->dev.row_idx = reinterpret_cast<uint16_t *>(base + o_ri);
    A->dev.col_ptr = reinterpret_cast<int32_t *>(base + o_cp);
    A->dev.col_idx = reinterpret_cast<uint16_t *>(base + o_ci);
    A->dev.blk_ptr = reinterpret_cast<int64_t *>(base + o_bp);
    A->dev.weights = base + o_w;
    A->dev.rowmask64 = reinterpret_cast<uint64_t *>(base + o_rm);
    A->dev.bytes = (int64_t)canon_end;
    if (A->mma.present) {
        A->mma.d_cptr = reinterpret_cast<int32_t *>(base + o_kp);
        A->mma.d_bptr = reinterpret_cast<int32_t *>(base + o_bp2);
        A->mma.d_recs = reinterpret_cast<unsigned char *>(base + o_af);
        A->mma.bytes = (int64_t)(mma_end - canon_end);
    }
    if (A->mmaw.present) {
        A->mmaw.d_cptr = reinterpret_cast<int32_t *>(base + o_wkp);
        A->mmaw.d_bptr = reinterpret_cast<int32_t *>(base + o_wbp);
        A->mmaw.d_recs = reinterpret_cast<unsigned char *>(base + o_waf);
        A->mmaw.bytes = (int64_t)(bytes(A->mmaw.cptr) + bytes(A->mmaw.bptr) + bytes(A->mmaw.recs));
    }
    if (A->gather.present) {
        A->gather.d_sptr = reinterpret_cast<int32_t *>(base + o_gs);
        A->gather.d_out_row = reinterpret_cast<int32_t *>(base + o_gq);
        A->gather.d_rows = reinterpret_cast<uint32_t *>(base + o_gr);
        A->gather.d_desc = reinterpret_cast<uint32_t *>(base + o_gd);
        A->gather.d_payload = reinterpret_cast<unsigned char *>(base + o_gp);
        A->gather.bytes = (int64_t)(o_gp + bytes(A->gather.payload) + 16 - o_gs);
    }
    if (A->gather32.present) {
        A->gather32.d_sptr = reinterpret_cast<int32_t *>(base + o_hs);
        A->gather32.d_out_row = reinterpret_cast<int32_t *>(base + o_hq);
        A->gather32.d_rows = reinterpret_cast<uint32_t *>(base + o_hr);
        A->gather32.d_desc = reinterpret_cast<uint32_t *>(base + o_hd);
        A->gather32.d_payload = reinterpret_cast<unsigned char *>(base + o_hp);
        A->gather32.bytes = (int64_t)(o_hp + bytes(A->gather32.payload) + 16 - o_hs);
    }
    if (A->gemv.present) {
        A->gemv.d_masks = reinterpret_cast<uint32_t *>(base + o_gm);
        A->gemv.d_woff = reinterpret_cast<uint32_t *>(base + o_go);
        A->gemv.bytes = (int64_t)(s.total - mma_end);
    }
    A->on_device = true;
    return GRIM_OK;
}

grim_status check_call(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, const float *Y, int64_t ldy) {
    if (!A || !X || !Y) return GRIM_ERR_NULL;
    if (N < 1 || ldx < N || ldy < N) return GRIM_ERR_SHAPE;
    if (N > (int64_t(1) << 30) || ldx > (int64_t(1) << 40) || ldy > (int64_t(1) << 40)) return GRIM_ERR_SHAPE;
    if (!A->on_device) return GRIM_ERR_DEVICE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != A->device) return GRIM_ERR_DEVICE;
    return GRIM_OK;
}

bool gemv_ok(const grim_bcr_matrix *A, int64_t N) {
    return A->gemv.present && N >= 1 && N <= 8 && A->K * N * dtype_size(A->dtype) <= kGemvMaxXBytes;
}

// do the byte ranges [a, a + na) and [b, b + nb) overlap?
bool ranges_overlap(const void *a, int64_t na, const void *b, int64_t nb) {
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + (uintptr_t)nb && b0 < a0 + (uintptr_t)na;
}

GemvDesc desc_of(const grim_bcr_matrix *A) {
    return GemvDesc{A->dev.weights, A->gemv.d_masks, A->gemv.d_woff, A->dev.strip_order};
}

}  // namespace

extern "C" {

grim_status grim_bcr_pack(const void *W_host, grim_dtype dt, int64_t M, int64_t K, int64_t ldw, int32_t BR, int32_t BC,
                          const int32_t *row_ptr, const uint16_t *row_idx, const int32_t *col_ptr,
                          const uint16_t *col_idx, const grim_bcr_options *opt, grim_bcr_matrix **out) {
    if (out) *out = nullptr;
    if (!out || !W_host || !row_ptr || !col_ptr) return GRIM_ERR_NULL;
    if (dt != GRIM_F32 && dt != GRIM_F16 && dt != GRIM_BF16) return GRIM_ERR_DTYPE;
    if (M < 1 || K < 1 || BR < 1 || BC < 1 || BR > 65535 || BC > 65535) return GRIM_ERR_SHAPE;
    if (M % BR || K % BC || ldw < K) return GRIM_ERR_SHAPE;
    if (M > (int64_t(1) << 31) - 1 || K > (int64_t(1) << 31) - 1) return GRIM_ERR_SHAPE;
    const int64_t nbr = M / BR, nbc = K / BC;
    if (nbr > (int64_t(1) << 30) / nbc) return GRIM_ERR_SHAPE;   // ptr arrays are 32-bit
    const int64_t nb = nbr * nbc;
    grim_status st = validate_sets(nb, BR, row_ptr, row_idx);
    if (st != GRIM_OK) return st;
    st = validate_sets(nb, BC, col_ptr, col_idx);
    if (st != GRIM_OK) return st;

    grim_bcr_matrix *A = nullptr;
    try {
        A = new grim_bcr_matrix();
        A->M = M; A->K = K; A->BR = BR; A->BC = BC; A->dtype = dt;
        A->nbr = nbr; A->nbc = nbc; A->nb = nb;
        A->reordered = !(opt && opt->no_reorder);
        // strip work = stored weights of the strip; heavier strips first, ties by index (Section 4.2)
        std::vector<int64_t> work(nbr, 0);
        for (int64_t s = 0; s < nbr; ++s)
            for (int64_t c = 0; c < nbc; ++c) {
                int64_t b = s * nbc + c;
                work[s] += int64_t(row_ptr[b + 1] - row_ptr[b]) * int64_t(col_ptr[b + 1] - col_ptr[b]);
            }
        A->strip_order.resize(nbr);
        std::iota(A->strip_order.begin(), A->strip_order.end(), 0);
        if (A->reordered)
            std::stable_sort(A->strip_order.begin(), A->strip_order.end(),
                             [&](int32_t a, int32_t b) { return work[a] > work[b]; });
        const int esz = dtype_size(dt);
        A->row_ptr.assign(nb + 1, 0);
        A->col_ptr.assign(nb + 1, 0);
        A->blk_ptr.assign(nb + 1, 0);
        A->rowmask64.assign(nb, 0);
        int64_t t = 0;
        for (int64_t p = 0; p < nbr; ++p) {
            int64_t s = A->strip_order[p];
            for (int64_t c = 0; c < nbc; ++c, ++t) {
                int64_t b = s * nbc + c;
                int32_t kr = row_ptr[b + 1] - row_ptr[b], kc = col_ptr[b + 1] - col_ptr[b];
                A->row_ptr[t + 1] = A->row_ptr[t] + kr;
                A->col_ptr[t + 1] = A->col_ptr[t] + kc;
                A->blk_ptr[t + 1] = A->blk_ptr[t] + int64_t(kr) * kc;
            }
        }
        A->nnz = A->blk_ptr[nb];
        A->row_idx.resize(A->row_ptr[nb]);
        A->col_idx.resize(A->col_ptr[nb]);
        A->weights.resize((size_t)A->nnz * esz);
        const unsigned char *W = static_cast<const unsigned char *>(W_host);
        t = 0;
        for (int64_t p = 0; p < nbr; ++p) {
            int64_t s = A->strip_order[p];
            for (int64_t c = 0; c < nbc; ++c, ++t) {
                int64_t b = s * nbc + c;
                int32_t kr = row_ptr[b + 1] - row_ptr[b], kc = col_ptr[b + 1] - col_ptr[b];
                const uint16_t *R = kr ? row_idx + row_ptr[b] : nullptr;
                const uint16_t *C = kc ? col_idx + col_ptr[b] : nullptr;
                for (int32_t i = 0; i < kr; ++i) {
                    A->row_idx[A->row_ptr[t] + i] = R[i];
                    if (BR <= 64) A->rowmask64[t] |= uint64_t(1) << R[i];
                }
                for (int32_t j = 0; j < kc; ++j) A->col_idx[A->col_ptr[t] + j] = C[j];
                unsigned char *dst = A->weights.data() + (size_t)A->blk_ptr[t] * esz;
                for (int32_t i = 0; i < kr; ++i) {
                    const unsigned char *src = W + ((s * BR + R[i]) * ldw + c * BC) * esz;
                    for (int32_t j = 0; j < kc; ++j) std::memcpy(dst + ((size_t)i * kc + j) * esz, src + (size_t)C[j] * esz, esz);
                }
            }
        }
        if (!(opt && opt->host_only == 1)) {
            // staged kernel: chunks of up to 256 rows, a 4-strip group's records within 16 KB (the producers move at
            // most 32 KB of X rows and 16 KB of records per chunk); wide-tile kernel: chunks of up to 128 or 192 rows, a
            // 16-strip group's records within 32 KB
            // (each layout is built from the canonical arrays alone: the three that write the most run side by side when
            // there is enough to write -- 4096 x 2048 at 10.7x: 11.6 -> 6.6 ms for the whole pack)
            const int32_t rows_opt = opt ? opt->chunk_rows : 0;
            auto mma = [&]() { build_mma_layout(A, A->mma, rows_opt, kMmaMaxChunkRows, 0, 16 * 1024, false); };
            auto wide = [&]() { build_mma_layout(A, A->mmaw, rows_opt, wide_max_chunk_rows(A->BR), 2, kWideMaxRecordBytes, true); };
            std::future<void> f1, f2;
            if (A->nnz >= 32 * 1024 && dt != GRIM_F32) {
                try {
                    f1 = std::async(std::launch::async, mma);
                    f2 = std::async(std::launch::async, wide);
                } catch (const std::system_error &) {       // no thread to be had
                }
            }
            build_gather_layout<1>(A, A->gather);
            build_gather32_layout(A);
            build_gemv_layout(A);
            if (f1.valid()) f1.get(); else mma();
            if (f2.valid()) f2.get(); else wide();
        }
    } catch (const std::bad_alloc &) {
        delete A;
        return GRIM_ERR_ALLOC;
    }
    if (!(opt && opt->host_only)) {
        st = upload(A);
        if (st != GRIM_OK) { delete A; return st; }
    }
    *out = A;
    return GRIM_OK;
}

grim_status grim_bcr_unpack(const grim_bcr_matrix *A, void *W_host_out, int64_t ldw) {
    if (!A || !W_host_out) return GRIM_ERR_NULL;
    if (ldw < A->K) return GRIM_ERR_SHAPE;
    const int esz = dtype_size(A->dtype);
    unsigned char *W = static_cast<unsigned char *>(W_host_out);
    for (int64_t i = 0; i < A->M; ++i) std::memset(W + i * ldw * esz, 0, (size_t)A->K * esz);
    int64_t t = 0;
    for (int64_t p = 0; p < A->nbr; ++p) {
        int64_t s = A->strip_order[p];
        for (int64_t c = 0; c < A->nbc; ++c, ++t) {
            int32_t kr = A->row_ptr[t + 1] - A->row_ptr[t], kc = A->col_ptr[t + 1] - A->col_ptr[t];
            const unsigned char *src = A->weights.data() + (size_t)A->blk_ptr[t] * esz;
            for (int32_t i = 0; i < kr; ++i) {
                int64_t r = s * A->BR + A->row_idx[A->row_ptr[t] + i];
                for (int32_t j = 0; j < kc; ++j) {
                    int64_t k = c * A->BC + A->col_idx[A->col_ptr[t] + j];
                    std::memcpy(W + (r * ldw + k) * esz, src + ((size_t)i * kc + j) * esz, esz);
                }
            }
        }
    }
    return GRIM_OK;
}

grim_status grim_bcr_unpack_layout(const grim_bcr_matrix *A, int32_t layout, void *W_host_out, int64_t ldw) {
    if (!A || !W_host_out) return GRIM_ERR_NULL;
    if (ldw < A->K) return GRIM_ERR_SHAPE;
    const int esz = dtype_size(A->dtype);
    unsigned char *W = static_cast<unsigned char *>(W_host_out);
    auto clear = [&]() { for (int64_t i = 0; i < A->M; ++i) std::memset(W + i * ldw * esz, 0, (size_t)A->K * esz); };
    auto put = [&](int64_t r, int64_t k, const void *src) { std::memcpy(W + (r * ldw + k) * esz, src, esz); };
    if (layout == 1 || layout == 4) {
        // staged matrix-core layouts: regions of [steps x header][payload] per (chunk, stored strip)
        const MmaLayout &L = layout == 1 ? A->mma : A->mmaw;
        if (!L.present) return GRIM_ERR_UNSUPPORTED;
        clear();
        const int32_t ng = L.ks / 8, hdr = L.ks * 2 + ng * 8;
        for (int32_t ch = 0; ch < L.nchunks; ++ch) {
            for (int64_t st = 0; st < A->nbr; ++st) {
                const size_t e = (size_t)ch * (A->nbr + 1) + st;
                const int32_t nst = L.cptr[e + 1] - L.cptr[e];
                const unsigned char *region = L.recs.data() + (size_t)L.bptr[e] * 16;
                for (int32_t s = 0; s < nst; ++s) {
                    const unsigned char *h = region + (size_t)s * hdr;
                    for (int32_t g = 0; g < ng; ++g) {
                        const uint16_t *hs = reinterpret_cast<const uint16_t *>(h) + g * 8;
                        const uint32_t *hd = reinterpret_cast<const uint32_t *>(h + L.ks * 2) + g * 2;
                        const uint32_t rowmask = hd[0];
                        const unsigned char *pw = region + (size_t)hd[1] * 16;
                        int32_t i = 0;
                        for (int32_t r = 0; r < A->BR; ++r) {
                            if (!((rowmask >> r) & 1u)) continue;
                            for (int32_t slot = 0; slot < 8; ++slot) {
                                const uint16_t srow = slot < 4 ? hs[2 * slot] : hs[2 * (slot - 4) + 1];
                                if (srow == (uint16_t)L.chunk_rows) continue;      // the zero row: padding
                                put((int64_t)A->strip_order[st] * A->BR + r, (int64_t)ch * L.chunk_rows + srow,
                                    pw + ((size_t)i * 8 + slot) * 2);
                            }
                            ++i;
                        }
                    }
                }
            }
        }
        return GRIM_OK;
    }
    if (layout == 2) {
        // row-gathering layout: per 16-row run a list of steps of four groups of 8 k slots
        const GatherLayout &L = A->gather;
        if (!L.present) return GRIM_ERR_UNSUPPORTED;
        clear();
        for (int64_t u = 0; u < L.nstrips; ++u) {
            for (int64_t s = L.sptr[(size_t)u]; s < L.sptr[(size_t)u + 1]; ++s) {
                for (int32_t g = 0; g < 4; ++g) {
                    const uint32_t rowmask = L.desc[(size_t)s * 8 + g * 2];
                    const unsigned char *pw = L.payload.data() + (size_t)L.desc[(size_t)s * 8 + g * 2 + 1] * 16;
                    int32_t i = 0;
                    for (int32_t r = 0; r < 16; ++r) {
                        if (!((rowmask >> r) & 1u)) continue;
                        const int32_t orow = L.out_row[(size_t)u * 16 + r];
                        for (int32_t j = 0; j < 8; ++j) {
                            const uint32_t k = L.rows[(size_t)s * 32 + (size_t)j * 4 + g];
                            if (k == 0xffffffffu) continue;
                            if (orow < 0 || k >= (uint32_t)A->K) return GRIM_ERR_INDEX;
                            put(orow, k, pw + ((size_t)i * 8 + j) * 2);
                        }
                        ++i;
                    }
                }
            }
        }
        return GRIM_OK;
    }
    if (layout == 3) {
        // SpMV layout: the compact weights with one row and one column bit mask per stored block
        const GemvLayout &G = A->gemv;
        if (!G.present) return GRIM_ERR_UNSUPPORTED;
        clear();
        for (int64_t t = 0; t < A->nb; ++t) {
            const uint32_t rm = G.masks[2 * (size_t)t], cm = G.masks[2 * (size_t)t + 1];
            const int32_t kc = __builtin_popcount(cm);
            const int64_t p = t / A->nbc, c = t % A->nbc;
            int32_t i = 0;
            for (int32_t r = 0; r < A->BR; ++r) {
                if (!((rm >> r) & 1u)) continue;
                int32_t j = 0;
                for (int32_t q = 0; q < A->BC; ++q) {
                    if (!((cm >> q) & 1u)) continue;
                    put((int64_t)A->strip_order[p] * A->BR + r, c * A->BC + q,
                        A->weights.data() + ((size_t)G.woff[(size_t)t] + (size_t)i * kc + j) * esz);
                    ++j;
                }
                ++i;
            }
        }
        return GRIM_OK;
    }
    return GRIM_ERR_SHAPE;
}

grim_status grim_bcr_export_bcrc(const grim_bcr_matrix *A, grim_bcrc **out) {
    if (out) *out = nullptr;
    if (!A || !out) return GRIM_ERR_NULL;
    if (A->M > 0x7fffffff || A->K > 0x7fffffff) return GRIM_ERR_SHAPE;
    grim_bcrc *B = nullptr;
    try {
        B = new grim_bcrc();
        B->M = A->M; B->K = A->K; B->dtype = A->dtype;
        const int esz = dtype_size(A->dtype);
        // stored position of every strip
        std::vector<int64_t> pos((size_t)A->nbr);
        for (int64_t p = 0; p < A->nbr; ++p) pos[(size_t)A->strip_order[p]] = p;
        // per original row: its kept global columns, and where each block's run of weights starts
        struct Run { int64_t w0; int32_t kc; };
        std::vector<std::vector<int32_t>> pattern((size_t)A->M);
        std::vector<std::vector<Run>> runs((size_t)A->M);
        for (int64_t s = 0; s < A->nbr; ++s) {
            for (int64_t c = 0; c < A->nbc; ++c) {
                const int64_t t = pos[(size_t)s] * A->nbc + c;
                const int32_t kr = A->row_ptr[t + 1] - A->row_ptr[t], kc = A->col_ptr[t + 1] - A->col_ptr[t];
                if (!kr || !kc) continue;
                for (int32_t i = 0; i < kr; ++i) {
                    const int64_t r = s * A->BR + A->row_idx[A->row_ptr[t] + i];
                    for (int32_t j = 0; j < kc; ++j)
                        pattern[(size_t)r].push_back((int32_t)(c * A->BC + A->col_idx[A->col_ptr[t] + j]));
                    runs[(size_t)r].push_back({A->blk_ptr[t] + (int64_t)i * kc, kc});
                }
            }
        }
        // groups in order of first appearance
        std::map<std::vector<int32_t>, int32_t> ids;
        std::vector<std::vector<int32_t>> members;
        for (int64_t r = 0; r < A->M; ++r) {
            auto it = ids.find(pattern[(size_t)r]);
            if (it == ids.end()) {
                it = ids.emplace(pattern[(size_t)r], (int32_t)members.size()).first;
                members.emplace_back();
            }
            members[(size_t)it->second].push_back((int32_t)r);
        }
        B->occurrence.push_back(0);
        B->column_stride.push_back(0);
        B->row_offset.push_back(0);
        B->weights.reserve(A->weights.size());
        for (const auto &grp : members) {
            const std::vector<int32_t> &cols = pattern[(size_t)grp[0]];
            B->compact_column.insert(B->compact_column.end(), cols.begin(), cols.end());
            B->column_stride.push_back((int64_t)B->compact_column.size());
            for (int32_t r : grp) {
                B->reorder.push_back(r);
                for (const Run &run : runs[(size_t)r]) {
                    const unsigned char *src = A->weights.data() + (size_t)run.w0 * esz;
                    B->weights.insert(B->weights.end(), src, src + (size_t)run.kc * esz);
                }
                B->row_offset.push_back((int64_t)(B->weights.size() / esz));
            }
            B->occurrence.push_back((int32_t)B->reorder.size());
        }
    } catch (const std::bad_alloc &) {
        delete B;
        return GRIM_ERR_ALLOC;
    }
    *out = B;
    return GRIM_OK;
}

grim_status grim_bcrc_arrays(const grim_bcrc *B, grim_bcrc_view *v) {
    if (!B || !v) return GRIM_ERR_NULL;
    v->M = B->M; v->K = B->K; v->dtype = B->dtype;
    v->ngroups = (int64_t)B->occurrence.size() - 1;
    v->nnz = B->row_offset.back();
    v->ncols = (int64_t)B->compact_column.size();
    v->reorder = B->reorder.data();
    v->row_offset = B->row_offset.data();
    v->occurrence = B->occurrence.data();
    v->column_stride = B->column_stride.data();
    v->compact_column = B->compact_column.data();
    v->weights = B->weights.data();
    return GRIM_OK;
}

void grim_bcrc_free(grim_bcrc *B) { delete B; }

grim_status grim_bcr_arrays(const grim_bcr_matrix *A, grim_bcr_view *v) {
    if (!A || !v) return GRIM_ERR_NULL;
    v->M = A->M; v->K = A->K; v->BR = A->BR; v->BC = A->BC; v->dtype = A->dtype; v->reordered = A->reordered;
    v->nbr = A->nbr; v->nbc = A->nbc; v->nb = A->nb; v->nnz = A->nnz;
    v->strip_order = A->strip_order.data();
    v->row_ptr = A->row_ptr.data();
    v->row_idx = A->row_idx.data();
    v->col_ptr = A->col_ptr.data();
    v->col_idx = A->col_idx.data();
    v->blk_ptr = A->blk_ptr.data();
    v->weights = A->weights.data();
    v->dev_bytes_canonical = A->on_device ? A->dev.bytes : 0;
    v->dev_bytes_mma = A->on_device && A->mma.present ? A->mma.bytes : 0;
    v->dev_bytes_gemv = A->on_device && A->gemv.present ? A->gemv.bytes : 0;
    return GRIM_OK;
}

// a few columns of a uniformly pruned matrix: the one-column SpMV kernel on a set of workgroups per column, while all
// sets fit the GPU in one round
// (`count`: products of this shape in the launch -- 2 for the two sides of a GRU step)
static bool columns_as_sets(const grim_bcr_matrix *A, int64_t N, int count) {
    return N > 1 && N <= 8 && gemv_ok(A, N) && A->BR <= 32 && A->BC <= 32 &&
           spmv_exact_applies(A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, A->K) &&
           spmv_column_sets_ok(count, A->nbr, (int32_t)N);
}

// Up to eight right-hand sides of a matrix the wave-per-strip SpMV kernels are not compiled for (blocks pruned at
// different rates, kept counts outside their pairs, too many columns for sets of workgroups): one padded 16-column tile
// of a row-gathering matrix-core kernel, at any alignment.  Against the workgroup-per-strip kernel bcr_spmv, whose cost
// grows with the columns: 4096 x 4096 of mixed rates at 1 / 2 / 5 / 8 columns 13.5 / 11.6 / 15.1 / 16 -> 6.3 / 5.4 / 6.1 /
// 5.1 us, 512 x 512 5.2 / 5.2 / 5.3 / 5.9 -> 5.2 / 4.7 / 4.7 / 4.2 us, fp32 4096 x 2048 12.5 / 9.0 / 11.5 / 13.6 ->
// 5.5 / 5.5 / 5.9 / 5.4 us.  Uniform blocks stay: one column of 4096 x 2048 4.3 us against 6.1.
static bool skinny_on_matrix_cores(const grim_bcr_matrix *A, const void *X_dev, int64_t N, int64_t ldx, int count = 1) {
    if (N > 8 || columns_as_sets(A, N, count)) return false;
    // (blocks the SpMV kernels do not take are left to the choice among the SpMM kernels)
    if (!gemv_ok(A, N) && !(N == 8 && ldx % 8 == 0 && reinterpret_cast<uintptr_t>(X_dev) % 16 == 0)) return false;
    if (N == 1 && gemv_ok(A, 1) && spmv_exact_applies(A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, A->K)) return false;
    if (N < 8 && gemv_ok(A, N) && spmv_many_strips_applies(count, A->nbr, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, A->K, A->BC, (int32_t)N))
        return false;
    if (A->dtype != GRIM_F32) return gather_any_applies(A, X_dev, N, ldx);
    if (!gather32_applies(A, X_dev)) return false;
    // Blocks of fewer than eight rows: a 16-row run is many times as long as the strips that the SpMV kernel takes side by side,
    // until there is a run to every compute unit (1 x 16 blocks, three columns: 1024 x 4096 25.6 us there, 54.5 here; 8192 x 1024
    // 82.0 and 26.8).
    if (A->BR < 8 && A->M < 4096) return false;
    // Two or three columns of a uniform matrix of twice as many runs, as long as they fit the SpMV kernel's memory twice: 8192 x
    // 4096 at three 13.9 us there, 16.1 here (four columns of 12288 x 4096 41.9 and 26.0).
    return !(N > 1 && N < 4 && A->gemv.uniform_kr > 0 && A->M >= 8192 && A->K >= 2048 && A->K * N <= 12 * 1024);
}
static grim_status launch_skinny(const grim_bcr_matrix *A, const void *X, int64_t N, int64_t ldx, float *Y, int64_t ldy, hipStream_t stream) {
    return A->dtype == GRIM_F32 ? launch_spmm_gather32(A, X, N, ldx, Y, ldy, stream) : launch_spmm_gather(A, X, N, ldx, Y, ldy, stream);
}

// which kernel family a grim_bcr_spmm_tuned call runs
enum SpmmRoute { ROUTE_NONE, ROUTE_SPMV, ROUTE_FMA, ROUTE_MMA, ROUTE_GATHER, ROUTE_GATHER32, ROUTE_WIDE };

// what the columns the wide-tile kernel leaves over (a multiple of eight, like N) cost on the kernels that take any N
static double rest_cost(const grim_bcr_matrix *A, int64_t n) {
    int tn = 0, g = 0;
    double best = A->mma.present ? mma_best_shape(A, n, 0, 0, &tn, &g) : -1.0;
    if (A->gather.present) {
        const double c = gather_cost(A, n);
        if (best < 0 || c < best) best = c;
    }
    return best;
}

// `wide_tn` / `wide_cols`: for ROUTE_WIDE, the tile width and the leading columns that kernel takes
static SpmmRoute spmm_route(const grim_bcr_matrix *A, const void *X_dev, int64_t N, int64_t ldx, const float *Y_dev,
                            int64_t ldy, int32_t tile_n, int32_t strips_per_wg, int32_t kernel, int *wide_tn,
                            int64_t *wide_cols) {
    if (kernel < 0 || kernel > 4 || tile_n < 0 || strips_per_wg < 0) return ROUTE_NONE;
    const bool free_choice = kernel == 0 && tile_n == 0 && strips_per_wg == 0;
    if (kernel == 3) return !tile_n && !strips_per_wg && gather_applies(A, X_dev, N, ldx) ? ROUTE_GATHER : ROUTE_NONE;
    if (kernel == 4) {
        *wide_tn = tile_n;
        *wide_cols = N;
        return !strips_per_wg && wide_applies(A, X_dev, N, ldx, Y_dev, ldy, tile_n) ? ROUTE_WIDE : ROUTE_NONE;
    }
    if (free_choice && skinny_on_matrix_cores(A, X_dev, N, ldx)) return A->dtype == GRIM_F32 ? ROUTE_GATHER32 : ROUTE_GATHER;
    if (free_choice && gemv_ok(A, N)) return ROUTE_SPMV;
    const bool mma = A->mma.present && kernel != 1;
    if (kernel == 2 && !mma) return ROUTE_NONE;
    if (free_choice) {
        // the matrix-core kernels that apply: take the one that moves fewer bytes through a compute unit
        int tn = 0, g = 0;
        const double staged = mma ? mma_best_shape(A, N, 0, 0, &tn, &g) : -1.0;
        const double gather = gather_applies(A, X_dev, N, ldx) ? gather_cost(A, N) : -1.0;
        const double wide = wide_plan(A, X_dev, N, ldx, Y_dev, ldy, rest_cost, wide_tn, wide_cols);
        if (wide >= 0 && (staged < 0 || wide < staged) && (gather < 0 || wide < gather)) return ROUTE_WIDE;
        if (gather >= 0 && (staged < 0 || gather < staged)) return ROUTE_GATHER;
        // (rows of X at any alignment: 360 products of 9 to 25087 columns, 64 x 576 to 1024 x 1024 and 512 x 4608, were quicker
        // there than staged or on the vector ALUs, by 1.0 to 50 times)
        if (gather < 0 && gather_any_applies(A, X_dev, N, ldx)) return ROUTE_GATHER;
        if (gather32_applies(A, X_dev) && gather32_quicker(A, N)) return ROUTE_GATHER32;
    }
    if (mma) return ROUTE_MMA;
    return A->BR > 64 ? ROUTE_NONE : ROUTE_FMA;
}

grim_status grim_bcr_spmm_tuned(const grim_bcr_matrix *A, const void *X_dev, int64_t N, int64_t ldx, float *Y_dev,
                                int64_t ldy, int32_t tile_n, int32_t strips_per_wg, int32_t kernel, void *hip_stream) {
    grim_status st = check_call(A, X_dev, N, ldx, Y_dev, ldy);
    if (st != GRIM_OK) return st;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    int wide_tn = 0;
    int64_t wide_cols = 0;
    switch (spmm_route(A, X_dev, N, ldx, Y_dev, ldy, tile_n, strips_per_wg, kernel, &wide_tn, &wide_cols)) {
        case ROUTE_SPMV: {
            GemvDesc d = desc_of(A);
            return launch_spmv(nullptr, d, nullptr, 1, A->M, A->K, A->BR, A->BC, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc,
                               A->gemv.vec, A->gemv.krmax, A->gemv.kcmax, X_dev, 0, (int32_t)N, ldx, Y_dev, 0, ldy, stream);
        }
        case ROUTE_GATHER: return launch_spmm_gather(A, X_dev, N, ldx, Y_dev, ldy, stream);
        case ROUTE_GATHER32: return launch_spmm_gather32(A, X_dev, N, ldx, Y_dev, ldy, stream);
        case ROUTE_WIDE: {
            // whole rounds of fat workgroups, the few columns left over on whatever suits them: in the same launch when
            // that is the row-gathering kernel in the form the combined kernel carries, else in a launch of their own
            const char *x_rest = static_cast<const char *>(X_dev) + wide_cols * dtype_size(A->dtype);
            if (wide_cols < N) {
                int tn2 = 0;
                int64_t cols2 = 0;
                if (spmm_route(A, x_rest, N - wide_cols, ldx, Y_dev + wide_cols, ldy, 0, 0, 0, &tn2, &cols2) == ROUTE_GATHER) {
                    st = launch_spmm_wide_with_rest(A, X_dev, N, ldx, Y_dev, ldy, wide_tn, wide_cols, stream);
                    if (st != GRIM_ERR_UNSUPPORTED) return st;
                }
            }
            st = launch_spmm_wide(A, X_dev, wide_cols, ldx, Y_dev, ldy, wide_tn, stream);
            if (st != GRIM_OK || wide_cols >= N) return st;
            return grim_bcr_spmm_tuned(A, x_rest, N - wide_cols, ldx, Y_dev + wide_cols, ldy, 0, 0, 0, hip_stream);
        }
        case ROUTE_MMA: {
            if (kernel == 0 && tile_n == 0 && strips_per_wg == 0) {
                // whole rounds of workgroups on the staged kernel, the few columns left over on whatever suits them
                int tn = 0, g = 0;
                const int64_t n_main = mma_whole_rounds(A, N, &tn, &g);
                if (n_main < N) {
                    st = launch_spmm_mma(A, X_dev, n_main, ldx, Y_dev, ldy, tn, g, stream);
                    if (st != GRIM_OK) return st;
                    const char *x_rest = static_cast<const char *>(X_dev) + n_main * dtype_size(A->dtype);
                    return grim_bcr_spmm_tuned(A, x_rest, N - n_main, ldx, Y_dev + n_main, ldy, 0, 0, 0, hip_stream);
                }
            }
            return launch_spmm_mma(A, X_dev, N, ldx, Y_dev, ldy, tile_n, strips_per_wg, stream);
        }
        case ROUTE_FMA: return launch_spmm_fma(A, X_dev, N, ldx, Y_dev, ldy, stream);
        case ROUTE_NONE: break;
    }
    return GRIM_ERR_UNSUPPORTED;
}

const char *grim_bcr_spmm_kernel_name(const grim_bcr_matrix *A, const void *X_dev, int64_t N, int64_t ldx, int32_t tile_n,
                                      int32_t strips_per_wg, int32_t kernel) {
    if (!A || !X_dev || N < 1 || ldx < N || !A->on_device) return "none";
    // (the output is taken to be 16-byte aligned with a leading dimension of N rounded up to 4, as allocators give it)
    int wide_tn = 0;
    int64_t wide_cols = 0;
    switch (spmm_route(A, X_dev, N, ldx, reinterpret_cast<const float *>(uintptr_t(256)), (N + 3) / 4 * 4, tile_n, strips_per_wg,
                       kernel, &wide_tn, &wide_cols)) {
        case ROUTE_SPMV: return "bcr_spmv";
        case ROUTE_WIDE: return "bcr_spmm_wide";
        case ROUTE_GATHER: return "bcr_spmm_gather";
        case ROUTE_MMA: return "bcr_spmm_mma";
        case ROUTE_GATHER32: return "bcr_spmm_gather32";
        case ROUTE_FMA: return "bcr_spmm_fma";
        case ROUTE_NONE: break;
    }
    return "none";
}

grim_status grim_bcr_spmm(const grim_bcr_matrix *A, const void *X_dev, int64_t N, int64_t ldx, float *Y_dev, int64_t ldy,
                          void *hip_stream) {
    return grim_bcr_spmm_tuned(A, X_dev, N, ldx, Y_dev, ldy, 0, 0, 0, hip_stream);
}

grim_status grim_bcr_spmv(const grim_bcr_matrix *A, const void *x_dev, int32_t batch, int64_t ldx, float *y_dev,
                          int64_t ldy, void *hip_stream) {
    if (!A || !x_dev || !y_dev) return GRIM_ERR_NULL;
    if (batch < 1 || batch > 8) return GRIM_ERR_SHAPE;
    grim_status st = check_call(A, x_dev, batch, ldx, y_dev, ldy);
    if (st != GRIM_OK) return st;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (skinny_on_matrix_cores(A, x_dev, batch, ldx)) return launch_skinny(A, x_dev, batch, ldx, y_dev, ldy, stream);
    if (gemv_ok(A, batch)) {
        GemvDesc d = desc_of(A);
        return launch_spmv(nullptr, d, nullptr, 1, A->M, A->K, A->BR, A->BC, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc,
                           A->gemv.vec, A->gemv.krmax, A->gemv.kcmax, x_dev, 0, batch, ldx, y_dev, 0, ldy, stream);
    }
    // blocks the SpMV kernels do not take (more than 32 rows or columns): whatever the SpMM entry point picks
    return grim_bcr_spmm_tuned(A, x_dev, batch, ldx, y_dev, ldy, 0, 0, 0, hip_stream);
}

static grim_status conv_call(const grim_bcr_matrix *A, const void *F_dev, int32_t Cin, int32_t H, int32_t W, int32_t kh,
                             int32_t kw, const float *bias_dev, int32_t relu, void *out_dev, int32_t odt, int64_t ldo,
                             void *hip_stream) {
    if (!A || !F_dev || !out_dev) return GRIM_ERR_NULL;
    if (Cin < 1 || H < 1 || W < 1 || kh < 1 || kw < 1 || kh % 2 == 0 || kw % 2 == 0) return GRIM_ERR_SHAPE;
    if ((int64_t)Cin * kh * kw != A->K || ldo < (int64_t)H * W) return GRIM_ERR_SHAPE;
    if (odt != GRIM_F32 && odt != GRIM_F16 && odt != GRIM_BF16) return GRIM_ERR_DTYPE;
    if (!A->on_device) return GRIM_ERR_DEVICE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != A->device) { (void)hipGetLastError(); return GRIM_ERR_DEVICE; }
    grim_status st = launch_conv_wide(A, F_dev, Cin, H, W, kh, kw, 1, 0, bias_dev, relu ? 1 : 0, out_dev, odt, ldo, 0,
                                      static_cast<hipStream_t>(hip_stream));
    if (st != GRIM_ERR_UNSUPPORTED) return st;
    return launch_conv_gather(A, F_dev, Cin, H, W, kh, kw, bias_dev, relu ? 1 : 0, out_dev, odt, ldo,
                              static_cast<hipStream_t>(hip_stream));
}

grim_status grim_bcr_conv2d(const grim_bcr_matrix *A, const void *F_dev, int32_t Cin, int32_t H, int32_t W, int32_t kh,
                            int32_t kw, float *Y_dev, int64_t ldy, void *hip_stream) {
    return conv_call(A, F_dev, Cin, H, W, kh, kw, nullptr, 0, Y_dev, GRIM_F32, ldy, hip_stream);
}

grim_status grim_bcr_conv2d_act(const grim_bcr_matrix *A, const void *F_dev, int32_t Cin, int32_t H, int32_t W, int32_t kh,
                                int32_t kw, const float *bias_dev, int32_t relu, void *out_dev, grim_dtype out_dt,
                                int64_t ldo, void *hip_stream) {
    return conv_call(A, F_dev, Cin, H, W, kh, kw, bias_dev, relu, out_dev, (int32_t)out_dt, ldo, hip_stream);
}

struct grim_bcr_conv_plan {
    const grim_bcr_matrix *A = nullptr;
    int32_t Cin = 0, H = 0, W = 0, kh = 0, kw = 0, stride = 1;
    int device = -1;
    uint32_t *d_words = nullptr;
    // the rows cut into runs of 64 (where that leaves fewer rows of the im2col matrix to form); `rows` are window-start words
    GatherLayout tall;
    RunSteps tall_steps;
    void *d_tall = nullptr;          // one allocation for all of it
    ConvDense dense;
    void *d_dense = nullptr;
};

// Runs of 64 rows pay once there are about as many (tile, run) pairs as two thirds of the compute units -- below that the
// four times as many 16-row workgroups are quicker (512 channels on one 28 x 28 map, 104 pairs: 13.6 -> 19.4 us) -- and, at
// stride 1, for strips of some length that name each row nearly twice and more.  Measured, 16-row against 64-row runs:
// 256 channels, 3 x 3, four 28 x 28 maps in 16 x 32 / 8 x 16 / 16 x 16 / 4 x 16 blocks (rows named 1.5 / 1.9 / 2.1 / 2.7
// times) 13.5 -> 13.7 (not taken), 18.1 -> 15.7, 18.1 -> 16.0, 26.1 -> 15.7 us; 128 channels on eight 56 x 56 maps 21.9 ->
// 26.1 (not taken), 32.3 -> 29.6, 32.4 -> 29.7, 41.7 -> 30.0; 1 x 1 with 8 steps 7.1 -> 7.5 (not taken).  At stride 2, where
// a window is two loads, 128 -> 256 channels from four 56 x 56 maps 12.5 -> 10.6, 16.0 -> 11.8, 16.2 -> 11.9, 20.4 -> 12.0
// and its 1 x 1 shortcut 7.0 -> 6.6, 7.6 -> 7.2, 7.8 -> 7.1, 8.8 -> 7.2.
static bool conv_on_tall_runs(const grim_bcr_matrix *A, const RunSteps &tall, int32_t H, int32_t W, int32_t stride, int32_t batch) {
    if (A->M <= 16 || tall.runs == 0 || tall.total * 4 > A->gather.nsteps * 3) return false;
    if (stride == 1 && (tall.longest < 12 || tall.total * 7 > A->gather.nsteps * 4)) return false;
    const int64_t Ho = (H + 1) / 2, Wp = ((W + 1) / 2 + 7) / 8 * 8;
    const int64_t positions = stride == 2 ? Ho * Wp : (int64_t)H * W;
    if ((positions + 63) / 64 * batch * tall.runs < 160) return false;
    // (where a batch on 16-row runs has the bits of its images one by one, it keeps them)
    return stride == 2 || !conv_batch_sums_as_one_image(A, positions, batch);
}

// The dense copy (bcr_conv_patch) where it is to be quicker than the kernel the layer would run on without it.  Microseconds, by the
// forms the three kernels run in (workgroups of eight waves with a compute unit each, or of four waves in rounds of two to a compute
// unit; a last round that is at most half full counts 0.7):
//   dense    0.38 per step of a wave, 0.72 or 0.66 per 64 tasks (pixels of a chunk) of a wave, 2.6 or 5 per workgroup, 3.5 per launch
//   64-row   1.07 or 1.03 per step of a wave (1.44 times that at stride 2), 4 or 5.35 per workgroup, 3.2 per launch
//   16-row   0.107 per step of a strip and 0.45 per strip (1.3 times that at stride 2) in rounds of 256, 5.7 per launch; a strip to a
//            wave 0.105 and 0.16, 9.3 per launch; four waves to a strip at stride 2 0.13 and 0.18; 32-position tiles, all of them at
//            once, 0.066 per step of the longest strip, 5.7 per launch
// Fitted to 518 layers of 32 to 512 channels, 3 x 3 and 5 x 5, on 2 to 32 maps of 7 x 7 to 64 x 64, the last three forms to 1667 of
// 3845 more on 1 to 24 maps of 5 x 5 to 112 x 112, each run with and without the dense copy; the estimates lie within 12 % (rms).  The
// dense copy has to be estimated 2 % ahead.  Of the 3845 layers 1594 get it, 32 of which lose 3 % or more, the worst 15 (with one form
// of 16-row runs 1728 and 140, the worst 65: small maps at stride 2 on 32-position tiles); in all 79.4 ms without, 67.3 with this
// rule, 66.5 with the quicker one each time.
// Without -> on the dense copy: 256 channels, 3 x 3, four 28 x 28 maps in 4 x 16 / 16 x 32 / mixed 32 x 32 blocks 16.5 / 13.7 / 11.9
// -> 11.2 / 11.2 / 11.1 us; 448 from seven 103 x 24 maps at stride 2 in 4 x 16 / 16 x 32 blocks 119 / 82 -> 36 / 36; 512 on eight
// 14 x 14 19.3 -> 17.4; 5 x 5, 192 on four 18 x 18 maps in 32 x 32 blocks 20.4 -> 18.9.  Not taken: 224 -> 160 on eight 47 x 47 maps in
// mixed 32 x 32 blocks 29.0 -> 39.9; 288 -> 224 on 26 of 17 x 17 in 16 x 32 blocks 25.2 -> 34.4; 160 -> 192 from five 56 x 56 at stride 2
// 11.0 -> 13.2; 320 -> 384 on five 35 x 35 31.6 -> 38.7; 320 -> 224 from seven 8 x 8 at stride 2 in 4 x 16 blocks 8.9 -> 12.7; 384 on four 68 x 68
// 74.7 -> 86.
constexpr int64_t kConvWholeRounds = 8;          // rounds of workgroups that are counted whole

static bool conv_on_dense_copy(const grim_bcr_matrix *A, const RunSteps &tall, int32_t H, int32_t W, int32_t kh, int32_t kw, int32_t stride, int32_t batch) {
    if (!A->gather.present || A->gather.nstrips == 0 || A->M <= 16) return false;
    const int64_t KK = (int64_t)kh * kw, Cin = A->K / KK;
    const int32_t octets = conv_patch_octets(Cin, H, W, kh, kw, stride);
    if (octets == 0) return false;
    const int64_t Ho = (H + stride - 1) / stride, Wo = (W + stride - 1) / stride;
    const int64_t chunks = (Cin + 8 * octets - 1) / (8 * octets), steps = (KK * octets + 3) / 4, runs = (A->M + 63) / 64;
    if (runs * chunks * steps > (1 << 16)) return false;                     // (256 MB)
    // (where a batch on 16-row runs has the bits of its images one by one, it keeps them)
    if (stride == 1 && conv_batch_sums_as_one_image(A, (int64_t)H * W, batch)) return false;
    auto rounds = [](int64_t n, int64_t launch, int64_t slots) {             // of n workgroups, `launch` with those that only pad
        const int64_t whole = launch / slots, rest = launch % slots;
        return n > kConvWholeRounds * slots ? (double)n / (double)slots : (double)whole + (rest == 0 ? 0.0 : 2 * rest <= slots ? 0.7 : 1.0);
    };
    const int64_t tiles = (Ho * Wo + 63) / 64 * batch;
    const int64_t row_tiles = stride == 2 ? (Ho * ((Wo + 7) / 8 * 8) + 63) / 64 * batch : tiles;       // (rows padded to pieces there)
    if (row_tiles > 0x7fffffff / 16) return false;                           // (refused by every launcher)
    int64_t launched = 0;
    xcd_map((int32_t)tiles, runs, &launched);
    const double tasks = (double)((patch_pixels(H, W, kh, kw, stride) / 8 * 2 * octets + 63) / 64);
    const int waves = patch_waves((int32_t)tiles, runs);
    const double share = (double)((chunks + waves - 1) / waves) * (double)steps, turned = (double)((chunks + waves - 1) / waves) * tasks;
    const double dense = 3.5 + (waves == 8 ? 2.6 + 0.375 * share + 0.72 * turned : rounds(tiles * runs, launched, 512) * (5.0 + 0.385 * share + 0.66 * turned));
    double without;
    if (conv_on_tall_runs(A, tall, H, W, stride, batch)) {
        const double step = (double)tall.total / (double)tall.runs * (stride == 2 ? 1.44 : 1.0);
        xcd_map((int32_t)row_tiles, tall.runs, &launched);
        const int64_t pairs = row_tiles * tall.runs;
        without = 3.2 + (pairs <= 256 ? rounds(pairs, launched, 256) * (4.0 + 1.07 * step / 8.0) : rounds(pairs, launched, 512) * (5.35 + 1.03 * step / 4.0));
    } else {
        const int64_t pairs = row_tiles * A->gather.nstrips;
        const int nt = conv_subtiles(A, stride == 2 ? Ho * ((Wo + 7) / 8 * 8) : Ho * Wo, batch, stride, true);
        const int strip_waves = conv_strip_waves(A, nt, pairs, stride);
        const double turns = pairs <= 1024 ? (double)((pairs + 255) / 256) : (double)pairs / 256.0;
        const double strip = (double)A->gather.nsteps / (double)A->gather.nstrips;
        if (nt == 2) without = 5.67 + 0.066 * (double)A->gather.max_steps;
        else if (stride == 1 && strip_waves == 1) without = 9.27 + turns * (0.105 * strip + 0.16);
        else if (stride == 2 && strip_waves == 4) without = 5.7 + turns * (0.1315 * strip + 0.18);
        else without = 5.7 + 0.107 * turns * (strip + 4.2) * (stride == 2 ? 1.3 : 1.0);
    }
    return dense * 1.02 <= without;
}

// Does `met` hold for some batch the plan can be called with?  The forms of the kernels, and with them what the rules answer, change
// with the batch up to kConvWholeRounds rounds of 512 workgroups on 64-row runs; beyond, every estimate is linear in the batch, so
// that what holds for any batch there holds for the first or for the last.
static bool conv_some_batch(const grim_bcr_conv_plan *P, bool (*met)(const grim_bcr_conv_plan *, int32_t)) {
    const int64_t Ho = (P->H + P->stride - 1) / P->stride, Wo = (P->W + P->stride - 1) / P->stride;
    const int64_t tiles = (Ho * ((Wo + 7) / 8 * 8) + 63) / 64, pairs = (Ho * Wo + 63) / 64 * ((P->A->M + 63) / 64);
    const int64_t last = std::max<int64_t>(1, (0x7fffffff / 16) / tiles), linear = std::min(last, kConvWholeRounds * 512 / pairs + 1);
    for (int64_t batch = 1; batch <= linear; ++batch)
        if (met(P, (int32_t)batch)) return true;
    return met(P, (int32_t)last);
}

static bool plan_on_dense_copy(const grim_bcr_conv_plan *P, int32_t batch) {
    return conv_on_dense_copy(P->A, P->tall_steps, P->H, P->W, P->kh, P->kw, P->stride, batch);
}
static bool plan_on_tall_runs(const grim_bcr_conv_plan *P, int32_t batch) {              // where it is not on a dense copy that it has
    return conv_on_tall_runs(P->A, P->tall_steps, P->H, P->W, P->stride, batch) && !(P->dense.present && plan_on_dense_copy(P, batch));
}

// The plan's dense copy of the weights (ConvDense); without memory for it the plan does without.
static void add_dense_layout(grim_bcr_conv_plan *P) {
    const grim_bcr_matrix *A = P->A;
    if (!conv_some_batch(P, plan_on_dense_copy)) return;
    ConvDense &D = P->dense;
    const int32_t octets = conv_patch_octets(P->Cin, P->H, P->W, P->kh, P->kw, P->stride);
    const int32_t KK = P->kh * P->kw;
    D.runs = (A->M + 63) / 64;
    D.octets = octets;
    D.chunks = (P->Cin + 8 * octets - 1) / (8 * octets);
    D.steps = (KK * octets + 3) / 4;
    const size_t run_values = (size_t)D.chunks * D.steps * kConvTallRuns * 512, run_rows = 16 * kConvTallRuns;
    std::vector<uint16_t> w;
    std::vector<int32_t> out_row;
    std::vector<uint32_t> place;                 // of column k inside a run, for row 0 of the first 16
    try {
        w.assign((size_t)D.runs * run_values, 0);
        out_row.assign((size_t)D.runs * run_rows, -1);
        place.resize((size_t)A->K);
    } catch (const std::bad_alloc &) {
        return;
    }
    for (int32_t c = 0, k = 0; c < P->Cin; ++c)
        for (int32_t tap = 0; tap < KK; ++tap, ++k) {
            const int32_t pair = tap * octets + c % (8 * octets) / 8;        // (tap, channel octet): four to a step
            place[(size_t)k] = (uint32_t)((((size_t)(c / (8 * octets)) * D.steps + pair / 4) * kConvTallRuns * 64 + pair % 4 * 16) * 8 + c % 8);
        }
    const uint16_t *src = reinterpret_cast<const uint16_t *>(A->weights.data());
    int64_t t = 0;
    for (int64_t p = 0; p < A->nbr; ++p) {
        for (int32_t r = 0; r < A->BR; ++r) out_row[(size_t)(p * A->BR + r)] = (int32_t)((int64_t)A->strip_order[p] * A->BR + r);
        for (int64_t c = 0; c < A->nbc; ++c, ++t) {
            const uint16_t *v = src + A->blk_ptr[t];
            for (int32_t i = A->row_ptr[t]; i < A->row_ptr[t + 1]; ++i) {
                const size_t row = (size_t)(p * A->BR + A->row_idx[i]);
                uint16_t *dst = w.data() + row / run_rows * run_values + (row % run_rows / 16 * 64 + row % 16) * 8;
                for (int32_t j = A->col_ptr[t]; j < A->col_ptr[t + 1]; ++j) dst[place[(size_t)(c * A->BC + A->col_idx[j])]] = *v++;
            }
        }
    }
    Slab s;
    const size_t o_w = s.add(w.size() * 2), o_q = s.add(out_row.size() * 4);
    char *base = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&base), s.total + 256) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (hipMemcpy(base + o_w, w.data(), w.size() * 2, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(base + o_q, out_row.data(), out_row.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(base);
        return;
    }
    P->d_dense = base;
    D.d_weights = reinterpret_cast<unsigned char *>(base + o_w);
    D.d_out_row = reinterpret_cast<int32_t *>(base + o_q);
    D.present = true;
}

// The layout of 64-row runs, if some batch would run on it.  A plan that cannot have it (no memory) does without.
static void add_tall_layout(grim_bcr_conv_plan *P) {
    const grim_bcr_matrix *A = P->A;
    GatherLayout &L = P->tall;
    try {
        if (!conv_some_batch(P, plan_on_tall_runs)) return;
        build_gather_layout<kConvTallRuns>(A, L);
        for (uint32_t &r : L.rows) r = conv_plan_word(r, P->H, P->W, P->kh, P->kw);
    } catch (const std::bad_alloc &) {
        L = GatherLayout();
        return;
    }
    if (!L.present) return;
    Slab s;
    auto bytes = [](const auto &v) { return v.size() * sizeof(v[0]); };
    const size_t o_s = s.add(bytes(L.sptr)), o_q = s.add(bytes(L.out_row)), o_r = s.add(bytes(L.rows)), o_d = s.add(bytes(L.desc)),
                 o_p = s.add(bytes(L.payload) + 16);
    char *base = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&base), s.total + 256) != hipSuccess) {
        (void)hipGetLastError();
        L = GatherLayout();
        return;
    }
    auto put = [&](size_t off, const void *src, size_t n) { return n == 0 || hipMemcpy(base + off, src, n, hipMemcpyHostToDevice) == hipSuccess; };
    if (!(put(o_s, L.sptr.data(), bytes(L.sptr)) && put(o_q, L.out_row.data(), bytes(L.out_row)) && put(o_r, L.rows.data(), bytes(L.rows)) &&
          put(o_d, L.desc.data(), bytes(L.desc)) && put(o_p, L.payload.data(), bytes(L.payload)))) {
        (void)hipGetLastError();
        (void)hipFree(base);
        L = GatherLayout();
        return;
    }
    P->d_tall = base;
    L.d_sptr = reinterpret_cast<int32_t *>(base + o_s);
    L.d_out_row = reinterpret_cast<int32_t *>(base + o_q);
    L.d_rows = reinterpret_cast<uint32_t *>(base + o_r);
    L.d_desc = reinterpret_cast<uint32_t *>(base + o_d);
    L.d_payload = reinterpret_cast<unsigned char *>(base + o_p);
    L.rows = {}; L.desc = {}; L.payload = {}; L.out_row = {};            // (the host copies have done their work)
}

grim_status grim_bcr_conv_plan_create(const grim_bcr_matrix *A, int32_t Cin, int32_t H, int32_t W, int32_t kh, int32_t kw,
                                      int32_t stride, grim_bcr_conv_plan **out) {
    if (!A || !out) return GRIM_ERR_NULL;
    *out = nullptr;
    if (Cin < 1 || H < 1 || W < 1 || kh < 1 || kw < 1 || kh % 2 == 0 || kw % 2 == 0) return GRIM_ERR_SHAPE;
    if ((int64_t)Cin * kh * kw != A->K || (stride != 1 && stride != 2)) return GRIM_ERR_SHAPE;
    if (!A->on_device) return GRIM_ERR_DEVICE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != A->device) { (void)hipGetLastError(); return GRIM_ERR_DEVICE; }
    if (!A->gather.present || kh * kw > 31 || (int64_t)Cin * H * W > (int64_t(1) << 26) || A->gather.rows.empty())
        return GRIM_ERR_UNSUPPORTED;
    std::vector<uint32_t> words(A->gather.rows.size());
    for (size_t i = 0; i < words.size(); ++i) words[i] = conv_plan_word(A->gather.rows[i], H, W, kh, kw);
    std::unique_ptr<grim_bcr_conv_plan> P(new (std::nothrow) grim_bcr_conv_plan);
    if (!P) return GRIM_ERR_ALLOC;
    P->A = A; P->Cin = Cin; P->H = H; P->W = W; P->kh = kh; P->kw = kw; P->stride = stride; P->device = dev;
    void *ptr = nullptr;
    if (hipMalloc(&ptr, words.size() * 4) != hipSuccess) { (void)hipGetLastError(); return GRIM_ERR_ALLOC; }
    if (hipMemcpy(ptr, words.data(), words.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(ptr);
        return GRIM_ERR_DEVICE;
    }
    P->d_words = static_cast<uint32_t *>(ptr);
    try {
        P->tall_steps = count_run_steps<kConvTallRuns>(A);
    } catch (const std::bad_alloc &) {           // (no runs: neither layout)
    }
    add_dense_layout(P.get());
    add_tall_layout(P.get());
    *out = P.release();
    return GRIM_OK;
}

void grim_bcr_conv_plan_free(grim_bcr_conv_plan *P) {
    if (!P) return;
    if (P->d_words) (void)hipFree(P->d_words);
    if (P->d_tall) (void)hipFree(P->d_tall);
    if (P->d_dense) (void)hipFree(P->d_dense);
    delete P;
}

grim_status grim_bcr_conv2d_plan(const grim_bcr_conv_plan *P, const void *F_dev, int32_t batch, int64_t f_image_stride,
                                 const float *bias_dev, int32_t relu, void *out_dev, grim_dtype out_dt, int64_t ldo,
                                 int64_t out_image_stride, void *hip_stream) {
    if (!P || !F_dev || !out_dev) return GRIM_ERR_NULL;
    const int64_t Ho = (P->H + P->stride - 1) / P->stride, Wo = (P->W + P->stride - 1) / P->stride;
    const int64_t M = P->A->M;
    if (batch < 1 || ldo < Ho * Wo) return GRIM_ERR_SHAPE;
    if (batch > 1 && (f_image_stride < (int64_t)P->Cin * P->H * P->W || out_image_stride < (M - 1) * ldo + Ho * Wo))
        return GRIM_ERR_SHAPE;
    if (out_dt != GRIM_F32 && out_dt != GRIM_F16 && out_dt != GRIM_BF16) return GRIM_ERR_DTYPE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != P->device) { (void)hipGetLastError(); return GRIM_ERR_DEVICE; }
    if (P->stride == 1) {
        const grim_status st = launch_conv_wide(P->A, F_dev, P->Cin, P->H, P->W, P->kh, P->kw, batch, f_image_stride, bias_dev,
                                                relu ? 1 : 0, out_dev, (int32_t)out_dt, ldo, out_image_stride,
                                                static_cast<hipStream_t>(hip_stream));
        if (st != GRIM_ERR_UNSUPPORTED) return st;
    }
    if (P->dense.present && plan_on_dense_copy(P, batch)) {
        const grim_status st = launch_conv_patch(P->A, P->dense, P->d_words, F_dev, P->Cin, P->H, P->W, P->kh, P->kw, bias_dev, relu ? 1 : 0, out_dev,
                                                 (int32_t)out_dt, ldo, static_cast<hipStream_t>(hip_stream), batch, P->stride, f_image_stride,
                                                 out_image_stride);
        if (st != GRIM_ERR_UNSUPPORTED) return st;
    }
    if (P->tall.present && conv_on_tall_runs(P->A, P->tall_steps, P->H, P->W, P->stride, batch)) {
        const grim_status st = launch_conv_tall(P->A, P->tall, P->d_words, F_dev, P->Cin, P->H, P->W, P->kh, P->kw, bias_dev, relu ? 1 : 0, out_dev,
                                                (int32_t)out_dt, ldo, static_cast<hipStream_t>(hip_stream), batch, P->stride, f_image_stride,
                                                out_image_stride);
        if (st != GRIM_ERR_UNSUPPORTED) return st;
    }
    return launch_conv_gather(P->A, F_dev, P->Cin, P->H, P->W, P->kh, P->kw, bias_dev, relu ? 1 : 0, out_dev, (int32_t)out_dt,
                              ldo, static_cast<hipStream_t>(hip_stream), batch, P->stride, f_image_stride, out_image_stride,
                              P->d_words);
}

const char *grim_bcr_conv2d_kernel_name(const grim_bcr_matrix *A, int32_t Cin, int32_t H, int32_t W, int32_t kh, int32_t kw,
                                        int32_t batch, int32_t stride) {
    if (!A || !A->on_device || Cin < 1 || H < 1 || W < 1 || kh < 1 || kw < 1 || batch < 1 || (int64_t)Cin * kh * kw != A->K)
        return "none";
    // operands as tests and benchmarks pass them: 16-byte aligned, dense images one after the other
    const int64_t HW = (int64_t)H * W;
    void *aligned = reinterpret_cast<void *>(uintptr_t(256));
    if (stride == 1 && conv_wide_applies(A, aligned, Cin, H, W, kh, kw, batch, Cin * HW, aligned, GRIM_F32, HW, A->M * HW))
        return "bcr_conv_wide";
    if (!A->gather.present) return "none";
    try {
        if (stride == 2 || (stride == 1 && batch > 1)) {
            const RunSteps tall = count_run_steps<kConvTallRuns>(A);
            if (conv_on_dense_copy(A, tall, H, W, kh, kw, stride, batch)) return "bcr_conv_patch";
            if (conv_on_tall_runs(A, tall, H, W, stride, batch)) return "bcr_conv_tall";
        }
    } catch (const std::bad_alloc &) {           // (a plan without memory for that layout does without it, too)
    }
    return "bcr_conv_gather";
}

grim_status grim_lstm_cell(const float *gates_dev, int64_t ldg, const float *bias_dev, float *c_dev, int64_t ldc,
                           void *h_dev, grim_dtype dt, int64_t ldh, float *h32_dev, int64_t ldh32, int64_t H,
                           int32_t batch, void *hip_stream) {
    if (!gates_dev || !c_dev) return GRIM_ERR_NULL;
    if (H < 1 || batch < 1 || ldg < batch || ldc < batch || (h_dev && ldh < batch) || (h32_dev && ldh32 < batch))
        return GRIM_ERR_SHAPE;
    if (H > (int64_t(1) << 40) / batch) return GRIM_ERR_SHAPE;
    if (dt != GRIM_F32 && dt != GRIM_F16 && dt != GRIM_BF16) return GRIM_ERR_DTYPE;
    return launch_lstm_cell(gates_dev, ldg, bias_dev, c_dev, ldc, h_dev, dt, ldh, h32_dev, ldh32, H, batch,
                            static_cast<hipStream_t>(hip_stream));
}

grim_status grim_bcr_lstm_step(const grim_bcr_matrix *A, const void *xh_dev, int32_t batch, int64_t ldx,
                               float *gates_dev, int64_t ldg, const float *bias_dev, float *c_dev, int64_t ldc,
                               void *h_dev, int64_t ldh, float *h32_dev, int64_t ldh32, void *hip_stream) {
    if (!A || !xh_dev || !gates_dev || !c_dev) return GRIM_ERR_NULL;
    if (A->M % 4 != 0) return GRIM_ERR_SHAPE;
    const int64_t H = A->M / 4;
    if (batch < 1 || ldc < batch || (h_dev && ldh < batch) || (h32_dev && ldh32 < batch)) return GRIM_ERR_SHAPE;
    if (A->gemv.present && spmv_cell_batch_ok(H, A->BR, batch)) {
        // One launch: the cell in the epilogue of the gate product, a set of workgroups per column of xh.  Workgroups
        // then write h while others may still read the input vectors, so the new h must not land in what this step reads.
        grim_status st0 = check_call(A, xh_dev, batch, ldx, gates_dev, ldg);
        if (st0 != GRIM_OK) return st0;
        const int esz = dtype_size(A->dtype);
        const bool aliased = h_dev && ranges_overlap(xh_dev, ((A->K - 1) * ldx + batch) * esz, h_dev, ((H - 1) * ldh + batch) * esz);
        if (!aliased) {
            // (a matrix stored in its original strip order spares the step kernel the look-up its weight fetch waits for)
            RnnCell cell{A->order_identity ? nullptr : A->dev.strip_pos, nullptr, bias_dev, nullptr, c_dev, h_dev, h32_dev, ldc, ldh, ldh32,
                         (int32_t)H, A->dtype};
            st0 = launch_spmv_cell(1, desc_of(A), nullptr, A->M, A->K, A->BR, A->BC, A->dtype, A->gemv.uniform_kr,
                                   A->gemv.uniform_kc, xh_dev, 0, batch, ldx, gates_dev, 0, ldg, cell, static_cast<hipStream_t>(hip_stream));
            if (st0 != GRIM_ERR_UNSUPPORTED) return st0;
        }
    }
    if (rnn_gather_applies(A, xh_dev, ldx, nullptr, nullptr, 0, H, batch)) {
        grim_status st0 = check_call(A, xh_dev, batch, ldx, gates_dev, ldg);
        if (st0 != GRIM_OK) return st0;
        if (!(h_dev && ranges_overlap(xh_dev, ((A->K - 1) * ldx + batch) * dtype_size(A->dtype), h_dev, ((H - 1) * ldh + batch) * dtype_size(A->dtype)))) {
            RnnCell cell{nullptr, nullptr, bias_dev, nullptr, c_dev, h_dev, h32_dev, ldc, ldh, ldh32, (int32_t)H, A->dtype};
            return launch_rnn_gather(A, xh_dev, ldx, gates_dev, ldg, nullptr, nullptr, 0, nullptr, 0, batch, cell, static_cast<hipStream_t>(hip_stream));
        }
    }
    grim_status st = batch <= 8 ? grim_bcr_spmv(A, xh_dev, batch, ldx, gates_dev, ldg, hip_stream)
                                : grim_bcr_spmm(A, xh_dev, batch, ldx, gates_dev, ldg, hip_stream);
    if (st != GRIM_OK) return st;
    return grim_lstm_cell(gates_dev, ldg, bias_dev, c_dev, ldc, h_dev, (grim_dtype)A->dtype, ldh, h32_dev, ldh32, H, batch,
                          hip_stream);
}

int32_t grim_bcr_rnn_step_launches(const grim_bcr_matrix *A, const grim_bcr_matrix *Ah, int32_t batch) {
    if (!A || batch < 1 || !A->on_device) return 0;
    // operands as allocators give them: aligned, a leading dimension of `batch`
    const void *aligned = reinterpret_cast<const void *>(uintptr_t(256));
    if (!Ah) {
        if (A->M % 4 != 0) return 0;
        const int64_t H = A->M / 4;
        const bool by_column = A->gemv.present && spmv_cell_batch_ok(H, A->BR, batch) &&
                               spmv_cell_applies(1, A->M, A->K, A->BR, A->BC, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, H);
        return by_column || rnn_gather_applies(A, aligned, batch, nullptr, nullptr, 0, H, batch) ? 1 : 2;
    }
    if (A->M != Ah->M || A->M % 3 != 0 || Ah->K != A->M / 3 || A->dtype != Ah->dtype || !Ah->on_device) return 0;
    const int64_t H = A->M / 3;
    const bool same = A->K == Ah->K && A->BR == Ah->BR && A->BC == Ah->BC && A->gemv.present && Ah->gemv.present;
    const bool by_column = spmv_cell_batch_ok(H, A->BR, batch) && same && A->gemv.uniform_kr == Ah->gemv.uniform_kr && A->gemv.uniform_kc == Ah->gemv.uniform_kc &&
                           spmv_cell_applies(2, A->M, A->K, A->BR, A->BC, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, H);
    if (by_column || rnn_gather_applies(A, aligned, batch, Ah, aligned, batch, H, batch)) return 1;
    // both products in one launch (the row-gathering kernel below 64 columns, SpMV kernels up to 8 columns when the matrices
    // have one shape), then the cell; otherwise a launch per product
    const bool one_launch = gather_pair_applies(A, aligned, Ah, aligned, batch, batch) || (same && gemv_ok(A, batch) && gemv_ok(Ah, batch));
    return one_launch ? 2 : 3;
}

// exchange words of the sequence kernel: allocated with the first sequence call on a matrix, freed with the matrix
static grim_status seq_exchange_of(const grim_bcr_matrix *A, void **out) {
    std::lock_guard<std::mutex> hold(A->seq_lock);
    if (!A->seq_exch) {
        void *ptr = nullptr;
        if (hipMalloc(&ptr, (size_t)seq_exchange_words(A->M) * 8) != hipSuccess) {
            (void)hipGetLastError();
            return GRIM_ERR_ALLOC;
        }
        A->seq_exch = ptr;
    }
    *out = A->seq_exch;
    return GRIM_OK;
}

static grim_status seq_check(const grim_bcr_matrix *A, const void *xs, int32_t T, int32_t batch, const void *h0,
                             const float *state, const void *hs, const int32_t *status) {
    if (!A || !xs || !h0 || !state || !hs || !status) return GRIM_ERR_NULL;
    if (T < 1 || batch < 1) return GRIM_ERR_SHAPE;
    if (!A->on_device) return GRIM_ERR_DEVICE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != A->device) return GRIM_ERR_DEVICE;
    return GRIM_OK;
}

int32_t grim_bcr_rnn_sequence_supported(const grim_bcr_matrix *A, const grim_bcr_matrix *Ah) {
    return grim_bcr_rnn_sequence_batch_supported(A, Ah, 1);
}

int32_t grim_bcr_rnn_sequence_batch_supported(const grim_bcr_matrix *A, const grim_bcr_matrix *Ah, int32_t batch) {
    if (!A || !A->on_device || !A->gemv.present) return 0;
    if (!Ah) {
        if (A->M % 4 != 0 || A->K <= A->M / 4) return 0;
        const int64_t H = A->M / 4;
        return rnn_seq_applies(1, A->BR, A->BC, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, A->K, 0, A->K - H, H, batch) ? 1 : 0;
    }
    if (!Ah->on_device || !Ah->gemv.present || A->M != Ah->M || A->M % 3 != 0 || Ah->K != A->M / 3) return 0;
    if (A->dtype != Ah->dtype || A->BR != Ah->BR || A->BC != Ah->BC || A->gemv.uniform_kr != Ah->gemv.uniform_kr ||
        A->gemv.uniform_kc != Ah->gemv.uniform_kc)
        return 0;
    return rnn_seq_applies(2, A->BR, A->BC, A->dtype, A->gemv.uniform_kr, A->gemv.uniform_kc, A->K, Ah->K, A->K, Ah->K, batch) ? 1 : 0;
}

grim_status grim_bcr_lstm_sequence(const grim_bcr_matrix *A, const void *xs_dev, int64_t ldxs, int32_t T,
                                   const float *bias_dev, const void *h0_dev, float *c_dev, void *hs_dev, int64_t ldhs,
                                   float *hs32_dev, int64_t ldhs32, int32_t *status_dev, uint32_t max_polls,
                                   void *hip_stream) {
    return grim_bcr_lstm_sequence_batch(A, xs_dev, ldxs, T, 1, bias_dev, h0_dev, c_dev, hs_dev, ldhs, hs32_dev, ldhs32,
                                        status_dev, max_polls, hip_stream);
}

grim_status grim_bcr_lstm_sequence_batch(const grim_bcr_matrix *A, const void *xs_dev, int64_t ldxs, int32_t T, int32_t batch,
                                         const float *bias_dev, const void *h0_dev, float *c_dev, void *hs_dev, int64_t ldhs,
                                         float *hs32_dev, int64_t ldhs32, int32_t *status_dev, uint32_t max_polls,
                                         void *hip_stream) {
    grim_status st = seq_check(A, xs_dev, T, batch, h0_dev, c_dev, hs_dev, status_dev);
    if (st != GRIM_OK) return st;
    if (A->M % 4 != 0 || A->K <= A->M / 4) return GRIM_ERR_SHAPE;
    const int64_t H = A->M / 4, I = A->K - H;
    if (ldxs < I || ldhs < H || (hs32_dev && ldhs32 < H)) return GRIM_ERR_SHAPE;
    if (!grim_bcr_rnn_sequence_batch_supported(A, nullptr, batch)) return GRIM_ERR_UNSUPPORTED;
    void *exch = nullptr;
    st = seq_exchange_of(A, &exch);
    if (st != GRIM_OK) return st;
    return launch_rnn_seq(1, desc_of(A), nullptr, A->dev.strip_pos, nullptr, A->BR, A->BC, A->dtype, A->gemv.uniform_kr,
                          A->gemv.uniform_kc, A->K, 0, I, H, T, batch, xs_dev, ldxs, h0_dev, bias_dev, nullptr, c_dev, hs_dev,
                          ldhs, hs32_dev, ldhs32, exch, status_dev, max_polls, static_cast<hipStream_t>(hip_stream));
}

grim_status grim_bcr_lstm_sequence_noalloc(const grim_bcr_matrix *A, const void *xs_dev, int64_t ldxs, int32_t T,
                                           const float *bias_dev, const void *h0_dev, float *c_dev, void *hs_dev,
                                           int64_t ldhs, float *hs32_dev, int64_t ldhs32, int32_t *status_dev,
                                           uint32_t max_polls, void *hip_stream) {
    grim_status st = seq_check(A, xs_dev, T, 1, h0_dev, c_dev, hs_dev, status_dev);
    if (st != GRIM_OK) return st;
    if (A->M % 4 != 0 || A->K <= A->M / 4) return GRIM_ERR_SHAPE;
    const int64_t H = A->M / 4, I = A->K - H;
    if (ldxs < I || ldhs < H || (hs32_dev && ldhs32 < H)) return GRIM_ERR_SHAPE;
    if (H > kSeqMaxH) return GRIM_ERR_UNSUPPORTED;                 // beyond the static exchange words
    if (!grim_bcr_rnn_sequence_supported(A, nullptr)) return GRIM_ERR_UNSUPPORTED;
    void *exch = nullptr;
    st = rnn_seq_static_exchange(&exch);
    if (st != GRIM_OK) return st;
    return launch_rnn_seq(1, desc_of(A), nullptr, A->dev.strip_pos, nullptr, A->BR, A->BC, A->dtype, A->gemv.uniform_kr,
                          A->gemv.uniform_kc, A->K, 0, I, H, T, 1, xs_dev, ldxs, h0_dev, bias_dev, nullptr, c_dev, hs_dev, ldhs,
                          hs32_dev, ldhs32, exch, status_dev, max_polls, static_cast<hipStream_t>(hip_stream));
}

grim_status grim_bcr_gru_sequence(const grim_bcr_matrix *Ai, const grim_bcr_matrix *Ah, const void *xs_dev, int64_t ldxs,
                                  int32_t T, const float *bias_i_dev, const float *bias_h_dev, const void *h0_dev,
                                  float *h32_dev, void *hs_dev, int64_t ldhs, float *hs32_dev, int64_t ldhs32,
                                  int32_t *status_dev, uint32_t max_polls, void *hip_stream) {
    return grim_bcr_gru_sequence_batch(Ai, Ah, xs_dev, ldxs, T, 1, bias_i_dev, bias_h_dev, h0_dev, h32_dev, hs_dev, ldhs,
                                       hs32_dev, ldhs32, status_dev, max_polls, hip_stream);
}

grim_status grim_bcr_gru_sequence_batch(const grim_bcr_matrix *Ai, const grim_bcr_matrix *Ah, const void *xs_dev, int64_t ldxs,
                                        int32_t T, int32_t batch, const float *bias_i_dev, const float *bias_h_dev,
                                        const void *h0_dev, float *h32_dev, void *hs_dev, int64_t ldhs, float *hs32_dev,
                                        int64_t ldhs32, int32_t *status_dev, uint32_t max_polls, void *hip_stream) {
    grim_status st = seq_check(Ai, xs_dev, T, batch, h0_dev, h32_dev, hs_dev, status_dev);
    if (st != GRIM_OK) return st;
    if (!Ah) return GRIM_ERR_NULL;
    if (Ai->M != Ah->M || Ai->M % 3 != 0 || Ah->K != Ai->M / 3) return GRIM_ERR_SHAPE;
    if (Ai->dtype != Ah->dtype) return GRIM_ERR_DTYPE;
    if (!Ah->on_device || Ah->device != Ai->device) return GRIM_ERR_DEVICE;
    const int64_t H = Ah->K, I = Ai->K;
    if (ldxs < I || ldhs < H || (hs32_dev && ldhs32 < H)) return GRIM_ERR_SHAPE;
    if (!grim_bcr_rnn_sequence_batch_supported(Ai, Ah, batch)) return GRIM_ERR_UNSUPPORTED;
    void *exch = nullptr;
    st = seq_exchange_of(Ah, &exch);
    if (st != GRIM_OK) return st;
    const GemvDesc dh = desc_of(Ah);
    return launch_rnn_seq(2, desc_of(Ai), &dh, Ai->dev.strip_pos, Ah->dev.strip_pos, Ai->BR, Ai->BC, Ai->dtype,
                          Ai->gemv.uniform_kr, Ai->gemv.uniform_kc, I, H, I, H, T, batch, xs_dev, ldxs, h0_dev, bias_i_dev, bias_h_dev,
                          h32_dev, hs_dev, ldhs, hs32_dev, ldhs32, exch, status_dev, max_polls,
                          static_cast<hipStream_t>(hip_stream));
}

grim_status grim_gru_cell(const float *gi_dev, int64_t ldgi, const float *gh_dev, int64_t ldgh, const float *bias_i_dev,
                          const float *bias_h_dev, float *h32_dev, int64_t ldh32, void *h_dev, grim_dtype dt, int64_t ldh,
                          int64_t H, int32_t batch, void *hip_stream) {
    if (!gi_dev || !gh_dev || !h32_dev) return GRIM_ERR_NULL;
    if (H < 1 || batch < 1 || ldgi < batch || ldgh < batch || ldh32 < batch || (h_dev && ldh < batch)) return GRIM_ERR_SHAPE;
    if (H > (int64_t(1) << 40) / batch) return GRIM_ERR_SHAPE;
    if (dt != GRIM_F32 && dt != GRIM_F16 && dt != GRIM_BF16) return GRIM_ERR_DTYPE;
    return launch_gru_cell(gi_dev, ldgi, gh_dev, ldgh, bias_i_dev, bias_h_dev, h32_dev, ldh32, h_dev, dt, ldh, H, batch,
                           static_cast<hipStream_t>(hip_stream));
}

grim_status grim_bcr_gru_step(const grim_bcr_matrix *Ai, const grim_bcr_matrix *Ah, const void *x_dev, int64_t ldx,
                              const void *hin_dev, int64_t ldhin, int32_t batch, float *gi_dev, int64_t ldgi,
                              float *gh_dev, int64_t ldgh, const float *bias_i_dev, const float *bias_h_dev,
                              float *h32_dev, int64_t ldh32, void *hout_dev, int64_t ldhout, void *hip_stream) {
    if (!Ai || !Ah || !x_dev || !hin_dev || !gi_dev || !gh_dev || !h32_dev) return GRIM_ERR_NULL;
    if (Ai->M != Ah->M || Ai->M % 3 != 0 || Ah->K != Ai->M / 3) return GRIM_ERR_SHAPE;
    if (Ai->dtype != Ah->dtype) return GRIM_ERR_DTYPE;
    const int64_t H = Ai->M / 3;
    if (batch < 1 || ldh32 < batch || (hout_dev && ldhout < batch)) return GRIM_ERR_SHAPE;
    grim_status st = check_call(Ai, x_dev, batch, ldx, gi_dev, ldgi);
    if (st == GRIM_OK) st = check_call(Ah, hin_dev, batch, ldhin, gh_dev, ldgh);
    if (st != GRIM_OK) return st;
    // Both products in one launch when the two matrices have one shape and the SpMV kernels take
    // them: the second operand / result is addressed as the first plus a stride (of either sign).
    const int esz = dtype_size(Ai->dtype);
    const ptrdiff_t xd = static_cast<const char *>(hin_dev) - static_cast<const char *>(x_dev);
    const ptrdiff_t yd = reinterpret_cast<const char *>(gh_dev) - reinterpret_cast<const char *>(gi_dev);
    // (few columns of a matrix the wave-per-strip kernels are not compiled for: on the matrix cores, as for a lone product)
    if (spmv_cell_batch_ok(H, Ai->BR, batch) && Ai->K == Ah->K && Ai->BR == Ah->BR && Ai->BC == Ah->BC && Ai->gemv.present && Ah->gemv.present &&
        Ai->gemv.uniform_kr == Ah->gemv.uniform_kr && Ai->gemv.uniform_kc == Ah->gemv.uniform_kc && ldx == ldhin && ldgi == ldgh &&
        xd % esz == 0 && yd % 4 == 0) {
        // One launch: both gate products with the cell in the epilogue.  The new state must not land in the vector
        // the hidden-side product reads (workgroups write it while others may still read).
        const bool aliased = hout_dev && (ranges_overlap(hin_dev, ((Ah->K - 1) * ldhin + batch) * esz, hout_dev, ((H - 1) * ldhout + batch) * esz) ||
                                          ranges_overlap(x_dev, ((Ai->K - 1) * ldx + batch) * esz, hout_dev, ((H - 1) * ldhout + batch) * esz));
        if (!aliased) {
            const GemvDesc di = desc_of(Ai), dh = desc_of(Ah);
            RnnCell cell{Ai->order_identity ? nullptr : Ai->dev.strip_pos, Ah->order_identity ? nullptr : Ah->dev.strip_pos, bias_i_dev, bias_h_dev, h32_dev, hout_dev, nullptr, ldh32, ldhout, 0,
                         (int32_t)H, Ai->dtype};
            st = launch_spmv_cell(2, di, &dh, Ai->M, Ai->K, Ai->BR, Ai->BC, Ai->dtype, Ai->gemv.uniform_kr, Ai->gemv.uniform_kc,
                                  x_dev, xd / esz, batch, ldx, gi_dev, yd / 4, ldgi, cell, static_cast<hipStream_t>(hip_stream));
            if (st != GRIM_ERR_UNSUPPORTED) return st;
        }
    }
    if (rnn_gather_applies(Ai, x_dev, ldx, Ah, hin_dev, ldhin, H, batch)) {
        const bool aliased = hout_dev && (ranges_overlap(hin_dev, ((Ah->K - 1) * ldhin + batch) * esz, hout_dev, ((H - 1) * ldhout + batch) * esz) ||
                                          ranges_overlap(x_dev, ((Ai->K - 1) * ldx + batch) * esz, hout_dev, ((H - 1) * ldhout + batch) * esz));
        if (!aliased) {
            RnnCell cell{nullptr, nullptr, bias_i_dev, bias_h_dev, h32_dev, hout_dev, nullptr, ldh32, ldhout, 0, (int32_t)H, Ai->dtype};
            return launch_rnn_gather(Ai, x_dev, ldx, gi_dev, ldgi, Ah, hin_dev, ldhin, gh_dev, ldgh, batch, cell, static_cast<hipStream_t>(hip_stream));
        }
    }
    const bool few_on_matrix_cores = ldx == ldhin && ldgi == ldgh && skinny_on_matrix_cores(Ai, x_dev, batch, ldx, 2) &&
                                       skinny_on_matrix_cores(Ah, hin_dev, batch, ldx, 2) &&
                                       gather_pair_applies(Ai, x_dev, Ah, hin_dev, batch, ldx);
    if (!few_on_matrix_cores && batch <= 8 && Ai->K == Ah->K && Ai->BR == Ah->BR && Ai->BC == Ah->BC && gemv_ok(Ai, batch) &&
        gemv_ok(Ah, batch) && ldx == ldhin && ldgi == ldgh && xd % esz == 0 && yd % 4 == 0) {
        const GemvDesc di = desc_of(Ai), dh = desc_of(Ah);
        const bool same = Ai->gemv.uniform_kr == Ah->gemv.uniform_kr && Ai->gemv.uniform_kc == Ah->gemv.uniform_kc;
        st = launch_spmv(nullptr, di, &dh, 2, Ai->M, Ai->K, Ai->BR, Ai->BC, Ai->dtype, same ? Ai->gemv.uniform_kr : -1,
                         same ? Ai->gemv.uniform_kc : -1, std::min(Ai->gemv.vec, Ah->gemv.vec),
                         std::max(Ai->gemv.krmax, Ah->gemv.krmax), std::max(Ai->gemv.kcmax, Ah->gemv.kcmax), x_dev, xd / esz,
                         batch, ldx, gi_dev, yd / 4, ldgi, static_cast<hipStream_t>(hip_stream));
    } else if (ldx == ldhin && ldgi == ldgh && gather_pair_applies(Ai, x_dev, Ah, hin_dev, batch, ldx)) {
        // fewer than 64 columns on the matrix cores: one launch of the row-gathering kernel, grid.y = product
        st = launch_spmm_gather(Ai, x_dev, batch, ldx, gi_dev, ldgi, static_cast<hipStream_t>(hip_stream), Ah, hin_dev, gh_dev);
    } else {
        st = grim_bcr_spmm(Ai, x_dev, batch, ldx, gi_dev, ldgi, hip_stream);
        if (st == GRIM_OK) st = grim_bcr_spmm(Ah, hin_dev, batch, ldhin, gh_dev, ldgh, hip_stream);
    }
    if (st != GRIM_OK) return st;
    return grim_gru_cell(gi_dev, ldgi, gh_dev, ldgh, bias_i_dev, bias_h_dev, h32_dev, ldh32, hout_dev, (grim_dtype)Ai->dtype,
                         ldhout, H, batch, hip_stream);
}

// The table of the matrices' row-gathering layouts, if all have one (without memory for it the group does without).
static void add_group_gather(grim_bcr_group *G, const grim_bcr_matrix *const *mats) {
    int64_t steps = 0;
    for (int32_t i = 0; i < G->count; ++i) {
        if (!mats[i]->gather.present || mats[i]->gather.nstrips != mats[0]->gather.nstrips) return;
        steps += mats[i]->gather.nsteps;
    }
    const size_t each = gather_entry_bytes();
    std::vector<unsigned char> table;
    try {
        table.resize(each * (size_t)G->count);
    } catch (const std::bad_alloc &) {
        return;
    }
    for (int32_t i = 0; i < G->count; ++i) gather_fill_entry(mats[i], table.data() + each * (size_t)i);
    if (hipMalloc(&G->d_gather, table.size()) != hipSuccess) { (void)hipGetLastError(); G->d_gather = nullptr; return; }
    if (hipMemcpy(G->d_gather, table.data(), table.size(), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(G->d_gather);
        G->d_gather = nullptr;
        return;
    }
    G->gather_runs = mats[0]->gather.nstrips;
    G->gather_steps = steps;
}

grim_status grim_bcr_group_create(const grim_bcr_matrix *const *mats, int32_t count, grim_bcr_group **out) {
    if (out) *out = nullptr;
    if (!mats || !out) return GRIM_ERR_NULL;
    if (count < 1 || count > 65535) return GRIM_ERR_SHAPE;   // grid.y = matrix
    for (int32_t i = 0; i < count; ++i)
        if (!mats[i]) return GRIM_ERR_NULL;
    const grim_bcr_matrix *A0 = mats[0];
    int dev = -1;
    if (!A0->on_device || hipGetDevice(&dev) != hipSuccess || dev != A0->device) return GRIM_ERR_DEVICE;
    if (!A0->gemv.present) return GRIM_ERR_UNSUPPORTED;
    grim_bcr_group *G = nullptr;
    std::vector<GemvDesc> table;
    try {
        G = new grim_bcr_group();
        table.resize(count);
    } catch (const std::bad_alloc &) {
        delete G;
        return GRIM_ERR_ALLOC;
    }
    G->count = count; G->M = A0->M; G->K = A0->K; G->BR = A0->BR; G->BC = A0->BC; G->dtype = A0->dtype;
    G->nbr = A0->nbr; G->nbc = A0->nbc; G->device = dev;
    G->uniform_kr = A0->gemv.uniform_kr; G->uniform_kc = A0->gemv.uniform_kc; G->vec = A0->gemv.vec;
    G->krmax = A0->gemv.krmax; G->kcmax = A0->gemv.kcmax;
    for (int32_t i = 0; i < count; ++i) {
        const grim_bcr_matrix *A = mats[i];
        if (A->M != G->M || A->K != G->K || A->BR != G->BR || A->BC != G->BC || A->dtype != G->dtype) { delete G; return GRIM_ERR_SHAPE; }
        if (!A->on_device || A->device != dev) { delete G; return GRIM_ERR_DEVICE; }
        if (!A->gemv.present) { delete G; return GRIM_ERR_UNSUPPORTED; }
        if (A->gemv.uniform_kr != G->uniform_kr || A->gemv.uniform_kc != G->uniform_kc) G->uniform_kr = G->uniform_kc = -1;
        G->vec = std::min(G->vec, A->gemv.vec);
        G->krmax = std::max(G->krmax, A->gemv.krmax);
        G->kcmax = std::max(G->kcmax, A->gemv.kcmax);
        table[i] = desc_of(A);
    }
    if (hipMalloc(reinterpret_cast<void **>(&G->d_table), sizeof(GemvDesc) * count) != hipSuccess) { (void)hipGetLastError(); delete G; return GRIM_ERR_ALLOC; }
    if (hipMemcpy(G->d_table, table.data(), sizeof(GemvDesc) * count, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError(); (void)hipFree(G->d_table); delete G; return GRIM_ERR_DEVICE;
    }
    add_group_gather(G, mats);
    *out = G;
    return GRIM_OK;
}

// Groups the wave-per-strip SpMV kernels are not compiled for, and small launches of those for several columns, on the matrix
// cores (16-bit types, one padded 16-column tile per run of 16 rows).  Before -> there: 64 of 2048 x 2048 of mixed rates at 1 / 8
// columns 54.3 / 168 -> 24.6 / 28.3 us; 39 of 960 x 1632 keeping 10 x 10 at 8 25.5 -> 9.2; 12 of 2048 x 512 in 8 x 32 blocks of
// mixed rates at 1 / 8 15.8 / 34.5 -> 4.9 / 5.3; 20 of 2048 x 4096 keeping 8 x 12 at 4 27.2 -> 19.0.
static bool group_on_matrix_cores(const grim_bcr_group *G, int32_t batch) {
    if (!G->d_gather || G->BR < 8) return false;
    if (batch == 1) return !spmv_exact_applies(G->dtype, G->uniform_kr, G->uniform_kc, G->K);
    if (spmv_many_strips_applies(G->count, G->nbr, G->dtype, G->uniform_kr, G->uniform_kc, G->K, G->BC, batch))
        return group_quicker_on_matrix_cores(G->count, G->nbr, G->nbc, G->uniform_kr, G->uniform_kc, G->K, G->gather_runs, G->gather_steps, batch);
    // (columns as sets of workgroups: the bits of a call for one matrix, which takes that form too)
    if (spmv_column_sets_ok(G->count, G->nbr, batch) && spmv_exact_applies(G->dtype, G->uniform_kr, G->uniform_kc, G->K)) return false;
    return true;
}

grim_status grim_bcr_spmv_batched(const grim_bcr_group *G, const void *x_dev, int64_t x_stride, int32_t batch, int64_t ldx,
                                  float *y_dev, int64_t y_stride, int64_t ldy, void *hip_stream) {
    if (!G || !x_dev || !y_dev) return GRIM_ERR_NULL;
    if (batch < 1 || batch > 8 || ldx < batch || ldy < batch || x_stride < 0 || y_stride < 0) return GRIM_ERR_SHAPE;
    if (G->K * batch * dtype_size(G->dtype) > kGemvMaxXBytes) return GRIM_ERR_UNSUPPORTED;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != G->device) return GRIM_ERR_DEVICE;
    if (group_on_matrix_cores(G, batch)) {
        const grim_status st = launch_spmm_gather_many(G, x_dev, x_stride, batch, ldx, y_dev, y_stride, ldy, static_cast<hipStream_t>(hip_stream));
        if (st != GRIM_ERR_UNSUPPORTED) return st;
    }
    GemvDesc none{nullptr, nullptr, nullptr, nullptr};
    return launch_spmv(G->d_table, none, nullptr, G->count, G->M, G->K, G->BR, G->BC, G->dtype, G->uniform_kr, G->uniform_kc, G->vec, G->krmax, G->kcmax,
                       x_dev, x_stride, batch, ldx, y_dev, y_stride, ldy, static_cast<hipStream_t>(hip_stream));
}

void grim_bcr_group_free(grim_bcr_group *G) {
    if (!G) return;
    if (G->d_table) (void)hipFree(G->d_table);
    if (G->d_gather) (void)hipFree(G->d_gather);
    delete G;
}

void grim_bcr_free(grim_bcr_matrix *A) {
    if (!A) return;
    if (A->seq_exch) (void)hipFree(A->seq_exch);
    if (A->on_device && A->dev.strip_order) (void)hipFree(A->dev.strip_order);   // base of the slab
    delete A;
}

const char *grim_status_str(grim_status s) {
    switch (s) {
        case GRIM_OK: return "GRIM_OK";
        case GRIM_ERR_NULL: return "GRIM_ERR_NULL: required pointer is NULL";
        case GRIM_ERR_SHAPE: return "GRIM_ERR_SHAPE: invalid shape, block size, leading dimension or batch";
        case GRIM_ERR_INDEX: return "GRIM_ERR_INDEX: malformed kept-row / kept-column index sets";
        case GRIM_ERR_DTYPE: return "GRIM_ERR_DTYPE: unknown element type";
        case GRIM_ERR_ALLOC: return "GRIM_ERR_ALLOC: allocation failed";
        case GRIM_ERR_DEVICE: return "GRIM_ERR_DEVICE: HIP failure, no GPU, wrong current device, or host-only matrix";
        case GRIM_ERR_UNSUPPORTED: return "GRIM_ERR_UNSUPPORTED: no kernel covers this request";
    }
    return "unknown grim_status";
}

}  // extern "C"
