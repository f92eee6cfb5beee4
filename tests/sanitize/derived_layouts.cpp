// csrc/bcr_pack.cpp with decoders for the two layouts that grim_bcr_unpack_layout does not reach: the fp32 row-gathering
// product's, and the runs of 64 rows that a convolution plan makes for itself.
#include "bcr_pack.cpp"

namespace {
// Runs of 16 R rows in steps of 4 groups of `slots` k slots, as the kernels read them; false where an index leaves the matrix
// or a row of a run is written to that does not exist.
template <int R>
bool decode(const grim_bcr_matrix *A, const grim::GatherLayout &L, int slots, bool slot_major, unsigned char *W, int64_t ldw) {
    const int64_t esz = A->dtype == GRIM_F32 ? 4 : 2;
    for (int64_t i = 0; i < A->M; ++i) std::memset(W + i * ldw * esz, 0, (size_t)(A->K * esz));
    if (L.sptr.size() != (size_t)L.nstrips + 1 || L.sptr[0] != 0 || L.sptr[(size_t)L.nstrips] != L.nsteps) return false;
    for (int64_t u = 0; u < L.nstrips; ++u) {
        const int32_t n = L.sptr[(size_t)u + 1] - L.sptr[(size_t)u];
        if (n < 0 || n > L.max_steps || (L.usteps > 0 && n != L.usteps)) return false;
        for (int64_t s = L.sptr[(size_t)u]; s < L.sptr[(size_t)u + 1]; ++s) {
            for (int g = 0; g < 4; ++g) {
                for (int m = 0; m < R; ++m) {
                    const uint32_t mask = L.desc[(size_t)(s * R + m) * 8 + g * 2];
                    const unsigned char *w = L.payload.data() + (size_t)L.desc[(size_t)(s * R + m) * 8 + g * 2 + 1] * 16;
                    if (mask >> 16) return false;
                    for (int r = 0; r < 16; ++r) {
                        if (!((mask >> r) & 1u)) continue;
                        if (w + 16 > L.payload.data() + L.payload.size()) return false;
                        const int32_t row = L.out_row[(size_t)(u * R + m) * 16 + r];
                        if (row < 0 || row >= A->M) return false;
                        for (int j = 0; j < slots; ++j) {
                            const uint32_t k = L.rows[(size_t)s * 4 * slots + (slot_major ? j * 4 + g : g * slots + j)];
                            const unsigned char *at = w + j * esz;
                            if (k != 0xffffffffu && k >= (uint64_t)A->K) return false;
                            static const unsigned char zero[4] = {};
                            if (k != 0xffffffffu && std::memcmp(at, zero, (size_t)esz)) std::memcpy(W + (row * ldw + k) * esz, at, (size_t)esz);
                            else if (k == 0xffffffffu && std::memcmp(at, zero, (size_t)esz)) return false;    // padding multiplies zeros
                        }
                        w += 16;
                    }
                }
            }
        }
    }
    return true;
}
}  // namespace

extern "C" {
// a staged layout's rows to a chunk, chunks and most 16-byte units a chunk holds for groups of 4, 8, 16, 32 strips
int grim_test_staged_sizes(const grim_bcr_matrix *A, int wide, int64_t *out) {
    const grim::MmaLayout &L = wide ? A->mmaw : A->mma;
    if (!L.present) return 1;
    out[0] = L.chunk_rows;
    out[1] = L.nchunks;
    for (int g = 0; g < 4; ++g) out[2 + g] = L.amax[g];
    return 0;
}
// 0: decoded into W; 1: the matrix has no such layout; 2: the layout is not in order
int grim_test_decode_gather32(const grim_bcr_matrix *A, unsigned char *W, int64_t ldw) {
    if (!A->gather32.present) return 1;
    return decode<1>(A, A->gather32, 4, false, W, ldw) ? 0 : 2;
}
int grim_test_decode_64_row_runs(const grim_bcr_matrix *A, unsigned char *W, int64_t ldw) {
    grim::GatherLayout L;
    build_gather_layout<4>(A, L);
    if (!L.present) return 1;
    // (the steps a plan counts before it builds them)
    const RunSteps n = count_run_steps<4>(A);
    if (n.runs != L.nstrips || n.total != L.nsteps || n.longest != L.max_steps) return 2;
    return decode<4>(A, L, 8, true, W, ldw) ? 0 : 2;
}
}
