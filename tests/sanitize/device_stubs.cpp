// Stand-ins for the kernel launchers, so that the host side of the library (validation, compaction, the
// derived layouts, their decoders, the BCRC export) links without any device code and can run under the
// address and undefined-behaviour sanitizers on a machine without a GPU.  Every launcher reports that
// there is no device; nothing here computes anything.
#include "bcr_matrix.hpp"
#include "conv_rules.hpp"

namespace grim {
grim_status launch_spmm_fma(const grim_bcr_matrix *, const void *, int64_t, int64_t, float *, int64_t, hipStream_t) { return GRIM_ERR_DEVICE; }
grim_status launch_spmm_mma(const grim_bcr_matrix *, const void *, int64_t, int64_t, float *, int64_t, int32_t, int32_t, hipStream_t) { return GRIM_ERR_DEVICE; }
bool mma_supported(const grim_bcr_matrix *) { return false; }
grim_status launch_spmm_wide(const grim_bcr_matrix *, const void *, int64_t, int64_t, float *, int64_t, int32_t, hipStream_t) { return GRIM_ERR_DEVICE; }
grim_status launch_spmm_wide_with_rest(const grim_bcr_matrix *, const void *, int64_t, int64_t, float *, int64_t, int32_t, int64_t, hipStream_t) { return GRIM_ERR_DEVICE; }
bool wide_applies(const grim_bcr_matrix *, const void *, int64_t, int64_t, const float *, int64_t, int32_t) { return false; }
double wide_plan(const grim_bcr_matrix *, const void *, int64_t, int64_t, const float *, int64_t, double (*)(const grim_bcr_matrix *, int64_t), int *, int64_t *) { return -1.0; }
grim_status launch_spmm_gather(const grim_bcr_matrix *, const void *, int64_t, int64_t, float *, int64_t, hipStream_t, const grim_bcr_matrix *, const void *, float *) { return GRIM_ERR_DEVICE; }
bool gather_pair_applies(const grim_bcr_matrix *, const void *, const grim_bcr_matrix *, const void *, int64_t, int64_t) { return false; }
bool gather_applies(const grim_bcr_matrix *, const void *, int64_t, int64_t) { return false; }
bool gather_any_applies(const grim_bcr_matrix *, const void *, int64_t, int64_t) { return false; }
bool gather32_quicker(const grim_bcr_matrix *, int64_t) { return false; }
bool gather32_applies(const grim_bcr_matrix *, const void *) { return false; }
grim_status launch_spmm_gather32(const grim_bcr_matrix *, const void *, int64_t, int64_t, float *, int64_t, hipStream_t) { return GRIM_ERR_DEVICE; }
// the convolutions' rules: the library's own where a test asks for them
static int g_conv_rules = 0;
extern "C" void grim_stub_conv_rules(int own) { g_conv_rules = own; }
bool gather_wave_per_strip(const grim_bcr_matrix *, int64_t, int64_t) { return false; }
grim_status launch_conv_gather(const grim_bcr_matrix *, const void *, int32_t, int32_t, int32_t, int32_t, int32_t, const float *, int32_t, void *, int32_t, int64_t, hipStream_t, int32_t, int32_t, int64_t, int64_t, const uint32_t *, int32_t, int64_t, int64_t) { return GRIM_ERR_DEVICE; }
grim_status launch_conv_tall(const grim_bcr_matrix *, const GatherLayout &, const uint32_t *, const void *, int32_t, int32_t, int32_t, int32_t, int32_t, const float *, int32_t, void *, int32_t, int64_t, hipStream_t, int32_t, int32_t, int64_t, int64_t) { return GRIM_ERR_DEVICE; }
bool conv_batch_sums_as_one_image(const grim_bcr_matrix *A, int64_t positions, int32_t batch) { return !g_conv_rules || conv_batch_sums_as_one(A, positions, batch); }
uint32_t conv_plan_word(uint32_t, int32_t, int32_t, int32_t, int32_t) { return 0; }
// octets a plan's dense copy is made with (0: none), as a test asks
static int g_patch_octets = 0;
int32_t conv_patch_octets(int64_t Cin, int32_t H, int32_t W, int32_t kh, int32_t kw, int32_t stride) { return g_conv_rules ? patch_octets(Cin, H, W, kh, kw, stride) : g_patch_octets; }
extern "C" void grim_stub_patch_octets(int octets) { g_patch_octets = octets; }
grim_status launch_conv_patch(const grim_bcr_matrix *, const ConvDense &, const uint32_t *, const void *, int32_t, int32_t, int32_t, int32_t, int32_t, const float *, int32_t, void *, int32_t, int64_t, hipStream_t, int32_t, int32_t, int64_t, int64_t) { return GRIM_ERR_UNSUPPORTED; }
size_t gather_entry_bytes() { return 8; }
void gather_fill_entry(const grim_bcr_matrix *A, void *entry) { __builtin_memcpy(entry, &A, 8); }
grim_status launch_spmm_gather_many(const grim_bcr_group *, const void *, int64_t, int64_t, int64_t, float *, int64_t, int64_t, hipStream_t) { return GRIM_ERR_DEVICE; }
bool conv_wide_applies(const grim_bcr_matrix *, const void *, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int64_t, const void *, int32_t, int64_t, int64_t) { return false; }
grim_status launch_conv_wide(const grim_bcr_matrix *, const void *, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int64_t, const float *, int32_t, void *, int32_t, int64_t, int64_t, hipStream_t) { return GRIM_ERR_UNSUPPORTED; }
double gather_cost(const grim_bcr_matrix *, int64_t) { return 0.0; }
double mma_best_shape(const grim_bcr_matrix *, int64_t, int32_t, int32_t, int *, int *) { return -1.0; }
int64_t mma_whole_rounds(const grim_bcr_matrix *, int64_t N, int *, int *) { return N; }
grim_status launch_spmv(const GemvDesc *, const GemvDesc &, const GemvDesc *, int32_t, int64_t, int64_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, const void *, int64_t, int32_t, int64_t, float *, int64_t, int64_t, hipStream_t) { return GRIM_ERR_DEVICE; }
bool spmv_cell_applies(int, int64_t, int64_t, int32_t, int32_t, int32_t, int32_t, int32_t, int64_t) { return false; }
grim_status launch_spmv_cell(int, const GemvDesc &, const GemvDesc *, int64_t, int64_t, int32_t, int32_t, int32_t, int32_t, int32_t, const void *, int64_t, int32_t, int64_t, float *, int64_t, int64_t, const RnnCell &, hipStream_t) { return GRIM_ERR_DEVICE; }
bool rnn_gather_applies(const grim_bcr_matrix *, const void *, int64_t, const grim_bcr_matrix *, const void *, int64_t, int64_t, int32_t) { return false; }
grim_status launch_rnn_gather(const grim_bcr_matrix *, const void *, int64_t, float *, int64_t, const grim_bcr_matrix *, const void *, int64_t, float *, int64_t, int32_t, const RnnCell &, hipStream_t) { return GRIM_ERR_DEVICE; }
grim_status rnn_seq_static_exchange(void **) { return GRIM_ERR_DEVICE; }
bool spmv_cell_batch_ok(int64_t, int32_t, int32_t) { return false; }
bool spmv_exact_applies(int32_t, int32_t, int32_t, int64_t) { return false; }
bool spmv_many_strips_applies(int64_t, int64_t, int32_t, int32_t, int32_t, int64_t, int32_t, int32_t) { return false; }
bool spmv_column_sets_ok(int64_t, int64_t, int32_t) { return false; }
bool rnn_seq_applies(int, int32_t, int32_t, int32_t, int32_t, int32_t, int64_t, int64_t, int64_t, int64_t, int32_t) { return false; }
grim_status launch_rnn_seq(int, const GemvDesc &, const GemvDesc *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t, int32_t, int32_t, int64_t, int64_t, int64_t, int64_t, int32_t, int32_t, const void *, int64_t, const void *, const float *, const float *, float *, void *, int64_t, float *, int64_t, void *, int32_t *, uint32_t, hipStream_t) { return GRIM_ERR_DEVICE; }
grim_status launch_lstm_cell(const float *, int64_t, const float *, float *, int64_t, void *, int32_t, int64_t, float *, int64_t, int64_t, int32_t, hipStream_t) { return GRIM_ERR_DEVICE; }
grim_status launch_gru_cell(const float *, int64_t, const float *, int64_t, const float *, const float *, float *, int64_t, void *, int32_t, int64_t, int64_t, int32_t, hipStream_t) { return GRIM_ERR_DEVICE; }
}  // namespace grim

// the HIP runtime calls the host side makes (allocation and upload of a packed matrix): no device here, unless a test asks for
// one made of host memory, whose allocations can be counted and made to fail
#include <cstdlib>
#include <cstring>
extern "C" {
static int g_device = 0, g_allocations_left = -1, g_live = 0;
// device: 1 = a device made of host memory; allocations_left: allocations that succeed from now on (-1: all)
void grim_stub_device(int device, int allocations_left) { g_device = device; g_allocations_left = allocations_left; }
int grim_stub_live_allocations() { return g_live; }
hipError_t hipGetDeviceCount(int *n) { if (n) *n = g_device; return g_device ? hipSuccess : hipErrorNoDevice; }
hipError_t hipGetDevice(int *d) { if (d) *d = g_device ? 0 : -1; return g_device ? hipSuccess : hipErrorNoDevice; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    *p = nullptr;
    if (!g_device) return hipErrorNoDevice;
    if (g_allocations_left == 0) return hipErrorOutOfMemory;
    if (g_allocations_left > 0) --g_allocations_left;
    *p = std::malloc(n);
    if (*p) ++g_live;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
    if (!g_device) return hipErrorNoDevice;
    if (p) --g_live;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) {
    if (!g_device) return hipErrorNoDevice;
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *src, size_t n, hipMemcpyKind) {
    if (!g_device) return hipErrorNoDevice;
    std::memcpy(d, src, n);
    return hipSuccess;
}
}
