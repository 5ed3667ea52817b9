// The library's host code (csrc/pced_api.cpp) over stand-ins for the HIP runtime,
// the BLAS library and the kernel launchers, so that what it plans, launches and
// copies can be checked without a GPU. Nothing here computes: every launch and
// runtime call is recorded by name with a few of its arguments, and device
// addresses are never dereferenced. Compiled by tests/test_host_path.py.
#include <rocblas/rocblas.h>

#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "pced_internal.h"

namespace {
struct Rec {
  std::string name;
  long v[8];
};
std::vector<Rec> g_recs;
std::string g_fail_name;  // the g_fail_in-th call of this name from now on fails
int g_fail_in = 0;

hipError_t note(const char* name, long a = 0, long b = 0, long c = 0, long d = 0, long e = 0, long f = 0, long g = 0, long h = 0) {
  g_recs.push_back(Rec{name, {a, b, c, d, e, f, g, h}});
  if (g_fail_in > 0 && g_fail_name == name && --g_fail_in == 0) return hipErrorUnknown;
  return hipSuccess;
}
constexpr uintptr_t kDeviceFrom = (uintptr_t)1 << 46;  // addresses from here on count as device memory
}  // namespace

extern "C" {
int rec_count() { return (int)g_recs.size(); }
const char* rec_name(int i) { return g_recs[i].name.c_str(); }
long rec_value(int i, int j) { return g_recs[i].v[j]; }
void rec_clear() { g_recs.clear(); }
void rec_fail(const char* name, int nth) { g_fail_name = name; g_fail_in = nth; }

hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
  return note(kind == hipMemcpyHostToDevice ? "copy_in" : "copy", (long)n, (long)(uintptr_t)dst, (long)(uintptr_t)src);
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return note("copy_2d"); }
hipError_t hipStreamSynchronize(hipStream_t) { return note("synchronize"); }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof *a);
  a->type = (uintptr_t)p >= kDeviceFrom ? hipMemoryTypeDevice : hipMemoryTypeHost;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)(uintptr_t)16; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded failure"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t*, size_t*, hipDeviceptr_t) { return hipErrorUnknown; }

rocblas_status rocblas_create_handle(rocblas_handle* h) { *h = (rocblas_handle)(uintptr_t)16; return rocblas_status_success; }
rocblas_status rocblas_destroy_handle(rocblas_handle) { return rocblas_status_success; }
rocblas_status rocblas_set_stream(rocblas_handle, hipStream_t) { return rocblas_status_success; }
const char* rocblas_status_to_string(rocblas_status) { return ""; }
rocblas_status rocblas_gemm_ex(rocblas_handle, rocblas_operation, rocblas_operation, rocblas_int m, rocblas_int n,
                               rocblas_int k, const void*, const void*, rocblas_datatype, rocblas_int, const void*,
                               rocblas_datatype, rocblas_int, const void*, const void*, rocblas_datatype, rocblas_int,
                               void*, rocblas_datatype, rocblas_int, rocblas_datatype, rocblas_gemm_algo, int32_t,
                               uint32_t) {
  note("library_gemm", m, n, k);
  return rocblas_status_success;
}
}  // extern "C"

namespace pced {
hipError_t launch_fill_i32(int32_t*, int32_t, size_t, hipStream_t) { return note("fill"); }
hipError_t launch_zero_bytes(void*, size_t, hipStream_t) { return note("zero"); }
hipError_t launch_load(const LoadArgs& a, int n_items, bool, hipStream_t, const Timing*) {
  return note("load", n_items, a.items != nullptr, a.layer0, a.n_layers, a.one_s, a.page0, a.one_len);
}
hipError_t launch_append(const AppendArgs& a, bool, hipStream_t, const Timing*) {
  return note("append", a.n_chunks, a.total_pages, a.n_seqs);
}
hipError_t launch_attn(const AttnArgs& a, int, bool, hipStream_t, const Timing*) {
  return note("attn", a.layer, a.launch_layers, a.n_chunks, a.kv_reread, a.tq, a.tq_T, a.split_stride, a.n_seqs);
}
hipError_t launch_attn_combine(const AttnArgs& a, int, bool, hipStream_t, const Timing*) {
  return note("combine", a.layer, a.launch_layers);
}
int attn_blocks_per_cu(int, bool) { return 8; }
hipError_t launch_pack_lm_head(const void*, void*, int, int, bool, hipStream_t) { return note("pack"); }
hipError_t launch_lmhead(const LmArgs&, bool, hipStream_t, const Timing*) { return note("lmhead"); }
hipError_t launch_beta(const BetaArgs&, int, int, bool, hipStream_t, const Timing*) { return note("beta"); }
hipError_t launch_fuse(const FuseArgs&, int, hipStream_t, const Timing*, const Timing*) { return note("fuse"); }
int fuse_slice(int, int, int) { return 512; }
int agg_slice(int, int, int, int) { return kAggSlice; }
hipError_t launch_beta_mean(const BetaArgs&, int, hipStream_t) { return note("beta_mean"); }
hipError_t launch_agg(const AggArgs&, int, int, hipStream_t, const Timing*) { return note("agg"); }
hipError_t launch_fuse_final(const FuseArgs&, int, hipStream_t, const Timing*) { return note("fuse_final"); }
int lmhead_fused_nblk(int, int, bool) { return 0; }
LmWidePlan lmhead_wide_plan(int, int, int) { return LmWidePlan{}; }
LmWidePlan lmhead_wide_plan_queries(const int32_t*, int, int, int, int) { return LmWidePlan{}; }
size_t lmhead_packed_rows(const LmWidePlan&) { return 0; }
hipError_t launch_synth(const SynthArgs&, int, hipStream_t, const Timing*) { return note("synth"); }
hipError_t launch_copy_rows(const void*, void*, size_t, hipStream_t) { return note("copy_rows"); }
hipError_t launch_stream_read(const void*, size_t, uint32_t*, int, hipStream_t) { return note("stream_read"); }
hipError_t launch_pack_tiles(const void*, void*, int, int, int, int, int, hipStream_t) { return note("pack_tiles"); }
hipError_t launch_gemm(const GemmArgs& a, GemmEpi epi, hipStream_t, const Timing*) { return note("gemm", a.M, epi); }
hipError_t launch_proj_epilogue(const GemmArgs& a, GemmEpi epi, hipStream_t, const Timing*) { return note("epilogue", a.M, epi); }
int proj_ksplit(int, int, int) { return 1; }
hipError_t launch_embed(const EmbedArgs&, int rows, hipStream_t, const Timing*) { return note("embed", rows); }
hipError_t launch_prefill_meta(const PrefillMetaArgs&, hipStream_t) { return note("prefill_meta"); }
hipError_t launch_read_cache(const ReadCacheArgs&, hipStream_t) { return note("read_cache"); }
hipError_t noalloc_scratch(void** out) { *out = nullptr; return hipErrorUnknown; }
hipError_t launch_rho(const float*, int, int, int, float, float, float*, hipStream_t) { return note("rho"); }
hipError_t launch_rope_table(float2*, int, int, double, hipStream_t) { return note("rope"); }
}  // namespace pced
