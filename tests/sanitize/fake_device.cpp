#include "fake_device.h"

#include <cstdlib>
#include <cstring>
#include <map>

#include "../../paper_1412_6367_amd/csrc/fused.h"
#include "../../paper_1412_6367_amd/csrc/plan_device.h"

namespace fake {
std::vector<std::string> calls;
azi::StreamLaunch stream;
azi::BandLaunch band;
const void *dark = nullptr, *norm = nullptr;
int64_t fail_in = -1, live = 0, uploaded = 0;
int encoded = 0;
static std::map<void*, size_t> sizes;
bool held(const void* p) {
    auto i = sizes.upper_bound(const_cast<void*>(p));
    if (i == sizes.begin()) return false;
    --i;
    return (const char*)p < (const char*)i->first + i->second;
}
static hipError_t note(const char* name) {
    calls.push_back(name);
    return hipSuccess;
}
}  // namespace fake

// azi::build_stream, linked with --wrap
extern "C" {
bool __real__ZN3azi12build_streamERKNS_10HostMatrixEiiillRNS_12StreamMatrixE(
    const azi::HostMatrix&, int32_t, int32_t, int32_t, int64_t, int64_t, azi::StreamMatrix&);
bool __wrap__ZN3azi12build_streamERKNS_10HostMatrixEiiillRNS_12StreamMatrixE(
    const azi::HostMatrix& m, int32_t h, int32_t w, int32_t px, int64_t pix, int64_t bin,
    azi::StreamMatrix& sm) {
    ++fake::encoded;
    return __real__ZN3azi12build_streamERKNS_10HostMatrixEiiillRNS_12StreamMatrixE(m, h, w, px, pix,
                                                                                  bin, sm);
}
hipError_t hipMalloc(void** p, size_t n) {
    if (fake::fail_in >= 0 && fake::fail_in-- == 0) return hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    fake::sizes[*p] = n;
    fake::live += (int64_t)n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    fake::live -= (int64_t)fake::sizes[p];
    fake::sizes.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    if (k == hipMemcpyHostToDevice) fake::uploaded += (int64_t)n;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(d, s, n, k);
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetSymbolAddress(void** p, const void* s) {
    *p = const_cast<void*>(s);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return fake::note("graph"); }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}

namespace azi {
using fake::note;
hipError_t launch_forward(const ForwardLaunch&, hipStream_t) { return note("forward"); }
hipError_t launch_backward(const BackwardLaunch&, hipStream_t) { return note("backward"); }
hipError_t launch_correct(const void*, int32_t, const int32_t*, const void* dark, const void* norm,
                          void*, int32_t, int64_t, hipStream_t) {
    fake::dark = dark;
    fake::norm = norm;
    return note("correct");
}
hipError_t launch_band(const BandLaunch& a, hipStream_t) {
    fake::band = a;
    return note("band");
}
int32_t runs_resident_per_cu(int32_t, int32_t, int32_t waves) { return 32 / waves; }
hipError_t launch_corr_pair(const void*, const void*, void*, int32_t, int64_t, hipStream_t) {
    return note("corr_pair");
}
hipError_t launch_dark_is_float(const double*, int64_t, int32_t*, hipStream_t) {
    return note("dark_is_float");
}
hipError_t launch_corr_record12(const double*, const double*, void*, int64_t, hipStream_t) {
    return note("corr_record12");
}
hipError_t launch_block(const BlockLaunch&, hipStream_t) { return note("block"); }
hipError_t launch_stage(const StageLaunch&, hipStream_t) { return note("stage"); }
hipError_t launch_norm(const void*, const void*, const void*, void*, int32_t, int64_t, hipStream_t) {
    return note("norm");
}
hipError_t launch_fused(const FusedLaunch&, hipStream_t) { return note("fused"); }
hipError_t launch_stream(const StreamLaunch& a, hipStream_t) {
    fake::stream = a;
    return note("stream");
}
hipError_t launch_stream_coef(const StreamCoefLaunch&, hipStream_t) { return note("stream_coef"); }
hipError_t launch_stream_adjoint(const StreamAdjointLaunch&, hipStream_t) {
    return note("stream_adjoint");
}
hipError_t launch_dark_kind(const void*, int32_t, int64_t, int32_t*, hipStream_t) {
    return note("dark_kind");
}
hipError_t launch_dark_store(const void*, int32_t, int32_t, void*, int64_t, hipStream_t) {
    return note("dark_store");
}
// The device builder's kernels: not for plans made here.
hipError_t launch_extents(const azi_geom&, int32_t, int32_t, double*, double*, double*, double*,
                          hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_minmax(const double*, const double*, int64_t, double*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_count(const azi_geom&, int32_t, int32_t, const double*, const double*, double,
                        double, int32_t, int32_t, int32_t*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_fill(const azi_geom&, int32_t, int32_t, const double*, const double*, double,
                       double, int32_t, int32_t, const int32_t*, int32_t*, double*, int32_t*,
                       hipStream_t) {
    return hipErrorNotSupported;
}
size_t scan_work_bytes(int64_t) { return 256; }
hipError_t launch_scan(const int32_t*, int64_t, int32_t*, int64_t*, void*, hipStream_t) {
    return hipErrorNotSupported;
}
size_t sort_work_bytes(int64_t) { return 256; }
hipError_t launch_sort(const int32_t*, int64_t, int, int32_t*, int32_t*, void*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_div(const int32_t*, int64_t, int32_t, int32_t*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_bounds(const int32_t*, int64_t, int32_t, int32_t*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_gather(const int32_t*, int64_t, int64_t, const int32_t*, const double*, int32_t*,
                         void*, int32_t, double*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_band_entries(const int32_t*, int64_t, int64_t, const int32_t*, const int32_t*,
                               const double*, int32_t, int32_t*, void*, int32_t, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_first(const int32_t*, const int32_t*, int64_t, int32_t*, int32_t*, hipStream_t) {
    return hipErrorNotSupported;
}
hipError_t launch_to_storage(const double*, int64_t, void*, int32_t, hipStream_t) {
    return hipErrorNotSupported;
}
}  // namespace azi
