// Stream encoding on the device: dispatch of the forward kernels, the
// coefficients put in stream order, and the per-pixel dark values of the
// folded stage.
#include <hip/hip_runtime.h>

#include "accum.h"
#include "correct.h"
#include "stream.h"
#include "stream_lane.h"

namespace azi {

hipError_t launch_stream(const StreamLaunch& a, hipStream_t s) {
    if (a.dtype == AZI_F64) return launch_stream_f64(a, s);
    if (a.accum == AZI_ACC_KAHAN32) return launch_stream_k32(a, s);
    return launch_stream_f32(a, s);
}

namespace {

// Every lane writes its pixel's coefficients to their stream positions.
template <class T, class S, bool kNorm>
__global__ __launch_bounds__(256) void k_stream_coef(const StreamTile* __restrict__ tiles,
                                                     const uint16_t* __restrict__ words,
                                                     const int32_t* __restrict__ gbase,
                                                     const int32_t* __restrict__ colptr,
                                                     const S* __restrict__ src,
                                                     const T* __restrict__ norm,
                                                     T* __restrict__ coef) {
    const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const StreamTile t = tiles[blockIdx.x];
    const int ng = StreamLane::blocks(t);
    for (int g = wave; g < ng; g += 4) {
        const StreamLane at(t, g, lane);
        int32_t base = gbase[t.g0 + g];
        for (int k = 0; k < kLanePix; ++k) {
            const int n = (int)(words[t.word0 + g * kBlockPix + kLanePix * lane + k] >>
                                kStreamCountShift);
            const int64_t p = t.pix0 + (at.inside(t) > k ? at.pixel(t) + k : 0);
            const int32_t k0 = colptr[p];
            double scale = 1.0;
            if constexpr (kNorm) scale = 1.0 / (double)norm[p];
            for (int j = 0; __ballot(n > j) != 0; ++j) {
                const uint64_t m = __ballot(n > j);
                const int rank = (int)__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (n > j) {
                    if constexpr (kNorm) coef[base + rank] = (T)((double)src[k0 + j] * scale);
                    else coef[base + rank] = (T)src[k0 + j];
                }
                base += (int32_t)__popcll(m);
            }
        }
    }
}

template <class T, class S>
hipError_t coef_launch(const StreamCoefLaunch& a, hipStream_t s) {
    const S* src = static_cast<const S*>(a.src);
    const T* norm = static_cast<const T*>(a.norm);
    T* coef = static_cast<T*>(a.coef);
    if (norm)
        hipLaunchKernelGGL((k_stream_coef<T, S, true>), dim3((unsigned)a.ntiles), dim3(256), 0, s,
                           a.tiles, a.words, a.gbase, a.colptr, src, norm, coef);
    else
        hipLaunchKernelGGL((k_stream_coef<T, S, false>), dim3((unsigned)a.ntiles), dim3(256), 0, s,
                           a.tiles, a.words, a.gbase, a.colptr, src, norm, coef);
    return hipGetLastError();
}

template <class T>
__global__ void k_dark_kind(const T* __restrict__ dark, int64_t n, int32_t* __restrict__ flags) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double d = (double)dark[i];
    // the flags only ever gain bits
    if (!(d >= 0.0 && d <= 65535.0 && d == floor(d))) atomicOr(flags, 1);
    if (!((double)(float)d == d)) atomicOr(flags, 2);
}

template <class T, class V>
__global__ void k_dark_store(const T* __restrict__ dark, int64_t n, V* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (V)dark[i];
}

__global__ void k_clear(int32_t* p) { *p = 0; }

template <class T>
hipError_t dark_store(const void* dark, int32_t kind, void* out, int64_t n, unsigned blocks,
                      hipStream_t s) {
    const T* d = static_cast<const T*>(dark);
    if (kind == kCorrRunDarkU16)
        hipLaunchKernelGGL((k_dark_store<T, uint16_t>), dim3(blocks), dim3(256), 0, s, d, n,
                           static_cast<uint16_t*>(out));
    else if (kind == kCorrRunDarkF32)
        hipLaunchKernelGGL((k_dark_store<T, float>), dim3(blocks), dim3(256), 0, s, d, n,
                           static_cast<float*>(out));
    else
        hipLaunchKernelGGL((k_dark_store<T, T>), dim3(blocks), dim3(256), 0, s, d, n,
                           static_cast<T*>(out));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stream_coef(const StreamCoefLaunch& a, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    if (a.dtype == AZI_F64) return coef_launch<double, double>(a, s);
    return a.src_f64 ? coef_launch<float, double>(a, s) : coef_launch<float, float>(a, s);
}

hipError_t launch_dark_kind(const void* dark, int32_t dtype, int64_t n, int32_t* flags,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, s, flags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n <= 0) return e;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (dtype == AZI_F64)
        hipLaunchKernelGGL((k_dark_kind<double>), dim3(blocks), dim3(256), 0, s,
                           static_cast<const double*>(dark), n, flags);
    else
        hipLaunchKernelGGL((k_dark_kind<float>), dim3(blocks), dim3(256), 0, s,
                           static_cast<const float*>(dark), n, flags);
    return hipGetLastError();
}

hipError_t launch_dark_store(const void* dark, int32_t dtype, int32_t kind, void* out, int64_t n,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    return dtype == AZI_F64 ? dark_store<double>(dark, kind, out, n, blocks, s)
                            : dark_store<float>(dark, kind, out, n, blocks, s);
}

}  // namespace azi
