// Stream encoding on the device: dispatch of the forward kernels, the
// coefficients put in stream order, the adjoint, and the per-pixel dark
// values of the folded stage.
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

// Every lane writes its pixels' coefficients to their stream positions.
template <class T, class S, bool kNorm>
__global__ __launch_bounds__(256) void k_stream_coef(
    const StreamTile* __restrict__ tiles, const uint16_t* __restrict__ words,
    const int32_t* __restrict__ gbase, const int32_t* __restrict__ colptr,
    const uint16_t* __restrict__ xpix, const int32_t* __restrict__ xsrc,
    const S* __restrict__ src, const T* __restrict__ norm, bool divide, T* __restrict__ coef) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    const StreamTile t = tiles[blockIdx.x];
    auto scale_of = [&](int64_t p) {
        if constexpr (kNorm) return divide ? (double)norm[p] : 1.0 / (double)norm[p];
        else return 1.0;
    };
    auto put = [&](int32_t& base, int n, int32_t k0, double scale) {
        for (int j = 0;; ++j) {
            const uint64_t m = __ballot(n > j);
            if (m == 0) break;
            const int rank = (int)__builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (n > j) {
                const S c = src[k0 + j];
                if constexpr (kNorm)
                    coef[base + rank] = (T)(divide ? (double)c / scale : (double)c * scale);
                else
                    coef[base + rank] = (T)c;
            }
            base += (int32_t)__popcll(m);
        }
    };
    const int ng = StreamLane::blocks(t);
    for (int g = wave; g < ng; g += 4) {
        const StreamLane at(t, g, lane);
        const int64_t e = (int64_t)t.word0 + g * kBlockPix + kLanePix * lane;
        int32_t base = gbase[t.g0 + g];
        int n[kLanePix];
        int32_t k0[kLanePix];
        double scale[kLanePix];
#pragma unroll
        for (int k = 0; k < kLanePix; ++k) {
            n[k] = (int)(words[e + k] >> kStreamCountShift);
            const int64_t p = t.pix0 + (at.inside(t) > k ? at.pixel(t) + k : 0);
            k0[k] = colptr[p];
            scale[k] = scale_of(p);
        }
#pragma unroll
        for (int k = 0; k < kLanePix; ++k) put(base, n[k], k0[k], scale[k]);
    }
    for (int u = wave; u < t.nx; u += 4) {
        const int n = (int)(words[(int64_t)t.word0 + ng * kBlockPix + u * kWave + lane] >>
                            kStreamCountShift);
        const int64_t x = (int64_t)(t.x0 + u) * kWave + lane;
        const int i = xpix[x];
        int32_t base = gbase[t.g0 + ng + u];
        put(base, n, xsrc[x],
            scale_of(t.pix0 + (i >> kStreamColBits) * t.w + (i & ((1 << kStreamColBits) - 1))));
    }
}

template <class T, class S>
hipError_t coef_launch(const StreamCoefLaunch& a, hipStream_t s) {
    const S* src = static_cast<const S*>(a.src);
    const T* norm = static_cast<const T*>(a.norm);
    T* coef = static_cast<T*>(a.coef);
    if (norm)
        hipLaunchKernelGGL((k_stream_coef<T, S, true>), dim3((unsigned)a.ntiles), dim3(256), 0, s,
                           a.tiles, a.words, a.gbase, a.colptr, a.xpix, a.xsrc, src, norm,
                           a.divide, coef);
    else
        hipLaunchKernelGGL((k_stream_coef<T, S, false>), dim3((unsigned)a.ntiles), dim3(256), 0, s,
                           a.tiles, a.words, a.gbase, a.colptr, a.xpix, a.xsrc, src, norm,
                           a.divide, coef);
    return hipGetLastError();
}

// One workgroup per tile of the forward; the tile's bins' v = gI / U + gW are
// formed once into LDS (one pass less than a vector formed beforehand, and
// the pixels' bins then come from LDS instead of the caches), the words and
// coefficients read as in the forward, every lane writing its four pixels'
// gradients together.  Workgroups past the tiles write the empty sums of the
// tiles whose pixels feed no bin (over the norm, as every pixel's: a masked
// pixel's norm of 0 gives NaN wherever it lies).  The products are added in ascending bins, as by k_csc_bwd: the
// same bits.  Bound by HBM: coefficients, words and gradient; k_csc_bwd read 8
// bytes of column pointer and first bin a pixel in the words' place.  Forward
// and gradient of 64 float32 images of 1e3 to 1e6 pixels: 98.3 us with
// k_csc_bwd behind the stream forward, 82.9 with this (78.5 by now).
template <class T, int NMAX, bool kOver, bool kNt>
__global__ __launch_bounds__(256) void k_stream_adjoint(
    const StreamTile* __restrict__ tiles, int32_t ntiles, const StreamTile* __restrict__ blanks,
    const uint16_t* __restrict__ words, const int32_t* __restrict__ gbase,
    const T* __restrict__ coef, const T* __restrict__ U, const T* __restrict__ gI,
    const T* __restrict__ gW, const T* __restrict__ norm, T* __restrict__ gx) {
    __shared__ double v[kStreamSlots + kStreamUnrolled];  // lanes read past their last bin
    if ((int32_t)blockIdx.x >= ntiles) {
        const StreamTile t = blanks[blockIdx.x - ntiles];
        for (int e = threadIdx.x; e < t.tw * t.th; e += 256) {
            const int r = e / t.tw;
            const int64_t p = t.pix0 + r * t.w + e - r * t.tw;
            gx[p] = norm ? (T)(0.0 / (double)norm[p]) : T(0);
        }
        return;
    }
    const StreamTile t = tiles[stream_tile_of(blockIdx.x, ntiles)];
    for (int i = threadIdx.x; i < t.nwin; i += 256) {
        const int b = t.wlo + i;
        double val = 0.0;
        if (gI) {
            const double u = (double)U[b];
            val = (u != 0.0) ? (double)gI[b] / u : 0.0;
        }
        if (gW) val = val + (double)gW[b];
        v[i] = val;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    const int ng = StreamLane::blocks(t);
    const int g0 = (ng * wave) >> 2, g1 = (ng * (wave + 1)) >> 2;
    const bool over = kOver && StreamLane::over(t, NMAX);
    StreamLane at(t, g0, lane);
    const int32_t bases = gbase[t.g0 + min(g0 + lane, ng - 1)];
    auto fetch = [&](int g) {
        const int e = t.word0 + min(g, ng - 1) * kBlockPix + kLanePix * lane;
        return ld<kNt>(reinterpret_cast<const uint64_t*>(words + e));
    };
    uint64_t word = fetch(g0);
    __syncthreads();
    for (int g = g0; g < g1; ++g) {
        T c[kLanePix][NMAX];
        int32_t more[kLanePix];
        int32_t base = __builtin_amdgcn_readlane(bases, g - g0);
        const uint64_t w4 = word;
        auto bits = [&](int k) { return (uint32_t)(w4 >> (16 * k)) & 0xffffu; };
#pragma unroll
        for (int k = 0; k < kLanePix; ++k) {
            const int n = (int)(bits(k) >> kStreamCountShift);
            more[k] = base = stream_coefs<kNt, NMAX>(base, n, coef, c[k]);
            if (over) base = stream_skip(base, n, NMAX);
        }
        word = fetch(g + 1);
        const int64_t p = t.pix0 + at.pixel(t);
        const int in = at.inside(t);
        at.next();
        Four<T> out;
#pragma unroll
        for (int k = 0; k < kLanePix; ++k) {
            const int n = (int)(bits(k) >> kStreamCountShift);
            const double* vb = v + (bits(k) & ((1u << kStreamCountShift) - 1));
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < NMAX; ++j) {
                const double s = __fma_rn((double)c[k][j], vb[j], acc);
                acc = n > j ? s : acc;
            }
            if (over) {
                for (int j = NMAX; __ballot(n > j) != 0; ++j) {
                    T cj[1];
                    more[k] = stream_coefs<kNt, 1>(more[k], n > j ? 1 : 0, coef, cj);
                    if (n > j) acc = __fma_rn((double)cj[0], vb[j], acc);
                }
            }
            if (norm && k < in) acc = acc / (double)norm[p + k];
            out.v[k] = (T)acc;
        }
        // the next words are waited for here: a wait after the stores would
        // be for the stores too
        asm volatile("" : "+v"(word));
        if (in >= kLanePix) {
            store_four(gx + p, out);
        } else {
#pragma unroll
            for (int k = 0; k < kLanePix; ++k)
                if (k < in) gx[p + k] = out.v[k];
        }
    }
}

template <class T, int NMAX, bool kOver, bool kNt>
hipError_t adjoint_launch(const StreamAdjointLaunch& a, hipStream_t s) {
    hipLaunchKernelGGL((k_stream_adjoint<T, NMAX, kOver, kNt>), dim3((unsigned)(a.ntiles + a.nblanks)),
                       dim3(256), 0, s, a.tiles, a.ntiles, a.blanks, a.words, a.gbase,
                       static_cast<const T*>(a.coef), static_cast<const T*>(a.U),
                       static_cast<const T*>(a.gI), static_cast<const T*>(a.gW),
                       static_cast<const T*>(a.norm), static_cast<T*>(a.gx));
    return hipGetLastError();
}

template <class T, bool kNt>
hipError_t adjoint_slots(const StreamAdjointLaunch& a, hipStream_t s) {
    if (a.slots == 2)
        return a.over ? adjoint_launch<T, 2, true, kNt>(a, s)
                      : adjoint_launch<T, 2, false, kNt>(a, s);
    if (a.slots == 3)
        return a.over ? adjoint_launch<T, 3, true, kNt>(a, s)
                      : adjoint_launch<T, 3, false, kNt>(a, s);
    return adjoint_launch<T, kStreamUnrolled, true, kNt>(a, s);
}

template <class T>
hipError_t adjoint_cached(const StreamAdjointLaunch& a, hipStream_t s) {
    return a.cached ? adjoint_slots<T, false>(a, s) : adjoint_slots<T, true>(a, s);
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

hipError_t launch_stream_adjoint(const StreamAdjointLaunch& a, hipStream_t s) {
    if (a.ntiles + a.nblanks <= 0) return hipSuccess;
    return a.dtype == AZI_F64 ? adjoint_cached<double>(a, s) : adjoint_cached<float>(a, s);
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
