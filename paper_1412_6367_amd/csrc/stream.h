// Launch wrappers of the stream kernels (host side): one-dimensional
// integration and its adjoint over the stream encoding (StreamMatrix).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace azi {

// Per-pixel correction of a stream launch, read in image order beside the
// raw count: none, the unit image (U of the plan), the (dark, 1 / norm)
// pairs or records of the fused stage, or dark alone (kCorrRunDark* kinds,
// one value per pixel here) where the coefficients carry 1 / norm.
constexpr int32_t kStreamPlain = -1, kStreamOnes = -2;

struct StreamLaunch {
    const StreamTile* tiles = nullptr;
    int32_t ntiles = 0;
    const uint16_t* words = nullptr;
    const int32_t* gbase = nullptr;
    const uint16_t* xpix = nullptr;    // two-dimensional matrices: pixels of the scattered items
    const void* coef = nullptr;        // storage type, 64 spare elements at the end
    const StreamChunk* chunks = nullptr;
    int32_t nchunks = 0;
    const StreamEnt* ents = nullptr;
    int64_t ents_per_chunk = 0;        // on average, and
    int32_t ents_most = 0;             // at most: these select the reduction's shape
    int32_t slots = 4;                 // coefficients a pixel keeps in registers: 2, 3 or 4
    bool over = true;                  // some pixel has more
    bool cached = false;               // words and coefficients through the caches (stream_cached)
    const void* img = nullptr;         // raw or corrected image (flat, img_dtype)
    int32_t img_dtype = AZI_F64;
    int64_t npix = 0;                  // pixels of img, four at least
    const void* corr = nullptr;
    int32_t corr_kind = kStreamPlain;
    void* parts = nullptr;             // 8 bytes per partial sum
    void* I = nullptr;
    void* W = nullptr;                 // may be null
    void* U = nullptr;                 // may be null
    double empty = 0.0;
    int32_t dtype = AZI_F64;
    int32_t accum = AZI_ACC_F64;
    const double* ufix = nullptr;      // U of every bin
    const double* wsub = nullptr;      // subtracted from W when set
    double* wfix_out = nullptr;        // only W (or U, of the unit image) is written, here
};

hipError_t launch_stream(const StreamLaunch& a, hipStream_t s);
// launch_stream for one storage type and accumulator.
hipError_t launch_stream_f64(const StreamLaunch& a, hipStream_t s);
hipError_t launch_stream_f32(const StreamLaunch& a, hipStream_t s);
hipError_t launch_stream_k32(const StreamLaunch& a, hipStream_t s);

// coef[gbase ...] = src[colptr[p] + j], in stream order; with `norm`
// (storage type, one value per pixel) times 1 / norm, rounded once more, or
// with `divide` over norm, rounded once.
// src holds doubles (src_f64) or the storage type.
struct StreamCoefLaunch {
    const StreamTile* tiles = nullptr;
    int32_t ntiles = 0;
    const uint16_t* words = nullptr;
    const int32_t* gbase = nullptr;
    const int32_t* colptr = nullptr;
    const uint16_t* xpix = nullptr;    // two-dimensional matrices: pixels of the scattered items
    const int32_t* xsrc = nullptr;     // and positions in src
    const void* src = nullptr;
    bool src_f64 = false;
    const void* norm = nullptr;
    bool divide = false;
    void* coef = nullptr;
    int32_t dtype = AZI_F64;
};
hipError_t launch_stream_coef(const StreamCoefLaunch& a, hipStream_t s);

// Adjoint: gx_p = sum_b A_bp (gI_b / U_b + gW_b).
struct StreamAdjointLaunch {
    const StreamTile* tiles = nullptr;
    int32_t ntiles = 0;
    const StreamTile* blanks = nullptr;  // pixels without entries: gx = 0
    int32_t nblanks = 0;
    const uint16_t* words = nullptr;
    const int32_t* gbase = nullptr;
    const void* coef = nullptr;
    int32_t slots = 4;                 // as in StreamLaunch
    bool over = true, cached = false;
    const void* U = nullptr;           // storage type
    const void* gI = nullptr;          // may be null
    const void* gW = nullptr;          // may be null
    const void* norm = nullptr;        // divide the result by it when non-null
    void* gx = nullptr;
    int32_t dtype = AZI_F64;
};
hipError_t launch_stream_adjoint(const StreamAdjointLaunch& a, hipStream_t s);

// *flags (device int32) = 1 if some dark[i] is not an integer in [0, 65535],
// plus 2 if some is not exactly a float.
hipError_t launch_dark_kind(const void* dark, int32_t dtype, int64_t n, int32_t* flags,
                            hipStream_t s);
// out[i] = dark[i] as uint16 (kCorrRunDarkU16), float (kCorrRunDarkF32) or
// the storage type (kCorrRunDark).
hipError_t launch_dark_store(const void* dark, int32_t dtype, int32_t kind, void* out, int64_t n,
                             hipStream_t s);

}  // namespace azi
