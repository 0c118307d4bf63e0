// The forward stream kernel and its reduction, instantiated per storage type
// and accumulator by stream_f64.hip, stream_f32.hip and stream_k32.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "accum.h"
#include "correct.h"
#include "stream.h"
#include "stream_lane.h"

namespace azi {

namespace {

struct NoCorr {};    // the image as it is, cast to the storage type
struct UnitImage {}; // every pixel 1

// One workgroup of four wavefronts per tile; wavefront w takes the w-th
// quarter of the tile's blocks of 64 lanes by four pixels.  Words, image and
// (packed, slot-major) coefficients are read once and coalesced: a lane's
// four words and four pixels with one load each, a block ahead; the block's
// coefficients, whose places the words give, together.  Every wavefront adds
// into its own copies of the tile's bin window in LDS by plain read - add -
// write: the encoding gives lanes that share a copy distinct first bins, so
// the j-th bins of the lanes' k-th pixels are distinct LDS elements, and a
// wavefront's LDS accesses complete in the order they are issued.  The
// workgroup then sums its copies in a fixed order and writes the window.
// kX: two-dimensional matrices, whose tiles end in scattered groups.
//
// Bound by HBM: 22.6 + 2 + 4 bytes a pixel of the 3162 x 3163 float64 frame
// (coefficients, words, int32 counts).  The bin-major run encoding reads 4
// bytes per run of a pixel in a band (1.45 runs a pixel) and gathers the
// frame again for every band.  That frame's pass, with the reduction: 75.0 ->
// 52.7 us (284 MB: 5.4 TB/s; a 1 GiB copy reaches 5.1); float32 and 1000
// bins 45.5 -> 29.9; 4e6 uint16 pixels, float32, 26.7 -> 16.4; the frame's map
// of 1000 x 360 bins 131 -> 65.6 (253 MB read).  The reduction stays a kernel of
// its own: finishing the bins in the last workgroup to arrive needs a release
// at device scope per workgroup, an L2 write-back each, and takes 12.4 -> 136
// us for 981 x 1043 pixels.
template <class T, class Acc, class RawT, class CorrT, int NMAX, bool kOver, bool kX, bool kNt>
__global__ __launch_bounds__(256) void k_stream(const StreamTile* __restrict__ tiles,
                                                const uint16_t* __restrict__ words,
                                                const int32_t* __restrict__ gbase,
                                                const T* __restrict__ coef,
                                                const RawT* __restrict__ img, int64_t npix,
                                                const CorrT* __restrict__ corr,
                                                const uint16_t* __restrict__ xpix,
                                                Acc* __restrict__ parts) {
    constexpr bool kUnit = std::is_same<CorrT, UnitImage>::value;
    constexpr bool kCorr = !kUnit && !std::is_same<CorrT, NoCorr>::value;
    __shared__ Acc acc[4][kStreamSlots];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    const StreamTile t = tiles[stream_tile_of(blockIdx.x, gridDim.x)];
    const int ng = StreamLane::blocks(t);
    const int g0 = (ng * wave) >> 2, g1 = (ng * (wave + 1)) >> 2;
    const int copies = StreamLane::copies(t);
    const bool over = kOver && StreamLane::over(t, NMAX);
    StreamLane at(t, g0, lane);
    const int32_t bases = gbase[t.g0 + min(g0 + lane, ng - 1)];
    // where the last four pixels of the image start: no lane reads past them
    const int64_t end = npix - kLanePix - t.pix0;
    uint64_t word = 0;
    Four<RawT> raw;
    Four<CorrT> cor;
    int shift = 0;
    auto fetch = [&](int g) {
        // past the wavefront's last block: the last one's words again, unused
        const int e = t.word0 + min(g, g1 - 1) * kBlockPix + kLanePix * lane;
        word = ld<kNt>(reinterpret_cast<const uint64_t*>(words + e));
        if constexpr (!kUnit) {
            const int64_t p = at.pixel(t);
            const int64_t q = p < end ? p : end;
            shift = (int)min(p - q, (int64_t)kLanePix);
            raw = load_four(img + t.pix0 + q);
            if constexpr (kCorr) cor = load_four(corr + t.pix0 + q);
        }
        at.next();
    };
    Acc* const own = acc[wave];
    Acc* const mine = own + (lane & (copies - 1)) * t.pitch;
    // the first scattered group of the wavefront: its words and pixel places
    // before, its pixels after the first block's requests
    uint16_t xword = 0, xat = 0;
    if constexpr (kX) {
        if (wave < t.nx) {
            xword = words[(int64_t)t.word0 + ng * kBlockPix + wave * kWave + lane];
            xat = xpix[(int64_t)(t.x0 + wave) * kWave + lane];
        }
    }
    auto xpixel = [&](uint16_t i) {
        return t.pix0 + (i >> kStreamColBits) * t.w + (i & ((1 << kStreamColBits) - 1));
    };
    RawT xraw{};
    CorrT xcor{};
    if (g0 < g1) fetch(g0);
    if constexpr (kX && !kUnit) {
        xraw = img[xpixel(xat)];
        if constexpr (kCorr) xcor = corr[xpixel(xat)];
    }
    for (int i = lane; i < t.pitch * copies; i += kWave) own[i].zero();
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
        T x[kLanePix];
#pragma unroll
        for (int k = 0; k < kLanePix; ++k) {
            if constexpr (kUnit) x[k] = T(1);
            else if constexpr (kCorr) x[k] = corr_apply((T)raw.v[k], cor.v[k]);
            else x[k] = (T)raw.v[k];
        }
        if constexpr (!kUnit) {
            // the image's last pixels, read from further back
            if (__ballot(shift > 0) != 0) {
#pragma unroll
                for (int k = 0; k < kLanePix; ++k) {
                    T v = x[k];
#pragma unroll
                    for (int s = 1; s < kLanePix; ++s)
                        if (k + s < kLanePix && shift == s) v = x[k + s];
                    x[k] = v;
                }
            }
        }
        fetch(g + 1);
#pragma unroll
        for (int k = 0; k < kLanePix; ++k) {
            const int n = (int)(bits(k) >> kStreamCountShift);
            Acc* p = mine + (bits(k) & ((1u << kStreamCountShift) - 1));
#pragma unroll
            for (int j = 0; j < NMAX; ++j) {
                if (n > j) {
                    Acc v = p[j];
                    v.add(c[k][j], x[k]);
                    p[j] = v;
                }
                lds_in_order();
            }
            if (over) {
                // pixels of more bins than are held
                for (int j = NMAX; __ballot(n > j) != 0; ++j) {
                    T cj[1];
                    more[k] = stream_coefs<kNt, 1>(more[k], n > j ? 1 : 0, coef, cj);
                    if (n > j) {
                        Acc v = p[j];
                        v.add(cj[0], x[k]);
                        p[j] = v;
                    }
                    lds_in_order();
                }
            }
        }
    }
    if constexpr (kX) {
        for (int u = wave; u < t.nx; u += 4) {
            if (u != wave) {
                xword = words[(int64_t)t.word0 + ng * kBlockPix + u * kWave + lane];
                if constexpr (!kUnit) {
                    xat = xpix[(int64_t)(t.x0 + u) * kWave + lane];
                    xraw = img[xpixel(xat)];
                    if constexpr (kCorr) xcor = corr[xpixel(xat)];
                }
            }
            const int n = xword >> kStreamCountShift;
            T c[NMAX];
            int32_t more = stream_coefs<kNt, NMAX>(gbase[t.g0 + ng + u], n, coef, c);
            T x;
            if constexpr (kUnit) x = T(1);
            else if constexpr (kCorr) x = corr_apply((T)xraw, xcor);
            else x = (T)xraw;
            Acc* p = mine + (xword & ((1 << kStreamCountShift) - 1));
#pragma unroll
            for (int j = 0; j < NMAX; ++j) {
                if (n > j) {
                    Acc v = p[j];
                    v.add(c[j], x);
                    p[j] = v;
                }
                lds_in_order();
            }
            if (over) {
                for (int j = NMAX; __ballot(n > j) != 0; ++j) {
                    T cj[1];
                    more = stream_coefs<kNt, 1>(more, n > j ? 1 : 0, coef, cj);
                    if (n > j) {
                        Acc v = p[j];
                        v.add(cj[0], x);
                        p[j] = v;
                    }
                    lds_in_order();
                }
            }
        }
    }
    // each wavefront's copies into its first, then the four wavefronts'
    if (copies > 1) {
        for (int b = lane; b < t.nwin; b += kWave) {
            Acc v = own[b];
            for (int k = 1; k < copies; ++k) v.merge(own[k * t.pitch + b]);
            own[b] = v;
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < t.nwin; b += 256) {
        Acc v = acc[0][b];
        for (int w = 1; w < 4; ++w) v.merge(acc[w][b]);
        parts[t.part0 + b] = v;
    }
}

// Finishes B of a chunk's bins per workgroup of B * L threads: L lanes a bin
// walk the chunk's list of tiles, four entries in flight each, and are
// merged in a fixed tree.  Bound by its two dependent loads (entries, sums):
// 4 to 4.3 us for 1000 bins of 1e6 to 4e6 pixels (40 to 90 tiles a chunk).
template <class T, class Acc, int B, int L>
__global__ __launch_bounds__(B* L) void k_stream_reduce(
    const StreamChunk* __restrict__ chunks, const StreamEnt* __restrict__ ents,
    const Acc* __restrict__ parts, T* __restrict__ I, T* __restrict__ W, T* __restrict__ U,
    double empty, const double* __restrict__ ufix, const double* __restrict__ wsub,
    double* __restrict__ wfix_out) {
    constexpr int kWaves = B * L / kWave;
    constexpr int kFlight = 4;
    __shared__ Acc s[kWaves][B];
    const StreamChunk ch = chunks[blockIdx.x / (kStreamChunk / B)];
    const int first = blockIdx.x % (kStreamChunk / B) * B;
    if (first >= ch.nbins) return;
    const int bi = threadIdx.x & (B - 1), li = threadIdx.x / B;
    const int b = ch.bin0 + first + bi;
    const bool last = threadIdx.x < B && first + bi < ch.nbins;
    RowFixed f;
    if (last) f = load_row_fixed(b, ufix, wsub);
    Acc a;
    a.zero();
    for (int k = ch.k0 + li; k < ch.k1; k += kFlight * L) {
        StreamEnt e[kFlight];
#pragma unroll
        for (int i = 0; i < kFlight; ++i) e[i] = ents[min(k + i * L, ch.k1 - 1)];
        Acc v[kFlight];
#pragma unroll
        for (int i = 0; i < kFlight; ++i) {
            const bool in = k + i * L < ch.k1 && b >= e[i].lo && b < e[i].hi;
            v[i] = parts[in ? e[i].base + b : 0];
            if (!in) v[i].zero();
        }
#pragma unroll
        for (int i = 0; i < kFlight; ++i) a.merge(v[i]);
    }
#pragma unroll
    for (int m = kWave / 2; m >= B; m >>= 1) a.merge(a.shfl_xor(m));
    if constexpr (kWaves > 1) {
        if ((threadIdx.x & (kWave - 1)) < B) s[threadIdx.x / kWave][bi] = a;
        __syncthreads();
        if (last)
            for (int w = 1; w < kWaves; ++w) a.merge(s[w][bi]);
    }
    if (last) write_row_u(b, a, I, W, U, empty, f, static_cast<double*>(nullptr), wfix_out);
}

// One lane per bin, for matrices none of whose chunks is reached by more than
// a few tiles (maps): 16 chunks a workgroup, outputs written by whole
// wavefronts.  360000 bins of a 3162 x 3163 frame: 7.1 us, 10.7 us with four
// lanes a bin and one chunk a workgroup; with lists of up to 40 tiles among
// short ones (512 images of 1e2 to 1e5 pixels) it is 3 us the slower one.
constexpr int kEachChunks = 256 / kStreamChunk;
template <class T, class Acc>
__global__ __launch_bounds__(256) void k_stream_reduce_each(
    const StreamChunk* __restrict__ chunks, int32_t nchunks, const StreamEnt* __restrict__ ents,
    const Acc* __restrict__ parts, T* __restrict__ I, T* __restrict__ W, T* __restrict__ U,
    double empty, const double* __restrict__ ufix, const double* __restrict__ wsub,
    double* __restrict__ wfix_out) {
    constexpr int kFlight = 4;
    const int c = blockIdx.x * kEachChunks + threadIdx.x / kStreamChunk;
    const int bi = threadIdx.x & (kStreamChunk - 1);
    if (c >= nchunks) return;
    const StreamChunk ch = chunks[c];
    if (bi >= ch.nbins) return;
    const int b = ch.bin0 + bi;
    const RowFixed f = load_row_fixed(b, ufix, wsub);
    Acc a;
    a.zero();
    for (int k = ch.k0; k < ch.k1; k += kFlight) {
        StreamEnt e[kFlight];
#pragma unroll
        for (int i = 0; i < kFlight; ++i) e[i] = ents[min(k + i, ch.k1 - 1)];
        Acc v[kFlight];
#pragma unroll
        for (int i = 0; i < kFlight; ++i) {
            const bool in = k + i < ch.k1 && b >= e[i].lo && b < e[i].hi;
            v[i] = parts[in ? e[i].base + b : 0];
            if (!in) v[i].zero();
        }
#pragma unroll
        for (int i = 0; i < kFlight; ++i) a.merge(v[i]);
    }
    write_row_u(b, a, I, W, U, empty, f, static_cast<double*>(nullptr), wfix_out);
}

template <class T, class Acc, class RawT, class CorrT, int NMAX, bool kOver, bool kX, bool kNt>
hipError_t stream_launch(const StreamLaunch& a, hipStream_t s) {
    hipLaunchKernelGGL((k_stream<T, Acc, RawT, CorrT, NMAX, kOver, kX, kNt>), dim3((unsigned)a.ntiles),
                       dim3(256), 0, s, a.tiles, a.words, a.gbase, static_cast<const T*>(a.coef),
                       static_cast<const RawT*>(a.img), a.npix, static_cast<const CorrT*>(a.corr),
                       a.xpix, static_cast<Acc*>(a.parts));
    return hipGetLastError();
}

template <class T, class Acc, class RawT, class CorrT, bool kNt>
hipError_t stream_slots_1d(const StreamLaunch& a, hipStream_t s) {
    if (a.slots == 2 && !a.over)
        return stream_launch<T, Acc, RawT, CorrT, 2, false, false, kNt>(a, s);
    if (a.slots == 2) return stream_launch<T, Acc, RawT, CorrT, 2, true, false, kNt>(a, s);
    if (a.slots == 3 && !a.over)
        return stream_launch<T, Acc, RawT, CorrT, 3, false, false, kNt>(a, s);
    if (a.slots == 3) return stream_launch<T, Acc, RawT, CorrT, 3, true, false, kNt>(a, s);
    return stream_launch<T, Acc, RawT, CorrT, kStreamUnrolled, true, false, kNt>(a, s);
}

template <class T, class Acc, class RawT, class CorrT>
hipError_t stream_slots(const StreamLaunch& a, hipStream_t s) {
    if constexpr (!std::is_same<CorrT, typename Pair2<T>::type>::value &&
                  !std::is_same<CorrT, Corr12>::value) {
        // two-dimensional matrices
        if (a.xpix && a.slots == 2)
            return stream_launch<T, Acc, RawT, CorrT, 2, true, true, true>(a, s);
        if (a.xpix) return stream_launch<T, Acc, RawT, CorrT, 3, true, true, true>(a, s);
        if constexpr (!std::is_same<CorrT, UnitImage>::value)
            if (a.cached) return stream_slots_1d<T, Acc, RawT, CorrT, false>(a, s);
    }
    return stream_slots_1d<T, Acc, RawT, CorrT, true>(a, s);
}

template <class T, class Acc, class RawT>
hipError_t stream_corr(const StreamLaunch& a, hipStream_t s) {
    switch (a.corr_kind) {
        case kStreamPlain: return stream_slots<T, Acc, RawT, NoCorr>(a, s);
        case kCorrPair: return stream_slots<T, Acc, RawT, typename Pair2<T>::type>(a, s);
        case kCorrRunDark: return stream_slots<T, Acc, RawT, RunDark<T>>(a, s);
        case kCorrRunDarkU16: return stream_slots<T, Acc, RawT, RunDark<uint16_t>>(a, s);
        default: break;
    }
    if constexpr (std::is_same<T, double>::value) {
        if (a.corr_kind == kCorrRecord12) return stream_slots<T, Acc, RawT, Corr12>(a, s);
        if (a.corr_kind == kCorrRunDarkF32) return stream_slots<T, Acc, RawT, RunDark<float>>(a, s);
    }
    return hipErrorInvalidValue;
}

template <class T, class Acc, int B, int L>
hipError_t stream_reduce(const StreamLaunch& a, hipStream_t s) {
    hipLaunchKernelGGL((k_stream_reduce<T, Acc, B, L>),
                       dim3((unsigned)(a.nchunks * (kStreamChunk / B))), dim3(B * L), 0, s,
                       a.chunks, a.ents, static_cast<const Acc*>(a.parts), static_cast<T*>(a.I),
                       static_cast<T*>(a.W), static_cast<T*>(a.U), a.empty, a.ufix, a.wsub,
                       a.wfix_out);
    return hipGetLastError();
}

template <class T, class Acc>
hipError_t stream_forward(const StreamLaunch& a, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (a.ntiles > 0) {
        if (a.corr_kind == kStreamOnes) {
            e = stream_slots<T, Acc, T, UnitImage>(a, s);
        } else {
            switch (a.img_dtype) {
                case AZI_I16: e = stream_corr<T, Acc, int16_t>(a, s); break;
                case AZI_U16: e = stream_corr<T, Acc, uint16_t>(a, s); break;
                case AZI_I32: e = stream_corr<T, Acc, int32_t>(a, s); break;
                case AZI_U32: e = stream_corr<T, Acc, uint32_t>(a, s); break;
                case AZI_F32: e = stream_corr<T, Acc, float>(a, s); break;
                case AZI_F64: e = stream_corr<T, Acc, double>(a, s); break;
                default: e = hipErrorInvalidValue;
            }
        }
        if (e != hipSuccess) return e;
    }
    if (a.nchunks <= 0) return hipSuccess;
    if (a.ents_per_chunk > 256) return stream_reduce<T, Acc, 4, 256>(a, s);
    if (a.ents_per_chunk > 32) return stream_reduce<T, Acc, 16, 64>(a, s);
    if (a.ents_per_chunk > 8) return stream_reduce<T, Acc, 16, 16>(a, s);
    if (a.ents_most > 16) return stream_reduce<T, Acc, 16, 4>(a, s);
    hipLaunchKernelGGL((k_stream_reduce_each<T, Acc>),
                       dim3((unsigned)((a.nchunks + kEachChunks - 1) / kEachChunks)), dim3(256), 0,
                       s, a.chunks, a.nchunks, a.ents, static_cast<const Acc*>(a.parts),
                       static_cast<T*>(a.I), static_cast<T*>(a.W), static_cast<T*>(a.U), a.empty,
                       a.ufix, a.wsub, a.wfix_out);
    return hipGetLastError();
}

}  // namespace
}  // namespace azi
