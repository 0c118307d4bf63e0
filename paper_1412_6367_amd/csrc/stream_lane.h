// Device helpers of the stream encoding (StreamMatrix) shared by its kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "correct.h"
#include "internal.h"

namespace azi {
namespace {

// Most coefficients of a pixel that a kernel holds in registers; the tiles of
// pixels of more bins than a kernel's take a loop.
constexpr int kStreamUnrolled = 4;
constexpr int kLanePix = 4;                  // neighbouring pixels of a lane
constexpr int kBlockPix = 64 * kLanePix;

// Four consecutive elements as one load (two or more where they exceed 16
// bytes), from an address aligned to the element alone.
template <class V> struct Four { V v[kLanePix]; };
template <class V> struct Vec4;
template <> struct Vec4<int16_t> { typedef int16_t type __attribute__((ext_vector_type(4), aligned(2))); };
template <> struct Vec4<uint16_t> { typedef uint16_t type __attribute__((ext_vector_type(4), aligned(2))); };
template <> struct Vec4<int32_t> { typedef int32_t type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec4<uint32_t> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec4<float> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
template <class V>
__device__ __forceinline__ Four<V> load_four(const V* p) {
    const typename Vec4<V>::type a = *reinterpret_cast<const typename Vec4<V>::type*>(p);
    return Four<V>{{a.x, a.y, a.z, a.w}};
}
typedef double StreamD2 __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ Four<double> load_four(const double* p) {
    const StreamD2 a = *reinterpret_cast<const StreamD2*>(p);
    const StreamD2 b = *reinterpret_cast<const StreamD2*>(p + 2);
    return Four<double>{{a.x, a.y, b.x, b.y}};
}
__device__ __forceinline__ void store_four(float* p, const Four<float>& a) {
    typename Vec4<float>::type v = {a.v[0], a.v[1], a.v[2], a.v[3]};
    *reinterpret_cast<typename Vec4<float>::type*>(p) = v;
}
__device__ __forceinline__ void store_four(double* p, const Four<double>& a) {
    StreamD2 lo = {a.v[0], a.v[1]}, hi = {a.v[2], a.v[3]};
    reinterpret_cast<StreamD2*>(p)[0] = lo;
    reinterpret_cast<StreamD2*>(p)[1] = hi;
}
template <class V>
__device__ __forceinline__ Four<RunDark<V>> load_four(const RunDark<V>* p) {
    const Four<V> a = load_four(reinterpret_cast<const V*>(p));
    return Four<RunDark<V>>{{{a.v[0]}, {a.v[1]}, {a.v[2]}, {a.v[3]}}};
}
__device__ __forceinline__ Four<float2> load_four(const float2* p) {
    return Four<float2>{{p[0], p[1], p[2], p[3]}};
}
__device__ __forceinline__ Four<double2> load_four(const double2* p) {
    return Four<double2>{{p[0], p[1], p[2], p[3]}};
}
__device__ __forceinline__ Four<Corr12> load_four(const Corr12* p) {
    return Four<Corr12>{{p[0], p[1], p[2], p[3]}};
}

// A lane's place in a tile, block after block.  The block's own place is the
// same for the whole wavefront.
struct StreamLane {
    int lgw, lrs;            // log2 of the lanes across and of the row stride
    int across;              // blocks across the tile
    int pr, pc;              // the block's row and column of blocks
    int r0, c0;              // the lane's first pixel within the block
    int at;                  // r0 * w + c0
    __device__ StreamLane(const StreamTile& t, int block, int lane) {
        lgw = (t.shape >> 4) & 15;
        lrs = (t.shape >> 8) & 15;
        const bool rows_minor = t.shape & kStreamRowsMinor;
        r0 = (rows_minor ? lane & ((64 >> lgw) - 1) : lane >> lgw) << lrs;
        c0 = kLanePix * (rows_minor ? lane >> (6 - lgw) : lane & ((1 << lgw) - 1));
        at = r0 * t.w + c0;
        across = blocks_across(t, lgw);
        pr = block / across;
        pc = block - pr * across;
    }
    __device__ static int blocks_across(const StreamTile& t, int lgw) {
        return (t.tw + (kLanePix << lgw) - 1) >> (2 + lgw);
    }
    __device__ static int blocks(const StreamTile& t) {
        const int lgw = (t.shape >> 4) & 15, lrs = (t.shape >> 8) & 15;
        const int lrows = 6 - lgw + lrs;
        return blocks_across(t, lgw) * ((t.th + (1 << lrows) - 1) >> lrows << lrs);
    }
    // Copies of the window, and whether a pixel of the tile has more than n bins.
    __device__ static int copies(const StreamTile& t) { return 1 << (t.shape & 15); }
    __device__ static bool over(const StreamTile& t, int n) {
        return (t.shape >> kStreamMostShift) > n;
    }
    // The block's first row and column in the tile.
    __device__ int row() const {
        return (pr >> lrs << (6 - lgw + lrs)) + (pr & ((1 << lrs) - 1));
    }
    __device__ int column() const { return pc << (2 + lgw); }
    // The lane's first pixel, counted from the tile's first.
    __device__ int pixel(const StreamTile& t) const { return row() * t.w + column() + at; }
    // Pixels of the lane that the tile has (0 or less: none).
    __device__ int inside(const StreamTile& t) const {
        return row() + r0 < t.th ? t.tw - column() - c0 : 0;
    }
    __device__ void next() {
        ++pc;
        const bool wrap = pc == across;
        pc = wrap ? 0 : pc;
        pr += wrap ? 1 : 0;
    }
};

// The tile of workgroup g of n.  Workgroup g runs on XCD g % 8; of every 64
// tiles each XCD takes 8 neighbours, which share the image lines at their
// edges in its L2.  Tiles differ in work with their place in the image, so an
// XCD's share is spread over it (one contiguous eighth of the tiles each:
// 1000 x 360 bins of a 3162 x 3163 frame 86 us a pass, a tile at a time 77 us
// with half as many bytes again read).
__device__ inline int64_t stream_tile_of(uint32_t g, uint32_t n) {
    return g < (n & ~63u) ? (g & ~63u) + (g & 7) * 8 + ((g >> 3) & 7) : g;
}

// The first N coefficients of one pixel of every lane (n bins each), those of
// the wavefront starting at base; returns where the next pixels' start when
// none has more than N bins.  Lanes without a j-th coefficient read their
// neighbour's, unused: no branch, no address outside the array and its spare
// elements.
// kNt: streamed past the caches (stream_cached has the rule).
template <bool kNt, int N, class T>
__device__ __forceinline__ int32_t stream_coefs(int32_t base, int n, const T* __restrict__ coef,
                                                T (&c)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const uint64_t m = __ballot(n > j);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        c[j] = ld<kNt>(coef + base + rank);
        base += (int32_t)__popcll(m);
    }
    return base;
}

// base past the j-th and further coefficients of the lanes' pixels.
__device__ __forceinline__ int32_t stream_skip(int32_t base, int n, int j) {
    for (;; ++j) {
        const uint64_t m = __ballot(n > j);
        if (m == 0) return base;
        base += (int32_t)__popcll(m);
    }
}

// Keeps the compiler from moving LDS accesses across: other lanes' elements
// are written in between.  (The hardware completes a wavefront's LDS
// accesses in order, so no wait is needed.)
__device__ __forceinline__ void lds_in_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace
}  // namespace azi
