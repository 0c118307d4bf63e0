// Host builder of the stream encoding (see StreamMatrix): tiles, words,
// block bases and the lists the reduction walks.  The coefficients are put
// in order on the device from the pixel-major entries.
#include <algorithm>
#include <cstdlib>
#include <limits>

#include "internal.h"

namespace azi {
namespace {

// Smallest k >= lk such that no two set lanes of `mask` agree modulo 2^k.
int32_t copies_for(uint64_t mask, int32_t lk) {
    for (; lk < 6; ++lk) {
        const int32_t K = 1 << lk;
        const uint64_t low = ((uint64_t)1 << K) - 1;
        uint64_t seen = 0;
        bool clash = false;
        for (int32_t s = 0; s < 64 && !clash; s += K) {
            const uint64_t part = (mask >> s) & low;
            clash = (seen & part) != 0;
            seen |= part;
        }
        if (!clash) break;
    }
    return lk;
}

struct Shape {
    int32_t lgw;
    bool rows_minor;
};
// Where the first bin changes along the rows, and where down the columns.
constexpr Shape kAlong[] = {{4, true}, {3, true}, {2, true}};
constexpr Shape kDown[] = {{3, false}, {2, false}, {1, false}};

struct Builder {
    const HostMatrix& m;
    const int32_t w;
    const int64_t pix_off, bin_off;
    StreamMatrix& sm;
    std::vector<uint64_t> lanes;          // per bin: lanes whose pixel starts there
    std::vector<int32_t> touched;
    std::vector<int32_t> first;           // the current tile's pixels, row-major: first bin
    std::vector<int32_t> count;           // and number of bins
    int32_t th = 0, tw = 0;

    int32_t across(Shape s) const { return (tw + (4 << s.lgw) - 1) >> (2 + s.lgw); }
    int32_t down(Shape s) const { return (th + (64 >> s.lgw) - 1) >> (6 - s.lgw); }

    // f(element of the tile, lane) for the k-th pixel of the lanes of block g
    // that feeds a bin, in lane order along or across the rows.
    template <class F>
    void each(Shape s, int32_t g, int32_t k, F&& f) const {
        const int32_t a = across(s), gh = 64 >> s.lgw, gw = 1 << s.lgw;
        const int32_t r0 = g / a * gh, c0 = g % a * gw * 4 + k;
        const int32_t nr = std::min(gh, th - r0);
        for (int32_t r = 0; r < nr; ++r) {
            const int32_t e = (r0 + r) * tw;
            for (int32_t l = 0; l < gw; ++l) {
                const int32_t c = c0 + 4 * l;
                if (c < tw && count[e + c] > 0)
                    f(e + c, s.rows_minor ? (l << (6 - s.lgw)) + r : (r << s.lgw) + l);
            }
        }
    }

    // The copies block g needs, at least lk.
    int32_t block_copies(Shape s, int32_t g, int32_t lk) {
        for (int32_t k = 0; k < 4; ++k) {
            touched.clear();
            each(s, g, k, [&](int32_t e, int32_t lane) {
                const int32_t b = first[e];
                if (!lanes[b]) touched.push_back(b);
                lanes[b] |= (uint64_t)1 << lane;
            });
            for (int32_t b : touched) {
                const uint64_t mask = lanes[b];
                lanes[b] = 0;
                if (mask & (mask - 1)) lk = copies_for(mask, lk);
            }
        }
        return lk;
    }

    void tile(int32_t i0, int32_t j0, int32_t rows, int32_t cols) {
        th = rows;
        tw = cols;
        const int32_t n = th * tw;
        int32_t lo = std::numeric_limits<int32_t>::max(), hi = -1;
        for (int32_t r = 0, e = 0; r < th; ++r) {
            int64_t p = (int64_t)(i0 + r) * w + j0;
            for (int32_t c = 0; c < tw; ++c, ++p, ++e) {
                const int32_t k0 = m.colptr[p], k1 = m.colptr[p + 1];
                count[e] = k1 - k0;
                if (k1 == k0) continue;
                first[e] = m.rowidx[k0];
                lo = std::min(lo, first[e]);
                hi = std::max(hi, first[e] + k1 - k0);
            }
        }
        const int64_t pix0 = pix_off + (int64_t)i0 * w + j0;
        if (hi < 0) {  // feeds no bin
            sm.blanks.push_back(StreamTile{pix0, w, tw, th, 0, 0, 0, 0, 0, 0, 0});
            return;
        }
        const int32_t nwin = hi - lo, pitch = nwin | 1;
        // which way the first bin changes, between the tile's edges
        int64_t along = 0, below = 0;
        for (int32_t r = 0; r < th; ++r)
            if (count[r * tw] && count[r * tw + tw - 1])
                along += std::abs(first[r * tw + tw - 1] - first[r * tw]);
        for (int32_t c = 0; c < tw; ++c)
            if (count[c] && count[n - tw + c]) below += std::abs(first[n - tw + c] - first[c]);
        const Shape* shapes = below * (tw - 1) * th > along * (th - 1) * tw ? kDown : kAlong;
        // the shape of the least work, copies estimated from three blocks:
        // about 240 issue slots a block and 4 for each image row it reads, 4
        // per 64 LDS elements cleared and merged by each of four wavefronts
        int64_t best = std::numeric_limits<int64_t>::max();
        Shape shape{-1, false};
        int32_t lk = 0;
        for (int k = 0; k < 3; ++k) {
            const Shape s = shapes[k];
            const int32_t ng = across(s) * down(s);
            if (ng > kStreamMaxBlocks) continue;
            int32_t l = 0;
            for (int32_t q = 0; q < 3; ++q)
                l = block_copies(s, (int32_t)((int64_t)(ng - 1) * q / 2), l);
            if ((int64_t)pitch << l > kStreamSlots) continue;
            const int64_t cost = (240 + 4 * (64 >> s.lgw)) * (int64_t)ng +
                                 16 * (((int64_t)pitch << l) / 64);
            if (cost < best) {
                best = cost;
                shape = s;
                lk = l;
            }
        }
        if (shape.lgw >= 0)
            for (int32_t g = 0; g < across(shape) * down(shape); ++g)
                lk = block_copies(shape, g, lk);
        if (shape.lgw < 0 || (int64_t)pitch << lk > kStreamSlots) {
            if (n == 1) {  // a single pixel always fits: one copy of its own bins
                shape = kAlong[0];
                lk = 0;
            } else if (rows >= cols) {
                tile(i0, j0, rows / 2, cols);
                tile(i0 + rows / 2, j0, rows - rows / 2, cols);
                return;
            } else {
                tile(i0, j0, rows, cols / 2);
                tile(i0, j0 + cols / 2, rows, cols - cols / 2);
                return;
            }
        }
        const int32_t ng = across(shape) * down(shape);
        sm.tiles.push_back(StreamTile{pix0, w, tw, th,
                                      lk | shape.lgw << 8 |
                                          (shape.rows_minor ? kStreamRowsMinor : 0),
                                      (int32_t)sm.words.size(), (int32_t)sm.gbase.size(),
                                      (int32_t)(bin_off + lo), nwin, pitch, (int32_t)sm.nparts});
        sm.nparts += nwin;
        sm.npix += n;
        const size_t word0 = sm.words.size();
        sm.words.resize(word0 + (size_t)ng * 256, 0);
        uint16_t* out = sm.words.data() + word0;
        for (int32_t g = 0; g < ng; ++g, out += 256) {
            int32_t sum = 0;
            for (int32_t k = 0; k < 4; ++k)
                each(shape, g, k, [&](int32_t e, int32_t lane) {
                    out[4 * lane + k] =
                        (uint16_t)((first[e] - lo) | (count[e] << kStreamCountShift));
                    sum += count[e];
                });
            sm.gbase.push_back((int32_t)sm.ncoef);
            sm.ncoef += sum;
        }
    }
};

}  // namespace

bool build_stream(const HostMatrix& m, int32_t h, int32_t w, int32_t tile_px, int64_t pix_off,
                  int64_t bin_off, StreamMatrix& sm) {
    constexpr int64_t kLimit = std::numeric_limits<int32_t>::max();
    if (m.two_d || m.npix < 4 || sm.ncoef + m.nnz() >= kLimit) return false;
    int32_t most = 0;
    for (int64_t p = 0; p < m.npix; ++p) {
        const int32_t k0 = m.colptr[p], k1 = m.colptr[p + 1];
        most = std::max(most, k1 - k0);
        if (k1 > k0 && m.rowidx[k1 - 1] != m.rowidx[k0] + (k1 - k0 - 1)) return false;
    }
    if (most > kStreamMaxCount) return false;
    sm.max_count = std::max(sm.max_count, most);
    const size_t t0 = sm.tiles.size();
    const int64_t px0 = sm.npix;
    // strips of equal width but for the rounding to 8 columns, and rows of
    // about tile_px pixels, a multiple of 16 (four blocks of 64 x 4 pixels,
    // one for each wavefront) where the image has them
    const int32_t strips = (w + 63) / 64;
    const int32_t strip = std::min(w, ((w + strips - 1) / strips + 7) / 8 * 8);
    int32_t rows = (std::min(tile_px, kStreamMaxPix) + strip / 2) / strip;
    rows = std::max(1, std::min(h, rows >= 16 ? rows / 16 * 16 : rows));
    Builder b{m, w, pix_off, bin_off, sm, std::vector<uint64_t>((size_t)m.npt, 0), {}, {}, {}};
    b.first.resize((size_t)rows * strip);
    b.count.resize((size_t)rows * strip);
    const int64_t plain = ((int64_t)(h + rows - 1) / rows) * ((w + strip - 1) / strip);
    for (int32_t i0 = 0; i0 < h; i0 += rows) {
        for (int32_t j0 = 0; j0 < w; j0 += strip) {
            b.tile(i0, j0, std::min(rows, h - i0), std::min(strip, w - j0));
            const int64_t ntiles = (int64_t)(sm.tiles.size() - t0);
            if (ntiles > 4 * plain && ntiles * kStreamMinPix > sm.npix - px0) return false;
            if (sm.nparts >= kLimit || (int64_t)sm.words.size() >= kLimit) return false;
        }
    }
    // the tiles that reach each chunk of bins, in tile order
    const int32_t nch = (m.npt + kStreamChunk - 1) / kStreamChunk;
    const size_t e0 = sm.ents.size();
    std::vector<int64_t> at((size_t)nch + 1, 0);
    auto span = [&](const StreamTile& t, int32_t& a, int32_t& z) {
        a = (int32_t)(t.wlo - bin_off) / kStreamChunk;
        z = (int32_t)(t.wlo - bin_off + t.nwin - 1) / kStreamChunk;
    };
    int32_t a, z;
    for (size_t k = t0; k < sm.tiles.size(); ++k) {
        span(sm.tiles[k], a, z);
        for (int32_t c = a; c <= z; ++c) at[c + 1]++;
    }
    for (int32_t c = 0; c < nch; ++c) at[c + 1] += at[c];
    if ((int64_t)e0 + at[nch] >= kLimit) return false;
    sm.ents.resize(e0 + (size_t)at[nch]);
    for (int32_t c = 0; c < nch; ++c)
        sm.chunks.push_back(StreamChunk{(int32_t)(bin_off + (int64_t)c * kStreamChunk),
                                        std::min(kStreamChunk, m.npt - c * kStreamChunk),
                                        (int32_t)(e0 + at[c]), (int32_t)(e0 + at[c + 1])});
    for (size_t k = t0; k < sm.tiles.size(); ++k) {
        const StreamTile& t = sm.tiles[k];
        span(t, a, z);
        for (int32_t c = a; c <= z; ++c)
            sm.ents[e0 + (size_t)at[c]++] = StreamEnt{t.part0 - t.wlo, t.wlo, t.wlo + t.nwin, 0};
    }
    return true;
}

}  // namespace azi
