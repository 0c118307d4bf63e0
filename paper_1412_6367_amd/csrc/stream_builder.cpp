// Host builder of the stream encoding (see StreamMatrix): tiles, words,
// block bases and the lists the reduction walks.  The coefficients are put
// in order on the device from the pixel-major entries.
#include <algorithm>
#include <cstdlib>
#include <iterator>
#include <limits>
#include <new>
#include <thread>

#include "internal.h"

namespace azi {
namespace {

constexpr int64_t kLimit = std::numeric_limits<int32_t>::max();

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
    int32_t lgw, lrs;
    bool rows_minor;
};
// Where the first bin changes along the rows, and where down the columns.
constexpr Shape kAlong[] = {{4, 0, true}, {3, 0, true}, {2, 0, true}};
constexpr Shape kDown[] = {{3, 0, false}, {2, 0, false}, {1, 0, false}, {3, 1, false}, {2, 1, false},
                           {2, 2, false}};

// A further run of a pixel (two-dimensional matrices).
struct Item {
    int32_t bin, count;   // first bin in the window, bins
    int32_t pix, src;     // StreamMatrix::xpix and xsrc
};

// Encodes tiles of one matrix; the positions of `sm` are its own (the caller
// puts the parts of several builders one after the other).
struct Builder {
    const HostMatrix& m;
    const int32_t w;
    const int64_t pix_off, bin_off;
    StreamMatrix sm;
    std::vector<uint64_t> lanes;          // per bin of the window: lanes whose pixel starts there
    std::vector<int32_t> touched;
    std::vector<uint64_t> seen;           // per bin and copy: the last access that met it
    uint64_t access = 0;
    std::vector<int32_t> first;           // the current tile's pixels, row-major: first bin of
    std::vector<int32_t> count;           // the window and number of bins,
    std::vector<int32_t> radial;          // first radial bin
    std::vector<int32_t> widx;            // two-dimensional: per wedge, its place in the window
    std::vector<int32_t> wedges;
    std::vector<Item> items;
    int32_t th = 0, tw = 0;
    int32_t wlast = 0, wrow = 0;          // a wedge and its first row

    Builder(const HostMatrix& m, int32_t w, int64_t pix_off, int64_t bin_off)
        : m(m), w(w), pix_off(pix_off), bin_off(bin_off) {
        // as many as a window may have (at its largest 0.36 MB to clear, 13 us for
        // every image of a batch)
        lanes.assign((size_t)std::min(kStreamSlots, m.npt), 0);
        seen.assign(lanes.size() << 6, 0);
        if (m.two_d) widx.assign((size_t)m.npt_azim, -1);
    }

    int32_t across(Shape s) const { return (tw + (4 << s.lgw) - 1) >> (2 + s.lgw); }
    int32_t down(Shape s) const {
        const int32_t l = 6 - s.lgw + s.lrs;
        return (th + (1 << l) - 1) >> l << s.lrs;
    }

    // f(element of the tile, lane) for the k-th pixel of the lanes of block g
    // that feeds a bin.
    template <class F>
    void each(Shape s, int32_t g, int32_t k, F&& f) const {
        const int32_t a = across(s), gh = 64 >> s.lgw, gw = 1 << s.lgw;
        const int32_t c0 = g % a * gw * 4 + k, q = g / a;
        const int32_t r0 = (q >> s.lrs << (6 - s.lgw + s.lrs)) + (q & ((1 << s.lrs) - 1));
        for (int32_t r = 0; r < gh && r0 + (r << s.lrs) < th; ++r) {
            const int32_t e = (r0 + (r << s.lrs)) * tw;
            for (int32_t l = 0; l < gw; ++l) {
                const int32_t c = c0 + 4 * l;
                if (c < tw && count[e + c] > 0)
                    f(e + c, s.rows_minor ? (l << (6 - s.lgw)) + r : (r << s.lgw) + l);
            }
        }
    }

    void touch(int32_t bin, int32_t lane) {
        if (!lanes[bin]) touched.push_back(bin);
        lanes[bin] |= (uint64_t)1 << lane;
    }
    // The copies the touched lanes need, at least lk; forgets them.
    int32_t settle(int32_t lk) {
        for (int32_t b : touched) {
            const uint64_t mask = lanes[b];
            lanes[b] = 0;
            if (mask & (mask - 1)) lk = copies_for(mask, lk);
        }
        touched.clear();
        return lk;
    }
    // Whether 2^lk copies are too few for block g.  Most blocks need no more
    // than those before them, and this costs a fifth of finding the number.
    bool clashes(Shape s, int32_t g, int32_t lk) {
        const int32_t low = (1 << lk) - 1;
        bool clash = false;
        for (int32_t k = 0; k < 4 && !clash; ++k) {
            ++access;
            each(s, g, k, [&](int32_t e, int32_t lane) {
                uint64_t& last = seen[(size_t)(first[e] << lk | (lane & low))];
                clash |= last == access;
                last = access;
            });
        }
        return clash;
    }
    // The copies block g needs, at least lk.
    int32_t block_copies(Shape s, int32_t g, int32_t lk) {
        if (!clashes(s, g, lk)) return lk;
        for (int32_t k = 0; k < 4; ++k) {
            each(s, g, k, [&](int32_t e, int32_t lane) { touch(first[e], lane); });
            lk = settle(lk);
        }
        return lk;
    }

    // Wedge of a row; the last one's rows are kept, neighbours mostly share it
    // (a division per entry was a third of this pass).
    int32_t wedge_of(int32_t row) {
        if (row < wrow || row - wrow >= m.npt_rad) {
            wlast = row / m.npt_rad;
            wrow = wlast * m.npt_rad;
        }
        return wlast;
    }
    // End of the run of a two-dimensional pixel's entries starting at k.
    int32_t run_end(int32_t k, int32_t k1) {
        wedge_of(m.rowidx[k]);
        const int32_t row = m.rowidx[k], most = std::min(k1 - k, wrow + m.npt_rad - row);
        int32_t n = 1;
        while (n < most && m.rowidx[k + n] == row + n) ++n;
        return k + n;
    }

    // Scattered groups of the sorted items: item i goes to group i % groups, so
    // that the items of one bin meet in one access only if there are more than
    // groups.
    int32_t xgroups() const { return 4 * (int32_t)((items.size() + 255) / 256); }
    int32_t item_copies(int32_t lk) {
        const size_t nx = (size_t)xgroups();
        for (size_t q = 0; q < nx; ++q) {
            for (size_t i = q; i < items.size(); i += nx) touch(items[i].bin, (int32_t)(i / nx));
            lk = settle(lk);
        }
        return lk;
    }

    void tile(int32_t i0, int32_t j0, int32_t rows, int32_t cols) {
        th = rows;
        tw = cols;
        const int32_t n = th * tw;
        if (first.size() < (size_t)n) {
            first.resize(n);
            count.resize(n);
            radial.resize(n);
        }
        int32_t lo = std::numeric_limits<int32_t>::max(), hi = -1, most = 0;
        wedges.clear();
        items.clear();
        for (int32_t r = 0, e = 0; r < th; ++r) {
            int64_t p = (int64_t)(i0 + r) * w + j0;
            for (int32_t c = 0; c < tw; ++c, ++p, ++e) {
                int32_t k0 = m.colptr[p];
                const int32_t k1 = m.colptr[p + 1];
                count[e] = 0;
                if (k1 == k0) continue;
                if (!m.two_d) {
                    count[e] = k1 - k0;
                    first[e] = radial[e] = m.rowidx[k0];
                    lo = std::min(lo, first[e]);
                    hi = std::max(hi, first[e] + k1 - k0);
                    most = std::max(most, k1 - k0);
                    continue;
                }
                bool main = true;
                while (k0 < k1) {
                    const int32_t z = run_end(k0, k1);
                    const int32_t wedge = wedge_of(m.rowidx[k0]), a = m.rowidx[k0] - wrow;
                    lo = std::min(lo, a);
                    hi = std::max(hi, a + z - k0);
                    most = std::max(most, z - k0);
                    if (widx[wedge] < 0) {
                        widx[wedge] = 0;
                        wedges.push_back(wedge);
                    }
                    if (main) {
                        count[e] = z - k0;
                        first[e] = m.rowidx[k0];
                        radial[e] = a;
                        main = false;
                    } else {
                        items.push_back(Item{m.rowidx[k0], z - k0, r << kStreamColBits | c, k0});
                    }
                    k0 = z;
                }
            }
        }
        for (int32_t k : wedges) widx[k] = -1;
        const int64_t pix0 = pix_off + (int64_t)i0 * w + j0;
        if (hi < 0) {  // feeds no bin
            sm.blanks.push_back(StreamTile{pix0, w, tw, th, 0, 0, 0, 0, 0, 0, 0, 0, 0});
            return;
        }
        const int32_t span = hi - lo;
        const int64_t nwin = m.two_d ? (int64_t)span * wedges.size() : span;
        if ((nwin | 1) > kStreamSlots) {
            halve(i0, j0, rows, cols, lo, span, rows < cols);
            return;
        }
        const int32_t pitch = (int32_t)nwin | 1;
        if (m.two_d) {
            std::sort(wedges.begin(), wedges.end());
            for (size_t k = 0; k < wedges.size(); ++k) widx[wedges[k]] = (int32_t)k * span;
            auto local = [&](int32_t row) {
                const int32_t at = widx[wedge_of(row)];
                return at + row - wrow - lo;
            };
            for (int32_t e = 0; e < n; ++e)
                if (count[e]) first[e] = local(first[e]);
            for (Item& it : items) it.bin = local(it.bin);
            for (int32_t k : wedges) widx[k] = -1;
            std::stable_sort(items.begin(), items.end(),
                             [](const Item& a, const Item& b) { return a.bin < b.bin; });
        } else {
            for (int32_t e = 0; e < n; ++e)
                if (count[e]) first[e] -= lo;
        }
        // which way the bins change, between the tile's edges
        int64_t along = 0, below = 0;
        for (int32_t r = 0; r < th; ++r)
            if (count[r * tw] && count[r * tw + tw - 1])
                along += std::abs(radial[r * tw + tw - 1] - radial[r * tw]);
        for (int32_t c = 0; c < tw; ++c)
            if (count[c] && count[n - tw + c]) below += std::abs(radial[n - tw + c] - radial[c]);
        const bool turn = below * (tw - 1) * th > along * (th - 1) * tw;
        const Shape* shapes = turn ? kDown : kAlong;
        const int nshapes = turn ? (int)std::size(kDown) : (int)std::size(kAlong);
        // the shape of the least work, copies estimated from three blocks:
        // about 240 issue slots a block and 4 for each image row it reads, 4
        // per 64 LDS elements cleared and merged by each of four wavefronts
        const int32_t xk = item_copies(0);
        int64_t best = std::numeric_limits<int64_t>::max();
        Shape shape{-1, 0, false};
        int32_t lk = 0;
        for (int k = 0; k < nshapes; ++k) {
            const Shape s = shapes[k];
            const int32_t ng = across(s) * down(s);
            if (ng > kStreamMaxBlocks) continue;
            int32_t l = block_copies(s, 0, xk);
            if (ng > 2) l = block_copies(s, (ng - 1) / 2, l);
            if (ng > 1) l = block_copies(s, ng - 1, l);
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
            if (n > 1) {
                // two-dimensional: across the direction in which the wedges lie
                halve(i0, j0, rows, cols, lo, span,
                      m.two_d && 2 * std::min(rows, cols) >= std::max(rows, cols) ? turn
                                                                                   : rows < cols);
                return;
            }
            // a pixel of its own: its runs have distinct bins, one copy serves
            shape = kAlong[0];
            lk = 0;
        }
        emit(pix0, shape, lk, lo, span, pitch, most);
    }

    // Half of the tile (of its columns or rows), then the other half; a single pixel (two-dimensional)
    // as many of its wedges at a time as a window holds.
    void halve(int32_t i0, int32_t j0, int32_t rows, int32_t cols, int32_t lo, int32_t span,
               bool columns) {
        if (rows * cols > 1) {
            if (!columns) {
                tile(i0, j0, rows / 2, cols);
                tile(i0 + rows / 2, j0, rows - rows / 2, cols);
            } else {
                tile(i0, j0, rows, cols / 2);
                tile(i0, j0 + cols / 2, rows, cols - cols / 2);
            }
            return;
        }
        if (span >= kStreamSlots) {  // refused by the caller
            sm.over[4] = -1;
            return;
        }
        const int64_t p = (int64_t)i0 * w + j0;
        const int32_t k1 = m.colptr[p + 1], most_wedges = (kStreamSlots - 1) / span;
        count[0] = 0;
        int32_t most = 0;
        wedges.clear();
        items.clear();
        auto flush = [&] {
            if (wedges.empty()) return;
            emit(pix_off + p, kAlong[0], 0, lo, span, ((int32_t)wedges.size() * span) | 1, most);
            wedges.clear();
            items.clear();
            most = 0;
        };
        for (int32_t k = m.colptr[p]; k < k1;) {
            const int32_t z = run_end(k, k1), wedge = wedge_of(m.rowidx[k]);
            if (wedges.empty() || wedges.back() != wedge) {
                if ((int32_t)wedges.size() == most_wedges) flush();
                wedges.push_back(wedge);
            }
            items.push_back(Item{((int32_t)wedges.size() - 1) * span + m.rowidx[k] - wrow - lo,
                                 z - k, 0, k});
            most = std::max(most, z - k);
            k = z;
        }
        flush();
    }

    void emit(int64_t pix0, Shape shape, int32_t lk, int32_t lo, int32_t span, int32_t pitch,
              int32_t most) {
        const int32_t ng = across(shape) * down(shape), nx = xgroups();
        const int32_t nwin = m.two_d ? span * (int32_t)wedges.size() : span;
        sm.tiles.push_back(StreamTile{
            pix0, w, tw, th,
            lk | shape.lgw << 4 | shape.lrs << 8 | (shape.rows_minor ? kStreamRowsMinor : 0) |
                std::min(most, kStreamMaxCount) << kStreamMostShift,
            (int32_t)sm.words.size(), (int32_t)sm.gbase.size(),
            m.two_d ? 0 : (int32_t)(bin_off + lo), nwin, pitch, (int32_t)sm.nparts, nx,
            (int32_t)(sm.xsrc.size() / 64)});
        if (most > kStreamMaxCount) sm.over[4] = -1;  // refused by the caller
        if (m.two_d) {
            for (size_t k = 0; k < wedges.size(); ++k) {
                const int32_t row = wedges[k] * m.npt_rad + lo;
                sm.segs.push_back(StreamEnt{(int32_t)sm.nparts + (int32_t)k * span, row, row + span, 0});
            }
        } else {
            sm.segs.push_back(StreamEnt{(int32_t)sm.nparts, (int32_t)(bin_off + lo),
                                        (int32_t)(bin_off + lo) + span, 0});
        }
        sm.nparts += nwin;
        sm.npix += th * tw;
        const size_t word0 = sm.words.size();
        sm.words.resize(word0 + (size_t)ng * 256 + (size_t)nx * 64, 0);
        uint16_t* out = sm.words.data() + word0;
        auto put = [&](uint16_t* at, int32_t bin, int32_t n, int32_t& sum) {
            *at = (uint16_t)(bin | n << kStreamCountShift);
            sum += n;
            for (int32_t k = 0; k < 4; ++k) sm.over[k] += n > k;
            if (sm.over[4] >= 0) sm.over[4] += n > 4;
        };
        for (int32_t g = 0; g < ng; ++g, out += 256) {
            int32_t sum = 0;
            for (int32_t k = 0; k < 4; ++k)
                each(shape, g, k, [&](int32_t e, int32_t lane) {
                    put(out + 4 * lane + k, first[e], count[e], sum);
                });
            sm.gbase.push_back((int32_t)sm.ncoef);
            sm.ncoef += sum;
        }
        const size_t x0 = sm.xsrc.size();
        sm.xsrc.resize(x0 + (size_t)nx * 64, 0);
        sm.xpix.resize(x0 + (size_t)nx * 64, 0);
        for (int32_t g = 0; g < nx; ++g, out += 64) {
            int32_t sum = 0;
            for (size_t lane = 0, i = g; i < items.size(); ++lane, i += nx) {
                put(out + lane, items[i].bin, items[i].count, sum);
                sm.xpix[x0 + 64 * (size_t)g + lane] = (uint16_t)items[i].pix;
                sm.xsrc[x0 + 64 * (size_t)g + lane] = items[i].src;
            }
            sm.gbase.push_back((int32_t)sm.ncoef);
            sm.ncoef += sum;
        }
    }
};

// Appends `part`, whose positions start at 0, to `sm`.
bool append(const StreamMatrix& part, StreamMatrix& sm) {
    if ((int64_t)(sm.words.size() + part.words.size()) >= kLimit ||
        sm.ncoef + part.ncoef >= kLimit || sm.nparts + part.nparts >= kLimit ||
        (int64_t)(sm.segs.size() + part.segs.size()) >= kLimit || part.over[4] < 0)
        return false;
    for (StreamTile t : part.tiles) {
        t.word0 += (int32_t)sm.words.size();
        t.g0 += (int32_t)sm.gbase.size();
        t.part0 += (int32_t)sm.nparts;
        t.x0 += (int32_t)(sm.xsrc.size() / 64);
        sm.tiles.push_back(t);
    }
    sm.blanks.insert(sm.blanks.end(), part.blanks.begin(), part.blanks.end());
    for (StreamEnt e : part.segs) {
        e.base += (int32_t)sm.nparts - e.lo;  // of the partial sum of bin b
        sm.segs.push_back(e);
    }
    for (int32_t g : part.gbase) sm.gbase.push_back(g + (int32_t)sm.ncoef);
    sm.words.insert(sm.words.end(), part.words.begin(), part.words.end());
    sm.xpix.insert(sm.xpix.end(), part.xpix.begin(), part.xpix.end());
    sm.xsrc.insert(sm.xsrc.end(), part.xsrc.begin(), part.xsrc.end());
    sm.ncoef += part.ncoef;
    sm.nparts += part.nparts;
    sm.npix += part.npix;
    for (int k = 0; k < 5; ++k) sm.over[k] += part.over[k];
    return true;
}

// One thread for every so many pixels of an instance, up to kBuildThreads
// (about 0.1 us a pixel, so 0.8 ms a thread where starting one takes 0.03; a
// 330 x 330 map of 100 x 36 bins takes 10 ms alone).
constexpr int64_t kThreadPix = (int64_t)1 << 13;
constexpr int32_t kBuildThreads = 16;

}  // namespace

bool build_stream(const HostMatrix& m, int32_t h, int32_t w, int32_t tile_px, int64_t pix_off,
                  int64_t bin_off, StreamMatrix& sm) {
    const int64_t nnz = (int64_t)m.rowidx.size();
    if (m.npix < 4 || sm.ncoef + nnz >= kLimit) return false;
    if (m.two_d && (m.npt_rad < 1 || pix_off || bin_off)) return false;
    // strips of equal width but for the rounding to 8 columns, and rows of
    // about tile_px pixels, a multiple of 16 (four blocks of 64 x 4 pixels,
    // one for each wavefront) where the image has them; of 64 for the wider
    // bins of two-dimensional matrices (blocks of 16 rows, every fourth)
    const int32_t strips = (w + 63) / 64;
    const int32_t strip = std::min(w, ((w + strips - 1) / strips + 7) / 8 * 8);
    int32_t rows = (std::min(tile_px, kStreamMaxPix) + strip / 2) / strip;
    rows = std::min(rows, 1 << (16 - kStreamColBits));
    const int32_t unit = m.two_d && rows >= 64 ? 64 : 16;
    rows = std::max(1, std::min(h, rows >= unit ? rows / unit * unit : rows));
    if (m.npix >= (int64_t)1 << kBandShift || stream_reach(rows, w) > kLimit) return false;
    const int32_t bands = (h + rows - 1) / rows;
    const int64_t per_band = (w + strip - 1) / strip;
    const int64_t units = bands * per_band;
    int64_t want = std::min({(int64_t)kBuildThreads, units, m.npix / kThreadPix});
    if (want > 1) want = std::min(want, (int64_t)std::thread::hardware_concurrency());
    const int32_t threads = (int32_t)std::max<int64_t>(1, want);
    std::vector<Builder> part;
    part.reserve(threads);
    for (int32_t k = 0; k < threads; ++k) part.emplace_back(m, w, pix_off, bin_off);
    std::vector<char> bad(threads, 0);
    // the k-th thread's tiles, along the bands; a matrix that will be refused
    // is given up early
    auto build = [&](int32_t k) {
        Builder& b = part[k];
        const int64_t a = units * k / threads, z = units * (k + 1) / threads;
        try {
            for (int64_t u = a; u < z && !bad[k]; ++u) {
                const int32_t i0 = (int32_t)(u / per_band) * rows;
                const int32_t j0 = (int32_t)(u % per_band) * strip;
                const int32_t i1 = std::min(i0 + rows, h), j1 = std::min(j0 + strip, w);
                for (int32_t i = i0; i < i1 && !m.two_d; ++i)
                    for (int64_t p = (int64_t)i * w + j0, e = p + (j1 - j0); p < e; ++p) {
                        const int32_t k0 = m.colptr[p], k1 = m.colptr[p + 1];
                        if (k1 - k0 > kStreamMaxCount ||
                            (k1 > k0 && m.rowidx[k1 - 1] != m.rowidx[k0] + (k1 - k0 - 1)))
                            bad[k] = 1;
                    }
                if (bad[k]) break;
                b.tile(i0, j0, i1 - i0, j1 - j0);
                const int64_t nt = (int64_t)b.sm.tiles.size();
                // what the whole matrix will be refused for, wherever its
                // tiles are: the answer does not depend on the threads
                if (nt > 4 * units && nt * kStreamMinPix > m.npix) bad[k] = 1;
                if ((int64_t)b.sm.words.size() >= kLimit || b.sm.nparts >= kLimit) bad[k] = 1;
            }
        } catch (...) {  // memory
            bad[k] = 2;
        }
    };
    // room first: nothing may throw past threads that run
    std::vector<std::thread> run;
    run.reserve(threads);
    for (int32_t k = 1; k < threads; ++k) {
        try {
            run.emplace_back(build, k);
        } catch (...) {  // no thread to be had: this one does it
            build(k);
        }
    }
    build(0);
    for (std::thread& t : run) t.join();
    for (char b : bad) {
        if (b == 2) throw std::bad_alloc();
        if (b) return false;
    }
    const size_t t0 = sm.tiles.size(), s0 = sm.segs.size();
    const int64_t px0 = sm.npix, parts0 = sm.nparts;
    if (threads > 1) {  // once, not as the parts come
        size_t nt = 0, nw = 0, ng = 0, nx = 0;
        for (const Builder& b : part) {
            nt += b.sm.tiles.size();
            nw += b.sm.words.size();
            ng += b.sm.gbase.size();
            nx += b.sm.xsrc.size();
        }
        sm.tiles.reserve(t0 + nt);
        sm.words.reserve(sm.words.size() + nw);
        sm.gbase.reserve(sm.gbase.size() + ng);
        sm.xsrc.reserve(sm.xsrc.size() + nx);
        sm.xpix.reserve(sm.xpix.size() + nx);
    }
    for (Builder& b : part) {
        if (!append(b.sm, sm)) return false;
        b.sm = StreamMatrix();
    }
    const int64_t ntiles = (int64_t)(sm.tiles.size() - t0);
    if (ntiles > 4 * per_band * bands && ntiles * kStreamMinPix > sm.npix - px0) return false;
    if (m.two_d && (sm.nparts - parts0) * 4 > nnz) return false;
    // the windows that reach each chunk of bins, in tile order
    const int32_t nch = (m.npt + kStreamChunk - 1) / kStreamChunk;
    const size_t e0 = sm.ents.size();
    std::vector<int64_t> at((size_t)nch + 1, 0);
    for (size_t k = s0; k < sm.segs.size(); ++k) {
        const StreamEnt& e = sm.segs[k];
        for (int64_t c = (e.lo - bin_off) / kStreamChunk; c * kStreamChunk < e.hi - bin_off; ++c)
            at[c + 1]++;
    }
    for (int32_t c = 0; c < nch; ++c) at[c + 1] += at[c];
    if ((int64_t)e0 + at[nch] >= kLimit) return false;
    sm.ents.resize(e0 + (size_t)at[nch]);
    for (int32_t c = 0; c < nch; ++c)
        sm.chunks.push_back(StreamChunk{(int32_t)(bin_off + (int64_t)c * kStreamChunk),
                                        std::min(kStreamChunk, m.npt - c * kStreamChunk),
                                        (int32_t)(e0 + at[c]), (int32_t)(e0 + at[c + 1])});
    for (size_t k = s0; k < sm.segs.size(); ++k) {
        const StreamEnt& e = sm.segs[k];
        for (int64_t c = (e.lo - bin_off) / kStreamChunk; c * kStreamChunk < e.hi - bin_off; ++c)
            sm.ents[e0 + (size_t)at[c]++] = e;
    }
    return true;
}

}  // namespace azi
