// Host-only driver of the stream encoding's builder: builds the matrix of the
// geometry given on the command line, encodes it, and checks the encoding
// against the matrix by walking it as the kernels do.  Prints "tiles N" or
// "refused"; any violation is reported and ends with status 1.
//   h w center_y center_x npt npt_azim unit split(0 none, 1 bbox, 2 full) tile_px [lo hi]
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_1412_6367_amd/csrc/internal.h"

using namespace azi;

#define CHECK(cond)                                              \
    do {                                                         \
        if (!(cond)) {                                           \
            std::printf("violated: %s (line %d)\n", #cond, __LINE__); \
            return 1;                                            \
        }                                                        \
    } while (0)

int main(int argc, char** argv) {
    if (argc < 10) return 2;
    azi_geom g{};
    g.h = std::atoi(argv[1]);
    g.w = std::atoi(argv[2]);
    g.center_y_px = std::atof(argv[3]);
    g.center_x_px = std::atof(argv[4]);
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    const int nrad = std::atoi(argv[5]), azim = std::atoi(argv[6]), unit = std::atoi(argv[7]);
    const int split = std::atoi(argv[8]);
    const double range[2] = {argc > 11 ? std::atof(argv[10]) : 0, argc > 11 ? std::atof(argv[11]) : 0};
    HostMatrix m;
    std::string err;
    if (build_matrix(g, nrad, azim, unit, split, argc > 11 ? range : nullptr, m, err) != AZI_OK)
        return 2;
    const int npt = m.npt;
    // a second instance's place in a batch: offsets in pixels, bins and positions
    StreamMatrix sm;
    // (two-dimensional matrices stand alone)
    const int64_t pix_off = azim ? 0 : 1000, bin_off = azim ? 0 : 300;
    sm.ncoef = 77;
    sm.nparts = 55;
    if (!build_stream(m, g.h, g.w, std::atoi(argv[9]), pix_off, bin_off, sm)) {
        std::printf("refused\n");
        return 0;
    }
    std::vector<int> seen((size_t)m.npix, 0);     // times a pixel has a word
    std::vector<int> used((size_t)m.nnz(), 0);    // times an entry has a coefficient
    std::vector<double> W((size_t)npt, 0.0), x((size_t)m.npix);
    for (int64_t p = 0; p < m.npix; ++p) x[p] = (double)((p * 7919) % 1009);
    for (const StreamTile& b : sm.blanks)
        for (int r = 0; r < b.th; ++r)
            for (int c = 0; c < b.tw; ++c) {
                const int64_t p = b.pix0 - pix_off + (int64_t)r * b.w + c;
                CHECK(m.colptr[p] == m.colptr[p + 1]);
                ++seen[p];
            }
    int64_t coef = 77, part = 55, word = 0, group = 0, xblock = 0;
    std::vector<double> parts;
    for (const StreamTile& t : sm.tiles) {
        const int lk = t.shape & 15, lgw = (t.shape >> 4) & 15, lrs = (t.shape >> 8) & 15;
        const bool rows = t.shape & kStreamRowsMinor;
        const int gw = 4 << lgw, gh = 64 >> lgw, K = 1 << lk;
        const int across = (t.tw + gw - 1) / gw;
        const int nb = across * ((t.th + (gh << lrs) - 1) / (gh << lrs)) << lrs;
        const int ng = nb + t.nx;  // blocks, then scattered groups
        CHECK(t.nx == 0 || (azim && t.x0 == xblock));
        CHECK(t.nwin >= 1 && t.pitch >= t.nwin && t.pitch * K <= kStreamSlots);
        CHECK(nb <= kStreamMaxBlocks && t.w == g.w && t.word0 == word && t.g0 == group);
        CHECK(t.part0 == part);
        std::vector<double> lds((size_t)t.pitch * K, 0.0);
        for (int b = 0; b < ng; ++b) {
            CHECK(sm.gbase[group + b] == coef);
            for (int k = 0; k < (b < nb ? 4 : 1); ++k) {
                std::vector<int> owner((size_t)t.pitch * K, -1);
                for (int l = 0; l < 64; ++l) {
                    const int q = b / across;  // every 2^lrs-th row belongs to one block
                    const int r = (q >> lrs) * (gh << lrs) + (q & ((1 << lrs) - 1)) +
                                  ((rows ? l & (gh - 1) : l >> lgw) << lrs);
                    const int c = b % across * gw + 4 * (rows ? l >> (6 - lgw) : l & ((1 << lgw) - 1)) + k;
                    const uint16_t wd = sm.words[b < nb ? word + 256 * b + 4 * l + k
                                                        : word + 256 * nb + 64 * (b - nb) + l];
                    const int n = wd >> kStreamCountShift;
                    const int rel = wd & ((1 << kStreamCountShift) - 1);
                    int64_t p, k0;
                    if (b < nb) {
                        if (r >= t.th || c >= t.tw) {
                            CHECK(wd == 0);
                            continue;
                        }
                        p = t.pix0 - pix_off + (int64_t)r * t.w + c;
                        k0 = m.colptr[p];
                        ++seen[p];
                        CHECK(azim || n == m.colptr[p + 1] - m.colptr[p]);
                    } else {
                        if (n == 0) continue;
                        const int64_t x = 64 * (xblock + b - nb) + l;
                        const int i = sm.xpix[x];
                        CHECK((i >> kStreamColBits) < t.th && (i & 63) < t.tw);
                        p = t.pix0 + (int64_t)(i >> kStreamColBits) * t.w + (i & 63);
                        k0 = sm.xsrc[x];
                        CHECK(k0 >= m.colptr[p] && k0 + n <= m.colptr[p + 1]);
                    }
                    CHECK(n <= (t.shape >> kStreamMostShift));
                    coef += n;
                    if (n == 0) continue;
                    CHECK(azim || t.wlo + rel - bin_off == m.rowidx[k0]);
                    CHECK(rel + n <= t.nwin);
                    for (int j = 0; j < n; ++j) ++used[k0 + j];
                    const int slot = (l & (K - 1)) * t.pitch + rel;
                    CHECK(owner[slot] < 0);  // no two lanes of an access in one element
                    owner[slot] = l;
                    for (int j = 0; j < n; ++j) lds[slot + j] += m.cdata[k0 + j] * x[p];
                }
            }
        }
        for (int b = 0; b < t.nwin; ++b) {
            double s = 0.0;
            for (int k = 0; k < K; ++k) s += lds[k * t.pitch + b];
            parts.push_back(s);
        }
        part += t.nwin;
        word += 256 * nb + 64 * t.nx;
        group += ng;
        xblock += t.nx;
    }
    CHECK(coef == sm.ncoef && coef == 77 + m.nnz() && part == sm.nparts);
    CHECK((int64_t)sm.words.size() == word && (int64_t)sm.gbase.size() == group);
    CHECK((int64_t)sm.xsrc.size() == 64 * xblock && sm.xpix.size() == sm.xsrc.size());
    for (int s : seen) CHECK(s == 1 || (azim && s > 1));  // a pixel may have several tiles
    for (int s : used) CHECK(s == 1);
    int64_t k = 0;
    int bin = (int)bin_off;
    for (const StreamChunk& c : sm.chunks) {
        CHECK(c.bin0 == bin && c.nbins >= 1 && c.nbins <= kStreamChunk && c.k0 == k);
        for (; k < c.k1; ++k)
            for (int b = std::max(c.bin0, sm.ents[k].lo);
                 b < std::min(c.bin0 + c.nbins, sm.ents[k].hi); ++b)
                W[b - bin_off] += parts[sm.ents[k].base + b - 55];
        bin += c.nbins;
    }
    CHECK(bin == bin_off + npt && k == (int64_t)sm.ents.size());
    for (int b = 0; b < npt; ++b) {
        double ref = 0.0;
        for (int32_t z = m.indptr[b]; z < m.indptr[b + 1]; ++z) ref += m.data[z] * x[m.indices[z]];
        CHECK(std::fabs(W[b] - ref) <= 1e-12 * std::fabs(ref));
    }
    std::printf("tiles %zu\n", sm.tiles.size());
    return 0;
}
