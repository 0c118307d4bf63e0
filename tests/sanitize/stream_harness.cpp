// Host-only driver of the stream encoding's builder: builds the matrix of the
// geometry given on the command line, encodes it, and checks the encoding
// against the matrix by walking it as the kernels do.  Prints "tiles N" or
// "refused"; any violation is reported and ends with status 1.
//   h w center_y center_x npt unit split(0 none, 1 bbox, 2 full) tile_px [lo hi]
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
    if (argc < 9) return 2;
    azi_geom g{};
    g.h = std::atoi(argv[1]);
    g.w = std::atoi(argv[2]);
    g.center_y_px = std::atof(argv[3]);
    g.center_x_px = std::atof(argv[4]);
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    const int npt = std::atoi(argv[5]), unit = std::atoi(argv[6]), split = std::atoi(argv[7]);
    const double range[2] = {argc > 10 ? std::atof(argv[9]) : 0, argc > 10 ? std::atof(argv[10]) : 0};
    HostMatrix m;
    std::string err;
    if (build_matrix(g, npt, 0, unit, split, argc > 10 ? range : nullptr, m, err) != AZI_OK) return 2;
    // a second instance's place in a batch: offsets in pixels, bins and positions
    StreamMatrix sm;
    const int64_t pix_off = 1000, bin_off = 300;
    sm.ncoef = 77;
    sm.nparts = 55;
    if (!build_stream(m, g.h, g.w, std::atoi(argv[8]), pix_off, bin_off, sm)) {
        std::printf("refused\n");
        return 0;
    }
    std::vector<int> seen((size_t)m.npix, 0);
    std::vector<double> W((size_t)npt, 0.0), x((size_t)m.npix);
    for (int64_t p = 0; p < m.npix; ++p) x[p] = (double)((p * 7919) % 1009);
    for (const StreamTile& b : sm.blanks)
        for (int r = 0; r < b.th; ++r)
            for (int c = 0; c < b.tw; ++c) {
                const int64_t p = b.pix0 - pix_off + (int64_t)r * b.w + c;
                CHECK(m.colptr[p] == m.colptr[p + 1]);
                ++seen[p];
            }
    int64_t coef = 77, part = 55, word = 0, group = 0;
    std::vector<double> parts;
    for (const StreamTile& t : sm.tiles) {
        const int lk = t.shape & 255, lgw = (t.shape >> 8) & 255;
        const bool rows = t.shape & kStreamRowsMinor;
        const int gw = 4 << lgw, gh = 64 >> lgw, K = 1 << lk;
        const int across = (t.tw + gw - 1) / gw, ng = across * ((t.th + gh - 1) / gh);
        CHECK(t.nwin >= 1 && t.pitch >= t.nwin && t.pitch * K <= kStreamSlots);
        CHECK(ng <= kStreamMaxBlocks && t.w == g.w && t.word0 == word && t.g0 == group);
        CHECK(t.part0 == part);
        std::vector<double> lds((size_t)t.pitch * K, 0.0);
        for (int b = 0; b < ng; ++b) {
            CHECK(sm.gbase[group + b] == coef);
            for (int k = 0; k < 4; ++k) {
                std::vector<int> owner((size_t)t.pitch * K, -1);
                for (int l = 0; l < 64; ++l) {
                    const int r = b / across * gh + (rows ? l & (gh - 1) : l >> lgw);
                    const int c = b % across * gw + 4 * (rows ? l >> (6 - lgw) : l & ((1 << lgw) - 1)) + k;
                    const uint16_t wd = sm.words[word + 256 * b + 4 * l + k];
                    const int n = wd >> kStreamCountShift;
                    const int rel = wd & ((1 << kStreamCountShift) - 1);
                    if (r >= t.th || c >= t.tw) {
                        CHECK(wd == 0);
                        continue;
                    }
                    const int64_t p = t.pix0 - pix_off + (int64_t)r * t.w + c;
                    CHECK(++seen[p] == 1);
                    CHECK(n == m.colptr[p + 1] - m.colptr[p] && n <= sm.max_count);
                    coef += n;
                    if (n == 0) continue;
                    CHECK(t.wlo + rel - bin_off == m.rowidx[m.colptr[p]]);
                    CHECK(rel + n <= t.nwin);
                    const int slot = (l & (K - 1)) * t.pitch + rel;
                    CHECK(owner[slot] < 0);  // no two lanes of an access in one element
                    owner[slot] = l;
                    for (int j = 0; j < n; ++j) lds[slot + j] += m.cdata[m.colptr[p] + j] * x[p];
                }
            }
        }
        for (int b = 0; b < t.nwin; ++b) {
            double s = 0.0;
            for (int k = 0; k < K; ++k) s += lds[k * t.pitch + b];
            parts.push_back(s);
        }
        part += t.nwin;
        word += 256 * ng;
        group += ng;
    }
    CHECK(coef == sm.ncoef && coef == 77 + m.nnz() && part == sm.nparts);
    CHECK((int64_t)sm.words.size() == word && (int64_t)sm.gbase.size() == group);
    for (int s : seen) CHECK(s == 1);
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
