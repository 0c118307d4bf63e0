// Host-only: images whose positions would not fit the stream kernels' 32 bits
// are refused before any of the matrix is read (these matrices have no
// arrays), and stream_reach bounds every position that the kernels' lanes
// form, walked over the block shapes.
#include <algorithm>
#include <cstdio>

#include "../../paper_1412_6367_amd/csrc/internal.h"

using namespace azi;

int main() {
    int bad = 0;
    const struct { int32_t h, w, azim; } refused[] = {
        {1, (1 << 27) - 1, 0},  // one row: 2^27 pixels are not reached, 127 rows of padding are
        {1, 1 << 25, 0},
        {1, 1 << 24, 12},
        {3, 1 << 24, 0},
        {1 << 14, 1 << 13, 0},  // 2^27 pixels
        {1 << 14, 1 << 13, 36},
        {1 << 27, 1, 0},
        {30000, 30000, 0},
    };
    for (const auto& c : refused) {
        HostMatrix m;
        m.npix = (int64_t)c.h * c.w;
        m.npt_rad = 16;
        m.two_d = c.azim > 0;
        m.npt_azim = std::max(c.azim, 1);
        m.npt = m.npt_rad * m.npt_azim;
        StreamMatrix sm;
        if (build_stream(m, c.h, c.w, c.azim ? 4096 : 3072, 0, 0, sm)) {
            std::printf("%d x %d encoded\n", c.h, c.w);
            bad = 1;
        }
    }
    // as StreamLane: lanes of 4 << lgw columns, 64 >> lgw rows, every 2^lrs-th
    const int shapes[][2] = {{4, 0}, {3, 0}, {2, 0}, {1, 0}, {3, 1}, {2, 1}, {2, 2}};
    for (int th : {1, 2, 15, 16, 17, 48, 63, 64, 65, 1023, 1024})
        for (int tw : {1, 5, 63, 64})
            for (const auto& s : shapes)
                for (int64_t w : {64ll, 1000000ll, 1ll << 24}) {
                    const int lgw = s[0], lrs = s[1], l = 6 - lgw + lrs;
                    const int64_t across = (tw + (4 << lgw) - 1) >> (2 + lgw);
                    // one block past the last: the first of the next row of blocks
                    const int64_t pr = (int64_t)((th + (1 << l) - 1) >> l << lrs);
                    int64_t row = 0;
                    for (int64_t q = 0; q <= pr; ++q)
                        row = std::max(row, (q >> lrs << l) + (q & ((1 << lrs) - 1)));
                    const int64_t r0 = (int64_t)((64 >> lgw) - 1) << lrs;
                    const int64_t c0 = 4 * ((1 << lgw) - 1) + 3;
                    const int64_t at = (row + r0) * w + ((across - 1) << (2 + lgw)) + c0;
                    if (at > stream_reach(th, (int32_t)w)) {
                        std::printf("past the reach: %d %d %d %d\n", th, tw, lgw, lrs);
                        bad = 1;
                    }
                }
    if (!bad) std::printf("ok\n");
    return bad;
}
