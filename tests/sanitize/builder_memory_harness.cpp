// Host-only: every allocation of the stream encoding's threaded builder fails
// in turn.  It gives the encoding it gives otherwise, or throws
// std::bad_alloc to its caller; it does not end the process.
//   npt npt_azim
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../../paper_1412_6367_amd/csrc/internal.h"

using namespace azi;

static std::atomic<long> fail_in{-1};

void* operator new(size_t n) {
    if (fail_in.load() >= 0 && fail_in.fetch_sub(1) == 0) throw std::bad_alloc();
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main(int argc, char** argv) {
    if (argc != 3) return 2;
    azi_geom g{};
    g.h = g.w = 256;  // eight threads
    g.center_y_px = 120.3;
    g.center_x_px = 131.6;
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    HostMatrix m;
    std::string err;
    if (build_matrix(g, std::atoi(argv[1]), std::atoi(argv[2]), 0, 1, nullptr, m, err) != AZI_OK)
        return 2;
    StreamMatrix ref;
    if (!build_stream(m, g.h, g.w, 1024, 0, 0, ref)) return 2;
    int thrown = 0;
    for (long k = 0;; ++k) {
        StreamMatrix sm;
        bool built = false;
        fail_in = k;
        try {
            built = build_stream(m, g.h, g.w, 1024, 0, 0, sm);
        } catch (const std::bad_alloc&) {
            ++thrown;
        }
        const bool over = fail_in.exchange(-1) >= 0;
        if (built && (sm.words != ref.words || sm.gbase != ref.gbase || sm.ncoef != ref.ncoef ||
                      sm.tiles.size() != ref.tiles.size() || sm.ents.size() != ref.ents.size())) {
            std::printf("another encoding after allocation %ld failed\n", k);
            return 1;
        }
        if (over) break;  // no allocation was the k-th
    }
    std::printf("ok, %d times out of memory\n", thrown);
    return 0;
}
