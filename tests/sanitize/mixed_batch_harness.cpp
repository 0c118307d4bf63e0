// Host-only: a batch of n images, the last one of h x w pixels (npt_azim 0:
// one-dimensional), which the stream encoding does not take.
//   n h w npt_azim -> "image <kernels>, N encoded"
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "fake_device.h"

static azi_plan* plan(int h, int w, int azim) {
    azi_geom g{};
    g.h = h;
    g.w = w;
    g.center_y_px = h * 0.5;
    g.center_x_px = w * 0.5;
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    azi_plan* p = nullptr;
    const int rc = azim ? azi_plan_create2d(&g, 4, azim, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr,
                                            AZI_F64, AZI_ACC_F64, &p)
                        : azi_plan_create(&g, 4, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr, AZI_F64,
                                          AZI_ACC_F64, &p);
    if (rc != AZI_OK || azi_plan_set_layout(p, AZI_LAYOUT_RUN) != AZI_OK) std::exit(2);
    azi_tiling t;
    azi_plan_get_tiling(p, &t, nullptr);
    t.tile_nnz = 0;
    t.band = 16;
    t.grid = 0;
    if (azi_plan_set_tiling(p, &t) != AZI_OK) std::exit(2);
    return p;
}

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    const int n = std::atoi(argv[1]);
    azi_plan* const one = plan(20, 30, 0);
    azi_plan* const last = plan(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]));
    std::vector<azi_plan*> plans(n, one);
    plans.back() = last;
    azi_batch* b = nullptr;
    if (azi_batch_create(plans.data(), n, 0, &b) != AZI_OK) return 2;
    std::vector<double> x((size_t)n * 600 + 600), I(1);
    fake::calls.clear();
    if (azi_batch_forward(b, x.data(), I.data(), nullptr, nullptr, 0.0, nullptr) != AZI_OK) return 2;
    std::printf("image");
    for (const std::string& c : fake::calls) std::printf(" %s", c.c_str());
    std::printf(", %d encoded\n", fake::encoded);
    azi_batch_destroy(b);
    azi_plan_destroy(one);
    azi_plan_destroy(last);
    return fake::live != 0;
}
