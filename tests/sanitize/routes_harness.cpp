// Host-only: which kernels a map's passes take, by its size.
//   h w npt npt_azim -> "image <kernel>, raw <kernels>"
#include <cstdio>
#include <cstdlib>

#include "fake_device.h"

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    azi_geom g{};
    g.h = std::atoi(argv[1]);
    g.w = std::atoi(argv[2]);
    g.center_y_px = g.h * 0.5;
    g.center_x_px = g.w * 0.5;
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    azi_plan* p = nullptr;
    if (azi_plan_create2d(&g, std::atoi(argv[3]), std::atoi(argv[4]), AZI_UNIT_R_M, AZI_SPLIT_BBOX,
                          nullptr, AZI_F64, AZI_ACC_F64, &p) != AZI_OK ||
        azi_plan_upload(p, 0) != AZI_OK)
        return 2;
    void* image = std::calloc((size_t)g.h * g.w, 8);
    double I[1];
    if (azi_plan_set_corrections(p, image, image, nullptr, nullptr, nullptr) != AZI_OK) return 2;
    fake::calls.clear();
    if (azi_integrate1d(p, image, I, nullptr, nullptr, 0.0, nullptr) != AZI_OK) return 2;
    std::printf("image");
    for (const std::string& c : fake::calls) std::printf(" %s", c.c_str());
    fake::calls.clear();
    if (azi_integrate1d_raw(p, image, AZI_I32, I, nullptr, nullptr, 0.0, nullptr) != AZI_OK) return 2;
    std::printf(", raw");
    for (const std::string& c : fake::calls) std::printf(" %s", c.c_str());
    std::printf("\n");
    azi_plan_destroy(p);
    std::free(image);
    return fake::live != 0;
}
