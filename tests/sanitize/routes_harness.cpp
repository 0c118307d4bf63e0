// Host-only: which kernels the passes of a plan, or of a batch of n like it, take.
//   h w npt npt_azim(0: one-dimensional) dtype(0 f64, 1 f32) n(0: the plan itself)
// prints "image <kernels>, raw <kernels>, backward <kernels>", of a batch its
// image and backward passes.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "fake_device.h"

static void list(const char* name) {
    std::printf("%s", name);
    for (const std::string& c : fake::calls) std::printf(" %s", c.c_str());
    fake::calls.clear();
}

int main(int argc, char** argv) {
    if (argc != 7) return 2;
    azi_geom g{};
    g.h = std::atoi(argv[1]);
    g.w = std::atoi(argv[2]);
    g.center_y_px = g.h * 0.5;
    g.center_x_px = g.w * 0.5;
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    const int npt = std::atoi(argv[3]), azim = std::atoi(argv[4]), n = std::atoi(argv[6]);
    const int32_t dtype = std::atoi(argv[5]) ? AZI_F32 : AZI_F64;
    azi_plan* p = nullptr;
    const int rc = azim ? azi_plan_create2d(&g, npt, azim, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr,
                                            dtype, AZI_ACC_F64, &p)
                        : azi_plan_create(&g, npt, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr, dtype,
                                          AZI_ACC_F64, &p);
    if (rc != AZI_OK) return 2;
    void* image = std::calloc((size_t)g.h * g.w * (n ? n : 1), 8);
    double I[1];
    if (n) {
        std::vector<azi_plan*> plans(n, p);
        azi_batch* b = nullptr;
        if (azi_batch_create(plans.data(), n, 0, &b) != AZI_OK) return 2;
        fake::calls.clear();
        if (azi_batch_forward(b, image, I, nullptr, nullptr, 0.0, nullptr) != AZI_OK) return 2;
        list("image");
        if (azi_batch_backward(b, I, I, nullptr, image, nullptr) != AZI_OK) return 2;
        list(", backward");
        azi_batch_destroy(b);
    } else {
        if (azi_plan_upload(p, 0) != AZI_OK ||
            azi_plan_set_corrections(p, image, image, nullptr, nullptr, nullptr) != AZI_OK)
            return 2;
        fake::calls.clear();
        if (azi_integrate1d(p, image, I, nullptr, nullptr, 0.0, nullptr) != AZI_OK) return 2;
        list("image");
        if (azi_integrate1d_raw(p, image, AZI_I32, I, nullptr, nullptr, 0.0, nullptr) != AZI_OK)
            return 2;
        list(", raw");
        if (azi_integrate1d_backward(p, I, I, nullptr, image, 0, nullptr) != AZI_OK) return 2;
        list(", backward");
    }
    std::printf("\n");
    azi_plan_destroy(p);
    std::free(image);
    return fake::live != 0;
}
