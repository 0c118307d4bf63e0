// Host-only: every allocation of azi_plan_set_corrections fails in turn.  A
// raw frame integrated after a failed call is corrected by what the plan says
// it holds: in the kernel from forms made for it, or by the correction pass;
// never from the image as it is.
//   two_d dtype(0 f64, 1 f32) stage(0 gather .. as azi_tiling; -1: the default)
#include <cstdio>
#include <cstdlib>

#include "fake_device.h"

int main(int argc, char** argv) {
    if (argc != 4) return 2;
    const bool two_d = std::atoi(argv[1]) != 0;
    const int32_t dtype = std::atoi(argv[2]) ? AZI_F32 : AZI_F64;
    azi_geom g{};
    g.h = two_d ? 1420 : 300;
    g.w = two_d ? 1420 : 280;
    g.center_y_px = g.h * 0.45;
    g.center_x_px = g.w * 0.55;
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    const size_t bytes = (size_t)g.h * g.w * 8;
    void* const image = std::calloc(1, bytes);
    double I[1];
    int failures = 0;
    bool wrong = false;
    azi_plan* p = nullptr;
    const int rc0 = two_d ? azi_plan_create2d(&g, 40, 12, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr,
                                              dtype, AZI_ACC_F64, &p)
                          : azi_plan_create(&g, 90, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr, dtype,
                                            AZI_ACC_F64, &p);
    if (rc0 != AZI_OK || azi_plan_upload(p, 0) != AZI_OK) return 2;
    if (std::atoi(argv[3]) >= 0) {
        azi_tiling t;
        azi_plan_get_tiling(p, &t, nullptr);
        t.stage = std::atoi(argv[3]);
        if (azi_plan_set_tiling(p, &t) != AZI_OK) return 2;
    }
    for (int k = 0;; ++k) {
        fake::fail_in = k;
        const int rc = azi_plan_set_corrections(p, image, image, nullptr, nullptr, nullptr);
        fake::fail_in = -1;
        fake::calls.clear();
        fake::dark = fake::norm = nullptr;
        fake::stream = azi::StreamLaunch();
        if (azi_integrate1d_raw(p, image, AZI_I32, I, nullptr, nullptr, 0.0, nullptr) != AZI_OK)
            return 2;
        if (rc == AZI_OK) {
            std::printf("ok: %d failures, then%s\n", failures,
                        fake::called("correct") ? " the correction pass" : " one pass");
            break;
        }
        ++failures;
        if (k < 2) continue;  // the copies of dark and norm themselves: neither is set
        const bool in_kernel = fake::stream.corr || fake::stream.wsub;
        const bool by_pass = fake::called("correct") && fake::dark && fake::norm;
        if (!in_kernel && !by_pass) {
            std::printf("uncorrected after allocation %d failed\n", k);
            wrong = true;
        }
    }
    fake::uploaded = 0;
    if (azi_plan_set_corrections(p, image, image, nullptr, nullptr, nullptr) != AZI_OK) return 2;
    if (two_d && fake::uploaded > 0) {
        std::printf("%lld bytes of the matrix copied again\n", (long long)fake::uploaded);
        wrong = true;
    }
    azi_plan_destroy(p);
    std::free(image);
    if (fake::live != 0) {
        std::printf("%lld bytes left\n", (long long)fake::live);
        return 1;
    }
    return wrong;
}
