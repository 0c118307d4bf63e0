// Host-only: a tiling is changed so that a plan or batch leaves the stream
// encoding and comes back, and every allocation on the way, on the device or
// the host, fails in turn.  A call that fails says so and throws nothing; the
// pass after it runs over an encoding that is whole and corrects raw frames.
//   map profile batch: 0 1 2
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>

#include "fake_device.h"

static std::atomic<long> new_in{-1};
void* operator new(size_t n) {
    if (new_in.load() >= 0 && new_in.fetch_sub(1) == 0) throw std::bad_alloc();
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return std::malloc(n ? n : 1); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

static int kind;
static azi_plan* p = nullptr;
static azi_batch* b = nullptr;
static void* image;

static int set(const azi_tiling& t) {
    return kind == 2 ? azi_batch_set_tiling(b, &t) : azi_plan_set_tiling(p, &t);
}

// What is wrong with the pass, or null.
static const char* pass(bool raw) {
    double I[1];
    fake::calls.clear();
    fake::stream = azi::StreamLaunch();
    fake::band = azi::BandLaunch();
    const int rc = kind == 2 ? azi_batch_forward(b, image, I, nullptr, nullptr, 0.0, nullptr)
                   : raw ? azi_integrate1d_raw(p, image, AZI_I32, I, nullptr, nullptr, 0.0, nullptr)
                         : azi_integrate1d(p, image, I, nullptr, nullptr, 0.0, nullptr);
    if (rc != AZI_OK) return "the pass fails";
    bool corrected = false;
    if (fake::called("stream")) {
        const azi::StreamLaunch& a = fake::stream;
        for (const void* q : {(const void*)a.tiles, (const void*)a.words, (const void*)a.gbase,
                              a.coef, (const void*)a.chunks, (const void*)a.ents,
                              (const void*)a.ufix, (const void*)a.parts})
            if (!fake::held(q)) return "a stream array is not there";
        corrected = a.corr || a.wsub;
    } else if (fake::called("band")) {
        const azi::BandLaunch& a = fake::band;
        for (const void* q : {(const void*)a.pieces, (const void*)a.packed, a.coef,
                              (const void*)a.bin_slot, (const void*)a.bin_count,
                              (const void*)a.parts, (const void*)a.gbase})
            if (!fake::held(q)) return "a run array is not there";
        corrected = a.corr || a.wsub_in;
    } else if (!fake::called("forward")) {
        return "nothing runs";
    }
    if (raw && !corrected && !fake::called("correct")) return "the frame is not corrected";
    return nullptr;
}

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    kind = std::atoi(argv[1]);
    azi_geom g{};
    g.h = kind == 0 ? 1420 : 200;
    g.w = kind == 0 ? 1420 : 180;
    g.center_y_px = g.h * 0.45;
    g.center_x_px = g.w * 0.55;
    g.pixel_y_m = g.pixel_x_m = 1e-4;
    g.dist_m = 0.1;
    g.wavelength_m = 1e-10;
    image = std::calloc(1, (size_t)g.h * g.w * 16);
    const int rc0 = kind == 0 ? azi_plan_create2d(&g, 40, 12, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr,
                                                  AZI_F64, AZI_ACC_F64, &p)
                              : azi_plan_create(&g, 90, AZI_UNIT_R_M, AZI_SPLIT_BBOX, nullptr,
                                                AZI_F64, AZI_ACC_F64, &p);
    if (rc0 != AZI_OK) return 2;
    azi_tiling on, off;
    if (kind == 2) {
        azi_plan* two[] = {p, p};
        if (azi_batch_create(two, 2, 0, &b) != AZI_OK) return 2;
        azi_batch_get_tiling(b, &on, nullptr);
    } else {
        if (azi_plan_upload(p, 0) != AZI_OK ||
            azi_plan_set_corrections(p, image, image, nullptr, nullptr, nullptr) != AZI_OK)
            return 2;
        azi_plan_get_tiling(p, &on, nullptr);
    }
    off = on;
    if (kind == 0) off.variant = 0;
    else off.tile_nnz = 2048;
    if (pass(kind < 2) || !fake::called("stream")) return 2;
    if (set(off) != AZI_OK || pass(kind < 2) || fake::called("stream")) return 2;
    int failed = 0;
    for (const bool leave : {true, false})
        for (const bool device : {true, false}) {
            for (long k = 0;; k += device || kind != 0 ? 1 : 41) {
                if (set(leave ? on : off) != AZI_OK) return 2;
                if (device) fake::fail_in = k;
                else new_in = k;
                int rc = AZI_OK;
                try {
                    rc = set(leave ? off : on);
                } catch (const std::exception&) {
                    std::printf("thrown out of the call\n");
                    return 1;
                }
                const bool over = device ? fake::fail_in >= 0 : new_in.load() >= 0;
                fake::fail_in = -1;
                new_in = -1;
                failed += rc != AZI_OK;
                for (int raw = 0; raw < (kind < 2 ? 2 : 1); ++raw)
                    if (const char* what = pass(raw)) {
                        std::printf("%s: %s, %s allocation %ld (status %d)\n", what,
                                    leave ? "leaving" : "entering", device ? "device" : "host", k, rc);
                        return 1;
                    }
                if (over) break;
            }
        }
    for (long k = 0; kind == 0; k += 37) {  // an upload: the encoder beside the copies
        new_in = k;
        int rc = AZI_OK;
        try {
            rc = azi_plan_upload(p, 0);
        } catch (const std::exception&) {
            std::printf("thrown out of the upload\n");
            return 1;
        }
        const bool over = new_in.exchange(-1) >= 0;
        if (rc != AZI_OK && rc != AZI_ENOMEM) return 2;
        if (azi_plan_upload(p, 0) != AZI_OK || pass(true)) {
            std::printf("not uploaded again after host allocation %ld\n", k);
            return 1;
        }
        if (over) break;
    }
    azi_batch_destroy(b);
    azi_plan_destroy(p);
    std::free(image);
    if (fake::live != 0) {
        std::printf("%lld bytes left\n", (long long)fake::live);
        return 1;
    }
    std::printf("ok, %d calls failed\n", failed);
    return 0;
}
