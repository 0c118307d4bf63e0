// A device without a GPU, for host-only tests of the C ABI's own logic: the
// runtime's memory calls on host memory, with a countdown after which
// allocations fail, and the library's kernel launches noted down instead of run.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../paper_1412_6367_amd/csrc/internal.h"
#include "../../paper_1412_6367_amd/csrc/kernels.h"
#include "../../paper_1412_6367_amd/csrc/stream.h"

namespace fake {
extern std::vector<std::string> calls;  // launches, in order
extern azi::StreamLaunch stream;        // arguments of the last launch_stream
extern azi::BandLaunch band;            // arguments of the last launch_band
extern const void *dark, *norm;         // arrays of the last launch_correct
extern int64_t fail_in;                 // allocations until one fails (negative: none does)
extern int encoded;                     // images given to build_stream
extern int64_t uploaded;                // bytes copied from the host
extern int64_t live;                    // bytes allocated
bool held(const void* p);               // p lies in an allocation
inline bool called(const char* name) {
    for (const std::string& c : calls)
        if (c == name) return true;
    return false;
}
}  // namespace fake
