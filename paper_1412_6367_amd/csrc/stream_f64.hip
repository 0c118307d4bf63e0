// Float64 storage, float64 sums.
#include "stream_forward.h"

namespace azi {
hipError_t launch_stream_f64(const StreamLaunch& a, hipStream_t s) {
    return stream_forward<double, AccWF64>(a, s);
}
}  // namespace azi
