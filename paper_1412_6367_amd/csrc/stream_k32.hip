// Float32 storage, Kahan float sums.
#include "stream_forward.h"

namespace azi {
hipError_t launch_stream_k32(const StreamLaunch& a, hipStream_t s) {
    return stream_forward<float, AccWK32>(a, s);
}
}  // namespace azi
