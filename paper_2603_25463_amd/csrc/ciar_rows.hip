// The streaming kernel's instances for large bf16 rows with a verifier row (next_by_lds in ciar_stream.h).
#include "ciar_stream.h"

namespace ciar {
namespace {

template <int THREADS, int NVEC>
hipError_t launch_tile(Mode mode, const RowArgs& a, StreamLaunch& s)
{
    return mode == Mode::Verify ? launch_stream_kernel<bf16_t, THREADS, NVEC, false, true, false>(a, s)
                                : launch_stream_kernel<bf16_t, THREADS, NVEC, true, true, false>(a, s);
}
template <int THREADS>
hipError_t launch_lanes(Mode mode, int vecs, const RowArgs& a, StreamLaunch& s)
{
    return vecs <= THREADS * 12 ? launch_tile<THREADS, 12>(mode, a, s) : launch_tile<THREADS, 16>(mode, a, s);
}

}  // namespace

// As many lanes as the row takes at sixteen vectors each.
hipError_t launch_both_rows(Mode mode, const RowArgs& a, StreamLaunch& s)
{
    const int vecs = (a.V + Elt<bf16_t>::kPerVec - 1) / Elt<bf16_t>::kPerVec;   // 16-byte vectors per row
    if (vecs <= 128 * 16) return launch_lanes<128>(mode, vecs, a, s);
    if (vecs <= 256 * 16) return launch_lanes<256>(mode, vecs, a, s);
    if (vecs <= 512 * 16) return launch_lanes<512>(mode, vecs, a, s);
    return hipErrorInvalidValue;
}

}  // namespace ciar
