// The streaming kernel's instances (ciar_stream.h) and which call takes which; those for large bf16 rows are ciar_rows.hip's.
#include "ciar_stream.h"

namespace ciar {
namespace {

template <typename T, int THREADS, int NVEC>
hipError_t launch_stream_cfg(Mode mode, const RowArgs& a, StreamLaunch& s)
{
    const bool rad = a.radius != nullptr;
    if (mode == Mode::Quantify && rad) {
        // (more than 64 tokens: radius_kernel's)
        if constexpr (NVEC == 1) {
            if (!radius_quantify_fits(a))
                return wide_radius(a) ? launch_stream_kernel<T, THREADS, 1, true, false, true, true>(a, s)
                                      : launch_stream_kernel<T, THREADS, 1, true, false, true>(a, s);
        }
        return hipErrorInvalidValue;
    }
    if (mode != Mode::Verify && wide_radius(a)) {
        // radii at which the widths crowd against 1: the variants that also accumulate their complements
        if (mode == Mode::Quantify) return launch_stream_kernel<T, THREADS, NVEC, true, false, false, true>(a, s);
        return rad ? launch_stream_kernel<T, THREADS, NVEC, true, true, true, true>(a, s)
                   : launch_stream_kernel<T, THREADS, NVEC, true, true, false, true>(a, s);
    }
    if (mode == Mode::Quantify) return launch_stream_kernel<T, THREADS, NVEC, true, false, false>(a, s);
    if (mode == Mode::Fused && rad) return launch_stream_kernel<T, THREADS, NVEC, true, true, true>(a, s);
    if constexpr (sizeof(T) == 2 && NVEC == 8) return hipErrorInvalidValue;    // (launch_both_rows')
    else return mode == Mode::Verify ? launch_stream_kernel<T, THREADS, NVEC, false, true, false>(a, s)
                                     : launch_stream_kernel<T, THREADS, NVEC, true, true, false>(a, s);
}

template <typename T>
hipError_t launch_stream_typed(Mode mode, const RowArgs& a, StreamLaunch& s)
{
    const int vecs = (a.V + Elt<T>::kPerVec - 1) / Elt<T>::kPerVec;   // 16-byte vectors per row
    if (mode == Mode::Verify || (!a.radius && !wide_radius(a) && (mode == Mode::Fused || s.finish_rows))) {
        if (sizeof(T) == 2 && vecs > 1024 && mode != Mode::Quantify) return launch_both_rows(mode, a, s);
        constexpr int kDtype = sizeof(T) == 4 ? 0 : 1;
        if (a.V > kTinyVocab && short_rows_fit(mode, kDtype, a, s.units)) return launch_short_rows(kDtype, mode, a, s);
    }
    if (vecs <= 256 * 1)  return launch_stream_cfg<T, 256, 1>(mode, a, s);
    if (vecs <= 256 * 2)  return launch_stream_cfg<T, 256, 2>(mode, a, s);
    if (vecs <= 256 * 4)  return launch_stream_cfg<T, 256, 4>(mode, a, s);
    if (vecs <= 256 * 8)  return launch_stream_cfg<T, 256, 8>(mode, a, s);
    if (vecs <= 256 * 16) {
        // Few rows: eight waves on a row keep the last rows of the launch short and the grid even; with many
        // rows the four-wave tile has less exchange overhead (measured).  For bf16 the four-wave tile would
        // hold 128 floats per lane and spill at four waves per SIMD: eight waves always.  The same goes for fp32 launches with a
        // verifier row, which keep both rows in the registers until the accept test is decided.
        if constexpr (sizeof(T) == 2) {
            return launch_stream_cfg<T, 512, 8>(mode, a, s);
        } else {
            if (mode != Mode::Quantify || a.N < 12 * (int64_t)s.units) return launch_stream_cfg<T, 512, 8>(mode, a, s);
            return wide_radius(a) ? launch_stream_kernel<T, 256, 16, true, false, false, true>(a, s)
                                  : launch_stream_kernel<T, 256, 16, true, false, false>(a, s);
        }
    }
    if (vecs <= 1024 * 8) return launch_stream_cfg<T, 1024, 8>(mode, a, s);
    return hipErrorInvalidValue;
}

}  // namespace

int max_vocab(int dtype) { return dtype == 0 ? 1024 * 8 * 4 : 1024 * 8 * 8; }

StreamPlan plan_stream(Mode mode, int dtype, const RowArgs& args, bool finish_rows)
{
    StreamLaunch L{false, finish_rows, nullptr, compute_units(), {0u, 0, false, 1, false, false, false}, nullptr, nullptr};
    if (args.N > 0) {
        if (dtype == 0) (void)launch_stream_typed<float>(mode, args, L);
        else (void)launch_stream_typed<bf16_t>(mode, args, L);
    }
    return L.plan;
}

hipError_t launch_stream(Mode mode, int dtype, const RowArgs& args, bool finish_rows, hipStream_t stream,
                         hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (args.N <= 0) return hipSuccess;
    StreamLaunch L{true, finish_rows, stream, compute_units(), {0u, 0, false, 1, false, false, false}, ev_start, ev_stop};
    return dtype == 0 ? launch_stream_typed<float>(mode, args, L)
                      : launch_stream_typed<bf16_t>(mode, args, L);
}

}  // namespace ciar
