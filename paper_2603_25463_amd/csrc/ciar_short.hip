// The streaming kernel's instances for short rows, one wave to a row or two (next_by_lds in
// ciar_stream.h).
#include "ciar_stream.h"

namespace ciar {
namespace {

template <typename T, int THREADS, int NVEC>
hipError_t launch_short_tile(Mode mode, const RowArgs& a, StreamLaunch& s)
{
    if (mode == Mode::Quantify) return launch_stream_kernel<T, THREADS, NVEC, true, false, false>(a, s);
    return mode == Mode::Verify ? launch_stream_kernel<T, THREADS, NVEC, false, true, false>(a, s)
                                : launch_stream_kernel<T, THREADS, NVEC, true, true, false>(a, s);
}
// vecs: 16-byte vectors per row
template <typename T>
hipError_t launch_short_rows_typed(Mode mode, int vecs, const RowArgs& a, StreamLaunch& s)
{
    if (vecs <= 64 * 2) return launch_short_tile<T, 64, 2>(mode, a, s);
    if (vecs <= 64 * 4) return launch_short_tile<T, 64, 4>(mode, a, s);
    if (vecs <= 64 * 8) return launch_short_tile<T, 64, 8>(mode, a, s);
    if constexpr (sizeof(T) == 2) {
        if (vecs <= 128 * 8) return launch_short_tile<T, 128, 8>(mode, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// How many rows it takes to pay, by the row's vectors (a call of few rows waits for one row's chain of instructions, and more
// lanes make it shorter; us, 256 lanes to a row / these, fused and verify-only):
//   bf16, up to 128 vectors: 1000 x 300 16.8 / 15.4 and 12.1 / 11.2, 40000 x 100 212 / 71 and 134 / 47, 530 x 1000 12.8 / 11.7, 64 x 600 12.0 / 12.5 and 10.9 / 11.2, 16384 x 1024 90 / 33 and 62 / 24;
//   up to 256: 1000 x 1672 14.1 / 13.4, 1150 x 1672 14.9 / 15.6, 1330 x 1500 15.9 / 15.4, 1282 x 1672 12.3 / 11.7 verified, 520 x 1100 13.1 / 13.5 and 11.3 / 11.0, 16384 x 2048 78 / 45 and 59 / 32;
//   up to 512: 1700 x 4096 18.0 / 18.5, 1900 x 4096 19.7 / 18.7, 2300 x 4096 21.3 / 22.2, 2300 x 2600 23.3 / 24.4, 2900 x 4096 24.7 / 24.1, verified 1700 x 3500 15.5 / 15.7,
//     1900 16.7 / 16.3, 2300 17.8 / 18.5, 2900 20.6 / 19.7, 16384 x 4096 97 / 70 and 72 / 53;
//   up to 1024: 2700 x 7000 35.9 / 36.5, 2900 x 5000 37.7 / 35.1, 2900 x 7500 39.5 / 37.6, 3300 x 8192 34.4 / 35.1, 3570 x 8192 36.0 / 37.2, 3900 x 8192 40.0 / 38.0, 2600 x 8192 24.0 / 23.0 verified, 16384 x 8192 139 / 120 and 103 / 93;
//   fp32, up to 256: 1700 x 800 15.0 / 15.4, 1900 x 800 16.3 / 15.5, 2300 x 800 16.9 / 17.3, 2600 x 600 18.4 / 17.5, rows of 1024 tokens 2060 15.9 / 14.9 and 2300 16.3 / 15.2, 1600 x 1024 12.6 / 10.9 verified, 16384 x 1024 65 / 35 and 52 / 29;
//   up to 512: 3100 x 1300 23.6 / 22.3, 3500 x 2048 22.6 / 23.2, 3900 x 2048 24.2 / 24.1 to 23.9 / 22.7, 3100 x 2048 18.6 / 17.0 verified, 16384 x 2048 75 / 55 and 61 / 49;
//   beyond that 128 lanes lose (4096 x 4096 31.2 / 37.2 and 27.8 / 28.9: the rows of twelve workgroups fill the LDS).
// (The gaps: four rows per compute unit are one to a SIMD, eight two.  The first rows beyond add a wave to a few SIMDs, and the call waits
// for those, where the four waves of the other tiles share them out.)
// Quantify-only: up to 512 vectors 700 x 1000 9.5 / 9.7, 2100 x 600 10.5 / 9.5, 1100 x 1672 9.6 / 9.8, 2060 x 1672 10.7 / 10.4, 2300 x 4096 12.1 / 13.1, 2900 x 2600 16.3 / 15.0, 16384 x 4096 59 / 40;
// above that from 32 rows per compute unit on (8500 x 8192 46.4 / 43.0); fp32 1600 x 800 9.5 / 9.8, 2300 x 800 10.0 / 9.7, 3200 x 2048 13.0 / 12.1.
bool short_rows_fit(Mode mode, int dtype, const RowArgs& a, int units)
{
    const int vecs = dtype == 0 ? (a.V + 3) / 4 : (a.V + 7) / 8;
    if (vecs > (dtype == 0 ? 512 : 1024)) return false;
    const double n = (double)a.N / units;
    const bool fused = mode == Mode::Fused, quantify = mode == Mode::Quantify;
    if (dtype != 0) {
        if (vecs <= 128) return n > (quantify ? 6 : 2);
        if (vecs <= 256) return quantify ? n > 6 : n > 3 && (!fused || n <= 4 || n > 5.25);
        if (vecs <= 512) return (n > 7 && n <= 8) || n > 11;
        return n > (quantify ? 32 : !fused ? 10 : a.V < 8192 ? 11 : 14);
    }
    if (vecs <= 256) return quantify ? n > 8 : n > (fused ? 7 : 6) && (!fused || n <= 8 || n > 9.5 || a.V == 1024);
    return n > (fused && vecs > 384 ? 15 : 12);
}

hipError_t launch_short_rows(int dtype, Mode mode, const RowArgs& a, StreamLaunch& s)
{
    return dtype == 0 ? launch_short_rows_typed<float>(mode, (a.V + 3) / 4, a, s) : launch_short_rows_typed<bf16_t>(mode, (a.V + 7) / 8, a, s);
}

}  // namespace ciar
