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
//   bf16, up to 128 vectors: 1000 x 300 16.8 / 15.4 and 12.1 / 11.2, 40000 x 100 212 / 71 and 134 / 47, 520 x 600 13.3 / 12.6 and 11.6 / 11.2, 64 x 600 12.0 / 12.5 and 10.9 / 11.2, 16384 x 1024 90 / 33 and 62 / 24;
//   up to 256: 1024 x 2048 14.4 / 13.3 and 12.0 / 11.1, 520 x 1100 13.1 / 13.5 and 11.3 / 11.0, 16384 x 2048 78 / 45 and 59 / 32;
//   up to 512: 2048 x 3000 23.3 / 21.2 and 17.1 / 16.2, 1024 x 3000 17.1 / 16.9 and 13.0 / 13.2, 16384 x 4096 97 / 70 and 72 / 53;
//   up to 1024: 4096 x 6000 49.6 / 42.2 and 36.9 / 31.7, 2048 x 6000 29.4 / 29.8 and 22.6 / 22.8, 16384 x 8192 139 / 120 and 103 / 93;
//   fp32, up to 256: 2048 x 600 16.9 / 16.4 and 14.5 / 12.1, 1024 x 600 13.3 / 14.2 and 11.9 / 11.6, 16384 x 1024 65 / 35 and 52 / 29;
//   up to 512: 4096 x 2048 25.5 / 23.7 and 21.5 / 18.8, 2048 x 2048 17.6 / 18.1 and 15.0 / 14.2, 16384 x 2048 75 / 55 and 61 / 49;
//   beyond that 128 lanes lose (4096 x 4096 31.2 / 37.2 and 27.8 / 28.9: the rows of twelve workgroups fill the LDS).
// Quantify-only: the same lines, but above 512 vectors from 32 rows per compute unit on (up to 256 vectors: 4096 x 1024 15.7 / 10.5, 2048 x 2048
// 10.5 / 10.2, 16384 x 2048 48 / 28; up to 512: 2048 x 4096 11.8 / 11.2, 4096 x 3000 20.2 / 17.4, 8192 x 4096 31.1 / 24.7, 16384 x 4096 59 / 40;
// 16384 x 8192 84 / 71; fp32 4096 x 2048 15.3 / 13.5).
bool short_rows_fit(Mode mode, int dtype, int vecs, int64_t rows)
{
    if (vecs > (dtype == 0 ? 512 : 1024)) return false;
    const int64_t units = compute_units();
    if (mode == Mode::Quantify && dtype != 0 && vecs > 512) return rows > 32 * units;
    if (dtype != 0) return vecs <= 128 ? rows > 2 * units : vecs <= 256 ? rows > 3 * units : vecs <= 512 ? rows > 6 * units : rows > 10 * units;
    return vecs <= 256 ? rows > 6 * units : rows > 12 * units;
}

hipError_t launch_short_rows(int dtype, Mode mode, const RowArgs& a, StreamLaunch& s)
{
    return dtype == 0 ? launch_short_rows_typed<float>(mode, (a.V + 3) / 4, a, s) : launch_short_rows_typed<bf16_t>(mode, (a.V + 7) / 8, a, s);
}

}  // namespace ciar
