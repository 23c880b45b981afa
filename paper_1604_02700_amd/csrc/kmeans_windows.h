// The windowed solver of the 1-D k-means programme (kmeans_windows.hip).
#pragma once

#include "common.h"

namespace gpic {

// The optimal segment starts first[0 .. ke] of the n sorted values sv (run
// flags, prefix sums SS of the values less *mean, as run_kmeans1d lays them
// out) with scratch phi (n float64), psum (a float64 per 2,048 values) and ws.
// *solved = 0: not solved (the caller runs the full programme); first is
// then unspecified.  Synchronises the stream.
hipError_t kmeans_windows(const double *sv, const int32_t *run, const double2 *SS, int64_t n,
                          const double *mean, int32_t ke, double *phi, double *psum, void *ws,
                          size_t ws_bytes, int64_t *first, hipStream_t s, int *solved);

} // namespace gpic
