// The windowed solver of the 1-D k-means programme (kmeans_windows.hip).
#pragma once

#include "common.h"

namespace gpic {

// The gaps between neighbouring sorted values, by size: gap / range in
// [2^-b, 2^(1-b)) goes to b (the last takes the smaller ones); their number,
// sum (in range / 2^60) and sum of square roots (in sqrt(range) / 2^40), in
// whole numbers, so that the order of the additions does not matter.
constexpr int kGapClasses = 64;
struct GapStats {
    double range;                        // largest value less the smallest
    double s2;                           // sum of squares about the mean
    unsigned long long count[kGapClasses], sum[kGapClasses], root[kGapClasses];
};

// Whether kmeans_windows may solve n values with up to k clusters.
bool kmeans_windows_apply(int64_t n, int64_t k);

// gs (device, its counts and sums zero) from the sorted values sv and the
// prefix sums SS of the values less their mean.
hipError_t launch_gap_stats(const double *sv, const double2 *SS, int64_t n, GapStats *gs,
                            hipStream_t s);

// The optimal segment starts first[0 .. ke] of the n sorted values sv (run
// flags, prefix sums SS of the values less *mean, as run_kmeans1d lays them
// out) with scratch phi (n float64), psum (a float64 per 2,048 values) and ws;
// gs: launch_gap_stats's, on the host.  *solved = 0: not solved (the caller
// runs the full programme); first is then unspecified.  Synchronises the
// stream.
hipError_t kmeans_windows(const double *sv, const int32_t *run, const double2 *SS, int64_t n,
                          const double *mean, int32_t ke, const GapStats &gs, double *phi,
                          double *psum, void *ws, size_t ws_bytes, int64_t *first,
                          hipStream_t s, int *solved);

} // namespace gpic
