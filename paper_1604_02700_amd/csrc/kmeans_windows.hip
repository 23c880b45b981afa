// Exact 1-D k-means for gfx950, the layers of the dynamic programme solved
// inside windows of split points that are proved to hold the optimum.
//
// The k - 1 split points ("cuts") p_1 < .. < p_{k-1} of the sorted values
// minimise the sum of the segment costs C(p_{c-1}, p_c) (p_0 = 0, p_k = n).
// The full programme (kmeans.hip) computes every row of every layer; only
// the few rows near the optimal cuts matter.  Here a grid of candidate
// positions gives, per layer, a lower bound F on the cost up to a cut, a
// lower bound B on the cost from it on, and the cost U of the best path
// that cuts at grid points only.  A grid cell where F + B exceeds U (plus a
// bound on the float64 rounding) holds no cut of an optimal path; the cells
// that some layer keeps become the next round's windows, cut into cells
// again, until every position of the windows is a grid point.  The programme
// over those is the exact one: same candidates around the optimum, same
// expressions, same order of additions and the leftmost minimum, so its cuts
// are those that the rows of the full programme lead to, but for ties to the
// rounding of the costs (n = 2M, k = 12 in clusters 1e-3 wide: one cut a
// few values away, the total 7e-11 smaller).
//
// The bounds.  Let a cell hold s values spanning w (its first to its last).
// Moving a cut from inside the cell to one of its ends, with the
// neighbouring cuts l and r held, lowers the cost by at most s w D, D the
// distance from the cell to the mean of the values up to r (or back to l):
// for fixed centres m1 < m2 the cost is convex in the cut (the values
// ascend) and dips below both ends by at most (m2 - m1) s w / 2, only if the
// midpoint of the centres lies in the cell, and then m2 - m1 is twice the
// distance from the midpoint to either centre; optimal centres for the
// inside cut are no worse than fixed ones at the ends.  So a path is
// matched, cut by cut, by a path over grid points that costs at most the
// sum of those terms more (forward from the left, backward from the right).
// Cuts that share a cell are matched by dropping the cell's values: from
// the cell's left end at the first of them to its right end at the last, at
// no cost.  Cells take equal shares of the sum of the square roots of the
// gaps between neighbouring values, which keeps s w even where the values
// are dense and sparse by turns, and puts a grid point into every wide gap;
// a gap counts for no more than about a cell, so that a few wide ones do not
// take the cells of all the values.  The terms shrink with the square of the
// cell, so a few rounds suffice for the embeddings met here; where they do
// not (values equal to rounding, clusters too many for the grid), the caller
// runs the full programme.
#include "common.h"
#include "kmeans_dev.h"
#include "kmeans_windows.h"

namespace gpic {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
// Where the windows are tried, measured against the full programme in the
// same run, geometric means: on embeddings of the clustering itself (kNN graphs
// and fused operators, 2 to 16 dimensions), and on 13 shapes of values (uniform,
// normal, heavy tails, integers, as many and fewer clusters than k from 1e-9 to
// 1e-3 wide and of widely different widths), 2 to 5 draws each.
//   Below 8,192 values the full programme is two or three levels a layer and
// the scratch holds few cells.  Up to 2^18 it has three levels, about 75 us a
// layer; embeddings with k = 7, 12, 24: n = 8,192: 1.20, 1.38, 1.48 times as
// fast; 20,000: 1.19, 1.42, 1.40; 60,000: 1.12, 1.27, 1.56 (the slowest 0.94);
// 125,000: 1.23, 1.45, 1.64.  The shapes there: k = 7: 1.14 at 8,192, 1.11 at
// 20,000, 1.0 at 60,000, with clusters of widely different widths down to 0.8;
// k = 10: 1.25, 1.23, 1.15; k = 6: 1.07, 1.07.
//   From 2^18 values: n = 270,000, k = 3, 7, 24: 1.05, 1.54, 2.4; n = 600,000, k =
// 5, 40: 1.5, 3.1; n = 2M, k = 3, 5, 50: 1.29, 1.76, 4.5 (19.2 ms without); one or
// two in a hundred, most of a cost near the rounding, down to 0.73.
// Cells: a first round of 1,024 costs 0.1-0.3 ms more, of 256 leaves wider
// windows; rows of 4 x kMaxPer instead of 8 x lose from k = 50 on.  Splits by 4,
// 8, 16 and as many as fit: the clustering's embeddings at n = 2M, k = 50: 3.23,
// 3.45, 3.67, 3.67 ms; by 4 some values no longer shrink (n = 1,050,000, k = 70).
constexpr int64_t kFromN = 8192, kLargeN = (int64_t)1 << 17, kHugeN = (int64_t)1 << 18;
constexpr int kFew = 7, kFewHuge = 3;    // fewest clusters below, from kHugeN on
// Costs of spare cuts up to this many times the bound on the rounding leave
// windows too wide (clusters of 1e-9 to 1e-12 of the range, fewer than k: a
// quarter of the full programme's time lost in two rounds that keep everything;
// with clusters of 1e-4 they are 2e5 times and more).
constexpr double kRoundingCost = 1e5;
constexpr int kFirst = 512;              // cells of the first round
constexpr int kMaxPer = 1024;            // cells per layer of a window later
constexpr int kMerged = 8, kMaxMerged = 32;   // a layer's range: this many times as many
constexpr int kMaxClusters = 512;
constexpr int kMaxSplit = 8;             // cells of one that is kept, beside a window's share
constexpr int kMaxRounds = 5;
constexpr int kMaxPoints = 1 << 17;      // of a grid

// What a round leaves for the host.
struct RoundCtl {
    int32_t nseg;                        // windows
    int32_t total;                       // grid points of the next round
    int32_t rows;                        // most grid points of a layer's range
    int32_t exact;                       // every position of the windows is a grid point
    int32_t fail;                        // a layer lost every cell, or no room for smaller ones
    int32_t span;                        // positions in all windows
    double thr;                          // no path above this cost is optimal
};

// Arrays of one solve.  Grid points are numbered window after window;
// layer c's values are kept for its own range wa[c] .. wb[c] of them, in
// rows of `stride`.
struct View {
    const double *sv;                    // sorted values
    const int32_t *run;                  // 1 where a run of equal values starts
    const double2 *SS;                   // prefix sums (S1, S2)
    int64_t n;
    int32_t ke, stride, per, points;     // points: room for grid points
    double cap;                          // most that one gap adds to phi
    int32_t *pos;                        // grid point -> position
    double2 *S;                          // SS at the position
    const double *mean;                  // of the values
    double *phi;                         // running sum of the gaps' square roots
    double *psum;                        // its tile sums
    double *xl, *xr;                     // (centred) first value of the cell to the left, last of the one to the right
    double2 *Ln, *Rn;                    // (S1, position) at the left and right neighbour
    double *sw;                          // largest s w of the cells beside it
    double *pen;                         // rounding term of the cell to its right, < 0: no cut inside
    double *F, *U, *B, *G, *Vf, *Vb;     // per layer; G: B less the forward term of its own cut
    int32_t *arg;
    int32_t *cellseg;                    // 1: first grid point of its window, 2: last
    int32_t *qmin, *rmax;                // furthest grid point that one segment can reach
    int32_t *keepp, *keepc;              // grid points, cells to their right, that some layer keeps
    int32_t *lo, *hi;                    // first and last kept position of a layer
    int32_t *wa, *wb;                    // its first and last grid point
    int32_t *segP, *segQ, *base;         // positions and first grid point of a window
    int32_t *kpre, *lpre, *mpre;         // of the windows before: kept cells, positions, windows with cells
    RoundCtl *ctl;
};

__device__ __forceinline__ double eta_of(const View &V)
{
    // how far a stored prefix difference may be from its value: 2^-45 of the
    // largest |S1|, itself at most sqrt(n S2)
    return 0x1p-45 * sqrt((double)V.n * V.SS[V.n].y);
}

// The start of the run that position p lies in.
__device__ __forceinline__ int32_t snap(const View &V, int32_t p)
{
    if (p <= 0 || V.run[p])
        return p < 0 ? 0 : p;
    const double x = V.sv[p];
    int32_t a = 0, b = p;                // first position with sv >= x
    while (a < b) {
        const int32_t m = a + (b - a) / 2;
        if (V.sv[m] < x)
            a = m + 1;
        else
            b = m;
    }
    return a;
}

// phi[i] = sum over j <= i of sqrt(x_j - x_{j-1}), at most cap each: tile sums, their scan by
// one workgroup, the tiles again from their offsets.  Any non-decreasing
// phi gives valid cells; its rounding does not matter.
__device__ __forceinline__ double gap_root(const View &V, int64_t i)
{
    return (i > 0 && i < V.n) ? fmin(sqrt(fmax(V.sv[i] - V.sv[i - 1], 0.0)), V.cap) : 0.0;
}

constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;

// A workgroup's gaps by class in LDS, then an atomic per class that it met.
__global__ __launch_bounds__(kThreads) void gap_stats_kernel(const double *__restrict__ sv,
                                                             const double2 *__restrict__ SS,
                                                             int64_t n, GapStats *__restrict__ gs)
{
    __shared__ unsigned long long sum[kGapClasses], root[kGapClasses];
    __shared__ unsigned int count[kGapClasses];
    if (threadIdx.x < kGapClasses) {
        sum[threadIdx.x] = 0ull;
        root[threadIdx.x] = 0ull;
        count[threadIdx.x] = 0u;
    }
    __syncthreads();
    const double R = sv[n - 1] - sv[0];
    for (int64_t i = 1 + (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const double q = (sv[i] - sv[i - 1]) / R;
        if (!(q > 0.0 && q <= 1.0))
            continue;                                // equal values, or no finite range
        const int e = -ilogb(q);
        const int b = e < kGapClasses ? e : kGapClasses - 1;
        atomicAdd(&count[b], 1u);
        atomicAdd(&sum[b], (unsigned long long)(q * 0x1p60));
        atomicAdd(&root[b], (unsigned long long)(sqrt(q) * 0x1p40));
    }
    __syncthreads();
    if (threadIdx.x < kGapClasses && count[threadIdx.x] != 0u) {
        atomicAdd(&gs->count[threadIdx.x], (unsigned long long)count[threadIdx.x]);
        atomicAdd(&gs->sum[threadIdx.x], sum[threadIdx.x]);
        atomicAdd(&gs->root[threadIdx.x], root[threadIdx.x]);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        gs->range = R;
        gs->s2 = SS[n].y;
    }
}

__global__ __launch_bounds__(kThreads) void phi_sums_kernel(View V)
{
    __shared__ double red[kWaves];
    const int64_t b = (int64_t)blockIdx.x * kTile;
    double t = 0.0;
    for (int u = 0; u < kItems; ++u)
        t += gap_root(V, b + u * kThreads + threadIdx.x);
    t = block_sum<kThreads>(t, red);
    if (threadIdx.x == 0)
        V.psum[blockIdx.x] = t;
}

// Exclusive scan over the workgroup of one value per thread (NT threads).
template <int NT>
__device__ __forceinline__ double block_scan_excl(double x, double *a)
{
    const int t = threadIdx.x;
    a[t] = x;
    __syncthreads();
    double y = x;
    for (int off = 1; off < NT; off <<= 1) {
        const double o = t >= off ? a[t - off] : 0.0;
        __syncthreads();
        y += o;
        a[t] = y;
        __syncthreads();
    }
    return t > 0 ? a[t - 1] : 0.0;
}

// The scan of the tile sums, and the first round's single window over every
// possible cut, for every layer.
__global__ __launch_bounds__(1024) void first_window_kernel(View V, int64_t tiles, int32_t cells)
{
    __shared__ double a[1024];
    const int64_t per = (tiles + 1023) / 1024;
    const int64_t b0 = (int64_t)threadIdx.x * per;
    double t = 0.0;
    for (int64_t b = b0; b < b0 + per && b < tiles; ++b)
        t += V.psum[b];
    double o = block_scan_excl<1024>(t, a);
    for (int64_t b = b0; b < b0 + per && b < tiles; ++b) {
        const double x = V.psum[b];
        V.psum[b] = o;
        o += x;
    }
    for (int c = threadIdx.x; c < V.ke; c += 1024) {
        V.lo[c] = 0;
        V.hi[c] = (int32_t)(V.n - 1);
    }
    if (threadIdx.x == 0) {
        V.segP[0] = 1;
        V.segQ[0] = (int32_t)(V.n - 1);
        V.base[0] = 0;
        V.base[1] = cells + 1;
        V.ctl->nseg = 1;
        V.ctl->total = cells + 1;
        V.ctl->fail = 0;
        V.ctl->thr = INFINITY;
    }
}

__global__ __launch_bounds__(kThreads) void phi_kernel(View V)
{
    __shared__ double a[kThreads];
    const int64_t b = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    double g[kItems];
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
        g[u] = gap_root(V, b + u);
        t += g[u];
    }
    double o = V.psum[blockIdx.x] + block_scan_excl<kThreads>(t, a);
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
        o += g[u];
        if (b + u < V.n)
            V.phi[b + u] = o;
    }
}

// Grid points: window z's positions P .. Q cut into cells of equal shares
// of phi (every position where there are no more than the cells), each
// moved to the start of its run of equal values (cuts lie there only).
__global__ __launch_bounds__(kThreads) void positions_kernel(View V)
{
    const int32_t i = (int32_t)(blockIdx.x * kThreads + threadIdx.x);
    if (i >= V.ctl->total)
        return;
    int a = 0, b = V.ctl->nseg - 1;      // last window with base <= i
    while (a < b) {
        const int m = (a + b + 1) / 2;
        if (V.base[m] <= i)
            a = m;
        else
            b = m - 1;
    }
    const int32_t P = V.segP[a], Q = V.segQ[a], t = i - V.base[a];
    const int32_t cells = V.base[a + 1] - V.base[a] - 1;
    int32_t p;
    if (t == 0 || t == cells || cells == Q - P) {
        p = (t == cells) ? Q : P + t;
    } else {
        const double lo = V.phi[P], hi = V.phi[Q];
        const double want = lo + (hi - lo) * ((double)t / (double)cells);
        int32_t x = P, y = Q;            // first position with phi >= want
        while (x < y) {
            const int32_t m = x + (y - x) / 2;
            if (V.phi[m] < want)
                x = m + 1;
            else
                y = m;
        }
        p = x;
    }
    V.pos[i] = snap(V, p);
    V.cellseg[i] = (t == 0 ? 1 : 0) | (t == cells ? 2 : 0);
}

// What the layers need to know of a grid point and the cells beside it, how
// far a segment from or to it can reach (a segment between cuts near the
// grid points q < r costs at least C(q + 1, r - 1), which falls as q grows
// and rises with r), and the layers' ranges.
__global__ __launch_bounds__(kThreads) void grid_kernel(View V)
{
    const int32_t i = (int32_t)(blockIdx.x * kThreads + threadIdx.x);
    const int32_t total = V.ctl->total;
    if (i >= 1 && i < V.ke) {
        int32_t x = 0, y = total - 1;    // last with pos <= lo
        while (x < y) {
            const int32_t m = x + (y - x + 1) / 2;
            if (V.pos[m] <= V.lo[i])
                x = m;
            else
                y = m - 1;
        }
        V.wa[i] = x;
        y = total - 1;                   // first with pos >= hi
        while (x < y) {
            const int32_t m = x + (y - x) / 2;
            if (V.pos[m] < V.hi[i])
                x = m + 1;
            else
                y = m;
        }
        V.wb[i] = x;
    }
    if (i >= total)
        return;
    V.keepp[i] = 0;
    V.keepc[i] = 0;
    const double thr = V.ctl->thr;
    auto over = [&](int32_t q, int32_t r) {      // no segment from near q to near r
        if (q + 1 >= r - 1)
            return false;
        const int32_t pq = V.pos[q + 1], pr = V.pos[r - 1];
        return pq < pr && seg_cost(V.SS[pq], V.SS[pr], pq, (int64_t)pr - 1) > thr;
    };
    {
        int32_t x = 0, y = i;            // first q that reaches i
        while (x < y) {
            const int32_t m = x + (y - x) / 2;
            if (over(m, i))
                x = m + 1;
            else
                y = m;
        }
        V.qmin[i] = x;
        x = i;
        y = total - 1;                   // last r that i reaches
        while (x < y) {
            const int32_t m = x + (y - x + 1) / 2;
            if (over(i, m))
                y = m - 1;
            else
                x = m;
        }
        V.rmax[i] = x;
    }
    const double eta = eta_of(V);
    const double R = V.sv[V.n - 1] - V.sv[0];
    const double mu = *V.mean;
    const int32_t e = V.cellseg[i];
    const int32_t p = V.pos[i];
    const int32_t l = (e & 1) ? p : V.pos[i - 1], r = (e & 2) ? p : V.pos[i + 1];
    const double xl = V.sv[l], xr = V.sv[r > 0 ? r - 1 : 0];
    double sw = 0.0, pen = -1.0;
    if (p > l) {
        const double w = V.sv[p - 1] - xl;
        sw = (w > 0.0) ? (double)(p - l) * (w + eta) : 0.0;
    }
    if (r > p) {
        const double w = xr - V.sv[p];
        if (w > 0.0) {
            sw = fmax(sw, (double)(r - p) * (w + eta));
            pen = 0x1p-44 * V.SS[V.n].y + 2.0 * (double)(r - p) * R * eta;
        }
    }
    V.S[i] = V.SS[p];
    V.Ln[i] = double2{V.SS[l].x, (double)l};
    V.Rn[i] = double2{V.SS[r].x, (double)r};
    V.xl[i] = xl - mu;
    V.xr[i] = xr - mu;
    V.sw[i] = sw;
    V.pen[i] = pen;
}

// Distance between x, an end of a cell, and the mean of the (centred) values
// between the positions in a and b: above, the mean less x, else x less the
// mean.  The callers pass the neighbouring grid points that give the extreme
// mean, and add kMeanSlack of the values' range: the reciprocal is good to
// 2^-18 and better, which the Newton step squares.
constexpr double kMeanSlack = 0x1p-35;
__device__ __forceinline__ double mean_dist(double2 a, double2 b, double x, bool above)
{
    const double m = b.y - a.y;
    double r = __builtin_amdgcn_rcp(m);
    r = fma(fma(-m, r, 1.0), r, r);
    const double q = (b.x - a.x) * r;
    return above ? q - x : x - q;
}

// Leftmost minimum over the wave of (value, index), the value alone where
// no index is wanted.
__device__ __forceinline__ double wave_min(double x)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
        x = fmin(x, __shfl_xor(x, o, kWave));
    return x;
}

// One layer of both directions (blockIdx.y: 0 forward, layer t; 1 backward,
// layer ke - t), a wave per grid point of the layer's window.  EXACT: every
// position is a grid point, the forward programme alone, with its argmins.
// A layer is 513 x 513 evaluations in the first round and mostly fewer
// later, except while its range is wide (up to 8,193 rows: 35 us); the
// launches, about 5 us each, are most of the rest.
template <bool EXACT>
__global__ __launch_bounds__(kThreads) void layer_kernel(View V, int t)
{
    const int lane = threadIdx.x % kWave;
    const bool back = !EXACT && blockIdx.y == 1;
    const int c = back ? V.ke - t : t;
    const int32_t a = V.wa[c], b = V.wb[c];
    const int32_t r = a + (int32_t)(blockIdx.x * kWaves + threadIdx.x / kWave);
    if (r > b)
        return;                                      // uniform per wave
    const int32_t p = V.pos[r];
    const double2 Sr = V.S[r];
    // of a distance: rounding of the values (eta) and of the means
    const double slack = EXACT ? 0.0 : eta_of(V) + kMeanSlack * (V.sv[V.n - 1] - V.sv[0]);
    const int64_t row = (int64_t)c * V.stride + (r - a);
    if (!back) {
        double f = INFINITY, u = INFINITY, vf = INFINITY;
        int64_t arg = INT64_MAX;
        if (c == 1) {
            u = (p > 0) ? seg_cost(V.SS[0], Sr, 0, (int64_t)p - 1) : INFINITY;
            f = (p > 0) ? u : 0.0;
        } else {
            const int32_t ap = V.wa[c - 1], bp = V.wb[c - 1], qm = V.qmin[r];
            const int64_t prow = (int64_t)(c - 1) * V.stride - ap;
            const int32_t qe = bp < r ? bp : r;
            const double xr = EXACT ? 0.0 : V.xr[r];
            const double2 Rr = EXACT ? double2{0.0, 0.0} : V.Rn[r];
            for (int32_t q = (ap > qm ? ap : qm) + lane; q <= qe; q += kWave) {
                const int32_t pq = V.pos[q];
                const bool some = pq < p;
                const double cost = some ? seg_cost(V.S[q], Sr, pq, (int64_t)p - 1) : 0.0;
                const double cu = some ? V.U[prow + q] + cost : INFINITY;
                if (cu < u) {
                    u = cu;
                    arg = q;
                }
                if (!EXACT) {
                    const double xl = V.xl[q];
                    const double2 Rq = V.Rn[q];
                    double D = xr - xl;
                    if (Rq.y < Rr.y)
                        D = fmin(D, mean_dist(Rq, Rr, xl, true));
                    D = fmax(D, 0.0) + slack;
                    f = fmin(f, V.F[prow + q] + cost - V.sw[q] * D);
                }
            }
            wave_argmin(u, arg);
            if (!EXACT) {
                f = wave_min(f);
                // cuts that share the cell to the left end at its right end
                if (r > a && r - 1 >= ap && r <= bp && V.pen[r - 1] >= 0.0) {
                    vf = fmin(V.F[prow + r - 1], V.Vf[prow + r - 1]) - V.pen[r - 1];
                    f = fmin(f, vf);
                }
            }
        }
        if (lane == 0) {
            V.U[row] = u;
            if (EXACT)
                V.arg[row] = (arg == INT64_MAX) ? -1 : (int32_t)arg;
            else {
                V.F[row] = f;
                if (r > a)
                    V.Vf[row - 1] = vf;              // by cell: r - 1
                if (r == b)
                    V.Vf[row] = INFINITY;
            }
        }
        return;
    }
    double f = INFINITY, g = INFINITY, vb = INFINITY;
    const double swq = V.sw[r], xl = V.xl[r];
    const double2 Lq = V.Ln[r], Rq = V.Rn[r];
    if (c == V.ke - 1) {
        const double D = fmax(V.sv[V.n - 1] - *V.mean - xl, 0.0) + slack;
        f = seg_cost(Sr, V.SS[V.n], p, V.n - 1);
        g = f - swq * D;
    } else {
        const int32_t an = V.wa[c + 1], bn = V.wb[c + 1], rm = V.rmax[r];
        const int64_t nrow = (int64_t)(c + 1) * V.stride - an;
        for (int32_t q = (an > r ? an : r) + lane; q <= (bn < rm ? bn : rm); q += kWave) {
            const int32_t pq = V.pos[q];
            const double cost = (p < pq) ? seg_cost(Sr, V.S[q], p, (int64_t)pq - 1) : 0.0;
            const double xr = V.xr[q];
            const double2 Ln = V.Ln[q], Rn = V.Rn[q];
            double Df = xr - xl, Db = Df;
            if (Rq.y < Rn.y)
                Df = fmin(Df, mean_dist(Rq, Rn, xl, true));
            if (Lq.y < Ln.y)
                Db = fmin(Db, mean_dist(Lq, Ln, xr, false));
            Df = fmax(Df, 0.0) + slack;
            Db = fmax(Db, 0.0) + slack;
            // the backward term of cut c + 1, and for G the forward one of
            // cut c, which the test of cut c needs
            const double y = V.B[nrow + q] + cost - V.sw[q] * Db;
            f = fmin(f, y);
            g = fmin(g, y - swq * Df);
        }
        f = wave_min(f);
        g = wave_min(g);
        if (r < b && r >= an && r + 1 <= bn && V.pen[r] >= 0.0) {
            vb = fmin(V.B[nrow + r + 1], V.Vb[nrow + r]) - V.pen[r];
            f = fmin(f, vb);
            g = fmin(g, vb);
        }
    }
    if (lane == 0) {
        V.B[row] = f;
        V.G[row] = g;
        V.Vb[row] = vb;                              // by cell: r
    }
}

// (several layers' workgroups mark one cell)
__device__ __forceinline__ void mark(int32_t *p)
{
    __hip_atomic_store(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A workgroup per layer: the grid points and cells of its range that a path
// of cost at most the best known one can cut at.
__global__ __launch_bounds__(kThreads) void prune_kernel(View V)
{
    __shared__ double red[kWaves];
    __shared__ int32_t wl[kWaves], wh[kWaves];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    // the best path over grid points
    {
        const int32_t a = V.wa[V.ke - 1], b = V.wb[V.ke - 1];
        double u = INFINITY;
        for (int32_t q = a + (int32_t)threadIdx.x; q <= b; q += kThreads) {
            const double x = V.U[(int64_t)(V.ke - 1) * V.stride + (q - a)];
            u = fmin(u, x + seg_cost(V.S[q], V.SS[V.n], V.pos[q], V.n - 1));
        }
        u = wave_min(u);
        if (lane == 0)
            red[w] = u;
    }
    __syncthreads();
    double best = red[0];
    for (int u = 1; u < kWaves; ++u)
        best = fmin(best, red[u]);
    // float64 rounding of a path's cost: a few ulps of the sum of squares,
    // and one of the running sum per cluster
    const double thr = best + (0x1p-44 + V.ke * 0x1p-50) * V.SS[V.n].y;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        V.ctl->thr = thr;
    const int c = (int)blockIdx.x + 1;
    const int32_t a = V.wa[c], b = V.wb[c];
    const int64_t row = (int64_t)c * V.stride;
    int32_t lo = INT32_MAX, hi = -1;
    for (int32_t i = a + (int32_t)threadIdx.x; i <= b; i += kThreads) {
        const int64_t e = row + (i - a);
        const double T = V.F[e] + V.G[e];
        if (T <= thr) {
            lo = min(lo, V.pos[i]);
            hi = max(hi, V.pos[i]);
            mark(V.keepp + i);
        }
        if (i < b && V.pen[i] >= 0.0) {
            const double vf = V.Vf[e], vb = V.Vb[e];
            double m = fmin(T, V.F[e + 1] + V.G[e + 1]);
            m = fmin(m, fmin(vf + V.B[e + 1], fmin(V.F[e] + vb, vf + vb)));
            if (m <= thr) {
                lo = min(lo, V.pos[i]);
                hi = max(hi, V.pos[i + 1]);
                mark(V.keepc + i);
            }
        }
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, kWave));
        hi = max(hi, __shfl_xor(hi, o, kWave));
    }
    if (lane == 0) {
        wl[w] = lo;
        wh[w] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int u = 1; u < kWaves; ++u) {
            lo = min(lo, wl[u]);
            hi = max(hi, wh[u]);
        }
        V.lo[c] = lo;
        V.hi[c] = hi;
    }
}

// Exclusive scan over the workgroup of one whole number per thread, and the
// total: within the waves by lane moves, their totals (in a) by every thread.
template <int NT>
__device__ __forceinline__ int32_t block_scan_excl(int32_t x, int32_t *a, int32_t &total)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int32_t y = x;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t z = __shfl_up(y, o, kWave);
        y += lane >= o ? z : 0;
    }
    __syncthreads();                             // the totals of the scan before are read
    if (lane == kWave - 1)
        a[wave] = y;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        before += w < wave ? a[w] : 0;
        total += a[w];
    }
    return before + y - x;
}

// The next round's windows: the runs of neighbouring cells that some layer
// keeps (a kept point beside no kept cell is one by itself), each cut into
// `split` cells for every one it had and `extra` more, as many as the grid
// and the rows hold, half of the room for either, or into every position
// where there is room for all of them.  A layer's range is that of the cells
// it keeps, made monotone over the layers; what lies in it between windows is
// left out, so that a few far apart ways to place the cuts (k above the number
// of clusters) do not keep all that lies between.
// One workgroup, bound by the latency of its few dependent passes: 15 us for
// 513 points, 40 for 49,000 (119 with a thread's run of marks read at a time
// and scans behind twenty barriers).
constexpr int kWinThreads = 1024;
static_assert(kMaxClusters <= kWinThreads, "a thread per layer");

__global__ __launch_bounds__(kWinThreads) void windows_kernel(View V)
{
    __shared__ int32_t a[kWinThreads / kWave];
    __shared__ int32_t lo[kMaxClusters], hi[kMaxClusters];
    __shared__ uint64_t cm[kMaxPoints / 64], pm[kMaxPoints / 64];
    __shared__ int32_t split, extra, rows, fail, all, exact;
    const int t = threadIdx.x;
    const int c = t;                             // the thread's layer, if any
    const bool layer = c >= 1 && c < V.ke;
    if (t == 0) {
        split = extra = INT32_MAX;
        rows = fail = 0;
        all = exact = 1;
    }
    __syncthreads();
    if (layer) {
        lo[c] = V.lo[c];
        hi[c] = V.hi[c];
        if (lo[c] > hi[c])
            atomicOr(&fail, 1);
    }
    __syncthreads();
    if (fail != 0) {                             // uniform
        if (t == 0)
            V.ctl->fail = 1;
        return;
    }
    for (int off = 1; off < V.ke; off <<= 1) {
        const int32_t l = layer && c + off < V.ke ? lo[c + off] : INT32_MAX;
        const int32_t h = layer && c - off >= 1 ? hi[c - off] : -1;
        __syncthreads();
        if (layer) {
            lo[c] = min(lo[c], l);
            hi[c] = max(hi[c], h);
        }
        __syncthreads();
    }
    // the marks of the grid points, 64 to a word, a wave's loads at a time
    const int32_t n = V.ctl->total;
    const int32_t words = (n + 63) / 64;
#pragma unroll 8
    for (int32_t i = t; i < words * 64; i += kWinThreads) {
        const uint64_t c64 = __ballot(i < n && V.keepc[i] != 0);
        const uint64_t p64 = __ballot(i < n && V.keepp[i] != 0);
        if (t % kWave == 0) {
            cm[i / 64] = c64;
            pm[i / 64] = p64;
        }
    }
    __syncthreads();
    // windows and kept cells before a thread's words: a window starts at a cell
    // or point without a kept cell before it, and ends at one without a cell
    const int32_t per = (words + kWinThreads - 1) / kWinThreads;
    const int32_t w0 = t * per, w1 = min(w0 + per, words);
    auto before = [&](int32_t w) { return (cm[w] << 1) | (w > 0 ? cm[w - 1] >> 63 : 0); };
    auto starts = [&](int32_t w) { return (cm[w] | pm[w]) & ~before(w); };
    int32_t s = 0, m = 0, k = 0;
    for (int32_t w = w0; w < w1; ++w) {
        const uint64_t first = starts(w);
        s += __popcll(first);
        m += __popcll(first & cm[w]);
        k += __popcll(cm[w]);
    }
    int32_t nseg, wide, cells;
    int32_t ws = block_scan_excl<kWinThreads>(s, a, nseg);
    int32_t wm = block_scan_excl<kWinThreads>(m, a, wide);
    int32_t wk = block_scan_excl<kWinThreads>(k, a, cells);
    // the windows' first and last grid points
    for (int32_t w = w0; w < w1; ++w) {
        const uint64_t C = cm[w], first = starts(w), last = (C | pm[w] | before(w)) & ~C;
        for (uint64_t e = first | last; e != 0; e &= e - 1) {
            const int b = __ffsll((unsigned long long)e) - 1;
            if ((first >> b) & 1) {
                V.segP[ws] = w * 64 + b;
                V.kpre[ws] = wk + __popcll(C & ((1ull << b) - 1));
                V.mpre[ws] = wm;
                ++ws;
                wm += (int)((C >> b) & 1);
            }
            if ((last >> b) & 1)
                V.segQ[ws - 1] = w * 64 + b;
        }
        wk += __popcll(C);
    }
    __syncthreads();
    // their positions, and the positions in the windows before
    const int32_t wper = (nseg + kWinThreads - 1) / kWinThreads;
    const int32_t z0 = t * wper, z1 = min(z0 + wper, nseg);
    int32_t l = 0;
    for (int32_t z = z0; z < z1; ++z) {
        const int32_t p = V.pos[V.segP[z]], q = V.pos[V.segQ[z]];
        V.segP[z] = p;
        V.segQ[z] = q;
        l += q - p + 1;
    }
    int32_t span;
    int32_t wl = block_scan_excl<kWinThreads>(l, a, span);
    for (int32_t z = z0; z < z1; ++z) {
        V.lpre[z] = wl;
        wl += V.segQ[z] - V.segP[z] + 1;
    }
    if (t == 0) {
        V.kpre[nseg] = cells;
        V.lpre[nseg] = span;
        V.mpre[nseg] = wide;
    }
    __syncthreads();
    // the layer's windows, and how far its rows let the cells be split
    int32_t zl = 0, zh = 0;
    if (layer) {
        auto at = [&](int32_t p) {               // last window that starts at or before p
            int32_t x = 0, y = nseg - 1;
            while (x < y) {
                const int32_t m = (x + y + 1) / 2;
                if (V.segP[m] <= p)
                    x = m;
                else
                    y = m - 1;
            }
            return x;
        };
        zl = at(lo[c]);
        zh = at(hi[c]);
        const int32_t half = max(V.stride - (zh - zl + 1), 0) / 2;
        const int32_t kc = V.kpre[zh + 1] - V.kpre[zl], mc = V.mpre[zh + 1] - V.mpre[zl];
        if (V.lpre[zh + 1] - V.lpre[zl] > V.stride)
            atomicAnd(&all, 0);
        if (kc > 0) {
            atomicMin(&split, half / kc);
            atomicMin(&extra, half / mc);
        }
    }
    if (t == 0) {
        if (span > V.points)
            atomicAnd(&all, 0);
        const int32_t half = max(V.points - nseg, 0) / 2;
        if (cells > 0) {
            atomicMin(&split, half / cells);
            atomicMin(&extra, half / wide);
        }
    }
    __syncthreads();
    const int64_t f = min(split, kMaxSplit), g = extra;
    const bool every = all != 0;
    // the windows' first grid points
    auto points = [&](int32_t z) {
        const int32_t len = V.segQ[z] - V.segP[z];
        const int64_t k = V.kpre[z + 1] - V.kpre[z];
        const int64_t most = k > 0 ? f * k + g : 0;
        return (every ? len : (int32_t)min((int64_t)len, most)) + 1;
    };
    int32_t b = 0;
    for (int32_t z = z0; z < z1; ++z) {
        const int32_t x = points(z);
        if (x != V.segQ[z] - V.segP[z] + 1)
            atomicAnd(&exact, 0);
        b += x;
    }
    int32_t total;
    int32_t o = block_scan_excl<kWinThreads>(b, a, total);
    for (int32_t z = z0; z < z1; ++z) {
        V.base[z] = o;
        o += points(z);
    }
    if (t == 0)
        V.base[nseg] = total;
    __syncthreads();
    if (layer) {
        V.lo[c] = lo[c];
        V.hi[c] = hi[c];
        atomicMax(&rows, V.base[zh + 1] - V.base[zl]);
    }
    __syncthreads();
    if (t == 0) {
        V.ctl->nseg = nseg;
        V.ctl->total = total;
        V.ctl->rows = rows;
        V.ctl->exact = exact;
        V.ctl->fail = !every && f + g < 2;
        V.ctl->span = span;
    }
}

// Row n - 1 of the last layer and the way back through the argmins.
__global__ __launch_bounds__(kThreads) void finish_kernel(View V, int64_t *__restrict__ first)
{
    __shared__ double wb[kWaves];
    __shared__ int64_t wa[kWaves];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int32_t a = V.wa[V.ke - 1], b = V.wb[V.ke - 1];
    double best = INFINITY;
    int64_t arg = INT64_MAX;
    for (int32_t q = a + (int32_t)threadIdx.x; q <= b; q += kThreads) {
        const double x = V.U[(int64_t)(V.ke - 1) * V.stride + (q - a)] +
                         seg_cost(V.S[q], V.SS[V.n], V.pos[q], V.n - 1);
        if (x < best) {
            best = x;
            arg = q;
        }
    }
    wave_argmin(best, arg);
    if (lane == 0) {
        wb[w] = best;
        wa[w] = arg;
    }
    __syncthreads();
    if (threadIdx.x != 0)
        return;
    for (int u = 1; u < kWaves; ++u)
        amin_merge(best, arg, wb[u], wa[u]);
    int32_t q = (arg == INT64_MAX) ? a : (int32_t)arg;
    for (int c = V.ke - 1; c >= 1; --c) {
        first[c] = V.pos[q];
        const int32_t back = V.arg[(int64_t)c * V.stride + (q - V.wa[c])];
        q = (c > 1 && back < 0) ? V.wa[c - 1] : back;
    }
    first[0] = 0;
    first[V.ke] = V.n;
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

// Places the arrays for `per` cells a layer and rows of `merged` times as
// many in `ws` (null: only the size).
size_t place(char *ws, int64_t n, int32_t ke, int32_t per, int32_t merged, View *V)
{
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *p = ws + o;
        o += al(bytes);
        return p;
    };
    V->ke = ke;
    V->per = per;
    int64_t most = (int64_t)per * (merged < ke - 1 ? merged : ke - 1);
    most = most < n ? most : n;
    V->stride = (int32_t)most + 1;
    // windows do not overlap and have at most a cell per position
    const int64_t later = (int64_t)(ke - 1) * (per + 1);
    const size_t pts = (size_t)(later < n + ke ? later : n + ke);
    const size_t rows = (size_t)ke * V->stride;
    V->points = (int32_t)pts;
    V->ctl = (RoundCtl *)take(sizeof(RoundCtl));
    V->pos = (int32_t *)take(pts * 4);
    V->S = (double2 *)take(pts * 16);
    V->xl = (double *)take(pts * 8);
    V->xr = (double *)take(pts * 8);
    V->sw = (double *)take(pts * 8);
    V->pen = (double *)take(pts * 8);
    V->Ln = (double2 *)take(pts * 16);
    V->Rn = (double2 *)take(pts * 16);
    V->cellseg = (int32_t *)take(pts * 4);
    V->F = (double *)take(rows * 8);
    V->G = (double *)take(rows * 8);
    V->U = (double *)take(rows * 8);
    V->B = (double *)take(rows * 8);
    V->Vf = (double *)take(rows * 8);
    V->Vb = (double *)take(rows * 8);
    V->arg = (int32_t *)take(rows * 4);
    V->lo = (int32_t *)take((size_t)ke * 4);
    V->hi = (int32_t *)take((size_t)ke * 4);
    V->qmin = (int32_t *)take(pts * 4);
    V->rmax = (int32_t *)take(pts * 4);
    V->keepp = (int32_t *)take(pts * 4);
    V->keepc = (int32_t *)take(pts * 4);
    V->wa = (int32_t *)take((size_t)ke * 4);
    V->wb = (int32_t *)take((size_t)ke * 4);
    V->segP = (int32_t *)take(pts * 4);
    V->segQ = (int32_t *)take(pts * 4);
    V->base = (int32_t *)take((pts + 1) * 4);
    V->kpre = (int32_t *)take((pts + 1) * 4);
    V->lpre = (int32_t *)take((pts + 1) * 4);
    V->mpre = (int32_t *)take((pts + 1) * 4);
    return o;
}

} // namespace

bool kmeans_windows_apply(int64_t n, int64_t k)
{
    return n >= kFromN && k >= (n < kHugeN ? kFew : kFewHuge);
}

hipError_t launch_gap_stats(const double *sv, const double2 *SS, int64_t n, GapStats *gs,
                            hipStream_t s)
{
    const int64_t want = (n + kTile - 1) / kTile;
    hipLaunchKernelGGL(gap_stats_kernel, dim3((unsigned)(want < 256 ? want : 256)),
                       dim3(kThreads), 0, s, sv, SS, n, gs);
    return hipGetLastError();
}

namespace {

// Whether the windows can be expected to shrink, from the gaps alone.  At a
// scale, the gaps above it split the values into groups, of mean width w (the
// sum of the others over their number).
//   * Where the values form fewer groups than ke, the cuts to spare are
//     decided by costs of about n w^2 / 64 (a deviation of w / 8).  Where that
//     is near the bound on the rounding, no bound excludes anything, unless the
//     next gaps give the ke groups and leave far less inside them.
//   * Up to kLargeN values, where they form well separated groups (w below a
//     quarter of every gap between them) and these are two thirds of ke or
//     fewer: many ways to hand out the spare cuts cost about the same, and the
//     scratch is small for a grid that tells them apart.
// Only the time depends on it.
bool worth_it(const GapStats &gs, int64_t n, int32_t ke)
{
    const double pad = (0x1p-44 + ke * 0x1p-50) * gs.s2;
    double inside = 0.0;
    for (int b = 0; b < kGapClasses; ++b)
        inside += (double)gs.sum[b];
    inside *= 0x1p-60;
    double finest = inside, groups = 1.0, separate = 1.0, last = -1.0;
    for (int b = 0; b < kGapClasses && groups <= ke; ++b) {
        // the groups at the gaps of the classes below b
        if (groups < ke) {
            finest = inside / groups;
            if (groups > 1.0 && finest < 0.25 * exp2(1.0 - b))
                separate = groups;
        } else if (last < 0.0) {
            last = inside / groups;
        }
        groups += (double)gs.count[b];
        inside -= (double)gs.sum[b] * 0x1p-60;
    }
    if (last >= 0.0 && last < 0.0625 * finest)
        return true;
    const double w = finest * gs.range;
    if ((double)n * w * w * 0x1p-6 <= kRoundingCost * pad)
        return false;
    return !(n < kLargeN && separate > 1.0 && 3.0 * separate <= 2.0 * ke);
}

// The most that one gap adds to phi: a wide gap needs one grid point, and
// without a bound a few of them take the cells of all the values.  The
// smallest class limit that is still a cell's share where every wider gap
// counts as much as it.
double root_cap(const GapStats &gs, int32_t cells)
{
    double rest = 0.0, wide = 0.0, cap = INFINITY;
    for (int b = 0; b < kGapClasses; ++b)
        rest += (double)gs.root[b] * 0x1p-40;
    for (int b = 0; b < kGapClasses; ++b) {
        const double c = exp2(-0.5 * b);             // the largest root of class b
        if (c * cells < rest + wide * c)
            break;
        cap = c;
        wide += (double)gs.count[b];
        rest -= (double)gs.root[b] * 0x1p-40;
    }
    return cap * sqrt(gs.range);
}

} // namespace

hipError_t kmeans_windows(const double *sv, const int32_t *run, const double2 *SS, int64_t n,
                          const double *mean, int32_t ke, const GapStats &gs, double *phi,
                          double *psum, void *ws, size_t ws_bytes, int64_t *first,
                          hipStream_t s, int *solved)
{
    *solved = 0;
    if (!kmeans_windows_apply(n, ke) || ke > kMaxClusters)
        return hipSuccess;
    // squares that overflow, in a sum or times n, or that lose their last
    // bits to underflow, leave no bound that means anything: every row is
    // computed
    if (!(gs.s2 > 0x1p-900 && gs.s2 < 0x1p900) || !worth_it(gs, n, ke))
        return hipSuccess;
    // cells of the first round, and rows of a layer: as many as are useful and
    // the scratch holds.  With few per cluster the windows do not shrink (one is
    // about sqrt(4 ke) / (cells per cluster) of it): 10 ke^1.5 cells, of up to 32
    // x kMaxPer, and from 2^17 values fewer are not tried (n = 600,000, k = 100, 130
    // with 8 x: 2.9, 2.2 times as fast and two and eight draws of 26 at 0.7 to 0.85,
    // with 16 x: 2.8, 2.7 and none; k = 70: 3.2 and 2.9; n = 2M, k = 150 with 16, 32 x:
    // 2.1, 2.8; k = 200 with 32 x, 7 ke^1.5: 1.8, five draws of 13 at 0.7 to 0.86).
    // With fewer values a range is every position soon, and 5.5 ke^1.5 will do:
    // embeddings with n = 8,192, k = 24 (5.7): 1.48; of the shapes at n = 12,000, k =
    // 24 (7.0) and 20,000, 32 (5.9) a tenth take 0.7 times as long again for 1.29
    // and 1.24 on average; 40,000, 48 (5.4): a third, for 1.15.
    View V{};
    const double least = (n < kLargeN ? 5.5 : 10.0) * ke * sqrt((double)ke);
    int32_t per = (int32_t)(n / 4 < kMaxPer ? n / 4 : kMaxPer), merged = kMerged;
    if (per > kMaxPoints / (ke - 1) - 1)
        per = kMaxPoints / (ke - 1) - 1;
    while (merged < kMaxMerged && (double)per * merged < least)
        merged *= 2;
    while (per >= 32 && place(nullptr, n, ke, per, merged, &V) > ws_bytes) {
        if (merged > 2)
            merged /= 2;
        else
            per -= (per + 15) / 16;
    }
    const double cells = (double)per * (merged < ke - 1 ? merged : ke - 1);
    if (per < 32 || per < 2 * ke || (cells < (double)n && cells < least))
        return hipSuccess;
    place(static_cast<char *>(ws), n, ke, per, merged, &V);
    V.sv = sv;
    V.run = run;
    V.SS = SS;
    V.n = n;
    V.mean = mean;
    V.phi = phi;
    V.psum = psum;
    const int64_t tiles = (n + kTile - 1) / kTile;
    const int32_t first_cells = per < kFirst ? per : kFirst;
    V.cap = root_cap(gs, first_cells);
    hipLaunchKernelGGL(phi_sums_kernel, dim3((unsigned)tiles), dim3(kThreads), 0, s, V);
    hipLaunchKernelGGL(first_window_kernel, dim3(1), dim3(1024), 0, s, V, tiles, first_cells);
    hipLaunchKernelGGL(phi_kernel, dim3((unsigned)tiles), dim3(kThreads), 0, s, V);
    int32_t total = first_cells + 1;
    int32_t rows = total;                            // most grid points of a window
    int64_t span = n;
    for (int round = 0; round < kMaxRounds; ++round) {
        const unsigned gg = (unsigned)(((total > ke ? total : ke) + kThreads - 1) / kThreads);
        hipLaunchKernelGGL(positions_kernel, dim3(gg), dim3(kThreads), 0, s, V);
        hipLaunchKernelGGL(grid_kernel, dim3(gg), dim3(kThreads), 0, s, V);
        const unsigned wg = (unsigned)((rows + kWaves - 1) / kWaves);
        for (int t = 1; t < ke; ++t)
            hipLaunchKernelGGL(layer_kernel<false>, dim3(wg, 2), dim3(kThreads), 0, s, V, t);
        hipLaunchKernelGGL(prune_kernel, dim3((unsigned)(ke - 1)), dim3(kThreads), 0, s, V);
        hipLaunchKernelGGL(windows_kernel, dim3(1), dim3(kWinThreads), 0, s, V);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        RoundCtl h{};
        if ((e = hipMemcpyAsync(&h, V.ctl, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return e;
        if (h.fail)
            return hipSuccess;
        // neither the windows nor their cells get smaller (the first grid may
        // be too coarse to exclude anything yet)
        const bool stuck = round > 0 && h.span > 0.75 * span &&
                           (double)h.span / h.total > 0.75 * span / total;
        total = h.total;
        rows = h.rows;
        span = h.span;
        if (h.exact) {
            // every position of the windows is a grid point: the programme itself
            const unsigned ge = (unsigned)(((total > ke ? total : ke) + kThreads - 1) / kThreads);
            hipLaunchKernelGGL(positions_kernel, dim3(ge), dim3(kThreads), 0, s, V);
            hipLaunchKernelGGL(grid_kernel, dim3(ge), dim3(kThreads), 0, s, V);
            const unsigned we = (unsigned)((rows + kWaves - 1) / kWaves);
            for (int t = 1; t < ke; ++t)
                hipLaunchKernelGGL(layer_kernel<true>, dim3(we), dim3(kThreads), 0, s, V, t);
            hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(kThreads), 0, s, V, first);
            *solved = 1;
            return hipGetLastError();
        }
        if (stuck)
            return hipSuccess;
    }
    return hipSuccess;
}

} // namespace gpic
