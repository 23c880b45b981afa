// Exact k-nearest-neighbour input graph for the sparse path, on gfx950.
//
// N(i) = the k points j != i with the smallest (||x_i - x_j||^2, j); edge
// {i, j} when j is in N(i) or i in N(j); weight exp(-||x_i - x_j||^2 /
// (2 sigma^2)) in float64, rounded once to float32; rows sorted by column.
// This is the graph the CSR power iteration takes as its affinity (the
// paper's method needs an affinity matrix; a kNN graph is its sparse form).
//
// Brute force in four steps, exact in the end:
//   1. bound: the points are put in Morton order of their quantised centred
//      coordinates and cut into tiles of 64 consecutive ones; for every row,
//      the k-th smallest float32 squared distance to the points of the 32
//      tiles whose boxes are centred nearest to its own tile's and of the
//      tiles next to it in Morton order, or, for rows whose bound is wide
//      against their tile's smallest, of the 32 tiles nearest to the row
//      itself; the k-th distance to any points bounds the true k-th
//      neighbour distance from above;
//   2. collect: squared distances on the fp32 matrix cores (Gram form over
//      the centred points augmented as [x_j, |x_j|^2, 1] .
//      [-2 x_i, 1, |x_i|^2]), appending every j that passes the row's bound
//      widened by the float32 error bounds of both forms to a per-row
//      candidate list.  In Morton order a tile of 64 consecutive points is
//      spatially compact; a pair of tiles whose bounding boxes are farther
//      apart than every bound of the row tile is skipped whole (no pair in
//      it can be a neighbour: its true distance exceeds the row's bound,
//      which is at least the true k-th neighbour distance), and so is each
//      block of 16 rows by 16 columns of the tiles that remain;
//   3. select: a wave per row recomputes the candidates' squared distances
//      in float64 and keeps the k smallest (ties to the smaller index); a
//      row whose list overflowed gets the k-th distance among the kept
//      candidates as its new bound and is collected again;
//   4. symmetrise: both directions of every kept pair as 64-bit keys
//      (row, column), radix sorted, duplicates dropped, CSR built, weights
//      from float64 distances.
// Supports d <= 16 and k <= 64.
#include "common.h"
#include "lanes.h"

namespace gpic {
namespace {

constexpr int kThreads = 256;
constexpr int kCap = 2048;                // candidate slots per row
constexpr int kPerLane = kCap / kWave;    // candidates per lane in the selection
constexpr int kRowsPerGroup = 64;         // collect: 4 waves x 16 rows
constexpr int kTileCols = 64;
constexpr float kEps32 = 5.9604645e-08f;  // 2^-24
constexpr int kMeanBlocks = 256;

typedef float floatx4 __attribute__((ext_vector_type(4)));

int64_t al(int64_t x) { return (x + 255) & ~(int64_t)255; }
int64_t padded_points(int64_t n) { return (n + kTileCols - 1) / kTileCols * kTileCols; }
// augmented dimension / 4, rounded up to an instantiated engine (3 or 5)
int ks_for(int d) { return (d + 2 + 3) / 4 <= 3 ? 3 : 5; }

// float64 squared distance summed over coordinates in order, without
// fused multiply-adds (the same value a plain C loop gives)
__device__ __forceinline__ double sq_dist64(const float *__restrict__ X, int d, int64_t i,
                                            int64_t j)
{
    double s = 0.0;
    for (int c = 0; c < d; ++c) {
        const double df = __dsub_rn((double)X[i * d + c], (double)X[j * d + c]);
        s = __dadd_rn(s, __dmul_rn(df, df));
    }
    return s;
}

// ------------------------------------------------------------ 1. bound

// The kNear tiles whose box centres lie nearest to a row tile's, nearest
// first (a workgroup per row tile): each thread keeps the nearest of every
// 256th tile -- neighbours in Morton order go to different threads -- and
// the 256 kept are ranked against each other.  With at most 256 tiles
// these are the nearest of all; else near enough (any tiles give a bound).
constexpr int kNear = 32;
constexpr int kWindow = 4;             // tiles on each side in Morton order

__global__ __launch_bounds__(kThreads) void near_tiles_kernel(const float *__restrict__ box,
                                                              int64_t nt, int d,
                                                              int32_t *__restrict__ near)
{
    __shared__ uint64_t key[kThreads];
    const int64_t row = blockIdx.x;
    float cr[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
        cr[c] = (c < d) ? 0.5f * box[c * nt + row] + 0.5f * box[(16 + c) * nt + row] : 0.0f;
    uint64_t best = ~0ull;
    for (int64_t t = threadIdx.x; t < nt; t += kThreads) {
        float s = 0.0f;
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (c < d) {
                const float g = 0.5f * box[c * nt + t] + 0.5f * box[(16 + c) * nt + t] - cr[c];
                s = fmaf(g, g, s);
            }
        // an overflowed or undefined distance ranks last
        s = (s < INFINITY) ? s : INFINITY;
        const uint64_t k = ((uint64_t)__float_as_uint(s) << 32) | (uint64_t)(uint32_t)t;
        best = (k < best) ? k : best;
    }
    key[threadIdx.x] = best;
    __syncthreads();
    int rank = 0;
    for (int u = 0; u < kThreads; ++u)
        rank += (key[u] < best) ? 1 : 0;
    // threads without a tile rank after every other, so the first
    // min(kNear, nt) places are filled
    if (best != ~0ull && rank < kNear)
        near[row * kNear + rank] = (int32_t)(best & 0xffffffffull);
}

// A wave per row tile, a thread per Morton position p, row i = perm[p]: the
// KT smallest float32 squared distances from x_i to the other points of the
// tile's near tiles and of its neighbours in Morton order, then tau_i = the
// k-th of them.  The k-th distance to any k other points bounds the true
// k-th neighbour distance from above, and these tiles hold at least k others
// (all points when there are no more than kNear tiles).  The Morton
// neighbours matter where a tile straddles a jump of the order: its box
// centre then lies far from all of its rows.  Bound by the insertions into the KT kept values, which
// a wave takes when any of its rows does: the nearer tiles first, and few
// of them.  (The k-th distance to 512 Morton neighbours and a sample of
// 65,536 points took 62 ms at n = 2M, k = 32, for a looser bound, 165
// candidates a row; these tiles 7 ms and 70 candidates.)
template <int D, int KT>
__global__ __launch_bounds__(kThreads) void knn_bound_kernel(
    const float *__restrict__ X, const int32_t *__restrict__ perm, int64_t n, int64_t nt, int k,
    const int32_t *__restrict__ near, float *__restrict__ tau, float *__restrict__ tmin)
{
    __shared__ float tile[kThreads / kWave][kWave * D];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int64_t row = (int64_t)blockIdx.x * (kThreads / kWave) + wave;
    if (row >= nt)
        return;                                  // uniform per wave, no barrier below
    const int64_t p = row * kTileCols + lane;
    const int64_t pc = p < n ? p : n - 1;
    const int64_t i = perm[pc];
    float xi[D];
#pragma unroll
    for (int c = 0; c < D; ++c)
        xi[c] = X[i * D + c];
    float best[KT];
#pragma unroll
    for (int u = 0; u < KT; ++u)
        best[u] = INFINITY;
    const int m = nt < kNear ? (int)nt : kNear;
    float *own = tile[wave];
    for (int a = -2 * kWindow - 1; a < m; ++a) {
        // the tiles within kWindow in Morton order, its own first, then the
        // near tiles that are not among them
        const int o = 2 * kWindow + 1 + a;       // 0, 1, 2, .. -> row, row - 1, row + 1, ..
        const int64_t t = (a < 0) ? row + ((o & 1) ? -(o + 1) / 2 : o / 2)
                                  : (int64_t)near[row * kNear + a];
        if (t < 0 || t >= nt || (a >= 0 && t >= row - kWindow && t <= row + kWindow))
            continue;                            // uniform per wave
        const int64_t q0 = t * kTileCols;
        const int cnt = (n - q0 < kTileCols) ? (int)(n - q0) : kTileCols;
        const int64_t pt = perm[q0 + lane < n ? q0 + lane : n - 1];
        float xj[D];
#pragma unroll
        for (int c = 0; c < D; ++c)
            xj[c] = X[pt * D + c];
        __builtin_amdgcn_wave_barrier();         // the wave's reads of the tile before
#pragma unroll
        for (int c = 0; c < D; ++c)
            own[lane * D + c] = xj[c];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int u = 0; u < cnt; ++u) {
            float s = 0.0f;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float df = xi[c] - own[u * D + c];
                s = fmaf(df, df, s);
            }
            if (q0 + u == pc)
                s = INFINITY;                    // not the row itself
            if (s < best[KT - 1]) {
#pragma unroll
                for (int w = KT - 1; w > 0; --w) {
                    const float lo = best[w - 1];
                    best[w] = (s < lo) ? lo : fminf(s, best[w]);
                }
                best[0] = fminf(s, best[0]);
            }
        }
    }
    float t = best[0];
#pragma unroll
    for (int u = 1; u < KT; ++u)
        if (u == k - 1)
            t = best[u];
    if (p < n)
        tau[i] = t;
    else
        t = INFINITY;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
        t = fminf(t, __shfl_xor(t, o, kWave));
    if (lane == 0)
        tmin[row] = t;
}

// The bound again for single rows, from the tiles nearest to the row itself:
// four workgroups per row tile take, one after another, the rows whose
// bound is more than kWide times the tile's smallest (flags null: before the
// first collection; the rows beyond a jump of the Morton order, mostly), or
// the flagged ones (their lists overflowed).  The smallest is tmin, formed
// with the bounds: a workgroup reads the bounds of its own rows alone, the
// others' being written meanwhile.  Nearest tiles by the distance
// from the point to the box centres as in near_tiles_kernel, then the k-th
// smallest of the distances to their 2,048 points by bisection on the bit
// patterns.  A wide bound costs its whole row tile a visit to most of a
// cluster.  ms per graph with kWide = 3, 6, 12: n = 2M, d = 8, k = 32: 141, 128,
// 135; d = 2, k = 5: 71, 30, 18; n = 200,000, d = 2, 8, 16 with k = 5: 4.3, 2.9,
// 2.5; 6.4, 4.5, 6.0; 7.2, 9.9, 9.7; with k = 32: 4.5, 4.4, 4.4; 10.6, 11.4, 11.6;
// 14.5, 15.2, 15.6; with k = 64 within 7 %; half of the points in 1,560 places, d
// = 6, k = 10: 10.2, 12.1, 13.9.  kNear = 16, 32, 64 at the first: 134, 128, 129;
// at the others 16 is up to 10 % faster and 64 up to 28 % slower, at n =
// 20,000, d = 16, k = 64: 2.9, 3.3, 4.0.
constexpr float kWide = 6.0f;
constexpr unsigned kRefineParts = 4;   // workgroups per row tile, each every 4th row

__global__ __launch_bounds__(kThreads) void refine_bound_kernel(
    const float *__restrict__ X, const int32_t *__restrict__ perm, const float *__restrict__ box,
    int64_t n, int64_t nt, int d, int k, const int *__restrict__ flags,
    const float *__restrict__ tmin, float *__restrict__ tau)
{
    constexpr int kW = kThreads / kWave;
    constexpr int kPts = kNear * kTileCols / kThreads;
    __shared__ uint64_t key[kThreads];
    __shared__ int32_t nb[kNear];
    __shared__ unsigned long long todo;
    __shared__ int cnt[2][kW];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int64_t p0 = (int64_t)(blockIdx.x / kRefineParts) * kTileCols;
    if (wave == 0) {
        const int64_t p = p0 + lane;
        const int64_t i = (p < n && lane % kRefineParts == blockIdx.x % kRefineParts)
                              ? (int64_t)perm[p] : -1;
        const bool want = i >= 0 && (flags != nullptr
                                         ? flags[i] != 0
                                         : tau[i] > kWide * tmin[blockIdx.x / kRefineParts]);
        const unsigned long long m = __ballot(want);
        if (lane == 0)
            todo = m;
    }
    __syncthreads();
    unsigned long long rows = todo;
    while (rows != 0) {                          // uniform over the workgroup
        const int r = __ffsll((long long)rows) - 1;
        rows &= rows - 1;
        const int64_t pc = p0 + r;
        const int64_t i = perm[pc];
        float xi[16];
#pragma unroll
        for (int c = 0; c < 16; ++c)
            xi[c] = (c < d) ? X[i * d + c] : 0.0f;
        uint64_t best = ~0ull;
        for (int64_t t = threadIdx.x; t < nt; t += kThreads) {
            float s = 0.0f;
#pragma unroll
            for (int c = 0; c < 16; ++c)
                if (c < d) {
                    const float g = 0.5f * box[c * nt + t] + 0.5f * box[(16 + c) * nt + t] - xi[c];
                    s = fmaf(g, g, s);
                }
            s = (s < INFINITY) ? s : INFINITY;
            const uint64_t kk = ((uint64_t)__float_as_uint(s) << 32) | (uint64_t)(uint32_t)t;
            best = (kk < best) ? kk : best;
        }
        key[threadIdx.x] = best;
        if (threadIdx.x < kNear)
            nb[threadIdx.x] = -1;
        __syncthreads();
        int rank = 0;
        for (int u = 0; u < kThreads; ++u)
            rank += (key[u] < best) ? 1 : 0;
        if (best != ~0ull && rank < kNear)
            nb[rank] = (int32_t)(best & 0xffffffffull);
        __syncthreads();
        // distances as bit patterns (non-negative floats compare as integers);
        // padding, the row itself and undefined ones last
        uint32_t v[kPts];
#pragma unroll
        for (int u = 0; u < kPts; ++u) {
            const int32_t t = nb[u * kW + wave];
            const int64_t q = (int64_t)t * kTileCols + lane;
            v[u] = 0x7f800000u;
            if (t >= 0 && q < n && q != pc) {
                const int64_t j = perm[q];
                float s = 0.0f;
                for (int c = 0; c < d; ++c) {
                    const float df = X[i * d + c] - X[j * d + c];
                    s = fmaf(df, df, s);
                }
                v[u] = (s < INFINITY) ? __float_as_uint(s) : 0x7f800000u;
            }
        }
        // smallest pattern with at least k values at or below it
        uint32_t a = 0, b = 0x7f800000u;
        for (int it = 0; a < b; ++it) {          // at most 31 steps
            const uint32_t m = a + (b - a) / 2;
            int c = 0;
#pragma unroll
            for (int u = 0; u < kPts; ++u)
                c += __popcll(__ballot(v[u] <= m));
            if (lane == 0)
                cnt[it & 1][wave] = c;
            __syncthreads();
            c = 0;
#pragma unroll
            for (int w = 0; w < kW; ++w)
                c += cnt[it & 1][w];
            if (c >= k)
                b = m;
            else
                a = m + 1;
        }
        if (threadIdx.x == 0)
            tau[i] = fminf(tau[i], __uint_as_float(a));
        __syncthreads();                         // key and nb are refilled for the next row
    }
}

// max_j |x_j|^2 (non-negative floats compare as their bit patterns)
__global__ __launch_bounds__(kThreads) void max_norm_kernel(const float *__restrict__ norm2,
                                                            int64_t n,
                                                            unsigned int *__restrict__ out)
{
    unsigned int m = 0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        m = max(m, __float_as_uint(norm2[i]));
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
        m = max(m, (unsigned int)__shfl_xor((int)m, o, kWave));
    if ((threadIdx.x % kWave) == 0)
        atomicMax(out, m);
}

// Collection threshold: the exact k-th neighbour distance is at most
// tau (1 + 4 (d + 2) eps32) (tau is a float32 difference-form value); a
// Gram-form value over the centred points x' = x - mean (rounded once), a
// float32 sum of KP terms whose magnitudes add up to at most
// 2 (|x'_i|^2 + |x'_j|^2), is below the exact squared distance by at most
// (2 KP + 20) eps32 (|x'_i|^2 + max |x'|^2) with margin (4 of it for the
// rounding of the centred coordinates).  Formed in float64 and rounded up.
// Rows not active get -1 (nothing passes).
__global__ __launch_bounds__(kThreads) void threshold_kernel(
    const float *__restrict__ tau, const double *__restrict__ kth,
    const float *__restrict__ norm2, const unsigned int *__restrict__ maxn, int64_t n,
    int d, int kp, const int *__restrict__ active, float *__restrict__ thr)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n)
        return;
    if (active != nullptr && !active[i]) {
        thr[i] = -1.0f;
        return;
    }
    const double eps = (double)kEps32;
    const double base = (kth != nullptr) ? fmin(kth[i], (double)tau[i]) : (double)tau[i];
    const double t = base * (1.0 + 4.0 * (d + 2) * eps) +
                     (2 * kp + 20) * eps * ((double)norm2[i] + (double)__uint_as_float(*maxn));
    float f = (float)t;
    if ((double)f < t)
        f = nextafterf(f, INFINITY);
    thr[i] = f;
}

// ------------------------------------------------------------ 2. collect

// Mean of the points per coordinate (float64): per-workgroup partial sums,
// then one workgroup adds them in order.
__global__ __launch_bounds__(kThreads) void mean_partials_kernel(const float *__restrict__ X,
                                                                 int64_t n, int d,
                                                                 double *__restrict__ part)
{
    __shared__ double red[kThreads / kWave];
    for (int c = 0; c < d; ++c) {
        double s = 0.0;
        for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n;
             p += (int64_t)gridDim.x * kThreads)
            s += (double)X[p * d + c];
        const double t = block_sum<kThreads>(s, red);
        if (threadIdx.x == 0)
            part[(int64_t)blockIdx.x * d + c] = t;
    }
}

__global__ void mean_finish_kernel(const double *__restrict__ part, int nb, int d, int64_t n,
                                   double *__restrict__ mu)
{
    const int c = threadIdx.x;
    if (c >= d)
        return;
    double s = 0.0;
    for (int b = 0; b < nb; ++b)
        s += part[(int64_t)b * d + c];
    mu[c] = s / (double)n;
}

// Augmented operands of the centred points x' = float32(x - mean):
// column xa[k * np + p] = [x'_p, |x'_p|^2, 1, 0...], row
// xb[p * KP + k] = [-2 x'_p, 1, |x'_p|^2, 0...]; |x'_p|^2 a float64 sum
// rounded once (also written to norm2).  Padding points are zeros.
// With perm, position p holds point perm[p] (norm2 stays indexed by point).
__global__ __launch_bounds__(kThreads) void knn_augment_kernel(
    const float *__restrict__ X, const double *__restrict__ mu, const int32_t *__restrict__ perm,
    int64_t n, int64_t np, int d, int KP, float *__restrict__ xa, float *__restrict__ xb,
    float *__restrict__ norm2)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= np)
        return;
    const int64_t pt = (p < n && perm != nullptr) ? (int64_t)perm[p] : p;
    float xc[16];
    double s = 0.0;
    for (int c = 0; c < 16; ++c) {
        xc[c] = 0.0f;
        if (c < d && p < n) {
            xc[c] = (float)((double)X[pt * d + c] - mu[c]);
            s = fma((double)xc[c], (double)xc[c], s);
        }
    }
    const float nrm = (float)s;
    if (p < n)
        norm2[pt] = nrm;
    for (int k = 0; k < KP; ++k) {
        float a = 0.0f, b = 0.0f;
        if (p < n) {
            if (k < d) {
                a = xc[k];
                b = -2.0f * a;
            } else if (k == d) {
                a = nrm;
                b = 1.0f;
            } else if (k == d + 1) {
                a = 1.0f;
                b = nrm;
            }
        }
        xa[k * np + p] = a;
        xb[p * KP + k] = b;
    }
}

// Morton key of point p: its centred coordinates quantised to b = min(64 / d,
// 32) bits over [-R, R] (R^2 = the largest |x - mean|^2), bits interleaved
// from the most significant down; the payload is the point's index.
__global__ __launch_bounds__(kThreads) void morton_key_kernel(
    const float *__restrict__ X, const double *__restrict__ mu,
    const unsigned int *__restrict__ maxn, int64_t n, int d, uint64_t *__restrict__ key,
    int32_t *__restrict__ idx)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= n)
        return;
    const double R = sqrt((double)__uint_as_float(*maxn));
    const int b = (64 / d < 32) ? 64 / d : 32;
    const double levels = ldexp(1.0, b);
    uint32_t q[16];
    for (int c = 0; c < d; ++c) {
        const double xc = (double)(float)((double)X[p * d + c] - mu[c]);
        double u = (R > 0.0) ? (xc + R) / (2.0 * R) * levels : 0.0;
        u = u < 0.0 ? 0.0 : (u > levels - 1.0 ? levels - 1.0 : u);
        q[c] = (uint32_t)u;
    }
    uint64_t k = 0;
    for (int l = b - 1; l >= 0; --l)
        for (int c = 0; c < d; ++c)
            k = (k << 1) | ((q[c] >> l) & 1u);
    key[p] = k;
    idx[p] = (int32_t)p;
}

// Bounding boxes of the raw coordinates of every block of 16 consecutive
// positions and of every tile of 64, coordinate-major so that neighbouring
// tiles' boxes are read together: the lowest values at [c nb + b], the
// highest at [(16 + c) nb + b] for the nb blocks (tiles).  A thread per
// (tile, coordinate); padding positions are left out (a block of them is
// empty: lowest +infinity, highest -infinity, never near anything).
constexpr int kBlock = 16;
constexpr int kBlocks = kTileCols / kBlock;

__global__ __launch_bounds__(kThreads) void tile_box_kernel(
    const float *__restrict__ X, const int32_t *__restrict__ perm, int64_t n, int d,
    int64_t ntiles, float *__restrict__ box, float *__restrict__ sub)
{
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= ntiles * 16)
        return;
    const int64_t t = e / 16;
    const int c = (int)(e % 16);
    if (c >= d)
        return;
    const int64_t nb = ntiles * kBlocks;
    float lo = INFINITY, hi = -INFINITY;
    for (int b = 0; b < kBlocks; ++b) {
        float l = INFINITY, h = -INFINITY;
        for (int64_t p = t * kTileCols + b * kBlock; p < t * kTileCols + (b + 1) * kBlock && p < n;
             ++p) {
            const float x = X[(int64_t)perm[p] * d + c];
            l = fminf(l, x);
            h = fmaxf(h, x);
        }
        sub[c * nb + t * kBlocks + b] = l;
        sub[(16 + c) * nb + t * kBlocks + b] = h;
        lo = fminf(lo, l);
        hi = fmaxf(hi, h);
    }
    box[c * ntiles + t] = lo;
    box[(16 + c) * ntiles + t] = hi;
}

// Whether two boxes are farther apart than any of the bounds (the largest
// being `cut`): the float32 squared gap is within 2e-6 of the exact one
// relatively (differences, squares and d <= 16 additions, each rounded
// once), so a gap above cut (1 + 8e-6) is truly above cut.
__device__ __forceinline__ float box_gap2(float lo, float hi, float rlo, float rhi, float s)
{
    const float g = fmaxf(fmaxf(lo - rhi, rlo - hi), 0.0f);
    return fmaf(g, g, s);
}

// 4 waves x 16 rows; all columns in tiles of 64 through double-buffered
// LDS (coordinate-major, XOR-swizzled as in the affinity engine);
// v_mfma_f32_16x16x4f32 with the A operand on the columns and the B operand
// on the wave's rows, so lane (m, g) holds row wrow0 + m and columns
// 16 q + 4 g + r of block q.  Every (i, j != i) whose squared distance
// passes thr_i is appended to row i's list (slots beyond kCap are counted,
// not written).  A row belongs to one workgroup, so its counter is in LDS
// until the end.  Bound by the matrix cores and the comparison of their
// results (1,260 tiles of 64 visited per row tile at n = 2M, d = 8, k = 32
// before the blocks' boxes, which leave 0.57 of the pairs).  Per graph there:
// 101 ms; 92 with the counters in LDS; 64 to 73, box to box, with tighter
// bounds, coordinate-major boxes and the blocks (52 for all rows, the rest
// for those whose lists overflowed).
template <int KS>
__global__ __launch_bounds__(kThreads) void knn_collect_kernel(
    const float *__restrict__ xa, int64_t np, const float *__restrict__ xb, int64_t n, int d,
    const int32_t *__restrict__ perm, const float *__restrict__ box,
    const float *__restrict__ sub, const float *__restrict__ thr, int *__restrict__ count,
    int32_t *__restrict__ cand)
{
    constexpr int KP = 4 * KS;
    constexpr int kRow4 = kTileCols / 4;
    static_assert(kRowsPerGroup == kTileCols, "a row group is one tile");
    __shared__ floatx4 xs[2][KP * kRow4];
    __shared__ int tl[kThreads];                 // column tiles of the current chunk
    __shared__ unsigned short tm[kThreads];      // their blocks: bit 4 wave + q
    __shared__ int wcnt[kThreads / kWave];
    __shared__ float wmax[kThreads / kWave];
    __shared__ float rbox[32];
    __shared__ float rsub[kBlocks][32];          // the waves' rows
    __shared__ int nrow[kRowsPerGroup];          // candidates per row so far
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
    const int g = lane >> 4;
    const int m = lane & 15;
    const int64_t wrow0 = (int64_t)blockIdx.x * kRowsPerGroup + wave * 16;
    const int64_t i = wrow0 + m;                 // position in Morton order
    const int64_t ic = i < n ? i : n - 1;
    const int64_t io = (i < n) ? (int64_t)perm[i] : -1;   // the point it holds
    const float t_i = (i < n) ? thr[io] : -1.0f;
    const bool active = t_i >= 0.0f;
    const float t_pass = active ? t_i : -INFINITY;
    if (threadIdx.x < kRowsPerGroup)
        nrow[threadIdx.x] = 0;

    // a workgroup with no active row has nothing to collect
    if (__syncthreads_or(active) == 0)
        return;

    // the largest bound among each wave's and the workgroup's rows (widened
    // for the float32 gaps), and the boxes of the rows
    const int64_t ntiles = (n + kTileCols - 1) / kTileCols;
    const int64_t nsub = ntiles * kBlocks;
    float wm = t_i;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
        wm = fmaxf(wm, __shfl_xor(wm, o, kWave));
    if (lane == 0)
        wmax[wave] = (wm >= 0.0f) ? wm * (1.0f + 8e-6f) : -1.0f;
    if (threadIdx.x < 32)
        rbox[threadIdx.x] = box[threadIdx.x * ntiles + blockIdx.x];
    if (threadIdx.x < 32 * kBlocks)
        rsub[threadIdx.x / 32][threadIdx.x % 32] =
            sub[(threadIdx.x % 32) * nsub + (int64_t)blockIdx.x * kBlocks + threadIdx.x / 32];
    __syncthreads();
    float cut = wmax[0];
#pragma unroll
    for (int w = 1; w < kThreads / kWave; ++w)
        cut = fmaxf(cut, wmax[w]);

    float bop[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        bop[s] = xb[ic * KP + 4 * s + g];

    constexpr int kPieces = KP * kRow4;
    constexpr int kPer = (kPieces + kThreads - 1) / kThreads;
    floatx4 stage[kPer];
    auto fetch = [&](int64_t jt) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int f = threadIdx.x + u * kThreads;
            if (kPieces % kThreads == 0 || f < kPieces)
                stage[u] = *reinterpret_cast<const floatx4 *>(
                    xa + (int64_t)(f / kRow4) * np + jt + 4 * (f % kRow4));
        }
    };
    auto commit = [&](int buf) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int f = threadIdx.x + u * kThreads;
            if (kPieces % kThreads == 0 || f < kPieces) {
                const int k = f / kRow4;
                xs[buf][k * kRow4 + ((f % kRow4) ^ (4 * (k & 3)))] = stage[u];
            }
        }
    };

    for (int64_t c0 = 0; c0 < ntiles; c0 += kThreads) {
    // this chunk's tiles that may hold neighbours, in order
    bool pass = false;
    const int64_t tt = c0 + threadIdx.x;
    if (tt < ntiles) {
        float lb = 0.0f;
        for (int c = 0; c < d; ++c)
            lb = box_gap2(box[c * ntiles + tt], box[(16 + c) * ntiles + tt], rbox[c],
                          rbox[16 + c], lb);
        pass = !(lb > cut);
    }
    const unsigned long long bal = __ballot(pass);
    if (lane == 0)
        wcnt[wave] = __popcll(bal);
    __syncthreads();
    int before = 0, cnt = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
        before += (w < wave) ? wcnt[w] : 0;
        cnt += wcnt[w];
    }
    if (pass)
        tl[before + __popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (kWave - lane))))] = (int)tt;
    __syncthreads();
    if (cnt == 0)
        continue;                                // uniform over the workgroup
    // which of a tile's 4 x 4 blocks may hold neighbours: 16 lanes a tile,
    // lane 4 w + q the rows of wave w and the columns of block q
    for (int u0 = 0; u0 < cnt; u0 += kThreads / 16) {
        const int u = u0 + threadIdx.x / 16, w = (threadIdx.x / 4) % 4, q = threadIdx.x % 4;
        bool near = false;
        if (u < cnt) {
            const int64_t b = (int64_t)tl[u] * kBlocks + q;
            float lb = 0.0f;
            for (int c = 0; c < d; ++c)
                lb = box_gap2(sub[c * nsub + b], sub[(16 + c) * nsub + b], rsub[w][c],
                              rsub[w][16 + c], lb);
            near = !(lb > wmax[w]);
        }
        const unsigned long long mask = __ballot(near);
        if (u < cnt && threadIdx.x % 16 == 0)
            tm[u] = (unsigned short)(mask >> (lane & ~15));
    }
    __syncthreads();
    fetch((int64_t)tl[0] * kTileCols);
    commit(0);
    __syncthreads();
    for (int u = 0; u < cnt; ++u) {
        const int buf = u & 1;
        const int64_t jt = (int64_t)tl[u] * kTileCols;
        if (u + 1 < cnt)
            fetch((int64_t)tl[u + 1] * kTileCols);
        const float *tile = reinterpret_cast<const float *>(xs[buf]) + g * kTileCols;
        const int blocks = __builtin_amdgcn_readfirstlane((tm[u] >> (4 * wave)) & 15);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!((blocks >> q) & 1))
                continue;                        // uniform per wave
            floatx4 cacc = {0.0f, 0.0f, 0.0f, 0.0f};
            const float *ap = tile + ((16 * q + m) ^ (16 * g));
#pragma unroll
            for (int s = 0; s < KS; ++s)
                cacc = __builtin_amdgcn_mfma_f32_16x16x4f32(ap[4 * s * kTileCols], bop[s],
                                                            cacc, 0, 0, 0);
            if (!(fminf(fminf(cacc[0], cacc[1]), fminf(cacc[2], cacc[3])) <= t_pass))
                continue;
            const int64_t j0 = jt + 16 * q + 4 * g;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j = j0 + r;
                if (cacc[r] <= t_pass && j < n && j != i) {
                    const int c = atomicAdd(&nrow[16 * wave + m], 1);
                    if (c < kCap)
                        cand[io * kCap + c] = perm[j];
                }
            }
        }
        if (u + 1 < cnt) {
            commit(buf ^ 1);
            __syncthreads();
        }
    }
    __syncthreads();                             // tl and xs are refilled next chunk
    }
    if (g == 0 && active)
        count[io] = nrow[16 * wave + m];
}

// ------------------------------------------------------------- 3. select

// The k smallest (distance, index) of a row's `kept` candidates, P per lane
// in registers: k rounds of a wave minimum, the winner's lane dropping it.
// Returns the last one's distance.
template <int P>
__device__ __forceinline__ double select_row(const float *__restrict__ X, int d, int k,
                                             int64_t i, int kept,
                                             const int32_t *__restrict__ cand,
                                             int32_t *__restrict__ nbr)
{
    const int lane = threadIdx.x % kWave;
    double dv[P];
    int32_t jv[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
        const int e = u * kWave + lane;
        jv[u] = (e < kept) ? cand[i * kCap + e] : INT32_MAX;
        dv[u] = (e < kept) ? sq_dist64(X, d, i, jv[u]) : INFINITY;
    }
    double last = 0.0;
    for (int t = 0; t < k; ++t) {
        double bd = INFINITY;
        int32_t bj = INT32_MAX;
#pragma unroll
        for (int u = 0; u < P; ++u)
            if (dv[u] < bd || (dv[u] == bd && jv[u] < bj)) {
                bd = dv[u];
                bj = jv[u];
            }
        argmin_step<32>(bd, bj);
        argmin_step<16>(bd, bj);
        argmin_step<8>(bd, bj);
        argmin_step<4>(bd, bj);
        argmin_step<2>(bd, bj);
        argmin_step<1>(bd, bj);
#pragma unroll
        for (int u = 0; u < P; ++u)
            if (jv[u] == bj)
                dv[u] = INFINITY, jv[u] = INT32_MAX;
        if (lane == 0)
            nbr[i * k + t] = bj;
        last = bd;
    }
    return last;
}

// A wave per active row: float64 squared distances of the kept candidates
// (at most kCap), then k rounds of a wave argmin over (distance, index).
// nbr[i k + t] are the k nearest in order; kth[i] is the k-th distance; a
// row whose list overflowed is flagged.  Every round visits each lane's
// registers, so a row takes as few as its list needs: 2, 4, 8 or all 32 per
// lane (n = 2M, k = 32, 32 per lane always: 57 ms with 165
// candidates a row on average; 19 by their number; 15 with 70).
__global__ __launch_bounds__(kThreads) void knn_select_kernel(
    const float *__restrict__ X, int64_t n, int d, int k, const int *__restrict__ active,
    int *__restrict__ count, const int32_t *__restrict__ cand, int32_t *__restrict__ nbr,
    double *__restrict__ kth, int *__restrict__ flags)
{
    const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kWave;
    const int lane = threadIdx.x % kWave;
    if (i >= n || (active != nullptr && !active[i]))
        return;                                             // uniform per wave
    const int cnt = count[i];
    const int kept = cnt < kCap ? cnt : kCap;
    double last;
    if (kept <= 2 * kWave)
        last = select_row<2>(X, d, k, i, kept, cand, nbr);
    else if (kept <= 4 * kWave)
        last = select_row<4>(X, d, k, i, kept, cand, nbr);
    else if (kept <= 8 * kWave)
        last = select_row<8>(X, d, k, i, kept, cand, nbr);
    else
        last = select_row<kPerLane>(X, d, k, i, kept, cand, nbr);
    if (lane == 0) {
        kth[i] = last;
        if (cnt > kCap || last == INFINITY)
            atomicAdd(&flags[0], 1);
    }
}

// rows to collect again (count reset): the overflowed ones, and any with
// fewer than k candidates (an infinite k-th distance widens its bound to
// everything, so it overflows next and then shrinks)
__global__ __launch_bounds__(kThreads) void knn_rearm_kernel(int64_t n, int *__restrict__ count,
                                                             const double *__restrict__ kth,
                                                             int *__restrict__ active)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n)
        return;
    const int again = count[i] > kCap || kth[i] == INFINITY;
    active[i] = again;
    if (again)
        count[i] = 0;
}

__global__ __launch_bounds__(kThreads) void fill_i32_kernel(int *__restrict__ a, int64_t n,
                                                            int v)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        a[i] = v;
}

// --------------------------------------------------------- 4. symmetrise

// Both directions of every kNN edge as (row, column) keys; with rank, in
// the node numbering rank[point] (the Morton position) instead of point
// indices.
__global__ __launch_bounds__(kThreads) void edge_keys_kernel(const int32_t *__restrict__ nbr,
                                                             int64_t n, int k, int bits,
                                                             const int32_t *__restrict__ rank,
                                                             uint64_t *__restrict__ key)
{
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= n * k)
        return;
    uint64_t a = (uint64_t)(e / k), b = (uint64_t)nbr[e];
    if (rank != nullptr) {
        a = (uint64_t)rank[a];
        b = (uint64_t)rank[b];
    }
    key[2 * e] = (a << bits) | b;
    key[2 * e + 1] = (b << bits) | a;
}

// rank[perm[p]] = p: the node number of every point in Morton numbering
__global__ __launch_bounds__(kThreads) void rank_kernel(const int32_t *__restrict__ perm,
                                                        int64_t n, int32_t *__restrict__ rank)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p < n)
        rank[perm[p]] = (int32_t)p;
}

// first[p] = 1 where sorted key p differs from key p - 1
__global__ __launch_bounds__(kThreads) void first_flags_kernel(const uint64_t *__restrict__ key,
                                                               int64_t m,
                                                               uint32_t *__restrict__ first)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p < m)
        first[p] = (p == 0 || key[p] != key[p - 1]) ? 1u : 0u;
}

// After an exclusive scan of the flags: column, row start and weight of
// every distinct key; row_ptr[n] = nnz.  With perm, node r is point
// perm[r] (the weight comes from the points' coordinates).
__global__ __launch_bounds__(kThreads) void build_csr_kernel(
    const uint64_t *__restrict__ key, const uint32_t *__restrict__ pos, int64_t m, int bits,
    const float *__restrict__ X, int64_t n, int d, double two_sigma2,
    const int32_t *__restrict__ perm, int64_t *__restrict__ row_ptr,
    int32_t *__restrict__ col, float *__restrict__ val)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= m)
        return;
    const uint64_t kp = key[p];
    const bool first = (p == 0 || kp != key[p - 1]);
    const uint64_t mask = (1ull << bits) - 1;
    const int64_t r = (int64_t)(kp >> bits), c = (int64_t)(kp & mask);
    if (p == m - 1)
        row_ptr[n] = (int64_t)pos[p] + (first ? 1 : 0);
    if (!first)
        return;
    const int64_t q = pos[p];
    col[q] = (int32_t)c;
    const int64_t pr = (perm != nullptr) ? (int64_t)perm[r] : r;
    const int64_t pc = (perm != nullptr) ? (int64_t)perm[c] : c;
    val[q] = (float)exp(-sq_dist64(X, d, pr, pc) / two_sigma2);
    if (p == 0 || (int64_t)(key[p - 1] >> bits) != r)
        row_ptr[r] = q;
}

int bits_for(int64_t n)
{
    int b = 1;
    while (((int64_t)1 << b) < n)
        ++b;
    return b;
}

struct KnnLayout {
    size_t xa, xb, mpart, mu, tau, norm2, maxn, thr, count, active, cand, nbr, kth, flags,
        keyA, keyB, first, hist, hsum, permA, permB, box, total;
};

KnnLayout knn_layout(int64_t n, int32_t k)
{
    KnnLayout L{};
    const int64_t np = padded_points(n);
    const int64_t m = 2 * n * (int64_t)k;
    size_t o = 0;
    auto take = [&](int64_t bytes) {
        const size_t at = o;
        o += (size_t)al(bytes);
        return at;
    };
    L.xa = take(np * 20 * 4);               // KP <= 20 for d <= 16
    L.xb = take(np * 20 * 4);
    L.mpart = take(kMeanBlocks * 16 * 8);
    L.mu = take(16 * 8);
    L.tau = take(n * 4);
    L.norm2 = take(n * 4);
    L.maxn = take(4);
    L.thr = take(n * 4);
    L.count = take(n * 4);
    L.active = take(n * 4);
    L.cand = take(n * (int64_t)kCap * 4);
    L.nbr = take(n * (int64_t)k * 4);
    L.kth = take(n * 8);
    L.flags = take(4);
    L.keyA = take(m * 8);
    L.keyB = take(m * 8);
    L.first = take(m * 4);
    L.hist = take((int64_t)radix_hist_bytes(m));
    L.hsum = take((int64_t)(radix_hsum_bytes(m) > scan_sums_bytes(m) ? radix_hsum_bytes(m)
                                                                      : scan_sums_bytes(m)));
    L.permA = take(n * 4);
    L.permB = take(n * 4);
    L.box = take(np / kTileCols * 32 * 4);
    L.total = o;
    return L;
}

template <int D>
void launch_bound(int KT, const float *X, const int32_t *perm, int64_t n, int k,
                  const int32_t *near, float *tau, float *tmin, hipStream_t s)
{
    const int64_t nt = (n + kTileCols - 1) / kTileCols;
    constexpr int kRowTiles = kThreads / kWave;
    const dim3 grid((unsigned)((nt + kRowTiles - 1) / kRowTiles));
    switch (KT) {
    case 8:
        hipLaunchKernelGGL((knn_bound_kernel<D, 8>), grid, dim3(kThreads), 0, s, X, perm, n, nt, k,
                           near, tau, tmin);
        break;
    case 16:
        hipLaunchKernelGGL((knn_bound_kernel<D, 16>), grid, dim3(kThreads), 0, s, X, perm, n, nt, k,
                           near, tau, tmin);
        break;
    case 32:
        hipLaunchKernelGGL((knn_bound_kernel<D, 32>), grid, dim3(kThreads), 0, s, X, perm, n, nt, k,
                           near, tau, tmin);
        break;
    default:
        hipLaunchKernelGGL((knn_bound_kernel<D, 64>), grid, dim3(kThreads), 0, s, X, perm, n, nt, k,
                           near, tau, tmin);
        break;
    }
}

} // namespace

size_t knn_graph_ws(int64_t n, int32_t k) { return knn_layout(n, k).total; }

hipError_t run_knn_graph(const float *X, int64_t n, int d, int k, float sigma,
                         int64_t *row_ptr, int32_t *col, float *val, int64_t *nnz_host,
                         int *status_host, void *ws, hipStream_t s, int32_t *perm_out)
{
    const KnnLayout L = knn_layout(n, k);
    char *w = static_cast<char *>(ws);
    float *xa = (float *)(w + L.xa), *xb = (float *)(w + L.xb);
    double *mpart = (double *)(w + L.mpart), *mu = (double *)(w + L.mu);
    float *tau = (float *)(w + L.tau), *norm2 = (float *)(w + L.norm2);
    unsigned int *maxn = (unsigned int *)(w + L.maxn);
    float *thr = (float *)(w + L.thr);
    int *count = (int *)(w + L.count), *active = (int *)(w + L.active);
    int32_t *cand = (int32_t *)(w + L.cand), *nbr = (int32_t *)(w + L.nbr);
    double *kth = (double *)(w + L.kth);
    int *flags = (int *)(w + L.flags);
    uint64_t *keyA = (uint64_t *)(w + L.keyA), *keyB = (uint64_t *)(w + L.keyB);
    uint32_t *first = (uint32_t *)(w + L.first);
    uint32_t *hist = (uint32_t *)(w + L.hist), *hsum = (uint32_t *)(w + L.hsum);
    const unsigned rows_grid = (unsigned)((n + kThreads - 1) / kThreads);
    *status_host = 0;

    if (d < 1 || d > 16)
        return hipErrorInvalidValue;
    const int KS = ks_for(d);
    const int64_t np = padded_points(n);
    hipLaunchKernelGGL(mean_partials_kernel, dim3(kMeanBlocks), dim3(kThreads), 0, s, X, n, d,
                       mpart);
    hipLaunchKernelGGL(mean_finish_kernel, dim3(1), dim3(64), 0, s, mpart, kMeanBlocks, d, n,
                       mu);
    const unsigned pgrid = (unsigned)((np + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(knn_augment_kernel, dim3(pgrid), dim3(kThreads), 0, s, X, mu,
                       (const int32_t *)nullptr, n, np, d, 4 * KS, xa, xb, norm2);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(kThreads), 0, s, (int *)maxn,
                       (int64_t)1, 0);
    hipLaunchKernelGGL(max_norm_kernel, dim3(1024), dim3(kThreads), 0, s, norm2, n, maxn);
    // Morton order of the points, the operands in that order, tile boxes
    int32_t *perm = (int32_t *)(w + L.permA), *permB = (int32_t *)(w + L.permB);
    uint64_t *mkA = keyA, *mkB = keyB;
    hipLaunchKernelGGL(morton_key_kernel, dim3(rows_grid), dim3(kThreads), 0, s, X, mu,
                       (const unsigned int *)maxn, n, d, mkA, perm);
    hipError_t e0 = radix_sort_u64(mkA, perm, mkB, permB, n, 64, hist, hsum, s);
    if (e0 != hipSuccess)
        return e0;
    hipLaunchKernelGGL(knn_augment_kernel, dim3(pgrid), dim3(kThreads), 0, s, X, mu,
                       (const int32_t *)perm, n, np, d, 4 * KS, xa, xb, norm2);
    const int64_t ntiles = np / kTileCols;
    float *box = (float *)(w + L.box);
    // the sort's keys are done with until the edges: the blocks' boxes, the
    // near tiles and the tiles' smallest bounds take their place (at most 11
    // bytes a point and 772 more; of 40, and the sort's counts, 1,024 or more)
    size_t at = L.keyA;
    float *sub = (float *)(w + at);
    at += (size_t)al(ntiles * kBlocks * 32 * 4);
    int32_t *near = (int32_t *)(w + at);
    at += (size_t)al(ntiles * kNear * 4);
    float *tmin = (float *)(w + at);
    if (at + (size_t)ntiles * 4 > L.permA)
        return hipErrorInvalidValue;             // not reached
    hipLaunchKernelGGL(tile_box_kernel, dim3((unsigned)((ntiles * 16 + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, X, (const int32_t *)perm, n, d, ntiles, box, sub);
    hipLaunchKernelGGL(near_tiles_kernel, dim3((unsigned)ntiles), dim3(kThreads), 0, s,
                       (const float *)box, ntiles, d, near);

    // 1. bound: the near tiles and the Morton neighbours for every row, the
    // tiles nearest to the row itself where that is wide
    const int KT = k <= 8 ? 8 : k <= 16 ? 16 : k <= 32 ? 32 : 64;
#define GPIC_BOUND(D)                                                          \
    case D:                                                                    \
        launch_bound<D>(KT, X, perm, n, k, near, tau, tmin, s);                \
        break;
    switch (d) {
        GPIC_BOUND(1) GPIC_BOUND(2) GPIC_BOUND(3) GPIC_BOUND(4) GPIC_BOUND(5) GPIC_BOUND(6)
        GPIC_BOUND(7) GPIC_BOUND(8) GPIC_BOUND(9) GPIC_BOUND(10) GPIC_BOUND(11)
        GPIC_BOUND(12) GPIC_BOUND(13) GPIC_BOUND(14) GPIC_BOUND(15) GPIC_BOUND(16)
    default:
        return hipErrorInvalidValue;
    }
#undef GPIC_BOUND
    hipLaunchKernelGGL(refine_bound_kernel, dim3((unsigned)ntiles * kRefineParts),
                       dim3(kThreads), 0, s, X,
                       (const int32_t *)perm, (const float *)box, n, ntiles, d, k,
                       (const int *)nullptr, (const float *)tmin, tau);
    hipLaunchKernelGGL(threshold_kernel, dim3(rows_grid), dim3(kThreads), 0, s, tau,
                       (const double *)nullptr, norm2, maxn, n, d, 4 * KS,
                       (const int *)nullptr, thr);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(4096), dim3(kThreads), 0, s, count, n, 0);

    // 2-3. collect and select, again for overflowed rows
    const int *act = nullptr;
    for (int round = 0;; ++round) {
        const dim3 cgrid((unsigned)((n + kRowsPerGroup - 1) / kRowsPerGroup));
        if (KS <= 3)
            hipLaunchKernelGGL(knn_collect_kernel<3>, cgrid, dim3(kThreads), 0, s, xa, np,
                               xb, n, d, (const int32_t *)perm, (const float *)box, (const float *)sub, thr, count,
                               cand);
        else
            hipLaunchKernelGGL(knn_collect_kernel<5>, cgrid, dim3(kThreads), 0, s, xa, np,
                               xb, n, d, (const int32_t *)perm, (const float *)box, (const float *)sub, thr, count,
                               cand);
        hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(kThreads), 0, s, flags, (int64_t)1,
                           0);
        hipLaunchKernelGGL(knn_select_kernel,
                           dim3((unsigned)((n * kWave + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, s, X, n, d, k, act, count, cand, nbr, kth,
                           flags);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        int bad = 0;
        if ((e = hipMemcpyAsync(&bad, flags, sizeof(int), hipMemcpyDeviceToHost, s)) !=
                hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return e;
        if (bad == 0)
            break;
        if (round == 8) {                   // bounds that do not shrink: give up
            *status_host = 1;
            return hipSuccess;
        }
        hipLaunchKernelGGL(knn_rearm_kernel, dim3(rows_grid), dim3(kThreads), 0, s, n,
                           count, (const double *)kth, active);
        hipLaunchKernelGGL(refine_bound_kernel, dim3((unsigned)ntiles * kRefineParts),
                       dim3(kThreads), 0, s, X,
                           (const int32_t *)perm, (const float *)box, n, ntiles, d, k,
                           (const int *)active, (const float *)tmin, tau);
        hipLaunchKernelGGL(threshold_kernel, dim3(rows_grid), dim3(kThreads), 0, s, tau,
                           (const double *)kth, norm2, maxn, n, d, 4 * KS,
                           (const int *)active, thr);
        act = active;
    }

    // 4. symmetrise (in Morton numbering when the caller takes the order:
    // the sort's spare index buffer holds the ranks)
    const int bits = bits_for(n);
    const int64_t mm = 2 * n * (int64_t)k;
    int32_t *rank = nullptr;
    if (perm_out != nullptr) {
        rank = permB;
        hipLaunchKernelGGL(rank_kernel, dim3(rows_grid), dim3(kThreads), 0, s,
                           (const int32_t *)perm, n, rank);
    }
    hipLaunchKernelGGL(edge_keys_kernel, dim3((unsigned)((n * k + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, nbr, n, k, bits, (const int32_t *)rank, keyA);
    int32_t *none_a = nullptr, *none_b = nullptr;
    hipError_t e = radix_sort_u64(keyA, none_a, keyB, none_b, mm, (2 * bits + 7) / 8 * 8,
                                  hist, hsum, s);
    if (e != hipSuccess)
        return e;
    const unsigned egrid = (unsigned)((mm + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(first_flags_kernel, dim3(egrid), dim3(kThreads), 0, s, keyA, mm, first);
    if ((e = exclusive_scan_u32(first, mm, hsum, s)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(build_csr_kernel, dim3(egrid), dim3(kThreads), 0, s, keyA, first, mm,
                       bits, X, n, d, 2.0 * (double)sigma * (double)sigma,
                       perm_out != nullptr ? (const int32_t *)perm : nullptr, row_ptr, col,
                       val);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    if (perm_out != nullptr &&
        (e = hipMemcpyAsync(perm_out, perm, (size_t)n * 4, hipMemcpyDeviceToDevice, s)) !=
            hipSuccess)
        return e;
    if ((e = hipMemcpyAsync(nnz_host, row_ptr + n, sizeof(int64_t), hipMemcpyDeviceToHost,
                            s)) != hipSuccess)
        return e;
    return hipStreamSynchronize(s);
}

} // namespace gpic
