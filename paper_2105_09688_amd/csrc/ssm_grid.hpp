// ssm_grid.hpp -- the interaction sums of one large system in three (or two)
// dimensions, by way of a grid, in O(N) operations.
//
// In the scaled coordinates s (Ys) the pair term of particle i is
//   K_i = sum_j (s_j - s_i) 2^(-|s_j - s_i|^2) = grad Phi(s_i) / (2 a),
//   Phi(x) = sum_j e^(-a |x - s_j|^2),  a = ln 2.
// On a grid of spacing g, and with a window psi of W nodes,
//   e^(-a x^2) = sum_u sum_v psi(x - u) t(u - v) psi(v)      per dimension,
//   t^(k) = G^(k) g / psi^(k)^2 on |k| <= pi / g   (G the Gaussian, ^ Fourier),
// up to the window's aliases and what the Gaussian has beyond pi / g.  So K is
//   spread : psi of every particle onto the grid,
//   convolve: with t along two axes and with t' / (2 a) along the third (three
//             components), and
//   gather : the three fields with psi at every particle,
// W^3 nodes a particle each way in place of N pairs.  psi is the window
// e^(beta (sqrt(1 - z^2) - 1)), |z| <= 1 (Barnett, Magland, af Klinteberg, "A
// parallel nonuniform fast Fourier transform library based on an exponential
// of semicircle kernel", SIAM J. Sci. Comput. 41, 2019).
//
// Two dimensions are taken as a third coordinate of 0: that makes 8 times (FP64
// 16 times) the nodes a particle needs, on sums that are bound by their launches.
//
// All of it is in double precision in every precision mode.  Node values are
// added up as integers in units of 2^-qb: integer sums do not depend on their
// order, so runs stay bitwise reproducible with atomic additions, and a resumed
// run equals an uninterrupted one.  In FP64 the unit is 2^-52 at every N, and
// the sums over the grid are in two words of 64 bits: what a unit cuts off are
// the window's tails, the same for all particles, which the convolution
// amplifies (with one word, 2^-46 at N = 50021 and 2^-44 at 2^18, the error was
// 6.8e-15 and 3e-14 of the root mean square of K).
//
// A cloud that is too wide for the grid, or holds a particle that is not
// finite, is summed by the pair kernels as before: k_grid_bin marks in SysDev
// which of the two the tick takes, and the other's kernels return at once.
// So is a cloud that has contracted against the kernel's width.  The grid's
// error is a fraction of Phi (FP64 4e-17 to 1e-16, FP32 modes 2e-9 to 3e-9);
// that of sums over pairs is one of K, and in a cluster of spread r (root mean
// square distance from the mean, scaled) K is r Phi.  k_grid_bin leaves clouds
// of less spread than GridWin::least to the pair kernels.  Several tight
// clusters, or a tight one and a few particles far away, have any spread: the
// last block of the gather compares the root mean square of K with the mean of
// Phi (the sums of which come from the third convolution) and marks the tick as
// the pair kernels' below the same ratio.
#pragma once

#include "ssm_kernels.hpp"

#include <cmath>
#include <vector>

namespace ssm {

constexpr int kGridCell = 8;     // nodes of a bin along each axis
constexpr int kGridAxis = 128;   // first nodes along an axis at most: 16 bins
constexpr int kGridBins = (kGridAxis / kGridCell) * (kGridAxis / kGridCell) * (kGridAxis / kGridCell);
constexpr int kGridTab = 176;    // offsets of the convolution tables: kGridAxis + W - 1, rounded up to whole products
constexpr int kGridRange = 256;  // blocks of k_grid_range at most
constexpr int kGridRow = 10;     // a row of k_grid_range: lo[3], -hi[3], sums of s - s_0 [3] and |s - s_0|^2
constexpr int kGridPer = 4;      // particles per thread of k_grid_bin and k_grid_scatter
constexpr double kGridAlpha = 0.69314718055994530942;  // a = ln 2

// Window and spacing of a precision.  Error of K against the exact sums,
// relative to its root mean square (normal clouds in two and three dimensions of
// standard deviation 0.1 to 2.6, N = 20000 to 2^18, this arithmetic on the CPU):
// FP64 1.9e-16 to 2.9e-16, sums over pairs in double there 2.5e-16 to 8.8e-16;
// FP32 modes 4e-9 to 1e-8 (the direct FP32 terms carry 2e-8 and their plain sums
// 5e-7).  What decides it in FP64 beside the unit: a spacing whose multiples are
// exact, so that a particle's distance from its nodes carries no rounding of its
// distance from the grid's corner; a window whose exponent cancels nothing and
// has exact constants (grid_psi); and 16 nodes (14 at 0.2 with those: 3e-16 at
// best, 5e-16 over the range, between the jump at a low window's edge and the
// aliases of a high one; 14 without them 2.5e-15).
template <typename T>
struct GridWin;
template <>
struct GridWin<float> {
    static constexpr int W = 8;
    static constexpr double step = 0.28, beta = 2.55 * 8;
    static constexpr double rate = beta * 1.44269504088896340736;  // psi = 2^(rate (sqrt(1 - z^2) - 1))
    static constexpr int chunk = 512;  // particles of a bin that a workgroup takes at a time
    static constexpr int wg = 512, gather_wg = 1024;
    static constexpr int64_t nodes = 1 << 20;
    static constexpr bool two = false;  // node sums in two words
    static constexpr int unit = 42;     // node sums in units of 2^-unit at most
    static constexpr double least = 0.1;    // least K / Phi: an error of 2e-8 of K, a direct FP32 term's
};
template <>
struct GridWin<double> {
    static constexpr int W = 16;
    static constexpr double step = 0.25, rate = 6.875;  // psi = 2^(-rate t^2 / (8 + sqrt(64 - t^2))), t = 8 z
    static constexpr long double beta = 55 * 0.693147180559945309417232121458176568L;
    static constexpr int chunk = 256;
    static constexpr int wg = 1024, gather_wg = 1024;
    static constexpr int64_t nodes = 1 << 21;
    static constexpr bool two = true;
    static constexpr int unit = 52;
    static constexpr double least = 0.125;  // 3e-16 of K
};

// The tick's grid: lowest coordinates, nodes and bins along each axis, chunks.
struct GridDom {
    double lo[3];
    int32_t n[3], nb[3];
    int32_t use;      // 0: the pair kernels take the tick
    int32_t nchunks;
    unsigned long long k2;      // kGridK2 bits: sum of |K / N|^2 in units of 2^-kb; above: blocks of the gather done
};

struct GridRec {      // a particle in its bin's order
    double f[3];      // its first node's distance ahead, in [0, 1) of a step
    int32_t i;
    int32_t cell;     // its first node's place in the bin: x | y << 4 | z << 8
};

struct GridChunk {
    int32_t start, len, bin, pad;
};

struct GridArgs {
    int64_t P, off;                 // component stride and first slot of the system
    int32_t N, qb;                  // particles; unit 2^-qb of the node sums
    int32_t dim;                    // 3, or 2: the third coordinate is 0
    int32_t kb;                     // unit 2^-kb of the sum of |K / N|^2
    double k2unit;                  // 2^kb / N^2
    int32_t nphi;                   // wavefronts of k_grid_conv
    double scale;                   // pair_scale
    double* range;                  // [kGridRange][kGridRow]
    double* phi;                    // [nphi] parts of the sum of Phi over the particles
    GridDom* dom;
    SysDev* sys;
    uint32_t* count;                // [kGridBins], zero between ticks
    int2* key;                      // [N] bin and place in it
    GridRec* rec;                   // [N]
    GridChunk* chunks;
    unsigned long long* grid;       // [nodes] (two words: [2][nodes], kGridLow), zero between ticks
    double *A, *B;                  // [3][nodes] each
    const double* tab;              // [2][2 kGridTab]: t and t' / (2 a) at offsets -kGridTab ..
    double* out;                    // pairsum
};

// ---------------------------------------------------------------------------
// Host: t and t' / (2 a) at the grid's offsets.  Gauss-Legendre panels in long
// double; psi's integral in z = sin(theta), where it is smooth.
// ---------------------------------------------------------------------------
inline std::vector<double> grid_table(int W, double step, long double beta)
{
    typedef long double L;
    const L pi = 3.14159265358979323846264338327950288L, a = 0.693147180559945309417232121458176568L;
    constexpr int G = 20, panels = 12, n = G * panels;
    L gx[G], gw[G];
    for (int i = 0; i < G; ++i) {
        L x = std::cos(pi * (i + 0.75L) / (G + 0.5L)), dp = 0;
        for (int it = 0; it < 50; ++it) {
            L p0 = 1, p1 = x;
            for (int k = 2; k <= G; ++k) {
                const L p2 = ((2 * k - 1) * x * p1 - (k - 1) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = G * (x * p1 - p0) / (x * x - 1);
            const L dx = p1 / dp;
            x -= dx;
            if (std::fabs(dx) < 1e-19L) break;
        }
        gx[i] = x;
        gw[i] = 2 / ((1 - x * x) * dp * dp);
    }
    std::vector<L> X(n), Wt(n);  // nodes of [0, 1]
    for (int p = 0; p < panels; ++p)
        for (int i = 0; i < G; ++i) {
            X[p * G + i] = (p + 0.5L * (gx[i] + 1)) / panels;
            Wt[p * G + i] = 0.5L * gw[i] / panels;
        }
    const L hw = (L)W * (L)step / 2, kmax = pi / (L)step;
    std::vector<L> zq(n), pq(n);
    for (int q = 0; q < n; ++q) {  // even in theta: twice the half range
        const L th = X[q] * pi / 2, c = std::cos(th);
        zq[q] = std::sin(th) * hw;
        pq[q] = std::exp(beta * (c - 1)) * c * Wt[q] * (pi / 2) * hw * 2;
    }
    std::vector<L> t(kGridTab, 0), td(kGridTab, 0);
    for (int q = 0; q < n; ++q) {
        const L k = X[q] * kmax;
        L ph = 0;
        for (int u = 0; u < n; ++u) ph += pq[u] * std::cos(k * zq[u]);
        const L th = std::sqrt(pi / a) * std::exp(-k * k / (4 * a)) * (L)step / (ph * ph) * Wt[q] * kmax * (L)step / pi;
        const L c1 = std::cos(k * (L)step), s1 = std::sin(k * (L)step);
        L c = 1, s = 0;
        for (int m = 0; m < kGridTab; ++m) {
            t[m] += th * c;
            td[m] -= th * k * s / (2 * a);
            const L cn = c * c1 - s * s1;
            s = s * c1 + c * s1;
            c = cn;
        }
    }
    std::vector<double> tab(4 * kGridTab, 0.0);
    for (int m = 0; m < kGridTab; ++m) {
        tab[kGridTab + m] = (double)t[m];
        tab[3 * kGridTab + m] = (double)td[m];
        if (m > 0) {
            tab[kGridTab - m] = (double)t[m];
            tab[3 * kGridTab - m] = -(double)td[m];
        }
    }
    return tab;
}

// ---------------------------------------------------------------------------
// k_grid_range: the cloud's extent and sums for its spread (about the first
// particle, s_0), a row per block.  A coordinate that is not finite leaves
// -infinity as its lower end.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_min_f64(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}

// A row from the threads' rows, in every thread (kBlk / 64 wavefronts).
__device__ __forceinline__ void block_row(double (&m)[kGridRow], double (*part)[kGridRow])
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < kGridRow; ++k) m[k] = k < 6 ? wave_min_f64(m[k]) : wave_sum(m[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kGridRow; ++k) part[wave][k] = m[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kGridRow; ++k)
        m[k] = k < 6 ? fmin(fmin(part[0][k], part[1][k]), fmin(part[2][k], part[3][k]))
                     : (part[0][k] + part[1][k]) + (part[2][k] + part[3][k]);
}

template <typename T>
__global__ __launch_bounds__(kBlk) void k_grid_range(GridArgs g, const T* __restrict__ Ys)
{
    __shared__ double part[kBlk / 64][kGridRow];
    double m[kGridRow], s0[3];
#pragma unroll
    for (int k = 0; k < kGridRow; ++k) m[k] = k < 6 ? INFINITY : 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) s0[k] = k < g.dim ? (double)Ys[k * g.P + g.off] : 0.0;
    // in 64 bits: with up to 2^31 - 1 particles the index past the last one is not an int
    for (int64_t i = (int64_t)blockIdx.x * kBlk + threadIdx.x; i < g.N; i += (int64_t)gridDim.x * kBlk)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double x = k < g.dim ? (double)Ys[k * g.P + g.off + i] : 0.0;
            const bool ok = fabs(x) < INFINITY;
            m[k] = fmin(m[k], ok ? x : -INFINITY);
            m[k + 3] = fmin(m[k + 3], ok ? -x : -INFINITY);
            m[k + 6] += x - s0[k];
            m[9] = fma(x - s0[k], x - s0[k], m[9]);
        }
    block_row(m, part);
    if (threadIdx.x < kGridRow) {
        double v = m[0];
#pragma unroll
        for (int k = 1; k < kGridRow; ++k) v = (int)threadIdx.x == k ? m[k] : v;
        g.range[blockIdx.x * kGridRow + threadIdx.x] = v;
    }
}

// A coordinate's first node (ceil of its place on the grid), and how far that
// lies ahead in steps.  With lo a multiple of a step that is a short binary
// fraction (FP64), the node's coordinate and its distance are exact; at the
// edges of a cell the distance may leave [0, 1) by the rounding of the place.
template <typename T>
__device__ __forceinline__ int grid_place(double s, double lo, double* f)
{
    constexpr double step = GridWin<T>::step;
    const double v = (s - lo) * (1.0 / step), c = ceil(v);
    *f = sizeof(T) == 8 ? (fma(c, step, lo) - s) * (1.0 / step) : c - v;
    return (int)c;
}

// The tick's grid from the blocks' ranges: the same in every block.
template <typename T>
__device__ __forceinline__ GridDom grid_domain(const GridArgs& g, int nrange, double (*part)[kGridRow])
{
    constexpr int W = GridWin<T>::W;
    constexpr double least = GridWin<T>::least;
    double m[kGridRow];
#pragma unroll
    for (int k = 0; k < kGridRow; ++k)
        m[k] = (int)threadIdx.x < nrange ? g.range[threadIdx.x * kGridRow + k] : k < 6 ? INFINITY : 0.0;
    block_row(m, part);
    GridDom d;
    d.use = 1;
    d.nchunks = 0;
    d.k2 = 0;
    const double inv = 1.0 / (double)g.N;
    const double spread2 = m[9] * inv - ((m[6] * inv) * (m[6] * inv) + (m[7] * inv) * (m[7] * inv) + (m[8] * inv) * (m[8] * inv));
    if (!(spread2 >= least * least)) d.use = 0;  // also where it is NaN
    int64_t nodes = 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        constexpr double step = GridWin<T>::step;
        d.lo[k] = m[k];
        if (sizeof(T) == 8 && fabs(m[k]) < 0x1.0p40) d.lo[k] = floor(m[k] * (1.0 / step)) * step;
        const double e = ceil((-m[k + 3] - d.lo[k]) * (1.0 / step));
        const bool fits = e < (double)kGridAxis;  // false for NaN and infinities
        const int cells = fits ? (int)e + 1 : 1;
        if (!fits) d.use = 0;
        d.n[k] = cells + W - 1;
        d.nb[k] = (cells + kGridCell - 1) / kGridCell;
        nodes *= d.n[k];
    }
    if (nodes > GridWin<T>::nodes) d.use = 0;
    return d;
}

// First of a thread's kGridPer particles, kBlk apart, in k_grid_bin and k_grid_scatter.
__host__ __device__ constexpr int64_t grid_first(uint32_t block, uint32_t thread)
{
    return (int64_t)block * (kBlk * kGridPer) + thread;
}
// the last block of the largest system: none of its threads' places wraps around
static_assert(grid_first(0x7ffffffeu / (kBlk * kGridPer), kBlk - 1) + (kGridPer - 1) * kBlk == 0x7fffffff, "");

// ---------------------------------------------------------------------------
// k_grid_bin: the particles' bins and their places in them.  A block counts
// 1024 particles in LDS and takes its places in each bin with one addition.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlk) void k_grid_bin(GridArgs g, int nrange, const T* __restrict__ Ys)
{
    __shared__ double part[kBlk / 64][kGridRow];
    __shared__ uint32_t hist[kGridBins];
    const int64_t i0 = grid_first(blockIdx.x, threadIdx.x);
    double s[kGridPer][3];
#pragma unroll
    for (int u = 0; u < kGridPer; ++u)
#pragma unroll
        for (int k = 0; k < 3; ++k) s[u][k] = k < g.dim ? (double)Ys[k * g.P + g.off + min(i0 + u * kBlk, (int64_t)g.N - 1)] : 0.0;
    const GridDom d = grid_domain<T>(g, nrange, part);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *g.dom = d;
        g.sys->by_grid = d.use;
    }
    if (!d.use) return;
    const int bins = d.nb[0] * d.nb[1] * d.nb[2];
    for (int b = threadIdx.x; b < bins; b += kBlk) hist[b] = 0;
    __syncthreads();
    int bin[kGridPer], place[kGridPer];
#pragma unroll
    for (int u = 0; u < kGridPer; ++u) {
        int c[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double f;
            c[k] = grid_place<T>(s[u][k], d.lo[k], &f) / kGridCell;
        }
        bin[u] = (c[0] * d.nb[1] + c[1]) * d.nb[2] + c[2];
        if (i0 + u * kBlk < g.N) place[u] = (int)atomicAdd(&hist[bin[u]], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += kBlk) {
        const uint32_t c = hist[b];
        if (c) hist[b] = atomicAdd(&g.count[b], c);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kGridPer; ++u)
        if (i0 + u * kBlk < g.N) g.key[i0 + u * kBlk] = make_int2(bin[u], place[u] + (int)hist[bin[u]]);
}

// Sums made for other uses than a tick leave no mark for the ticks after them.
__global__ void k_grid_leave(GridArgs g)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) g.sys->by_grid = 0;
}

// Exclusive sums of v over the block's threads; *total: their sum.
__device__ __forceinline__ int block_scan(int v, int* wsum, int* total)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlk / 64; ++w) {
        if (w < wave) base += wsum[w];
        tot += wsum[w];
    }
    *total = tot;
    return base + x - v;
}

// ---------------------------------------------------------------------------
// k_grid_scatter: the particles in the order of their bins, and (block 0) the
// list of chunks: at most GridWin::chunk particles of one bin each.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlk) void k_grid_scatter(GridArgs g, const T* __restrict__ Ys)
{
    constexpr int kRun = kGridBins / kBlk, C = GridWin<T>::chunk;
    __shared__ int start[kGridBins];
    __shared__ int wsum[kBlk / 64];
    const GridDom d = *g.dom;
    if (!d.use) return;
    const int bins = d.nb[0] * d.nb[1] * d.nb[2];
    int c[kRun], sum = 0;
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
        const int b = threadIdx.x * kRun + q;
        c[q] = b < bins ? (int)g.count[b] : 0;
        sum += c[q];
    }
    int total;
    int at = block_scan(sum, wsum, &total);
    int nch = 0;
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
        start[threadIdx.x * kRun + q] = at;
        at += c[q];
        nch += (c[q] + C - 1) / C;
    }
    if (blockIdx.x == 0) {
        int ch = block_scan(nch, wsum, &total);
        for (int q = 0; q < kRun; ++q) {
            const int b = threadIdx.x * kRun + q;
            for (int a = 0; a < c[q]; a += C) g.chunks[ch++] = GridChunk{start[b] + a, min(C, c[q] - a), b, 0};
        }
        if (threadIdx.x == 0) g.dom->nchunks = total;
    }
    __syncthreads();
    const int64_t i0 = grid_first(blockIdx.x, threadIdx.x);
#pragma unroll
    for (int u = 0; u < kGridPer; ++u) {
        const int64_t i = i0 + u * kBlk;
        if (i >= g.N) break;
        const int2 k = g.key[i];
        GridRec r;
        r.i = (int32_t)i;
        r.cell = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double s = a < g.dim ? (double)Ys[a * g.P + g.off + i] : 0.0;
            r.cell |= (grid_place<T>(s, d.lo[a], &r.f[a]) % kGridCell) << (4 * a);
        }
        g.rec[start[k.x] + k.y] = r;
    }
}

// psi at node m of a particle's W, f in [0, 1) the first node's distance.  FP64:
// sqrt(1 - z^2) - 1 as -z^2 / (1 + sqrt(1 - z^2)), whose difference would lose
// beta roundings at the window's peak, and by t = z W / 2, so that no constant
// is rounded: an error that all particles share is not averaged.
template <typename T>
__device__ __forceinline__ double grid_psi(int m, double f)
{
    constexpr int W = GridWin<T>::W;
    constexpr double rate = GridWin<T>::rate;
    const double t = (double)(m - W / 2) + f;
    if constexpr (sizeof(T) == 4) {
        const double z = t * (2.0 / W);
        return exp2_fast(fma(rate, sqrt(fmax(fma(-z, z, 1.0), 0.0)), -rate));
    }
    const double q = W / 2 + sqrt(fmax(fma(-t, t, W * W / 4.0), 0.0)), r = rcp_fast(q);
    return exp2_fast(-rate * (t * t * fma(fma(-q, r, 1.0), r, r)));
}

// A bin's nodes in LDS: kGridCell + W - 1 along each axis.  W = 8: rows of 16,
// odd ones turned by 8, so that the 8 x 8 nodes of a wavefront meet every bank
// equally often.
template <typename T>
struct GridTile {
    static constexpr int E = kGridCell + GridWin<T>::W - 1;
    static constexpr int pitch = GridWin<T>::W == 8 ? 16 : E;
    static constexpr int size = E * E * pitch;
    static __device__ __forceinline__ int at(int x, int y, int z)
    {
        const int row = x * E + y;
        return row * pitch + (pitch == 16 ? (z ^ ((y & 1) << 3)) : z);
    }
};

// Weights of `n` particles from rec into w, 3 W (+ pad) each, by the threads t, t + nt, ...
template <typename T, int PITCH>
__device__ __forceinline__ void grid_weights(const GridRec* __restrict__ rec, int n, double* w, int t, int nt)
{
    constexpr int W = GridWin<T>::W;
    for (int q = t; q < n * 3 * W; q += nt) {
        const int p = q / (3 * W), r = q - p * (3 * W), a = r / W, m = r - a * W;
        w[p * PITCH + r] = grid_psi<T>(m, rec[p].f[a]);
    }
}

// ---------------------------------------------------------------------------
// k_grid_spread: a workgroup adds a chunk's particles into its bin's nodes in
// LDS, a wavefront one particle at a time (lanes: y and z), then into the grid.
// A value, at most 1, is rounded to units of 2^-qb by adding 2^(52 - qb), whose
// own bits are taken off again.  Bound by LDS atomics: W^3 / 64 a particle.
// Two words: the tile's sums are whole (256 particles of 2^52 units), the grid
// takes their kGridLow lower bits and the others, 0 at most nodes, apart; neither
// word can overflow below 2^31 particles.
// ---------------------------------------------------------------------------
constexpr int kGridLow = 38;

template <typename T>
__global__ __launch_bounds__(GridWin<T>::wg) void k_grid_spread(GridArgs g)
{
    constexpr int W = GridWin<T>::W, WG = GridWin<T>::wg, PB = W == 8 ? 8 : 2, R = W * W / 64;
    typedef GridTile<T> Tile;
    constexpr int E = Tile::E;
    __shared__ unsigned long long tile[Tile::size];
    __shared__ double wts[WG / 64][PB * 3 * W];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const GridDom d = *g.dom;
    if (!d.use) return;
    // at W = 8 the added bits stay in: a power of two, they are above bit 51, and
    // a chunk's sum of a node is below 2^51 (GridWin::unit)
    const double magic = ldexp(1.0, 52 - g.qb);
    const unsigned long long mbits = W == 8 ? 0 : (unsigned long long)__double_as_longlong(magic);
    constexpr unsigned long long keep = W == 8 ? (1ull << 52) - 1 : ~0ull;
    double* w = wts[wave];
    for (int ch = blockIdx.x; ch < d.nchunks; ch += gridDim.x) {
        const GridChunk c = g.chunks[ch];
        const int bx = c.bin / (d.nb[1] * d.nb[2]), by = c.bin / d.nb[2] % d.nb[1], bz = c.bin % d.nb[2];
        for (int q = threadIdx.x; q < Tile::size; q += WG) tile[q] = 0;
        __syncthreads();
        for (int p0 = wave * PB; p0 < c.len; p0 += WG / 64 * PB) {
            const GridRec* __restrict__ rec = g.rec + c.start + p0;
            const int n = min(PB, c.len - p0);
            const int cells = rec[min(lane, n - 1)].cell;
            grid_weights<T, 3 * W>(rec, n, w, lane, 64);
            wave_lds_fence();
            for (int p = 0; p < n; ++p) {
                const int cell = __builtin_amdgcn_readlane(cells, p);
                const int x0 = cell & 15, y0 = (cell >> 4) & 15, z0 = cell >> 8;
                double wyz[R];
                int at[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int y = lane / W + 64 / W * r, z = lane % W;
                    wyz[r] = w[p * 3 * W + W + y] * w[p * 3 * W + 2 * W + z];
                    at[r] = Tile::at(x0, y0 + y, z0 + z);
                }
#pragma unroll
                for (int x = 0; x < W; ++x) {
                    const double wx = w[p * 3 * W + x];
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        atomicAdd(&tile[at[r] + x * E * Tile::pitch],
                                  (unsigned long long)__double_as_longlong(fma(wx, wyz[r], magic)) - mbits);
                }
            }
            wave_lds_fence();
        }
        __syncthreads();
        for (int q = threadIdx.x; q < E * E * E; q += WG) {
            const int x = q / (E * E), y = q / E % E, z = q % E;
            const unsigned long long v = tile[Tile::at(x, y, z)] & keep;
            if (v) {  // nodes outside the grid hold nothing
                const int64_t node = ((int64_t)(bx * kGridCell + x) * d.n[1] + by * kGridCell + y) * d.n[2] + bz * kGridCell + z;
                if constexpr (GridWin<T>::two) {
                    const unsigned long long low = v & ((1ull << kGridLow) - 1), high = v >> kGridLow;
                    if (low) atomicAdd(&g.grid[node], low);
                    if (high) atomicAdd(&g.grid[GridWin<T>::nodes + node], high);
                } else {
                    atomicAdd(&g.grid[node], v);
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// k_grid_conv: one axis, the slowest of its input, which becomes the fastest
// of its output; three launches come back to the grid's own order.
//   pass 0: grid -> A = {t, t'}     pass 1: A -> B = {tt, tt', t't}
//   pass 2: B -> A = {t't t, t t' t, t t t'}, the three components' fields
// A pass is the product [lines x n] [n x n] with the Toeplitz matrix t(a - b),
// so it runs on the FP64 matrix instruction: a wavefront makes 16 lines x 32
// outputs, its table operands from LDS.  The wait for the input, four products
// of 4 nodes ahead, is what is left of its time.  On the vector units (4
// outputs a thread) the three passes took 54 us at 65^3 nodes and 87 us at
// 95^3, on it 24 and 33 us.
// Pass 1 also clears the bins' counts for the next tick, pass 2 the grid, whose
// product with t t t of it is the sum of Phi over the particles.
// ---------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));

// A node's sum in units of 2^-qb.
template <bool TWO>
__device__ __forceinline__ double grid_sum(const unsigned long long* raw, int64_t at, int64_t nodes)
{
    if constexpr (TWO) return fma((double)(long long)raw[nodes + at], (double)(1ull << kGridLow), (double)(long long)raw[at]);
    else return (double)(long long)raw[at];
}

template <int PASS, bool TWO>
__global__ __launch_bounds__(kBlk) void k_grid_conv(GridArgs g, int64_t nodes)
{
    constexpr int NIN = PASS + 1, NOUT = PASS == 0 ? 2 : 3, NACC = PASS == 2 ? 4 : NOUT, NT = 2, U = 4;
    __shared__ double tab[4 * kGridTab];
    const GridDom d = *g.dom;
    if (!d.use) return;
    for (int q = threadIdx.x; q < 4 * kGridTab; q += kBlk) tab[q] = g.tab[q];
    __syncthreads();
    const int n = d.n[PASS], inner = d.n[(PASS + 1) % 3] * d.n[(PASS + 2) % 3];
    const double* __restrict__ in = PASS == 1 ? g.A : g.B;
    const unsigned long long* __restrict__ raw = g.grid;
    double* __restrict__ out = PASS == 1 ? g.B : g.A;
    const double unit = ldexp(1.0, -g.qb);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int col = lane & 15, kk = lane >> 4;
    double phi = 0.0;
    const int qt = (inner + 15) / 16, work = qt * ((n + 16 * NT - 1) / (16 * NT));
    for (int it = blockIdx.x * (kBlk / 64) + wave; it < work; it += gridDim.x * (kBlk / 64)) {
        const int a0 = it / qt * (16 * NT), q0 = it % qt * 16;
        const int qc = min(q0 + col, inner - 1);
        const double* t = tab + kGridTab + a0 + col - kk;
        double sum[PASS == 2 ? NT : 1][4];  // the nodes' sums, on their way meanwhile
        if constexpr (PASS == 2) {
#pragma unroll
            for (int c = 0; c < NT; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    sum[c][r] = grid_sum<TWO>(g.grid, (int64_t)min(q0 + 4 * r + kk, inner - 1) * n + min(a0 + 16 * c + col, n - 1), nodes);
        }
        f64x4 acc[NACC][NT];
#pragma unroll
        for (int o = 0; o < NACC; ++o)
#pragma unroll
            for (int c = 0; c < NT; ++c) acc[o][c] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int b = 0; b < n; b += 4 * U) {
            double x[U][NIN];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = b + 4 * u + kk;
                const int64_t at = (int64_t)min(k, n - 1) * inner + qc;
#pragma unroll
                for (int f = 0; f < NIN; ++f) {
                    if constexpr (PASS == 0) x[u][f] = grid_sum<TWO>(raw, at, nodes);
                    else x[u][f] = in[f * nodes + at];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool live = b + 4 * u + kk < n;
#pragma unroll
                for (int f = 0; f < NIN; ++f) x[u][f] = live ? x[u][f] : 0.0;
#pragma unroll
                for (int c = 0; c < NT; ++c) {
                    const double tv = t[16 * c - b - 4 * u], dv = t[2 * kGridTab + 16 * c - b - 4 * u];
                    auto mul = [&](f64x4& z, double xv, double bv) { z = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, bv, z, 0, 0, 0); };
                    if constexpr (PASS == 0) {
                        mul(acc[0][c], x[u][0], tv);
                        mul(acc[1][c], x[u][0], dv);
                    } else if constexpr (PASS == 1) {
                        mul(acc[0][c], x[u][0], tv);
                        mul(acc[1][c], x[u][0], dv);
                        mul(acc[2][c], x[u][1], tv);
                    } else {
                        mul(acc[0][c], x[u][2], tv);
                        mul(acc[1][c], x[u][1], tv);
                        mul(acc[2][c], x[u][0], dv);
                        mul(acc[3][c], x[u][0], tv);
                    }
                }
            }
        }
        // value r of a lane: line 4 r + lane / 16, output lane % 16
#pragma unroll
        for (int o = 0; o < NOUT; ++o)
#pragma unroll
            for (int c = 0; c < NT; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = q0 + 4 * r + kk, a = a0 + 16 * c + col;
                    if (q < inner && a < n) out[o * nodes + (int64_t)q * n + a] = PASS == 0 ? acc[o][c][r] * unit : acc[o][c][r];
                }
        if constexpr (PASS == 2) {
#pragma unroll
            for (int c = 0; c < NT; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = q0 + 4 * r + kk, a = a0 + 16 * c + col;
                    if (q >= inner || a >= n) continue;
                    const int64_t at = (int64_t)q * n + a;  // the grid's own order again; nobody else has this node
                    phi = fma(acc[3][c][r], sum[c][r], phi);
                    g.grid[at] = 0;
                    if constexpr (TWO) g.grid[nodes + at] = 0;
                }
        }
    }
    if constexpr (PASS == 2) {
        phi = wave_sum(phi);
        if (lane == 0) g.phi[blockIdx.x * (kBlk / 64) + wave] = phi * unit;
    }
    if constexpr (PASS == 1) {
        const int bins = d.nb[0] * d.nb[1] * d.nb[2];
        for (int q = blockIdx.x * kBlk + threadIdx.x; q < bins; q += gridDim.x * kBlk) g.count[q] = 0;
    }
}

// |K / N|^2 of a component in units of 2^-kb (integers: no order), K / N <= 0.52;
// rounded as the spread rounds its values.
__device__ __forceinline__ unsigned long long grid_k2(const GridArgs& g, double K)
{
    return (unsigned long long)__double_as_longlong(fma(K * K, g.k2unit, 0x1.0p52)) & ((1ull << 52) - 1);
}

// The end of the gather: the blocks' sums of grid_k2 added up, and by the last
// of the `blocks` (< 1024) blocks the choice that the pair kernels after it read.
// Sum and count share a word, so that one atomic and no fence orders them.
constexpr int kGridK2 = 54;

template <typename T, int WG>
__device__ __forceinline__ void grid_judge(const GridArgs& g, unsigned long long k2, int blocks)
{
    __shared__ unsigned long long sums[WG / 64];
    __shared__ double parts[WG / 64];
    __shared__ int last;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) k2 += __shfl_xor(k2, o);
    if (lane == 0) sums[wave] = k2;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < WG / 64; ++w) k2 += sums[w];
        const unsigned long long was = atomicAdd(&g.dom->k2, k2 + (1ull << kGridK2));
        last = (int)(was >> kGridK2) == blocks - 1;
        k2 += was & ((1ull << kGridK2) - 1);
    }
    __syncthreads();
    if (!last) return;
    double p = 0.0;
    for (int q = threadIdx.x; q < g.nphi; q += WG) p += g.phi[q];
    p = wave_sum(p);
    if (lane == 0) parts[wave] = p;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < WG / 64; ++w) p += parts[w];
        const double n = (double)g.N, least = GridWin<T>::least;
        const double kk = ldexp((double)k2, -g.kb) / n;  // mean of |K / N|^2
        p /= n * n;                                       // mean of Phi / N
        if (!(kk >= least * least * p * p)) g.sys->by_grid = 0;
    }
}

// ---------------------------------------------------------------------------
// k_grid_gather: the pair term of a chunk's particles from the three fields at
// their bin's nodes, `group` lanes per particle, one for each z.  The nodes
// are staged through LDS, the next ones read into registers meanwhile.
//
// W = 8: all fields at once, {F0, F1} of a node and {F2(x), F2(x + 1)} side by
// side.  A particle's 16 lanes are 8 z of two neighbouring rows, and rows of
// 16 nodes, odd ones turned by 8, put them on all 64 banks once; they are the
// lanes that a 16-byte LDS read serves together (of a half wavefront the quads
// 0, 3, 5, 6 and 1, 2, 4, 7).  N = 2^18: 140 us before (a
// field at a time in single doubles, 8 lanes a particle: 43 % of the LDS cycles
// were conflicts), 82 us
// ---------------------------------------------------------------------------
template <int W, int WG, int E>
struct GridNodes {  // which nodes of the grid a thread stages
    static constexpr int per = (E * E * E + WG - 1) / WG;
    int at[per];    // -1: outside the grid
    __device__ __forceinline__ void set(const GridDom& d, int bin)
    {
        const int ox = bin / (d.nb[1] * d.nb[2]) * kGridCell, oy = bin / d.nb[2] % d.nb[1] * kGridCell, oz = bin % d.nb[2] * kGridCell;
#pragma unroll
        for (int u = 0; u < per; ++u) {
            const int q = threadIdx.x + u * WG, x = q / (E * E), y = q / E % E, z = q % E;
            const bool in = ox + x < d.n[0] && oy + y < d.n[1] && oz + z < d.n[2] && q < E * E * E;
            at[u] = in ? ((ox + x) * d.n[1] + oy + y) * d.n[2] + oz + z : -1;
        }
    }
    __device__ __forceinline__ double load(const double* __restrict__ F, int u) const
    {
        const double v = F[max(at[u], 0)];
        return at[u] < 0 ? 0.0 : v;
    }
};

__global__ __launch_bounds__(GridWin<float>::gather_wg) void k_grid_gather8(GridArgs g, int64_t nodes)
{
    constexpr int W = 8, WG = GridWin<float>::gather_wg, E = kGridCell + W - 1, SP = 18, ROW = 16;
    __shared__ double2 t01[E * E * ROW];
    __shared__ double2 t2[E * E * ROW];
    __shared__ double stage[WG / 64][4 * SP];
    const GridDom d = *g.dom;
    if (!d.use || (int)blockIdx.x >= d.nchunks) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int quad = lane >> 2, odd = (quad >> 2) & 1;
    const int z = (quad & 2) * 2 + (lane & 3), grp = (__popc(quad & 7) & 1) + 2 * (lane >> 5);
    double* __restrict__ st = stage[wave] + grp * SP;
    unsigned long long k2 = 0;
    GridNodes<W, WG, E> nd;
    double next[nd.per][3];
    GridChunk c = g.chunks[blockIdx.x];
    nd.set(d, c.bin);
#pragma unroll
    for (int u = 0; u < nd.per; ++u)
#pragma unroll
        for (int f = 0; f < 3; ++f) next[u][f] = nd.load(g.A + f * nodes, u);
    for (int ch = blockIdx.x; ch < d.nchunks; ch += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < nd.per; ++u) {
            const int q = threadIdx.x + u * WG;
            if (q < E * E * E) {
                const int row = q / E, at = row * ROW + ((q - row * E) ^ ((row % E & 1) << 3));
                t01[at] = make_double2(next[u][0], next[u][1]);
                t2[at].x = next[u][2];
                if (row >= E) t2[at - E * ROW].y = next[u][2];
            }
        }
        __syncthreads();
        const GridRec* __restrict__ rec = g.rec + c.start;
        const int len = c.len;
        if (ch + (int)gridDim.x < d.nchunks) {
            c = g.chunks[ch + gridDim.x];
            nd.set(d, c.bin);
#pragma unroll
            for (int u = 0; u < nd.per; ++u)
#pragma unroll
                for (int f = 0; f < 3; ++f) next[u][f] = nd.load(g.A + f * nodes, u);
        }
        for (int p0 = wave * 4; p0 < len; p0 += WG / 16) {
            const GridRec r = rec[min(p0 + grp, len - 1)];
            double wx[W], wy[W / 2];
            wave_lds_fence();
            st[odd ? W + (z & 1) * 4 + z / 2 : z] = grid_psi<float>(z, odd ? r.f[1] : r.f[0]);  // wx, then wy: even ones, odd ones
            const double wz = grid_psi<float>(z, r.f[2]);
            const int y0 = ((r.cell >> 4) & 15) + odd;
            const int base = ((r.cell & 15) * E + y0) * ROW + (((r.cell >> 8) + z) ^ ((y0 & 1) << 3));
            wave_lds_fence();
#pragma unroll
            for (int m = 0; m < W; ++m) wx[m] = st[m];
#pragma unroll
            for (int m = 0; m < W / 2; ++m) wy[m] = st[W + 4 * odd + m];
            double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int x = 0; x < W; x += 2) {
                double s[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
#pragma unroll
                for (int y = 0; y < W / 2; ++y) {
                    const double2 a = t01[base + (x * E + 2 * y) * ROW], b = t01[base + ((x + 1) * E + 2 * y) * ROW],
                                  e = t2[base + (x * E + 2 * y) * ROW];
                    s[0][0] = fma(wy[y], a.x, s[0][0]);
                    s[0][1] = fma(wy[y], a.y, s[0][1]);
                    s[0][2] = fma(wy[y], e.x, s[0][2]);
                    s[1][0] = fma(wy[y], b.x, s[1][0]);
                    s[1][1] = fma(wy[y], b.y, s[1][1]);
                    s[1][2] = fma(wy[y], e.y, s[1][2]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) acc[k] = fma(wx[x + 1], s[1][k], fma(wx[x], s[0][k], acc[k]));
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                acc[k] *= wz;
                acc[k] += dpp64<kDppXor1>(acc[k]);
                acc[k] += dpp64<kDppXor2>(acc[k]);
                acc[k] += dpp64<kDppMirror>(acc[k]);  // the quad of the other four z
                acc[k] += __shfl_xor(acc[k], 20);     // the other rows
            }
            if (!odd && z < g.dim && p0 + grp < len) {
                const double K = z == 0 ? acc[0] : z == 1 ? acc[1] : acc[2];
                g.out[z * g.P + g.off + r.i] = g.scale * K;
                k2 += grid_k2(g, K);
            }
        }
    }
    grid_judge<float, WG>(g, k2, min((int)gridDim.x, d.nchunks));
}

// W = 16: a field at a time in 97 KB, 16 lanes a particle, one for each z.  A
// lane keeps its three weights of each of its particles.  N = 50021: 231 us of a
// tick of 280; with 14 nodes and two workgroups a compute unit 152 of 250 (same
// trace).  Chunks of 128 and 64, a field's chunk as a work item of its own, the
// next field's nodes read ahead, and 32 lanes a particle without bank conflicts
// were all slower or the same: staging and waiting bound it.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(GridWin<double>::gather_wg) void k_grid_gather16(GridArgs g, int64_t nodes)
{
    typedef GridWin<double> Win;
    constexpr int W = Win::W, WG = Win::gather_wg, E = GridTile<double>::E, ROW = GridTile<double>::pitch, SP = 2 * W + 2,
                  Q = Win::chunk / (WG / 16);
    __shared__ double tile[GridTile<double>::size];
    __shared__ double stage[WG / 64][4 * SP];
    const GridDom d = *g.dom;
    if (!d.use || (int)blockIdx.x >= d.nchunks) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int z = lane & 15, grp = lane >> 4;
    unsigned long long k2 = 0;
    const int tx = threadIdx.x / (E * E), ty = threadIdx.x / E % E, tz = threadIdx.x % E;
    double* __restrict__ st = stage[wave] + grp * SP;
    for (int ch = blockIdx.x; ch < d.nchunks; ch += gridDim.x) {
        const GridChunk c = g.chunks[ch];
        const GridRec* __restrict__ rec = g.rec + c.start + wave * 4;
        const int len = c.len - wave * 4;  // particles from this wavefront's first on
        const int ox = c.bin / (d.nb[1] * d.nb[2]) * kGridCell, oy = c.bin / d.nb[2] % d.nb[1] * kGridCell,
                  oz = c.bin % d.nb[2] * kGridCell;
        double w[Q][3];
        int base[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q * (WG / 16) >= len) break;
            const GridRec r = rec[min(q * (WG / 16) + grp, len - 1)];
#pragma unroll
            for (int a = 0; a < 3; ++a) w[q][a] = grid_psi<double>(z, r.f[a]);
            base[q] = ((r.cell & 15) * E + ((r.cell >> 4) & 15)) * ROW + (r.cell >> 8) + z;
        }
#pragma unroll 1
        for (int f = 0; f < g.dim; ++f) {
            const double* __restrict__ F = g.A + f * nodes;
            __syncthreads();
            // node t of the tile, then t + WG, ...: x, y and z move on by WG's digits
            int x = tx, y = ty, zz = tz;
#pragma unroll 6
            for (int t = threadIdx.x; t < E * E * E; t += WG) {
                const bool in = ox + x < d.n[0] && oy + y < d.n[1] && oz + zz < d.n[2];
                const double v = F[in ? ((ox + x) * d.n[1] + oy + y) * d.n[2] + oz + zz : 0];
                tile[(x * E + y) * ROW + zz] = in ? v : 0.0;
                zz += WG % E;
                y += WG / E % E + (zz >= E);
                zz -= zz >= E ? E : 0;
                x += WG / (E * E) + (y >= E);
                y -= y >= E ? E : 0;
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int p = q * (WG / 16) + grp;
                if (q * (WG / 16) >= len) break;
                wave_lds_fence();
                st[z] = w[q][0];
                st[W + z] = w[q][1];
                wave_lds_fence();
                double wy[W], acc = 0.0;
#pragma unroll
                for (int m = 0; m < W; ++m) wy[m] = st[W + m];
#pragma unroll 2
                for (int x = 0; x < W; ++x) {
                    double s = 0.0;
#pragma unroll
                    for (int y = 0; y < W; ++y) s = fma(wy[y], tile[base[q] + (x * E + y) * ROW], s);
                    acc = fma(st[x], s, acc);
                }
                acc *= w[q][2];
                acc += dpp64<kDppXor1>(acc);
                acc += dpp64<kDppXor2>(acc);
                acc += dpp64<kDppHalfMirror>(acc);
                acc += dpp64<kDppMirror>(acc);
                if (z == 0 && p < len) {
                    g.out[f * g.P + g.off + rec[p].i] = g.scale * acc;
                    k2 += grid_k2(g, acc);
                }
            }
        }
    }
    grid_judge<double, WG>(g, k2, min((int)gridDim.x, d.nchunks));
}

}  // namespace ssm
