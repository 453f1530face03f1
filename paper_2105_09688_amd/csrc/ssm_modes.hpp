// ssm_modes.hpp -- the interaction sums in one dimension, in O(N) operations.
//
// In the scaled coordinate s (Ys) the pair term of particle x is
//   K(x) = sum_j q(s_j - x),   q(z) = z 2^(-z^2) = z e^(-a z^2),  a = ln 2.
// By Poisson summation, for every period L (k_m = 2 pi m / L),
//   sum_p q(z + p L) = sum_{m >= 1} c_m sin(k_m z),
//   c_m = (2 pi / L) / sqrt(4 pi a) (k_m / a) e^(-k_m^2 / (4 a)),
// exactly.  With L = D + G, D the extent of the system's cloud, the images
// p != 0 stay below G 2^(-G^2) for every pair, and the modes k_m > kmax below
// 0.68 e^(-kmax^2 / (4 a)).  G and kmax are taken so that both lie under the
// rounding of the sums they replace (mode_limits), so what is left is
//   K(x) = sum_{m <= M} c_m (S_m cos k_m x - C_m sin k_m x),
//   C_m + i S_m = sum_j e^(i k_m s_j)   (positions from the cloud's centre):
// one pass over the particles for the 2 M sums and one to evaluate them,
// M = kmax L / (2 pi), in place of N^2 / 2 exponentials.  All of it runs in
// double precision in every precision mode.
//
// The modes grow with the cloud's extent, and a context whose cloud is drawn too
// wide for them keeps the pair kernels (modes_pay in ssm.hip).  A cloud that
// becomes too wide for its particle count later (mode_cap), or holds a particle
// that is not finite, is summed directly in place of its modes (mode_direct):
// every ordered pair, as the small-system kernel does, so NaN and infinities
// spread as they do there; further blocks of k_modes, which return at once
// otherwise, take shares of the sources where the rows alone leave compute units
// idle.
//
// An exact tick is two launches: k_modes (the sums' partial rows; the Brownian
// increments and the means of mu^Y, which do not depend on them, in further
// blocks) and k_update_modes (adds the rows, evaluates, updates, solves the
// next implicit step and leaves the new cloud's range).  At N = 2^16 a tick
// takes 9.5 us where the symmetric pair sums alone took 345 (FP32-compensated)
// or 1300 us (FP64); it is bound by the two dependent launches and the
// latencies inside them, the arithmetic being about 1 us of the chip.  The domain depends on
// the current positions only, so a resumed run equals an uninterrupted one
// bit for bit.
#pragma once

#include "ssm_small.hpp"

namespace ssm {

constexpr int kModeChunk = 8;                  // modes between reductions over a wavefront
constexpr int kModeCap = 1024;                 // modes of a system at most
constexpr int kModeVals = 2 * kModeCap;        // values of a partial row at most: per chunk C_m x 8, S_m x 8
constexpr double kModeAlpha = 0.69314718055994530942;  // a = ln 2
constexpr double kTwoPi = 6.283185307179586476925286766559;

// Gap G and largest wavenumber kmax of a precision: image and truncation
// errors of one pair term, whose largest value is 0.52, below 5e-18 in FP64
// (a twentieth of a rounding) and 1e-11 in the FP32 modes (the direct sums'
// terms carry 3e-8 to 1e-7 there).
struct ModeLimits {
    double gap, kmax;
};

__host__ __device__ constexpr ModeLimits mode_limits(bool fp64) { return fp64 ? ModeLimits{7.8, 10.46} : ModeLimits{6.3, 8.35}; }

// Value v of partial row `row` is at mode_at(row, v): the 16 values of a chunk
// side by side, the rows of a chunk one after the other.  A system's rows are
// then read from consecutive addresses; rows of kModeVals doubles, 16 KiB
// apart, all met the same cache channels (the 256 rows of N = 2^16: 3.2 us of
// k_update_modes' 8).
__host__ __device__ constexpr int64_t mode_at(int64_t row, int v, int64_t rows)
{
    return ((v >> 4) * rows + row) * 16 + (v & 15);
}

// Particles [i0, i0 + n) of a system, n <= 256 P, into partial row `row`.
struct ModeItem {
    int32_t sys, row, i0, n;
};

// A system's domain this tick: centre, 1 / L and the number of modes, a
// multiple of kModeChunk (0: direct sums).
struct ModeDom {
    double c, inv_L;
    int32_t M, pad;
};

// Most modes that k_modes takes for a system of N particles; beyond, its direct
// sums are the cheaper: a mode costs 0.11 us of a tick and those take, FP64 and
// FP32, 21 and 15 us at N = 300, 38 and 27 at 4096, 66 and 42 at 8191, 190 and 57
// at 16384, beside 9 us of both.
__host__ __device__ constexpr int mode_cap(int32_t N, bool fp64)
{
    const float m = fp64 ? 190.0f + 5.5e-6f * (float)N * (float)N : 145.0f + 1.4e-6f * (float)N * (float)N;
    const float few = N > 64 ? (float)N : 64.0f, top = m < few ? m : few;
    return top < (float)kModeCap ? (int)top : kModeCap;
}

// The domain of the cloud between lo and hi, of at most `cap` modes.
__device__ __forceinline__ ModeDom mode_domain(double lo, double hi, int cap, bool fp64)
{
    const ModeLimits lim = mode_limits(fp64);
    const double L = (hi - lo) + lim.gap;
    const double m = ceil(lim.kmax / kTwoPi * L);
    ModeDom d{0.5 * (lo + hi), 1.0 / L, 0, 0};
    // an infinite range, or one that overflows, fails the comparison
    if (m <= (double)cap) d.M = ((int)m + kModeChunk - 1) / kModeChunk * kModeChunk;
    return d;
}

// A system's domain from its blocks' ranges; every thread of a kBlk block gets it.
__device__ __forceinline__ ModeDom system_domain(const SysDev& S, const float2* __restrict__ rng, bool fp64, float2* red)
{
    float lo = INFINITY, hi = -INFINITY;
    for (int b = threadIdx.x; b < S.nblk; b += kBlk) {
        const float2 r = rng[S.blk0 + b];
        lo = fminf(lo, r.x);
        hi = fmaxf(hi, r.y);
    }
    wave_range(lo, hi);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_float2(lo, hi);
    __syncthreads();
    lo = fminf(fminf(red[0].x, red[1].x), fminf(red[2].x, red[3].x));
    hi = fmaxf(fmaxf(red[0].y, red[1].y), fmaxf(red[2].y, red[3].y));
    return mode_domain((double)lo, (double)hi, mode_cap(S.N, fp64), fp64);
}

// cos and sin of 2 pi t for |t| <= 1/2: quadrant k = rint(4 t), the rest by
// the Taylor series of sincos_angle on [-pi/4, pi/4].
__device__ __forceinline__ void sincos_turn(double t, double* sn, double* cs)
{
    constexpr double sin_c[8] = {-0x1.5555555555555p-3, 0x1.1111111111111p-7, -0x1.a01a01a01a01ap-13,
                                 0x1.71de3a556c734p-19, -0x1.ae64567f544e4p-26, 0x1.6124613a86d09p-33,
                                 -0x1.ae7f3e733b81fp-41, 0x1.952c77030ad4ap-49};
    constexpr double cos_c[8] = {-0x1.0000000000000p-1, 0x1.5555555555555p-5, -0x1.6c16c16c16c17p-10,
                                 0x1.a01a01a01a01ap-16, -0x1.27e4fb7789f5cp-22, 0x1.1eed8eff8d898p-29,
                                 -0x1.93974a8c07c9dp-37, 0x1.ae7f3e733b81fp-45};
    const double k = rint(4.0 * t);
    const double r = fma(k, -0.25, t) * kTwoPi;
    const double r2 = r * r;
    double ps = sin_c[7], pc = cos_c[7];
#pragma unroll
    for (int j = 6; j >= 0; --j) {
        ps = fma(ps, r2, sin_c[j]);
        pc = fma(pc, r2, cos_c[j]);
    }
    const double sr = fma(r * r2, ps, r);
    const double cr = fma(r2, pc, 1.0);
    const int q = (int)k & 3;
    const double a = (q & 1) ? cr : sr;
    const double b = (q & 1) ? sr : cr;
    *sn = (q & 2) ? -a : a;
    *cs = ((q + 1) & 2) ? -b : b;
}

// A particle's place on the domain in turns, hi + lo: the phase of mode m is m
// times that, exact to the roundings of the last product.
struct Turn {
    double hi, lo;
};

__device__ __forceinline__ Turn mode_turn(double s, const ModeDom& d)
{
    const double x = s - d.c, b = x - s, xl = (s - (x - b)) - (d.c + b);  // x + xl = s - c
    const double t = x * d.inv_L;
    return Turn{t, fma(x, d.inv_L, -t) + xl * d.inv_L};
}

// e^(2 pi i m t).  The powers of a particle's e^(2 pi i t) by repeated products
// carry its rounding m times: FP64 clouds of more than kModePlain modes take
// every kModeAnchor-th power from here, in the sums and in the evaluation
// (relative RMS error at 536 modes 5.5e-15 without, 6.4e-16 with, sums over
// pairs 2.2e-16; at 80 modes 2e-16 in either case).  Only in the kernels of
// contexts whose cloud is drawn wider than half of that (WIDE): their code costs
// a tick of narrow ones 0.4 of 7 us.
constexpr int kModePlain = 64, kModeAnchor = 16;

__device__ __forceinline__ void mode_power(const Turn& t, int m, double* im, double* re)
{
    const double k = (double)m;
    sincos_turn(fma(k, t.lo, fma(k, t.hi, -rint(k * t.hi))), im, re);
}

// (re, im) = (re, im) z
__device__ __forceinline__ void rotate(double& re, double& im, double zr, double zi)
{
    const double t = im * zi;
    im = fma(re, zi, im * zr);
    re = fma(re, zr, -t);
}

// The next kModeChunk modes of a thread's P particles: their current powers w
// added up and moved on by z, and the 16 sums over each row of lanes (C_m x 8,
// S_m x 8) left in lanes 0 .. 15 of it.
template <int P>
__device__ __forceinline__ double mode_chunk(double (&wr)[P], double (&wi)[P], const double (&zr)[P], const double (&zi)[P])
{
    double acc[2 * kModeChunk];
#pragma unroll
    for (int u = 0; u < kModeChunk; ++u) {
        double c = wr[0], sn = wi[0];
#pragma unroll
        for (int p = 1; p < P; ++p) {
            c += wr[p];
            sn += wi[p];
        }
        acc[u] = c;
        acc[kModeChunk + u] = sn;
#pragma unroll
        for (int p = 0; p < P; ++p) rotate(wr[p], wi[p], zr[p], zi[p]);
    }
    return row_scatter(acc);
}

// The modes from value v0 on up to v1 (kModeChunk values of a pair of 16) of a
// block's particles into their rows of lanes.  ANCHOR: with the powers of
// mode_power; `in(p)` says whether the thread has a particle p, place(p) where.
template <int P, bool ANCHOR, typename Row, typename In, typename Place>
__device__ __forceinline__ void mode_values(int v0, int v1, const ModeDom& d, double (&wr)[P], double (&wi)[P],
                                            const double (&zr)[P], const double (&zi)[P], Row&& row, In&& in, Place&& place)
{
    for (int v = v0; v < v1; v += 2 * kModeChunk) {
        if constexpr (ANCHOR) {
            if (v > 0 && v % (2 * kModeAnchor) == 0) {
#pragma unroll
                for (int p = 0; p < P; ++p)
                    if (in(p)) mode_power(mode_turn(place(p), d), v / 2 + 1, &wi[p], &wr[p]);
            }
        }
        row(v - v0 + (threadIdx.x & 15)) = mode_chunk<P>(wr, wi, zr, zi);
    }
}

// Whether a system takes the anchored forms.
template <typename T, bool WIDE>
__device__ __forceinline__ bool mode_anchored(const ModeDom& d)
{
    static_assert(!WIDE || sizeof(T) == 8, "FP32 modes: the plain powers are exact enough");
    return WIDE && d.M > kModePlain;
}

// p = p z + g
__device__ __forceinline__ void horner(double& pr, double& pi, double zr, double zi, const double2 g)
{
    const double t = fma(pr, zr, fma(-pi, zi, g.x));
    pi = fma(pr, zi, fma(pi, zr, g.y));
    pr = t;
}

// The direct sum of the thread's target ys over share q of Q of its system's
// sources, in tiles of kDirectTile staged in LDS (compensated within a tile in
// FP32, the tiles' sums added in double).
constexpr int kDirectTile = 1024;

template <typename T>
__device__ __forceinline__ double mode_direct(const SysDev& S, const T* __restrict__ Ys, T ys, int q, int Q, T* src)
{
    double tot = 0.0;
    const int64_t len = ((int64_t)S.N + Q * kBlk - 1) / (Q * kBlk) * kBlk;
    const int64_t j1 = min((q + 1) * len, (int64_t)S.N);
    for (int64_t j0 = q * len; j0 < j1; j0 += kDirectTile) {
        const int n = (int)min((int64_t)kDirectTile, j1 - j0);
        __syncthreads();
        for (int p = threadIdx.x; p < n; p += kBlk) src[p] = Ys[S.off + j0 + p];
        __syncthreads();
        const T yi[1] = {ys};
        T out[1];
        small_pairs<T, 1, sizeof(T) == 4>(src, 0, 0, n, yi, out);
        tot += (double)out[0];
    }
    return tot;
}

// ---------------------------------------------------------------------------
// One partial row of the mode sums: the block's particles, P per thread.
// Wavefront rows of 16 lanes leave their sums in LDS (kRowVals at a time,
// enough for the 64 modes that almost every cloud stays below; rows 16 doubles
// further apart than that, so that two of them meet no bank twice), added in
// a fixed order.  A system without modes gets its particles' direct sums here
// instead, in pairsum, or, each of Q > 1 blocks of a row its share of the
// sources, in the row's own place (value q 256 P + j for particle j; Q P <= 8, so
// that they fit): the kernel that evaluates also moves the particles.
// ---------------------------------------------------------------------------
constexpr int kRowVals = 128;
constexpr int kModeRowsLds = kBlk / 16;  // rows of 16 lanes in a block

template <typename T, int P, bool WIDE>
__device__ __forceinline__ void mode_block(const ModeItem& it, const SysDev& S, const T* __restrict__ Ys,
                                           const float2* __restrict__ rng, ModeDom* __restrict__ dom,
                                           double* __restrict__ part, int64_t nrows_tot, int q, int Q,
                                           double* __restrict__ pairsum)
{
    __shared__ __align__(32) double rows[kModeRowsLds][kRowVals + 16];
    static_assert(sizeof(rows) >= kDirectTile * sizeof(T), "the direct sums stage their sources there");
    __shared__ float2 red[kBlk / 64];
    // the positions are on their way while the domain is reduced
    T s[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int j = min(p * kBlk + (int)threadIdx.x, it.n - 1);
        s[p] = Ys[S.off + it.i0 + j];
    }
    const ModeDom d = system_domain(S, rng, sizeof(T) == 8, red);
    if (q == 0 && it.row == S.mode_row0 && threadIdx.x == 0) dom[it.sys] = d;
    if (d.M == 0) {  // block-uniform
#pragma unroll 1
        for (int p = 0; p < P; ++p) {
            const int j = p * kBlk + (int)threadIdx.x;
            const T ys = j < it.n ? Ys[S.off + it.i0 + j] : (T)0;
            const double K = mode_direct(S, Ys, ys, q, Q, reinterpret_cast<T*>(&rows[0][0]));
            if (j >= it.n) continue;
            if (Q == 1) pairsum[S.off + it.i0 + j] = K * S.pair_scale;
            else part[mode_at(it.row, q * kBlk * P + j, nrows_tot)] = K;
        }
        return;
    }
    if (q > 0) return;
    double zr[P], zi[P], wr[P], wi[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const bool valid = p * kBlk + (int)threadIdx.x < it.n;
        if (mode_anchored<T, WIDE>(d)) mode_power(mode_turn((double)s[p], d), 1, &zi[p], &zr[p]);
        else sincos_turn(((double)s[p] - d.c) * d.inv_L, &zi[p], &zr[p]);
        wr[p] = valid ? zr[p] : 0.0;
        wi[p] = valid ? zi[p] : 0.0;
    }
    for (int v0 = 0; v0 < 2 * d.M; v0 += kRowVals) {
        const int v1 = min(v0 + kRowVals, 2 * d.M);
        auto row = [&](int v) -> double& { return rows[threadIdx.x >> 4][v]; };
        auto in = [&](int p) { return p * kBlk + (int)threadIdx.x < it.n; };
        auto place = [&](int p) { return (double)s[p]; };
        if (mode_anchored<T, WIDE>(d)) mode_values<P, WIDE>(v0, v1, d, wr, wi, zr, zi, row, in, place);
        else mode_values<P, false>(v0, v1, d, wr, wi, zr, zi, row, in, place);
        __syncthreads();
        for (int v = threadIdx.x; v < v1 - v0; v += kBlk) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < kModeRowsLds; ++q) t += rows[q][v];
            part[mode_at(it.row, v0 + v, nrows_tot)] = t;
        }
        if (v1 < 2 * d.M) __syncthreads();
    }
}

// n_modes blocks of mode sums and n_modes (Q - 1) for the further shares of direct
// sums (next to each other, so that they lie on as many compute units: N = 8191
// FP64 67 us, 100 with the shares last), then (up to n_main) the Brownian sums,
// then job.n blocks of system means.
template <typename T, int P, int LP, bool ONE, bool WIDE>
__global__ __launch_bounds__(kBlk) void k_modes(int n_modes, int Q, int n_main, SysDev one, const ModeItem* __restrict__ mitems,
                                                const BlkItem* __restrict__ items, const SysDev* __restrict__ sys,
                                                Coef cf, int64_t Pn, const T* __restrict__ Ys,
                                                const float2* __restrict__ rng, ModeDom* __restrict__ dom,
                                                double* __restrict__ part, int64_t nrows_tot,
                                                double* __restrict__ pairsum, int64_t tick_arg,
                                                const int64_t* __restrict__ tick_dev, const double* __restrict__ win,
                                                double* __restrict__ dW, YMeanJob job)
{
    if ((int)blockIdx.x < n_modes * Q) {
        const int q = Q == 1 ? 0 : (int)blockIdx.x / n_modes, row = (int)blockIdx.x - q * n_modes;
        if constexpr (ONE) {
            const int i0 = row * kBlk * P;
            mode_block<T, P, WIDE>(ModeItem{0, row, i0, min(kBlk * P, one.N - i0)}, one, Ys, rng, dom, part, nrows_tot, q, Q, pairsum);
        } else {
            const ModeItem it = mitems[row];
            mode_block<T, P, WIDE>(it, sys[it.sys], Ys, rng, dom, part, nrows_tot, q, Q, pairsum);
        }
    } else if ((int)blockIdx.x < n_main)
        brownian_block<1, LP, (sizeof(T) == 4)>(blockIdx.x - n_modes * Q, items, sys, cf, Pn, tick_arg, tick_dev, win, dW);
    else
        ymean_block<1>(blockIdx.x - n_main, job, sys, tick_arg, tick_dev);
}

// The thread's share of the sums over a system's rows of the values
// v0 + 32 q + 2 l, + 1 (l = threadIdx.x % 16, q < 2): rows threadIdx.x / 16 +
// 16 u.  Sixteen rows of both at a time (indexes past the end repeat the last
// row and count nothing), so that 256 rows are one round trip to memory.
struct RowBatch {
    double2 v[2][16];
};

__device__ __forceinline__ RowBatch row_batch(const double* __restrict__ part, int64_t nrows_tot, const SysDev& S, int v0,
                                              int r0)
{
    RowBatch b;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double2* p = reinterpret_cast<const double2*>(
            part + mode_at(S.mode_row0, v0 + 32 * q + 2 * (int)(threadIdx.x & 15), nrows_tot));
#pragma unroll
        for (int u = 0; u < 16; ++u) b.v[q][u] = p[(int64_t)min(r0 + 16 * u, S.mode_rows - 1) * 8];
    }
    return b;
}

__device__ __forceinline__ void add_batch(const RowBatch& b, int r0, int nrows, double2 (&a)[2])
{
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const bool in = r0 + 16 * u < nrows;
            a[q].x += in ? b.v[q][u].x : 0.0;
            a[q].y += in ? b.v[q][u].y : 0.0;
        }
}

// k_mode_total: the rows of each listed system added up once, into one row of
// `tot` per system (`vals` apart), 16 values at a time by 16 threads each.  Launched where
// the blocks of k_update_modes would together read many more rows than the
// systems have.
__global__ __launch_bounds__(kBlk) void k_mode_total(const int32_t* __restrict__ sys_list, const SysDev* __restrict__ sys,
                                                     const ModeDom* __restrict__ dom, const double* __restrict__ part,
                                                     int64_t nrows_tot, int vals, double* __restrict__ tot)
{
    __shared__ double stage[kBlk / 16][16];
    const int s = sys_list[blockIdx.x];
    const SysDev S = sys[s];
    const int V = 2 * dom[s].M;
    const int w = threadIdx.x >> 4, l = threadIdx.x & 15;
    for (int v0 = blockIdx.y * 16; v0 < V; v0 += gridDim.y * 16) {
        const double* p = part + mode_at(S.mode_row0, v0 + l, nrows_tot);
        double a = 0.0;
        int r = w;
        for (; r + 7 * 16 < S.mode_rows; r += 8 * 16) {
            double q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = p[(int64_t)(r + u * 16) * 16];
#pragma unroll
            for (int u = 0; u < 8; ++u) a += q[u];
        }
        for (; r < S.mode_rows; r += 16) a += p[(int64_t)r * 16];
        stage[w][l] = a;
        __syncthreads();
        if (threadIdx.x < 16) {
            double t = 0.0;
#pragma unroll
            for (int u = 0; u < kBlk / 16; ++u) t += stage[u][l];
            tot[(int64_t)s * vals + v0 + l] = t;
        }
        __syncthreads();
    }
}

// Value v of a system's sums, C_m or S_m, times c_m into the coefficients
// g_m = c_m (S_m + i C_m).
__device__ __forceinline__ void mode_coef(const ModeDom& d, int v, double sum, double2* g)
{
    const double delta = kTwoPi * d.inv_L;
    const double c0 = delta * 0.3388303758015525;  // 1 / sqrt(4 pi a)
    const int m = (v >> 4) * kModeChunk + (v & 7);  // from 0
    const double k = (double)(m + 1) * delta;
    // e^(-k^2 / (4 a)) = 2^(-k^2 / (4 a^2))
    const double c = c0 * (k * 1.4426950408889634) * exp2_fast<double>(k * k * -0.5203422452514019);
    double* gm = reinterpret_cast<double*>(g + m);
    gm[(v & 8) ? 0 : 1] = c * sum;
}

// The coefficients of a system from its rows, kCoefVals values (32 modes) a
// round; `first` are the first round's rows, fetched before the domain is
// known, since the rows are long enough for any.
constexpr int kCoefVals = 64;

__device__ __forceinline__ void mode_coefs(const ModeDom& d, const double* __restrict__ part, int64_t nrows_tot,
                                           const SysDev& S, const RowBatch& first, double2* g, double (*stage)[kCoefVals])
{
    const int w = threadIdx.x >> 4;
    for (int v0 = 0; v0 < 2 * d.M; v0 += kCoefVals) {
        double2 a[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
        if (v0 == 0) add_batch(first, w, S.mode_rows, a);
        for (int r0 = v0 == 0 ? w + 256 : w; r0 < S.mode_rows; r0 += 256)
            add_batch(row_batch(part, nrows_tot, S, v0, r0), r0, S.mode_rows, a);
#pragma unroll
        for (int q = 0; q < 2; ++q)
            *reinterpret_cast<double2*>(&stage[w][32 * q + 2 * (threadIdx.x & 15)]) = a[q];
        __syncthreads();
        const int v = v0 + (int)threadIdx.x;
        if (threadIdx.x < kCoefVals && v < 2 * d.M) {
            double t = 0.0;
#pragma unroll
            for (int u = 0; u < kBlk / 16; ++u) t += stage[u][threadIdx.x];
            mode_coef(d, v, t, g);
        }
        __syncthreads();
    }
}

// sum_m Re(g_m z^m) of P particles by Horner's rule; mode_eval_anchored: in
// pieces that begin at the powers of mode_power.
template <int P>
__device__ __forceinline__ void mode_eval(int M, const double2* g, const double (&zr)[P], const double (&zi)[P], double (&K)[P])
{
    double pr[P], pi[P];
#pragma unroll
    for (int p = 0; p < P; ++p) pr[p] = pi[p] = 0.0;
    constexpr int kUnrolled = P == 1 ? 8 : 4;
#pragma unroll kUnrolled
    for (int m = M - 1; m >= 0; --m) {
        const double2 gm = g[m];
#pragma unroll
        for (int p = 0; p < P; ++p) horner(pr[p], pi[p], zr[p], zi[p], gm);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) K[p] = fma(pr[p], zr[p], -pi[p] * zi[p]);
}

template <int P>
__device__ __forceinline__ void mode_eval_anchored(const ModeDom& d, const double2* g, const double (&s)[P],
                                                   double (&K)[P])
{
    double zr[P], zi[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        mode_power(mode_turn(s[p], d), 1, &zi[p], &zr[p]);
        K[p] = 0.0;
    }
    for (int a = 0; a < d.M; a += kModeAnchor) {
        double pr[P], pi[P];
#pragma unroll
        for (int p = 0; p < P; ++p) pr[p] = pi[p] = 0.0;
        for (int m = min(a + kModeAnchor, d.M) - 1; m >= a; --m) {
            const double2 gm = g[m];
#pragma unroll
            for (int p = 0; p < P; ++p) horner(pr[p], pi[p], zr[p], zi[p], gm);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            double wr, wi;
            mode_power(mode_turn(s[p], d), a + 1, &wi, &wr);
            K[p] += fma(pr[p], wr, -pi[p] * wi);
        }
    }
}

// The scaled pair term of one block's particles (each thread its own), from
// the rows of its system (TOTALS: from the one row that k_mode_total made of
// them; the sixteen loads in flight of the other form would cost the large
// contexts half of their wavefronts); stored in pairsum too, for whoever reads
// the exact term after the tick (the surrogate's check, the training sampler).
template <bool TOTALS>
struct ModeLds {
    double2 g[kModeCap];
    double stage[TOTALS ? 1 : kBlk / 16][kCoefVals];
};

// Where the shares of direct sums of a context lie: its partial rows, of `per`
// particles, Q > 1 shares each; `vals` values from one row of totals to the next.
struct DirectRows {
    const double* part;
    int per, Q, vals;
};

// Values of a partial row that hold the sums of a system of N particles.
__host__ __device__ constexpr int mode_vals(int32_t N, bool fp64)
{
    return (mode_cap(N, fp64) + kModeChunk - 1) / kModeChunk * 2 * kModeChunk;
}

// The scaled pair term of particle i of a system without modes: the shares added up.
__device__ __forceinline__ double direct_pair(const DirectRows& dr, const SysDev& S, int i, int64_t nrows_tot)
{
    const int row = i / dr.per, j = i - row * dr.per;
    double K = 0.0;
    for (int q = 0; q < dr.Q; ++q) K += dr.part[mode_at(S.mode_row0 + row, q * dr.per + j, nrows_tot)];
    return K * S.pair_scale;
}

template <typename T, bool TOTALS, bool WIDE>
__device__ __forceinline__ double mode_pair(const BlkItem it, const SysDev& S, const T* __restrict__ Ys,
                                            const ModeDom* __restrict__ dom, const double* __restrict__ part,
                                            int64_t nrows_tot, const DirectRows& dr,
                                            double* __restrict__ pairsum, ModeLds<TOTALS>& lds)
{
    const int i = it.blk * kBlk + threadIdx.x;
    const int64_t at = S.off + min(i, S.N - 1);
    const ModeDom d = dom[it.sys];
    const T ys = Ys[at];
    double zr, zi;
    if constexpr (TOTALS) {
        const double* row = part + (int64_t)it.sys * dr.vals;
        double a = row[threadIdx.x];
        if (d.M == 0) return pairsum[at];  // block-uniform; contexts with totals have Q = 1
        for (int v = threadIdx.x; v < 2 * d.M; v += kBlk) {
            if (v >= kBlk) a = row[v];
            mode_coef(d, v, a, lds.g);
        }
        sincos_turn(((double)ys - d.c) * d.inv_L, &zi, &zr);
        __syncthreads();
    } else {
        const RowBatch first = row_batch(part, nrows_tot, S, 0, threadIdx.x >> 4);
        if (d.M == 0) {
            if (dr.Q == 1) return pairsum[at];
            const double K = direct_pair(dr, S, min(i, S.N - 1), nrows_tot);
            if (i < S.N) pairsum[at] = K;
            return K;
        }
        sincos_turn(((double)ys - d.c) * d.inv_L, &zi, &zr);
        mode_coefs(d, part, nrows_tot, S, first, lds.g, lds.stage);
    }
    const double z0[1] = {zr}, z1[1] = {zi}, s0[1] = {(double)ys};
    double k0[1];
    if (mode_anchored<T, WIDE>(d)) mode_eval_anchored<1>(d, lds.g, s0, k0);
    else mode_eval<1>(d.M, lds.g, z0, z1, k0);
    const double K = k0[0] * S.pair_scale;
    if (i < S.N) pairsum[at] = K;
    return K;
}

// k_update_modes: k_update with the pair term evaluated here (d = 1).  ONE: a
// context of one system, passed as an argument, whose blocks are numbered by
// blockIdx: two loads less in the chain of dependent ones.
//
// At N = 8191 and 2^16 (one wavefront per SIMD) the kernel is that chain.  By
// its own clock it took 15500 cycles, of which 7700 until the rows had
// arrived, in six waits one after the other; 2700 in the implicit solve; 1100
// in the block's reductions.  Every load is issued before the first wait now.
template <typename T, bool TOTALS, bool ONE, bool WIDE>
__global__ __launch_bounds__(kBlk) void k_update_modes(SysDev one, const BlkItem* __restrict__ items,
                                                       const SysDev* __restrict__ sys, Coef cf, int64_t P, int64_t tick_arg,
                                                       const int64_t* __restrict__ tick_dev, T* __restrict__ X,
                                                       T* __restrict__ Y, T* Ys, const ModeDom* __restrict__ dom,
                                                       const double* __restrict__ part, int64_t nrows_tot,
                                                       DirectRows dr,
                                                       double* __restrict__ pairsum, const double* __restrict__ dWbuf,
                                                       const double* __restrict__ ymean, double* __restrict__ psumX,
                                                       double* __restrict__ psumY, int64_t nblk_tot, Flags* flags,
                                                       int32_t* __restrict__ nmax, float2* __restrict__ rng)
{
    __shared__ double red[kRedLds];
    __shared__ __align__(16) ModeLds<TOTALS> lds;
    const BlkItem it = ONE ? BlkItem{0, (int)blockIdx.x} : items[blockIdx.x];
    const SysDev S = ONE ? one : sys[it.sys];
    const int i = it.blk * kBlk + threadIdx.x;
    const UpdateIn<1> u = load_update<T, 1>(it.sys, S.off + min(i, S.N - 1), P, Y, dWbuf, ymean);
    touch_coefs(cf);
    const double pair[1] = {mode_pair<T, TOTALS, WIDE>(it, S, Ys, dom, part, nrows_tot, dr, pairsum, lds)};
    const int64_t n = step_of(tick_of(tick_dev, tick_arg), S.stride);
    update_block<T, 1>(it, S, cf, P, n, pair, u, X, Y, Ys, psumX, psumY, nblk_tot, flags, nmax, rng, red);
}

// k_mode_eval: the pair term alone into pairsum (the training sampler).
template <typename T, bool TOTALS, bool WIDE>
__global__ __launch_bounds__(kBlk) void k_mode_eval(const BlkItem* __restrict__ items, const SysDev* __restrict__ sys,
                                                    const T* __restrict__ Ys, const ModeDom* __restrict__ dom,
                                                    const double* __restrict__ part, int64_t nrows_tot,
                                                    DirectRows dr,
                                                    double* __restrict__ pairsum)
{
    __shared__ __align__(16) ModeLds<TOTALS> lds;
    const BlkItem it = items[blockIdx.x];
    (void)mode_pair<T, TOTALS, WIDE>(it, sys[it.sys], Ys, dom, part, nrows_tot, dr, pairsum, lds);
}

}  // namespace ssm
