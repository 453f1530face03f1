// ssm_solo.hpp -- runs of small one-dimensional systems, one workgroup each.
//
// With the interaction by its modes (ssm_modes.hpp) a tick of a system of up
// to kSoloMax particles is so little work that a compute unit does it in less
// time than the barriers of the tiled kernel (ssm_small.hpp) or one launch
// take.  k_solo runs all ticks of an ssm_step call of one system in one
// workgroup: positions stay in registers, P particles a thread, and what the
// particles share (range, means, mode sums) goes through LDS, three workgroup
// barriers a tick.  Systems never meet, so no launch needs its workgroups to
// be resident together.
//
// The Brownian increments depend on no state.  k_solo_draw makes them for all
// ticks of the launch beforehand on the whole chip: inside the workgroup they
// would be the larger part of its work (at 1000 particles and 16 fine steps
// about 10 us a tick on one compute unit, 0.4 us spread over all).
//
// A tick of the small case (10 systems of 1000) took 18.6 us in FP64 and 8.6
// in FP32-compensated by the tiled kernel; 6.0 and 5.2 here, four wavefronts
// on one compute unit, bound by their issue (512 threads of two particles took
// 6.5 and 5.6, 1024 of one 9.8 and 9.3: the reductions of the mode sums are
// paid per wavefront).
#pragma once

#include "ssm_modes.hpp"

namespace ssm {

constexpr int kSoloMax = 2048;  // particles of a system at most: 512 threads of 4

// Most modes that k_solo takes for a system of N particles.  On its one compute
// unit a mode costs 0.06 + 6.6e-5 N us of a tick and the direct sums, FP64 and
// FP32, 30 and 17 us at N = 300, 181 and 93 at 1000, 626 and 168 at 2048.
__host__ __device__ constexpr int solo_cap(int32_t N, bool fp64)
{
    const int m = fp64 ? N : N / 2, top = fp64 ? kModeCap : 640;
    return m < 64 ? 64 : m < top ? m : top;
}

template <typename T>
struct SoloArgs {
    const SysDev* sys;
    Coef cf;
    int64_t P;            // slots
    int64_t t0, n;        // ticks t0 .. t0 + n - 1
    T* X;
    T* Y;
    T* Ys;
    const double* dW;     // [n][P] increments of the steps on those ticks
    Flags* flags;
    int32_t* nmax;
};

// The increments of ticks t0 .. t0 + n - 1 (blockIdx.y) of the listed blocks:
// dW[p][slot] where the system steps on tick t0 + p, as k_brownian_sum draws
// them for a system without a shared window.
template <int LP, bool F32>
__global__ __launch_bounds__(kBlk) void k_solo_draw(const BlkItem* __restrict__ items, const SysDev* __restrict__ sys,
                                                    Coef cf, int64_t P, int64_t t0, double* __restrict__ dW)
{
    const BlkItem it = items[blockIdx.x / LP];
    const SysDev S = sys[it.sys];
    const int64_t t = t0 + blockIdx.y;
    if (S.stride > 1 && t % S.stride != 0) return;
    const int q = threadIdx.x % LP;
    const int i = it.blk * kBlk + (int)(blockIdx.x % LP) * (kBlk / LP) + threadIdx.x / LP;
    double zs[kMaxD] = {0.0, 0.0, 0.0, 0.0};
    if (i < S.N) {
        const uint64_t q0 = (uint64_t)step_of(t, S.stride) * (uint64_t)S.r;
        stream_sum<1, F32>(cf.seed, (uint32_t)i, (uint64_t)S.ens, q0, q0 + (uint64_t)S.r, q0 / 4 + q, LP, zs);
    }
    lane_butterfly<LP, 1>(zs);
    if (q == 0 && i < S.N) dW[(int64_t)blockIdx.y * P + S.off + i] = cf.sqrt_hf * zs[0];
}

// Sums and range over a workgroup of WG threads, in every thread: the
// wavefronts' partial values meet in LDS, added in wavefront order.
template <int WG>
struct SoloRed {
    double a[2][WG / 64];
    float2 r[WG / 64];
};

// Largest Newton count of the thread's particles; failures and particles that
// are not finite are counted (flags may be null: the first solve of a launch
// repeats one that has been counted).
template <int P>
__device__ __forceinline__ int solo_solve(const SysDev& S, const Coef& cf, const bool (&valid)[P], const double (&x)[P],
                                          double xbar, double m2, double (&y)[P], Flags* flags)
{
    const double shift = S.h * cf.v_lam * xbar;
    const double alpha = 1.0 - S.h * (cf.v_rho - cf.v_kappa * m2);
    const double ha = S.h * (cf.v_cw ? cf.v_ak[0] : cf.v_a);
    double w[P];
    int it[P];
#pragma unroll
    for (int p = 0; p < P; ++p) w[p] = valid[p] ? x[p] + shift : 0.0;
    implicit_scalar<P>(w, alpha, ha, cf.newton_max_iter, y, it);
    int top = 0, fails = 0, bad = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        fails += (int)__popcll(__ballot(it[p] == -1));
        bad += (int)__popcll(__ballot(it[p] == -2));
        top = max(top, it[p]);
    }
    if (flags && (threadIdx.x & 63) == 0) {
        if (fails) atomicAdd(&flags->newton_fail, fails);
        if (bad) atomicAdd(&flags->nonfinite, bad);
    }
    return top;
}

template <typename T, bool PAIR, int WG, int P, bool WIDE>
__global__ __launch_bounds__(WG) void k_solo(SoloArgs<T> a)
{
    constexpr int kRows = WG / 16, kW = WG / 64;
    __shared__ __align__(32) double rows[PAIR ? kRows : 1][kRowVals + 16];
    __shared__ __align__(16) double2 g[PAIR ? kModeCap : 1];
    __shared__ SoloRed<WG> red;
    static_assert(!PAIR || sizeof(rows) >= WG * P * sizeof(T), "the direct sums stage the positions there");

    const SysDev S = a.sys[blockIdx.x];
    const Coef& cf = a.cf;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool valid[P];
    int64_t at[P];
    double x[P], y[P];
    int64_t step = (a.t0 + S.stride - 1) / S.stride;            // first step of the launch
    const int64_t end = (a.t0 + a.n + S.stride - 1) / S.stride;  // past its last
    if (step >= end) return;  // no step of this system falls on these ticks
    double dw[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = p * WG + (int)threadIdx.x;
        valid[p] = i < S.N;
        at[p] = S.off + min(i, S.N - 1);
        x[p] = (double)a.X[at[p]];
        dw[p] = a.dW[(step * S.stride - a.t0) * a.P + at[p]];
    }
    int top = 0;

    // moments of mu^X from the workgroup's particles, for a v that depends on them
    const bool mean_x = cf.v_lam != 0.0, mean_x2 = cf.v_kappa != 0.0;
    auto moments = [&](double& xbar, double& m2) {
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            s1 += valid[p] ? x[p] : 0.0;
            s2 += valid[p] ? x[p] * x[p] : 0.0;
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        __syncthreads();
        if (lane == 0) {
            red.a[0][wave] = s1;
            red.a[1][wave] = s2;
        }
        __syncthreads();
        s1 = s2 = 0.0;
#pragma unroll
        for (int w = 0; w < kW; ++w) {
            s1 += red.a[0][w];
            s2 += red.a[1][w];
        }
        xbar = mean_x ? s1 / (double)S.N : 0.0;
        m2 = mean_x2 ? s2 / (double)S.N : 0.0;
        __syncthreads();
    };

    // Y* of the first step, solved here from X, so that a run split over
    // launches or resumed from a saved state takes the same values
    {
        double xbar = 0.0, m2 = 0.0;
        if (!cf.fused) moments(xbar, m2);
        top = solo_solve<P>(S, cf, valid, x, xbar, m2, y, nullptr);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) y[p] = (double)(T)y[p];

    for (; step < end; ++step) {
        // the next step's increments are on their way during this one
        const int64_t nxt = min(step + 1, end - 1) * S.stride - a.t0;
        double dwn[P], ys[P];
#pragma unroll
        for (int p = 0; p < P; ++p) dwn[p] = a.dW[nxt * a.P + at[p]];
        // 1. mean of mu^Y, range of the scaled positions
        double sum = 0.0;
        float2 r = make_float2(INFINITY, -INFINITY);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            ys[p] = (double)(T)(cf.coord_scale * y[p]);
            sum += valid[p] ? y[p] : 0.0;
            if constexpr (PAIR) {
                const float2 q = position_range(valid[p], ys[p]);
                r.x = fminf(r.x, q.x);
                r.y = fmaxf(r.y, q.y);
            }
        }
        sum = wave_sum(sum);
        if constexpr (PAIR) wave_range(r.x, r.y);
        if (lane == 0) {
            red.a[0][wave] = sum;
            red.r[wave] = r;
        }
        __syncthreads();
        sum = 0.0;
#pragma unroll
        for (int w = 0; w < kW; ++w) {
            sum += red.a[0][w];
            if constexpr (PAIR) {
                r.x = fminf(r.x, red.r[w].x);
                r.y = fmaxf(r.y, red.r[w].y);
            }
        }
        const double ybar = sum / (double)S.N;
        double pair[P];
#pragma unroll
        for (int p = 0; p < P; ++p) pair[p] = 0.0;
        if constexpr (PAIR) {
            const ModeDom d = mode_domain((double)r.x, (double)r.y, solo_cap(S.N, sizeof(T) == 8), sizeof(T) == 8);
            if (d.M > 0) {
                // 2. the mode sums, as mode_block's, and their coefficients
                double zr[P], zi[P], wr[P], wi[P];
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    if (mode_anchored<T, WIDE>(d)) mode_power(mode_turn(ys[p], d), 1, &zi[p], &zr[p]);
                    else sincos_turn((ys[p] - d.c) * d.inv_L, &zi[p], &zr[p]);
                    wr[p] = valid[p] ? zr[p] : 0.0;
                    wi[p] = valid[p] ? zi[p] : 0.0;
                }
                for (int v0 = 0; v0 < 2 * d.M; v0 += kRowVals) {
                    const int v1 = min(v0 + kRowVals, 2 * d.M);
                    auto row = [&](int v) -> double& { return rows[threadIdx.x >> 4][v]; };
                    auto in = [&](int p) { return valid[p]; };
                    auto place = [&](int p) { return ys[p]; };
                    if (mode_anchored<T, WIDE>(d)) mode_values<P, WIDE>(v0, v1, d, wr, wi, zr, zi, row, in, place);
                    else mode_values<P, false>(v0, v1, d, wr, wi, zr, zi, row, in, place);
                    __syncthreads();
                    for (int v = threadIdx.x; v < v1 - v0; v += WG) {
                        double t = 0.0;
#pragma unroll
                        for (int q = 0; q < kRows; ++q) t += rows[q][v];
                        mode_coef(d, v0 + v, t, g);
                    }
                    __syncthreads();
                }
                // 3. evaluated, all of the thread's particles by the same coefficients
                if (mode_anchored<T, WIDE>(d)) mode_eval_anchored<P>(d, g, ys, pair);
                else mode_eval<P>(d.M, g, zr, zi, pair);
#pragma unroll
                for (int p = 0; p < P; ++p) pair[p] *= S.pair_scale;
            } else {
                // direct sums over the positions in LDS
                T* src = reinterpret_cast<T*>(&rows[0][0]);
#pragma unroll
                for (int p = 0; p < P; ++p) src[p * WG + threadIdx.x] = (T)ys[p];
                __syncthreads();
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const T yi[1] = {(T)ys[p]};
                    T out[1];
                    small_pairs<T, 1, sizeof(T) == 4>(src, 0, 0, S.N, yi, out);
                    pair[p] = (double)out[0] * S.pair_scale;
                }
                __syncthreads();
            }
        }
        // 4. the update (2.4), as update_block
#pragma unroll
        for (int p = 0; p < P; ++p) {
            double b = cf.b_c0 * y[p] + cf.b_lam * ybar + pair[p];
            if (cf.has_lin) {
                b += cf.b_const[0];
                b += cf.b_mat[0] * y[p];
                b += cf.b_mean[0] * ybar;
            }
            const double sig = cf.s0[0] + cf.s1[0] * y[p] + cf.s2[0] * ybar;
            x[p] = (double)(T)((y[p] + S.h * b) + sig * dw[p]);
            dw[p] = dwn[p];
        }
        // 5. the implicit step (2.3) of the next step
        double xbar = 0.0, m2 = 0.0;
        if (!cf.fused) moments(xbar, m2);
        else if constexpr (!PAIR) __syncthreads();  // red is written again by the next step
        top = max(top, solo_solve<P>(S, cf, valid, x, xbar, m2, y, a.flags));
#pragma unroll
        for (int p = 0; p < P; ++p) y[p] = (double)(T)y[p];
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (!valid[p]) continue;
        a.X[at[p]] = (T)x[p];
        a.Y[at[p]] = (T)y[p];
        a.Ys[at[p]] = (T)(cf.coord_scale * y[p]);
    }
    top = wave_max(top);
    // the counts have a slot for every 64 particles of the system
    if (lane == 0 && wave * 64 < S.N) atomicMax(a.nmax + (int64_t)S.blk0 * kSlotsPerBlk + wave, top);
}

}  // namespace ssm
