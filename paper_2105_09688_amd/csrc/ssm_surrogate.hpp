// ssm_surrogate.hpp -- learned surrogate of the interaction drift (not in the
// paper): random-Fourier-feature moments of mu^Y and a small MLP
//   [hi(y) (d), lo(y) (d), C_1..C_K, S_1..S_K] -> 64 -> 64 -> 64 -> d,
// SiLU hidden layers, where hi(y) = bf16(y) and lo(y) = bf16(y - hi(y)) carry
// the position to about 16 significant bits through the BF16 input layer,
// BF16 operands with FP32 accumulation on the matrix cores (MFMA), trained
// on (y, moments, exact pair term) samples by hand-written kernels with Adam.
//
// Matrix-core tiles: v_mfma_f32_16x16x32_bf16.  For one wavefront (lane l):
//   A (16 x 32): lane holds A[l % 16][8 (l / 16) + 0..7]
//   B (32 x 16): lane holds B[8 (l / 16) + 0..7][l % 16]
//   D (16 x 16): lane holds D[4 (l / 16) + 0..3][l % 16]
// A wavefront always works on 16 samples (rows); features are columns.
#pragma once

#include <cstddef>

#include "ssm_kernels.hpp"

namespace ssm {

constexpr int kRff = 16;         // frequencies; 2 kRff moments
constexpr int kHid = 64;         // hidden width
constexpr int kKpad = 64;        // input features padded: 2 d + 2 kRff <= 40 -> 64
constexpr int kOutPad = 16;      // outputs padded to one 16-column tile
constexpr int kStride = 72;      // LDS/global row stride (bf16) of 64-wide rows (bank spread)
constexpr int kStrideT4 = 40;    // row stride of the transposed output layer (32 used)
constexpr int kRffWaves = 4;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Inference layout (k_mlp_infer, k_mlp_apply).  The products run transposed,
// D = W (16 outputs x K) * act^T (K x 16 samples): each lane then holds, for
// its sample l % 16, the outputs 16 nt + 4 (l / 16) + i of every output tile
// nt, which are exactly the eight K entries it must supply to the next layer's
// B operand once the next layer's input columns are taken in the order
//   K slice ks, entry k (0..31)  <->  input feature (2 ks + (k % 8) / 4) 16 + 4 (k / 8) + k % 4.
// So an activation never leaves its lane; the permutation is applied to the
// weights once, when they are packed, and every A operand is stored in lane
// order (lane l's 8 BF16 at [l]), one conflict-free 16-byte LDS read each.
// Layer 1 takes only the position columns [hi(y), lo(y)] on the matrix cores;
// the moment columns act on per-system constants, so their product with the
// moments is a per-system bias computed in FP32 (W1m below).
struct MlpInfer {
    bf16x8 W1[4][64];         // [out tile][lane]: W1[16 nt + l % 16][k], k = 8 (l / 16) + j < 2 d, else 0
    bf16x8 W2[4][2][64];      // [out tile][K slice][lane], permuted input columns
    bf16x8 W3[4][2][64];
    bf16x8 W4[2][64];         // [K slice][lane]: rows l % 16 < d
    float W1m[kHid][2 * kRff];  // moment columns of W1 (BF16 values) as float
};

// Packed device weights: BF16 row-major [out][in] rows padded to kStride, and
// the transposes needed by the backward pass; FP32 biases; the inference layout.
struct MlpPacked {
    __bf16 W1[kHid * kStride];      // [64 out][64 in (d + 2K used)]
    __bf16 W2[kHid * kStride];
    __bf16 W3[kHid * kStride];
    __bf16 W4[kOutPad * kStride];   // [16 out (d used)][64 in]
    __bf16 W2t[kHid * kStride];     // [64 in][64 out]
    __bf16 W3t[kHid * kStride];
    __bf16 W4t[kHid * kStrideT4];   // [64 in][32 out (d used)]
    float b1[kHid], b2[kHid], b3[kHid], b4[kOutPad];
    MlpInfer inf;
};

// Flat master layout (FP32), as the oracle's: W1[64][in] b1[64] W2[64][64] b2
// W3[64][64] b3 W4[d][64] b4[d], in = 2 d + 2 kRff network inputs.  Sample
// rows handed to the library are "raw": [y (d), moments (2 kRff)].
__host__ __device__ constexpr int mlp_in(int d) { return 2 * d + 2 * kRff; }
__host__ __device__ constexpr int raw_in(int d) { return d + 2 * kRff; }

__device__ __forceinline__ __bf16 bf_hi(float y) { return (__bf16)y; }
__device__ __forceinline__ __bf16 bf_lo(float y) { return (__bf16)(y - (float)(__bf16)y); }
__host__ __device__ constexpr int64_t mlp_params(int d)
{
    return (int64_t)kHid * mlp_in(d) + kHid + 2 * ((int64_t)kHid * kHid + kHid) + (int64_t)d * kHid + d;
}

struct MlpOffsets {
    int64_t W1, b1, W2, b2, W3, b3, W4, b4;
};

__host__ __device__ inline MlpOffsets mlp_offsets(int d)
{
    MlpOffsets o{};
    const int in = mlp_in(d);
    o.W1 = 0;
    o.b1 = o.W1 + (int64_t)kHid * in;
    o.W2 = o.b1 + kHid;
    o.b2 = o.W2 + kHid * kHid;
    o.W3 = o.b2 + kHid;
    o.b3 = o.W3 + kHid * kHid;
    o.W4 = o.b3 + kHid;
    o.b4 = o.W4 + (int64_t)d * kHid;
    return o;
}

__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// sigma(z) = 1 / (1 + e^-z) with the hardware reciprocal (v_rcp_f32, 1 ulp)
// instead of a correctly rounded division: the network's activations carry
// about 16 significant bits, and the division was most of SiLU's cost.  For
// z -> -inf, e^-z -> inf and the reciprocal gives 0.
__device__ __forceinline__ float sigmoid_f(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_f(z); }

__device__ __forceinline__ float silu_prime_f(float z)
{
    const float s = sigmoid_f(z);
    return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// Fresh master weights: each weight matrix uniform on +-sqrt(6 / (fan_in +
// fan_out)), biases zero.  Parameter p takes word p % 4 of the Philox block
// with counter (p / 4, 0, 0, 5 * 2^32) under key (seed, 0) (stream tag 5).
// ---------------------------------------------------------------------------
__global__ void k_mlp_init(uint64_t seed, int d, float* __restrict__ master)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const MlpOffsets o = mlp_offsets(d);
    if (p >= mlp_params(d)) return;
    int fan_in = 0, fan_out = 0;
    if (p < o.b1) { fan_in = mlp_in(d); fan_out = kHid; }
    else if (p >= o.W2 && p < o.b2) { fan_in = kHid; fan_out = kHid; }
    else if (p >= o.W3 && p < o.b3) { fan_in = kHid; fan_out = kHid; }
    else if (p >= o.W4 && p < o.b4) { fan_in = kHid; fan_out = d; }
    float v = 0.0f;
    if (fan_in > 0) {
        const Block4 b = philox4x64_10((uint64_t)(p / 4), 0ull, 0ull, (uint64_t)5 << 32, seed, 0ull);
        const double u = unit_open(b.w[p % 4]);
        v = (float)(sqrt(6.0 / (double)(fan_in + fan_out)) * (2.0 * u - 1.0));
    }
    master[p] = v;
}

// ---------------------------------------------------------------------------
// master (flat FP32) -> packed BF16 (+ transposes), zero padding
// ---------------------------------------------------------------------------
__global__ void k_mlp_pack(const float* __restrict__ master, int d, MlpPacked* __restrict__ P)
{
    const MlpOffsets o = mlp_offsets(d);
    const int in = mlp_in(d);
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    // t indexes a (row, col) of a 64 x 72 grid, reused for every matrix
    if (t >= kHid * kStride) return;
    const int r = t / kStride, c = t % kStride;
    auto bf = [](float x) { return (__bf16)x; };
    P->W1[t] = bf((c < in) ? master[o.W1 + (int64_t)r * in + c] : 0.0f);
    P->W2[t] = bf((c < kHid) ? master[o.W2 + (int64_t)r * kHid + c] : 0.0f);
    P->W3[t] = bf((c < kHid) ? master[o.W3 + (int64_t)r * kHid + c] : 0.0f);
    P->W2t[t] = bf((c < kHid) ? master[o.W2 + (int64_t)c * kHid + r] : 0.0f);  // [in r][out c]
    P->W3t[t] = bf((c < kHid) ? master[o.W3 + (int64_t)c * kHid + r] : 0.0f);
    if (r < kOutPad) P->W4[t] = bf((r < d && c < kHid) ? master[o.W4 + (int64_t)r * kHid + c] : 0.0f);
    if (c < kStrideT4) P->W4t[r * kStrideT4 + c] = bf((c < d) ? master[o.W4 + (int64_t)c * kHid + r] : 0.0f);
    if (c == 0) {
        P->b1[r] = master[o.b1 + r];
        P->b2[r] = master[o.b2 + r];
        P->b3[r] = master[o.b3 + r];
        if (r < kOutPad) P->b4[r] = (r < d) ? master[o.b4 + r] : 0.0f;
    }
}

// The inference layout of master (flat FP32) weights: A operands in lane
// order with the permuted input columns of layers 2-4, and the moment columns
// of W1 as float (of their BF16 values).
__host__ __device__ constexpr int infer_feature(int ks, int k) { return (2 * ks + (k % 8) / 4) * 16 + 4 * (k / 8) + k % 4; }

__global__ void k_mlp_pack_infer(const float* __restrict__ master, int d, MlpInfer* __restrict__ P)
{
    const MlpOffsets o = mlp_offsets(d);
    const int in = mlp_in(d);
    const int nW1 = 4 * 64 * 8, nW2 = 4 * 2 * 64 * 8, nW4 = 2 * 64 * 8, nM = kHid * 2 * kRff;
    const int total = nW1 + 2 * nW2 + nW4 + nM;
    // element stores through scalar pointers (flat index = the array's own
    // [..][lane][j] order): one thread per BF16 value, no shared 16-byte word
    __bf16* w1 = (__bf16*)P->W1;
    __bf16* w2 = (__bf16*)P->W2;
    __bf16* w3 = (__bf16*)P->W3;
    __bf16* w4 = (__bf16*)P->W4;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        int q = e;
        if (q < nW1) {
            const int nt = q / 512, l = (q / 8) % 64, j = q % 8, k = 8 * (l / 16) + j;
            w1[q] = (__bf16)((k < 2 * d) ? master[o.W1 + (int64_t)(16 * nt + l % 16) * in + k] : 0.0f);
            continue;
        }
        q -= nW1;
        if (q < 2 * nW2) {
            const int layer = q / nW2;
            q %= nW2;
            const int nt = q / 1024, ks = (q / 512) % 2, l = (q / 8) % 64, j = q % 8;
            const int f = infer_feature(ks, 8 * (l / 16) + j);
            const int64_t base = layer == 0 ? o.W2 : o.W3;
            (layer == 0 ? w2 : w3)[q] = (__bf16)master[base + (int64_t)(16 * nt + l % 16) * kHid + f];
            continue;
        }
        q -= 2 * nW2;
        if (q < nW4) {
            const int ks = q / 512, l = (q / 8) % 64, j = q % 8, m = l % 16;
            const int f = infer_feature(ks, 8 * (l / 16) + j);
            w4[q] = (__bf16)((m < d) ? master[o.W4 + (int64_t)m * kHid + f] : 0.0f);
            continue;
        }
        q -= nW4;
        const int r = q / (2 * kRff), c = q % (2 * kRff);
        P->W1m[r][c] = (float)(__bf16)master[o.W1 + (int64_t)r * in + 2 * d + c];
    }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two floats -> packed BF16 (one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pk_bf16(float a, float b)
{
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The training kernel's weights in LDS: the front of MlpPacked, as it is.
struct TrainLds {
    __bf16 W1[kHid * kStride], W2[kHid * kStride], W3[kHid * kStride], W4[kOutPad * kStride];
    __bf16 W2t[kHid * kStride], W3t[kHid * kStride], W4t[kHid * kStrideT4];
    float b[3 * kHid + kOutPad];
};
constexpr int kTrainCopies = (sizeof(TrainLds) / 16 + 255) / 256;  // 16-byte pieces a thread of 256 copies
static_assert(sizeof(TrainLds) % 16 == 0 && sizeof(TrainLds) == offsetof(MlpPacked, inf), "one flat copy");

// One dense layer for the wavefront's 16 samples: acc[nt] = A (16 x 64) * W^T
// for NT column tiles; W is LDS [NT*16][kStride] (row = output feature).
template <int NT>
__device__ __forceinline__ void dense_tiles(const __bf16* W, const bf16x8 a[2], f32x4 acc[NT])
{
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 b = *(const bf16x8*)&W[(nt * 16 + (l & 15)) * kStride + ks * 32 + 8 * (l >> 4)];
            c = mfma_bf16(a[ks], b, c);
        }
        acc[nt] = c;
    }
}
// Write 16 x (16 NT) values held in D layout into an LDS tile [16][kStride]
// as BF16, then read them back in A layout (two K slices of 32).
template <int NT>
__device__ __forceinline__ void d_to_a(const f32x4 v[NT], __bf16* tile, bf16x8 a[2])
{
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[(4 * (l >> 4) + i) * kStride + nt * 16 + (l & 15)] = (__bf16)v[nt][i];
    wave_lds_fence();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) a[ks] = *(const bf16x8*)&tile[(l & 15) * kStride + ks * 32 + 8 * (l >> 4)];
    wave_lds_fence();
}

// Input features of one sample in A layout (training): lane l holds features
// k = 32 ks + 8 (l / 16) + 0..7 of sample l % 16:  u = [hi(y), lo(y), m_0..m_{2K-1}, 0...],
// from a raw row r = [y (d), m (2K)] in global memory.  load_input_row fetches
// the values that the lane's features come from, build_input_row makes them.
template <int D>
__device__ __forceinline__ void load_input_row(const float* r, float (&u)[2][8])
{
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = ks * 32 + 8 * (l >> 4) + i;
            u[ks][i] = r[min(k < D ? k : k - D, raw_in(D) - 1)];
        }
}

template <int D>
__device__ __forceinline__ void build_input_row(const float (&u)[2][8], bf16x8 a[2])
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // only the first eight features (lanes of group 0) hold positions, only the last 32 padding
            float v = u[ks][i];
            if (ks == 0 && i >= D && i < 2 * D) v = g == 0 ? v - (float)bf_hi(v) : v;
            if (ks == 1) v = 8 * g + i < mlp_in(D) - 32 ? v : 0.0f;
            a[ks][i] = (__bf16)v;
        }
}

// Forward pass of the wavefront's 16 samples.  Returns the output tile
// (D layout, columns 0..d-1 valid, bias added), the pre-activations z1..z3 and
// the activations h1..h3 (D layout) for the backward pass.
__device__ __forceinline__ void mlp_forward16(const __bf16* sW1, const __bf16* sW2, const __bf16* sW3,
                                              const __bf16* sW4, const float* sb, bf16x8 a[2],
                                              __bf16* tile, f32x4 z[3][4], f32x4 h[3][4], f32x4& out)
{
    const int l = threadIdx.x & 63;
    const __bf16* Ws[3] = {sW1, sW2, sW3};
#pragma unroll
    for (int layer = 0; layer < 3; ++layer) {
        f32x4 acc[4];
        dense_tiles<4>(Ws[layer], a, acc);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const float bias = sb[layer * kHid + nt * 16 + (l & 15)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float zz = acc[nt][i] + bias;
                z[layer][nt][i] = zz;
                h[layer][nt][i] = silu_f(zz);
            }
        }
        d_to_a<4>(h[layer], tile, a);
    }
    f32x4 o[1];
    dense_tiles<1>(sW4, a, o);
    const float b4 = sb[3 * kHid + (l & 15)];
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = o[0][i] + b4;
}

// ---------------------------------------------------------------------------
// RFF moments: per-block sums of cos / sin(omega_k . y), FP32 terms added in
// double, then one block per (system, moment) adds its partials in order.  A
// wavefront's 32 sums are left by two reduce-scatters over its rows of lanes
// (256 values per moment one after the other in 32 threads took 19 us at
// N = 2^20; with the draws in further blocks 69 us of two launches are 63).
// ---------------------------------------------------------------------------
struct RffFreq {
    float w[kRff][kMaxD];  // omega_k (already divided by ell)
};

template <typename T, int D>
__device__ __forceinline__ void rff_block(int vb, const BlkItem* __restrict__ items, const SysDev* __restrict__ sys,
                                          int64_t P, const T* __restrict__ Y, const RffFreq& fq,
                                          double* __restrict__ part /*[nblk_tot][2K]*/)
{
    static_assert(kRff == 16, "a row of lanes per kind of moment");
    __shared__ double red[kBlk / 64][2 * kRff];
    const BlkItem it = items[vb];
    const SysDev S = sys[it.sys];
    const int i = it.blk * kBlk + threadIdx.x;
    const bool valid = i < S.N;
    float y[D];
#pragma unroll
    for (int k = 0; k < D; ++k) y[k] = valid ? (float)Y[k * P + S.off + i] : 0.0f;
    double c[kRff], s[kRff];
#pragma unroll
    for (int q = 0; q < kRff; ++q) {
        float ph = 0.0f;
#pragma unroll
        for (int k = 0; k < D; ++k) ph = fmaf(fq.w[q][k], y[k], ph);
        float sn, cs;
        __sincosf(ph, &sn, &cs);
        c[q] = valid ? (double)cs : 0.0;
        s[q] = valid ? (double)sn : 0.0;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double cv = row_scatter(c), sv = row_scatter(s);
    cv += __shfl_xor(cv, 16);
    sv += __shfl_xor(sv, 16);
    cv += __shfl_xor(cv, 32);
    sv += __shfl_xor(sv, 32);
    if (lane < 2 * kRff) red[wave][lane] = lane < kRff ? cv : sv;
    __syncthreads();
    if (threadIdx.x < 2 * kRff)
        part[(int64_t)(S.blk0 + it.blk) * (2 * kRff) + threadIdx.x] =
            (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

template <typename T, int D>
__global__ __launch_bounds__(kBlk) void k_rff_partial(const BlkItem* __restrict__ items,
                                                      const SysDev* __restrict__ sys, int64_t P,
                                                      const T* __restrict__ Y, RffFreq fq, double* __restrict__ part)
{
    rff_block<T, D>(blockIdx.x, items, sys, P, Y, fq, part);
}

// A network tick's moments and, in further blocks, what else does not depend
// on the network: the Brownian sums and the means of mu^Y.
template <typename T, int D, int LP>
__global__ __launch_bounds__(kBlk) void k_rff_prep(int n_rff, int n_main, const BlkItem* __restrict__ items,
                                                   const SysDev* __restrict__ sys, Coef cf, int64_t P,
                                                   const T* __restrict__ Y, RffFreq fq, double* __restrict__ part,
                                                   int64_t tick_arg, const int64_t* __restrict__ tick_dev,
                                                   const double* __restrict__ win, double* __restrict__ dW, YMeanJob job)
{
    if ((int)blockIdx.x < n_rff)
        rff_block<T, D>(blockIdx.x, items, sys, P, Y, fq, part);
    else if ((int)blockIdx.x < n_main)
        brownian_block<D, LP, (sizeof(T) == 4)>(blockIdx.x - n_rff, items, sys, cf, P, tick_arg, tick_dev, win, dW);
    else
        ymean_block<D>(blockIdx.x - n_main, job, sys, tick_arg, tick_dev);
}

// Sum over a system's block partials part[(blk0 + b) * stride + q], b < nblk:
// thread t adds b = t, t + kBlk, ... in order, then a fixed-order tree over
// the block.  All threads of the block must call it.
__device__ __forceinline__ double sum_block_partials(const double* __restrict__ part, int64_t blk0, int64_t nblk,
                                                     int stride, int q, double* red)
{
    double acc = 0.0;
    for (int64_t b = threadIdx.x; b < nblk; b += kBlk) acc += part[(blk0 + b) * stride + q];
    return block_sum(acc, red);
}

// grid (listed systems, 2K), kBlk threads: mom[sys][q] = (1/N) sum of its block partials
__global__ __launch_bounds__(kBlk) void k_rff_final(const int32_t* __restrict__ sys_list,
                                                    const SysDev* __restrict__ sys,
                                                    const double* __restrict__ part, float* __restrict__ mom)
{
    __shared__ double red[kRedLds];
    const int s = sys_list[blockIdx.x];
    const SysDev S = sys[s];
    const int q = blockIdx.y;
    const double t = sum_block_partials(part, S.blk0, S.nblk, 2 * kRff, q, red);
    if (threadIdx.x == 0) mom[(int64_t)s * (2 * kRff) + q] = (float)(t / (double)S.N);
}

// ---------------------------------------------------------------------------
// Inference (split precision).  Every activation enters the matrix cores as
// hi + lo with hi = bf16(v) and lo = bf16(v - hi) (about 16 significant bits),
// each product as W hi + W lo; the weights stay BF16 (the network is trained
// with them), so the network stays a smooth function of its inputs (plain
// BF16 activations add rounding noise of order 1e-3 relative that changes
// from one step to the next).  A wavefront runs two 16-sample tiles at a
// time in the transposed layout of MlpInfer.
// ---------------------------------------------------------------------------
// hi / lo B operands of 8 values (4 from each of two output tiles).
__device__ __forceinline__ void split8(const f32x4& a, const f32x4& b, bf16x8& hi, bf16x8& lo)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 h, l;
    const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t hp = pk_bf16(v[2 * q], v[2 * q + 1]);
        h[q] = hp;
        l[q] = pk_bf16(v[2 * q] - __uint_as_float(hp << 16), v[2 * q + 1] - __uint_as_float(hp & 0xffff0000u));
    }
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}

// The hidden layers run on scaled values u = -log2(e) z (pre-activations)
// and a~ = -log2(e) a (activations): every hidden layer's input and bias
// carry the factor, so its output is u directly (the product is linear), and
//   a~ = -log2(e) z sigma(z) = u / (1 + 2^u)
// with the hardware exp2 and reciprocal (sigma(z) = 1 / (1 + e^-z)).  The
// factor enters before the hi / lo split, so it costs no precision.  Layer 1
// scales its output (its inputs hi(y), lo(y) are features of their own, with
// their own weights, and are taken as they are); the output layer undoes the
// factor once.
constexpr float kNegLog2e = -1.4426950408889634f;
constexpr float kNegLn2 = -0.6931471805599453f;

__device__ __forceinline__ float silu_scaled(float u) { return u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u)); }

// SiLU of a layer's four output tiles (scaled), split into the next layer's
// operands (K slice 0: tiles 0, 1; slice 1: tiles 2, 3).
__device__ __forceinline__ void act_split(f32x4 (&acc)[4], bf16x8 (&hi)[2], bf16x8 (&lo)[2])
{
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[nt][i] = silu_scaled(acc[nt][i]);
    split8(acc[0], acc[1], hi[0], lo[0]);
    split8(acc[2], acc[3], hi[1], lo[1]);
}

// LDS copy of the inference weights and biases (-log2(e) b2, -log2(e) b3, -log2(e) b4).
struct InferLds {
    bf16x8 W1[4][64];
    bf16x8 W2[4][2][64];
    bf16x8 W3[4][2][64];
    bf16x8 W4[2][64];
    float b[2 * kHid + kOutPad];
};

__device__ __forceinline__ void load_infer(const MlpPacked* __restrict__ P, InferLds& L)
{
    const uint4* src[4] = {(const uint4*)P->inf.W1, (const uint4*)P->inf.W2, (const uint4*)P->inf.W3,
                           (const uint4*)P->inf.W4};
    uint4* dst[4] = {(uint4*)L.W1, (uint4*)L.W2, (uint4*)L.W3, (uint4*)L.W4};
    const int n[4] = {4 * 64, 8 * 64, 8 * 64, 2 * 64};
#pragma unroll
    for (int m = 0; m < 4; ++m)
        for (int q = threadIdx.x; q < n[m]; q += blockDim.x) dst[m][q] = src[m][q];
    for (int q = threadIdx.x; q < 2 * kHid + kOutPad; q += blockDim.x)
        L.b[q] = kNegLog2e * (q < kHid ? P->b2[q] : q < 2 * kHid ? P->b3[q - kHid] : P->b4[q - 2 * kHid]);
}

// acc[nt][i] = v[16 nt + 4 (l / 16) + i]: a bias vector in the D layout.
__device__ __forceinline__ void bias_tiles(const float* v, f32x4 (&acc)[4])
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[nt] = *(const f32x4*)&v[16 * nt + 4 * g];
}

// One hidden layer (64 -> 64) for two tiles; acc in: bias, out: pre-activation.
__device__ __forceinline__ void hidden_layer2(const bf16x8 (*W)[2][64], const bf16x8 (&h0)[2], const bf16x8 (&l0)[2],
                                              const bf16x8 (&h1)[2], const bf16x8 (&l1)[2], f32x4 (&a0)[4],
                                              f32x4 (&a1)[4])
{
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 w = W[nt][ks][l];
            a0[nt] = mfma_bf16(w, l0[ks], a0[nt]);
            a1[nt] = mfma_bf16(w, l1[ks], a1[nt]);
            a0[nt] = mfma_bf16(w, h0[ks], a0[nt]);
            a1[nt] = mfma_bf16(w, h1[ks], a1[nt]);
        }
}

// The network for two tiles of 16 samples.  yin[t][c]: coordinate c of the
// lane's sample l % 16 in tile t; c1[t]: layer 1's bias plus its moment part
// for tile t, in the D layout.  out[t]: D layout of the output tile (lane l,
// l < 16: components 0..3 of sample l; bias added).
template <int D>
__device__ __forceinline__ void mlp_infer_pair(const InferLds& L, const float (&yin)[2][kMaxD], f32x4 (&c1)[2][4],
                                               f32x4 (&out)[2])
{
    const int l = threadIdx.x & 63;
    const int g = l >> 4;
    // layer 1: K slice [hi(y), lo(y), 0 ...]; lanes of group 0 hold the entries
    bf16x8 x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            __bf16 v = (__bf16)0.0f;
            if (g == 0 && j < 2 * D) {
                const float y = yin[t][j < D ? j : j - D];
                v = j < D ? (__bf16)y : (__bf16)(y - (float)(__bf16)y);
            }
            x[t][j] = v;
        }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const bf16x8 w = L.W1[nt][l];
        c1[0][nt] = mfma_bf16(w, x[0], c1[0][nt]);
        c1[1][nt] = mfma_bf16(w, x[1], c1[1][nt]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) c1[t][nt][i] *= kNegLog2e;
    bf16x8 h0[2], l0[2], h1[2], l1[2];
    act_split(c1[0], h0, l0);
    act_split(c1[1], h1, l1);
    f32x4 a0[4], a1[4];
    bias_tiles(&L.b[0], a0);
    bias_tiles(&L.b[0], a1);
    hidden_layer2(L.W2, h0, l0, h1, l1, a0, a1);
    act_split(a0, h0, l0);
    act_split(a1, h1, l1);
    bias_tiles(&L.b[kHid], a0);
    bias_tiles(&L.b[kHid], a1);
    hidden_layer2(L.W3, h0, l0, h1, l1, a0, a1);
    act_split(a0, h0, l0);
    act_split(a1, h1, l1);
    out[0] = out[1] = *(const f32x4*)&L.b[2 * kHid + 4 * g];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 w = L.W4[ks][l];
        out[0] = mfma_bf16(w, l0[ks], out[0]);
        out[1] = mfma_bf16(w, l1[ks], out[1]);
        out[0] = mfma_bf16(w, h0[ks], out[0]);
        out[1] = mfma_bf16(w, h1[ks], out[1]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[t][i] *= kNegLn2;
}

// Layer 1's bias plus its moment columns times the moments m (FP32, ascending
// moment index), for output feature o.
__device__ __forceinline__ float layer1_const(const MlpPacked* __restrict__ P, int o, const float* m)
{
    float a = P->b1[o];
#pragma unroll 8
    for (int q = 0; q < 2 * kRff; ++q) a = fmaf(P->inf.W1m[o][q], m[q], a);
    return a;
}

// ---------------------------------------------------------------------------
// k_mlp_infer: surrogate pair term for every particle of the listed blocks
// (256 particles each): surr[k][slot] (FP32) for k < d.  Wavefront w takes
// the tiles 4 w .. 4 w + 3 of a block, two at a time.
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(256) void k_mlp_infer(const BlkItem* __restrict__ items, int n_items,
                                                   const SysDev* __restrict__ sys, int64_t P,
                                                   const T* __restrict__ Y, const float* __restrict__ mom,
                                                   const MlpPacked* __restrict__ W, float* __restrict__ surr,
                                                   double* __restrict__ part /*[nblk_tot][kMaxD]*/)
{
    __shared__ InferLds L;
    __shared__ __align__(16) float c1s[kHid];
    __shared__ double red[4][D];
    load_infer(W, L);
    const int wave = threadIdx.x >> 6;
    const int l = threadIdx.x & 63;
    int cur_sys = -1;
    for (int itx = blockIdx.x; itx < n_items; itx += gridDim.x) {
        const BlkItem it = items[itx];
        const SysDev S = sys[it.sys];
        if (it.sys != cur_sys) {  // block-uniform
            __syncthreads();
            if (threadIdx.x < kHid) c1s[threadIdx.x] = layer1_const(W, threadIdx.x, mom + (int64_t)it.sys * (2 * kRff));
            cur_sys = it.sys;
        }
        __syncthreads();
        double tot[D];
#pragma unroll
        for (int k = 0; k < D; ++k) tot[k] = 0.0;
#pragma unroll 1
        for (int tp = 0; tp < 2; ++tp) {
            const int i0 = it.blk * kBlk + (4 * wave + 2 * tp) * 16;
            if (i0 >= S.N) break;  // wave-uniform
            float yin[2][kMaxD] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int i = i0 + 16 * t + (l & 15);
#pragma unroll
                for (int k = 0; k < D; ++k) yin[t][k] = (i < S.N) ? (float)Y[k * P + S.off + i] : 0.0f;
            }
            f32x4 c1[2][4], out[2];
            bias_tiles(c1s, c1[0]);
            bias_tiles(c1s, c1[1]);
            mlp_infer_pair<D>(L, yin, c1, out);
            if (l < 16) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int i = i0 + 16 * t + l;
                    if (i < S.N)
#pragma unroll
                        for (int k = 0; k < D; ++k) {
                            surr[(int64_t)k * P + S.off + i] = out[t][k];
                            tot[k] += (double)out[t][k];
                        }
                }
            }
        }
        // the block's sums, for the mean that the tick takes off (k_surr_final)
#pragma unroll
        for (int k = 0; k < D; ++k) {
            tot[k] += dpp64<kDppXor1>(tot[k]);
            tot[k] += dpp64<kDppXor2>(tot[k]);
            tot[k] += dpp64<kDppHalfMirror>(tot[k]);
            tot[k] += dpp64<kDppMirror>(tot[k]);
            if (l == 0) red[wave][k] = tot[k];
        }
        __syncthreads();
        if (threadIdx.x < D)
            part[(int64_t)(S.blk0 + it.blk) * kMaxD + threadIdx.x] =
                (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
    }
}

// Inference on explicit raw rows U [n][d + 2K] -> out [n][d]: the same
// network, with layer 1's moment part computed per row (each lane for its
// sample and its 16 output features).
template <int D>
__global__ __launch_bounds__(256) void k_mlp_apply(const float* __restrict__ U, int64_t n,
                                                   const MlpPacked* __restrict__ W, float* __restrict__ out)
{
    __shared__ InferLds L;
    load_infer(W, L);
    __syncthreads();
    const int wave = threadIdx.x >> 6;
    const int l = threadIdx.x & 63;
    const int g = l >> 4;
    constexpr int in = raw_in(D);
    for (int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * 32; r0 < n; r0 += (int64_t)gridDim.x * 128) {
        float yin[2][kMaxD] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
        f32x4 c1[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t row = r0 + 16 * t + (l & 15);
            float m[2 * kRff];
#pragma unroll
            for (int q = 0; q < 2 * kRff; ++q) m[q] = row < n ? U[row * in + D + q] : 0.0f;
#pragma unroll
            for (int k = 0; k < D; ++k) yin[t][k] = row < n ? U[row * in + k] : 0.0f;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) c1[t][nt][i] = layer1_const(W, 16 * nt + 4 * g + i, m);
        }
        f32x4 o[2];
        mlp_infer_pair<D>(L, yin, c1, o);
        if (l < 16) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int64_t row = r0 + 16 * t + l;
                if (row < n)
#pragma unroll
                    for (int k = 0; k < D; ++k) out[row * D + k] = o[t][k];
            }
        }
    }
}

// Sampled training pairs of one system: u = [y_i, moments], t = exact pair term
// at particle i, for n draws of i (Philox tag 4, counter (q, 0, 1)).
template <typename T, int D>
__global__ void k_gather_samples(const SysDev* __restrict__ sys, int s, int64_t P, const T* __restrict__ Y,
                                 const double* __restrict__ pairsum, const float* __restrict__ mom, int64_t n,
                                 uint64_t seed, float* __restrict__ U, float* __restrict__ Tt)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const SysDev S = sys[s];
    const Block4 rb = philox4x64_10((uint64_t)q, 0ull, 1ull, 4ull << 32, seed, 0ull);
    const int64_t i = (int64_t)(rb.w[0] % (uint64_t)S.N);
    const int64_t slot = S.off + i;
    const int in = raw_in(D);
#pragma unroll
    for (int k = 0; k < D; ++k) {
        U[q * in + k] = (float)Y[k * P + slot];
        Tt[q * D + k] = (float)pairsum[k * P + slot];
    }
    for (int m = 0; m < 2 * kRff; ++m) U[q * in + D + m] = mom[(int64_t)s * (2 * kRff) + m];
}

// ---------------------------------------------------------------------------
// Training, two launches a step.  k_train_fwdbwd: samples drawn with
// replacement by Philox (tag 4) from the sample set; forward, loss and
// back-propagated deltas.  k_train_wgrad: weight gradients, Adam, packing.
// ---------------------------------------------------------------------------
// Row `row` of minibatch `step`: a uniform draw (with replacement) from the
// sample set, Philox stream tag 4; or row itself for sequential batches.
__device__ __forceinline__ int64_t sample_index(int row, int64_t step, uint64_t seed, int64_t n, int sequential)
{
    if (sequential) return (int64_t)row % n;
    const Block4 rb = philox4x64_10((uint64_t)row, (uint64_t)step, 0ull, 4ull << 32, seed, 0ull);
    return (int64_t)(rb.w[0] % (uint64_t)n);
}

// Activations and deltas between the two kernels of a training step, in BF16,
// already in the order of the matrix-core operands that k_train_wgrad reads:
// per 32 samples and tile of 16 features, lane l holds feature l % 16 of the
// samples 8 (l / 16) .. + 7 (16 bytes).
struct TrainBufs {
    __bf16* act[4];    // act[0]: inputs; act[1..3]: SiLU outputs, 4 tiles each
    __bf16* delta[4];  // delta[0..2]: dL/dz of hidden layers 1..3, 4 tiles; delta[3]: dL/dy, 1 tile
    float* loss_part;  // [B / 64]
};

// The four samples 4 (l / 16) + r of a wavefront's 16 (samples b0 ..) at
// feature l % 16 of a tile: eight bytes of an operand in TrainBufs.
__device__ __forceinline__ void store_operand(__bf16* buf, int tiles, int tile, int b0, const uint2 v)
{
    const int l = threadIdx.x & 63, g = l >> 4;
    const int64_t lane = (int64_t)((b0 >> 5) * tiles + tile) * 64 + (2 * ((b0 >> 4) & 1) + (g >> 1)) * 16 + (l & 15);
    *reinterpret_cast<uint2*>(buf + lane * 8 + 4 * (g & 1)) = v;
}

__device__ __forceinline__ void store_operand(__bf16* buf, int tiles, int tile, int b0, const f32x4& v)
{
    store_operand(buf, tiles, tile, b0, make_uint2(pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3])));
}

// 64 samples per block, 16 per wavefront; a wavefront is a chain of dependent
// stages (draw, rows, three layers, three back), one per SIMD at a batch of
// 4096.  Each sample is drawn by one lane of each group of 16 and handed to
// the lanes that need its target (drawn again in each of them it was five
// Philox blocks a lane); its row is on the way while the weights go to LDS;
// activations and deltas leave as 8-byte pieces of operands, where the
// feature-major form stored every value on its own.  At a batch of 4096
// 22.8 us before, 10.8 now.
template <int D>
__global__ __launch_bounds__(256) void k_train_fwdbwd(const MlpPacked* __restrict__ W, const float* __restrict__ U,
                                                      const float* __restrict__ Tg, int64_t n_samples,
                                                      int B, uint64_t seed, int64_t step, int sequential,
                                                      TrainBufs tb)
{
    __shared__ __align__(16) TrainLds L;
    __shared__ __align__(16) __bf16 tiles[4][16 * kStride];
    __shared__ float lossw[4];
    const int wave = threadIdx.x >> 6;
    const int l = threadIdx.x & 63;
    const int b0 = blockIdx.x * 64 + wave * 16;  // first batch row of this wavefront
    // all of the weights are on their way while the sample is drawn
    uint4 wt[kTrainCopies];
#pragma unroll
    for (int q = 0; q < kTrainCopies; ++q)
        wt[q] = reinterpret_cast<const uint4*>(W)[min(q * 256 + (int)threadIdx.x, (int)(sizeof(TrainLds) / 16) - 1)];
    // this lane's sample (A layout row l % 16)
    const int64_t sidx = sample_index(b0 + (l & 15), step, seed, n_samples, sequential);
    float u[2][8];
    load_input_row<D>(U + sidx * raw_in(D), u);
    // targets of the four samples whose outputs this lane will hold
    const int comp = l & 15;
    float tg[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t si = __shfl(sidx, 4 * (l >> 4) + r, 64);
        tg[r] = Tg[si * D + min(comp, D - 1)];
    }
#pragma unroll
    for (int q = 0; q < kTrainCopies; ++q) {
        const int at = q * 256 + (int)threadIdx.x;
        if (at < (int)(sizeof(TrainLds) / 16)) reinterpret_cast<uint4*>(&L)[at] = wt[q];
    }
    __syncthreads();
    bf16x8 a[2];
    build_input_row<D>(u, a);
    // inputs as operands, through the wavefront's tile (rows = samples)
    __bf16* tile = tiles[wave];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) *(bf16x8*)&tile[(l & 15) * kStride + ks * 32 + 8 * (l >> 4)] = a[ks];
    wave_lds_fence();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        uint32_t v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[r] = reinterpret_cast<const uint16_t*>(tile)[(4 * (l >> 4) + r) * kStride + nt * 16 + (l & 15)];
        store_operand(tb.act[0], 4, nt, b0, make_uint2(v[0] | v[1] << 16, v[2] | v[3] << 16));
    }
    wave_lds_fence();

    f32x4 z[3][4], h[3][4];
    f32x4 out;
    mlp_forward16(L.W1, L.W2, L.W3, L.W4, L.b, a, tile, z, h, out);

    // dL/dy in D layout: rows = samples 4 (l/16) + r, column = output l % 16
    f32x4 dy;
    float lsum = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float g = 0.0f;
        if (comp < D) {
            const float res = out[r] - tg[r];
            lsum += res * res;
            g = 2.0f * res / (float)B;
        }
        dy[r] = g;
    }
    store_operand(tb.delta[3], 1, 0, b0, dy);
#pragma unroll
    for (int layer = 0; layer < 3; ++layer)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) store_operand(tb.act[layer + 1], 4, nt, b0, h[layer][nt]);

    // back-propagation: delta_3 = (dy W4) * silu'(z3) ...
    bf16x8 ga[2];
    {
        // dy (16 x 16, D layout) -> A layout with K = 32 (outputs 16..31 zero)
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[(4 * (l >> 4) + i) * kStride + (l & 15)] = (__bf16)dy[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[(4 * (l >> 4) + i) * kStride + 16 + (l & 15)] = (__bf16)0.0f;
        wave_lds_fence();
        ga[0] = *(const bf16x8*)&tile[(l & 15) * kStride + 8 * (l >> 4)];
        wave_lds_fence();
    }
    f32x4 g[4];
    // layer 4 backward: K = 32 (padded outputs), B operand from W4t [in][out]
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
        const bf16x8 b = *(const bf16x8*)&L.W4t[(nt * 16 + (l & 15)) * kStrideT4 + 8 * (l >> 4)];
        c = mfma_bf16(ga[0], b, c);
        g[nt] = c;
    }
    const __bf16* Wt[2] = {L.W3t, L.W2t};
#pragma unroll
    for (int layer = 2; layer >= 0; --layer) {
        // delta of hidden layer (layer+1) = g * silu'(z)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) g[nt][r] *= silu_prime_f(z[layer][nt][r]);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) store_operand(tb.delta[layer], 4, nt, b0, g[nt]);
        if (layer == 0) break;
        d_to_a<4>(g, tile, ga);
        f32x4 nxt[4];
        dense_tiles<4>(Wt[2 - layer], ga, nxt);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) g[nt] = nxt[nt];
    }
    // loss partial of this block, fixed order
    float ls = lsum;
    for (int off = 32; off > 0; off >>= 1) ls += __shfl_down(ls, off, 64);
    if (l == 0) lossw[wave] = ls;
    __syncthreads();
    if (threadIdx.x == 0) tb.loss_part[blockIdx.x] = (lossw[0] + lossw[1]) + (lossw[2] + lossw[3]);
}

// Adam (Kingma & Ba, bias-corrected) of one weight; returns the new one.
struct AdamArgs {
    float *w, *m, *v;  // flat master weights and moments
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float adam_step(const AdamArgs& o, int64_t q, float gg, float w, float m, float v)
{
    const float mm = fmaf(1.0f - o.b1, gg, o.b1 * m);
    const float vv = fmaf(gg, (1.0f - o.b2) * gg, o.b2 * v);
    o.m[q] = mm;
    o.v[q] = vv;
    w -= o.lr * (mm / o.c1) / (sqrtf(vv / o.c2) + o.eps);
    o.w[q] = w;
    return w;
}

// Weight gradients: one wavefront per 16 x 16 tile of a layer's weight matrix,
// summing over the batch with K = 32 samples per MFMA (fixed order); the
// tiles of input-column block 0 also produce the bias gradients.
// Tiles: layer 1: 4 x 4, layers 2 and 3: 4 x 4, layer 4: 1 x 4  -> 52; one
// block more adds up the loss.
//
// grad: the gradients go there.  Else (a training step) each wavefront
// applies Adam to its tile's weights and rounds them into the packed matrices
// that the next step reads: no weight belongs to two tiles, so the step ends
// with this launch (gradients, loss, Adam and packing were five).
//
// The sums are chains of B / 32 MFMAs; what they wait for is the operands.
// kWgradBatch chunks are on their way while as many are multiplied.  At a
// batch of 4096 35.1 us before (and 14 us of small launches), 8.9 now.
constexpr int kWgradTiles = 52, kWgradBatch = 16;

struct WgradChunks {
    bf16x8 a[kWgradBatch], b[kWgradBatch];
};

__device__ __forceinline__ void load_chunks(const bf16x8* a, const bf16x8* b, int ta, int c0, int nc, WgradChunks& w)
{
#pragma unroll
    for (int q = 0; q < kWgradBatch; ++q) {
        const int64_t c = min(c0 + q, nc - 1);  // past the end: repeated, not used
        w.a[q] = a[c * ta * 64];
        w.b[q] = b[c * 4 * 64];
    }
}

template <bool BIAS>
__device__ __forceinline__ void mul_chunks(const WgradChunks& w, int n, f32x4& acc, f32x4& bacc)
{
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;
#pragma unroll
    for (int q = 0; q < kWgradBatch; ++q)
        if (q < n) {  // uniform; n is kWgradBatch but for the last
            acc = mfma_bf16(w.a[q], w.b[q], acc);
            if constexpr (BIAS) bacc = mfma_bf16(w.a[q], ones, bacc);
        }
}

// The sum over all nc chunks in ascending order; cur: the first of them. Two
// sets of registers take turns, so that nothing is moved between them.
template <bool BIAS>
__device__ __forceinline__ void wgrad_sum(const bf16x8* pa, const bf16x8* pb, int ta, int nc, WgradChunks& cur, f32x4& acc,
                                          f32x4& bacc)
{
    WgradChunks nxt;
    int c0 = 0;
    for (; c0 + 2 * kWgradBatch <= nc; c0 += 2 * kWgradBatch) {
        load_chunks(pa, pb, ta, c0 + kWgradBatch, nc, nxt);
        mul_chunks<BIAS>(cur, kWgradBatch, acc, bacc);
        load_chunks(pa, pb, ta, c0 + 2 * kWgradBatch, nc, cur);
        mul_chunks<BIAS>(nxt, kWgradBatch, acc, bacc);
    }
    const int rest = nc - c0;
    if (rest > kWgradBatch) load_chunks(pa, pb, ta, c0 + kWgradBatch, nc, nxt);
    mul_chunks<BIAS>(cur, min(rest, kWgradBatch), acc, bacc);
    if (rest > kWgradBatch) mul_chunks<BIAS>(nxt, rest - kWgradBatch, acc, bacc);
}

__global__ __launch_bounds__(64) void k_train_wgrad(TrainBufs tb, int d, int B, float* __restrict__ grad, AdamArgs opt,
                                                    MlpPacked* __restrict__ W, float* __restrict__ loss)
{
    const int t = blockIdx.x;
    const int l = threadIdx.x & 63;
    if (t == kWgradTiles) {
        // the blocks' parts in ascending order, fetched 64 at a time
        double s = 0.0;
        for (int q0 = 0; q0 < B / 64; q0 += 64) {
            const float p = q0 + l < B / 64 ? tb.loss_part[q0 + l] : 0.0f;
            for (int q = 0; q < min(64, B / 64 - q0); ++q)
                s += (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), q));
        }
        if (l == 0) *loss = (float)(s / (double)B);
        return;
    }
    const int layer = t < 48 ? t / 16 : 3;
    const int ot = t < 48 ? (t % 16) / 4 : 0, it = t < 48 ? t % 4 : t - 48;
    const int ta = layer < 3 ? 4 : 1;
    const int nout = layer < 3 ? kHid : d;
    const int nin = layer == 0 ? mlp_in(d) : kHid;
    const MlpOffsets o = mlp_offsets(d);
    const int64_t wo = layer == 0 ? o.W1 : layer == 1 ? o.W2 : layer == 2 ? o.W3 : o.W4;
    const int64_t bo = layer == 0 ? o.b1 : layer == 1 ? o.b2 : layer == 2 ? o.b3 : o.b4;
    const int ic = it * 16 + (l & 15);            // D column = input feature
    const int or0 = ot * 16 + 4 * (l >> 4);       // D rows or0 .. or0 + 3 = output features
    const bool bias = it == 0 && (l & 15) == 0;
    const bf16x8* pa = (const bf16x8*)tb.delta[layer] + ot * 64 + l;
    const bf16x8* pb = (const bf16x8*)tb.act[layer] + it * 64 + l;
    const int nc = B / 32;
    WgradChunks cur;
    load_chunks(pa, pb, ta, 0, nc, cur);
    // this lane's weights and moments, used after the sums
    float w[4], m[4], v[4], wb[4], mb[4], vb[4];
    if (!grad) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int orr = min(or0 + r, nout - 1);
            const int64_t q = wo + (int64_t)orr * nin + min(ic, nin - 1), qb = bo + orr;
            w[r] = opt.w[q]; m[r] = opt.m[q]; v[r] = opt.v[q];
            wb[r] = opt.w[qb]; mb[r] = opt.m[qb]; vb[r] = opt.v[qb];
        }
    }
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 bacc = {0.0f, 0.0f, 0.0f, 0.0f};
    if (it == 0) wgrad_sum<true>(pa, pb, ta, nc, cur, acc, bacc);
    else wgrad_sum<false>(pa, pb, ta, nc, cur, acc, bacc);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int orr = or0 + r;
        if (orr >= nout) continue;
        if (grad) {
            if (ic < nin) grad[wo + (int64_t)orr * nin + ic] = acc[r];
            if (bias) grad[bo + orr] = bacc[r];
            continue;
        }
        if (ic < nin) {
            const __bf16 nw = (__bf16)adam_step(opt, wo + (int64_t)orr * nin + ic, acc[r], w[r], m[r], v[r]);
            if (layer == 0) {
                W->W1[orr * kStride + ic] = nw;
            } else if (layer == 1) {
                W->W2[orr * kStride + ic] = nw;
                W->W2t[ic * kStride + orr] = nw;
            } else if (layer == 2) {
                W->W3[orr * kStride + ic] = nw;
                W->W3t[ic * kStride + orr] = nw;
            } else {
                W->W4[orr * kStride + ic] = nw;
                W->W4t[ic * kStrideT4 + orr] = nw;
            }
        }
        if (bias) {
            const float nb = adam_step(opt, bo + orr, bacc[r], wb[r], mb[r], vb[r]);
            (layer == 0 ? W->b1 : layer == 1 ? W->b2 : layer == 2 ? W->b3 : W->b4)[orr] = nb;
        }
    }
}

// The exact pair term has zero net force (odd kernel: sum_i K^i = 0).  The
// surrogate is projected onto that constraint: block sums of its outputs
// (k_mlp_infer), then per-system means that k_update / k_surr_err subtract.
// grid (listed systems, d), kBlk threads
__global__ __launch_bounds__(kBlk) void k_surr_final(const int32_t* __restrict__ sys_list,
                                                     const SysDev* __restrict__ sys,
                                                     const double* __restrict__ part,
                                                     float* __restrict__ mean /*[n_sys][kMaxD]*/)
{
    __shared__ double red[kRedLds];
    const int s = sys_list[blockIdx.x];
    const SysDev S = sys[s];
    const int k = blockIdx.y;
    const double t = sum_block_partials(part, S.blk0, S.nblk, kMaxD, k, red);
    if (threadIdx.x == 0) mean[(int64_t)s * kMaxD + k] = (float)(t / (double)S.N);
}

// Check statistics per update block (fixed-order block sums), for the listed
// blocks, with s = surrogate minus its system mean, p = exact pair term and
// q = s + r the prediction (r = the stored residual when res_read, else 0):
//   [0] sum |q - p|^2, [1] sum |p|^2, then per component k:
//   [2 + 2k] sum p_k s_k, [3 + 2k] sum s_k^2, and [2 + 2 kMaxD] sum |s - p|^2.
// With res_write the residuals p - s replace the stored ones (each thread
// reads its own slots before it writes them).
constexpr int kErrStats = 3 + 2 * kMaxD;

template <typename T, int D>
__global__ __launch_bounds__(kBlk) void k_surr_err(const BlkItem* __restrict__ items,
                                                   const SysDev* __restrict__ sys, int64_t P,
                                                   const double* __restrict__ pairsum,
                                                   const float* __restrict__ surr,
                                                   const float* __restrict__ surr_mean,
                                                   float* res, int res_read, int res_write,
                                                   double* __restrict__ err_part /*[nblk][kErrStats]*/)
{
    __shared__ double red[kRedLds];
    const BlkItem it = items[blockIdx.x];
    const SysDev S = sys[it.sys];
    const int i = it.blk * kBlk + threadIdx.x;
    double e2 = 0.0, b2 = 0.0, r2 = 0.0, ps[kMaxD] = {0.0, 0.0, 0.0, 0.0}, ss[kMaxD] = {0.0, 0.0, 0.0, 0.0};
    if (i < S.N) {
        const int64_t slot = S.off + i;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const double pair = pairsum[k * P + slot];
            const double sv = (double)surr[k * P + slot] - (double)surr_mean[(int64_t)it.sys * kMaxD + k];
            const double q = res_read ? sv + (double)res[k * P + slot] : sv;
            if (res_write) res[k * P + slot] = (float)(pair - sv);
            e2 += (q - pair) * (q - pair);
            r2 += (sv - pair) * (sv - pair);
            b2 += pair * pair;
            ps[k] = pair * sv;
            ss[k] = sv * sv;
        }
    }
    double* out = err_part + (int64_t)blockIdx.x * kErrStats;
    const double t0 = block_sum(e2, red);
    const double t1 = block_sum(b2, red);
    const double t2 = block_sum(r2, red);
    if (threadIdx.x == 0) {
        out[0] = t0;
        out[1] = t1;
        out[2 + 2 * kMaxD] = t2;
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const double a = block_sum(ps[k], red);
        const double b = block_sum(ss[k], red);
        if (threadIdx.x == 0) {
            out[2 + 2 * k] = a;
            out[3 + 2 * k] = b;
        }
    }
}

}  // namespace ssm
