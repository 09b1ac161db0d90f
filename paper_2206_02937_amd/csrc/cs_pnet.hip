// cs_pnet.hip -- the paper's own learned component (Sec. 3.2): a small dense
// network that predicts, for a candidate lepton-photon pair, the probability
// of interaction against the cell's majorant, y' = P / P_max, in place of the
// analytic Klein-Nishina evaluation.
//
// Nine inputs per pair (FP32 rows): photon momentum k (3), lepton momentum p
// (3), P_max, w_e, w_g.  Widths 9 -> 9 -> 12 -> 9 -> 1, ReLU hidden layers
// (ReLU'(0) = 0), sigmoid output.  Parameters: per layer W[n_out][n_in]
// row-major, then b[n_out] (337 floats).  FP32 arithmetic, one pair per lane:
// the layers are too narrow for matrix-core tiles along the batch (9 x 9 of
// 16 x 12), but their weight gradients, sums over the pairs of delta times
// activation, fit one 16 x 16 tile each with the pairs as the contraction.
//
//   k_pnet_target     y = P / P_max = s(x) (1 - beta . k_hat) / 2 in FP64
//                     (the training target and the analytic reference)
//   k_pnet_fwd        y' per pair
//   k_pnet_grad_block forward and backward per pair, the weight gradients on
//                     FP32 MFMA, summed over a workgroup's pairs into
//                     per-workgroup partials
//   k_pnet_reduce     fixed-order sum of the partials over the workgroups,
//                     divided by n (gradient of the mean loss) and the loss
//   k_pnet_adam       one Adam step (Kingma & Ba; bias corrections from the
//                     host)
#include <hip/hip_runtime.h>

#include "cs_block.h"
#include "cs_device.h"
#include "cs_internal.h"

namespace cs {

constexpr int kPnetThreads = 256;
// parameter offsets of the four layers
constexpr int kW1 = 0, kB1 = 81, kW2 = 90, kB2 = 198, kW3 = 210, kB3 = 318, kW4 = 327, kB4 = 336;
constexpr int kPnetParams = 337;
constexpr int kPnetPart = kPnetParams + 1;  // per-workgroup partials: the gradient, then the loss

__global__ __launch_bounds__(kPnetThreads) void k_pnet_target(const float* in, int64_t n, float* y) {
    const int64_t i = (int64_t)blockIdx.x * kPnetThreads + threadIdx.x;
    if (i >= n) return;
    const float* r = in + 9 * i;
    const d3 k = {(double)r[0], (double)r[1], (double)r[2]};
    const d3 p = {(double)r[3], (double)r[4], (double)r[5]};
    const XFlux xf = x_flux(p, k, dot(p, p), dot(k, k));
    y[i] = xf.x > 0.0 ? (float)(0.5 * sigma_ratio(xf.x) * xf.flux) : 0.0f;
}

// The parameters are the same for every lane and do not change while a kernel
// runs, so they are read through the constant address space: scalar loads,
// and each multiply-add takes its weight from a scalar register.  (From LDS,
// the 337 broadcast reads per wave keep the LDS busy twice as long as the
// multiply-adds keep the vector ALUs; k_pnet_fwd uses them all the same where
// there are too few waves to wait for scalar loads.)
typedef const __attribute__((address_space(4))) float* cfptr;

// The forward pass of one pair: pre-activations and activations kept for the
// backward pass.
struct PnetActs {
    float a0[9], a1[9], a2[12], a3[9];
    float y;
};

template <typename Params>
__device__ __forceinline__ void pnet_forward(Params P, PnetActs& s) {
#pragma unroll
    for (int m = 0; m < 9; ++m) {
        float z = P[kB1 + m];
#pragma unroll
        for (int q = 0; q < 9; ++q) z = fmaf(P[kW1 + 9 * m + q], s.a0[q], z);
        s.a1[m] = fmaxf(z, 0.0f);
    }
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        float z = P[kB2 + i];
#pragma unroll
        for (int m = 0; m < 9; ++m) z = fmaf(P[kW2 + 9 * i + m], s.a1[m], z);
        s.a2[i] = fmaxf(z, 0.0f);
    }
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        float z = P[kB3 + j];
#pragma unroll
        for (int i = 0; i < 12; ++i) z = fmaf(P[kW3 + 12 * j + i], s.a2[i], z);
        s.a3[j] = fmaxf(z, 0.0f);
    }
    float z = P[kB4];
#pragma unroll
    for (int j = 0; j < 9; ++j) z = fmaf(P[kW4 + j], s.a3[j], z);
    s.y = 1.0f / (1.0f + expf(-z));
}

// A pair's nine inputs (rows of 36 bytes, 4-byte aligned).
__device__ __forceinline__ void load_pair(const float* row, float (&x)[9]) { __builtin_memcpy(x, row, sizeof(x)); }

// Pairs from and up to which the parameters come from LDS (LDS true) and not by
// scalar loads: eight waves per SIMD are 2^19 pairs, and the waves of a second
// round that is not full have too few others beside them.  Analytic ratio and
// forward together, us, by LDS / by scalar loads: 500,000 pairs 15.4 / 15.9, 700,000
// 19.4 / 19.7, 2^20 25.5 / 25.4, 1.2 M 32.1 / 30.3, 2^22 97.7 / 89.9; the forward
// alone 300,000 6.5 / 5.9.  (Loads of a pair that is clamped, not left out, past
// the end made the scalar form 0.3-0.9 us longer.)
constexpr int64_t kPnetLdsMin = 3 << 17, kPnetLdsMax = 1 << 20;

template <bool LDS>
__global__ __launch_bounds__(kPnetThreads) void k_pnet_fwd(const float* params, const float* in, int64_t n,
                                                         float* y) {
    const int64_t i = (int64_t)blockIdx.x * kPnetThreads + threadIdx.x;
    PnetActs s;
    if constexpr (LDS) {
        __shared__ float s_p[kPnetParams];
        for (int q = threadIdx.x; q < kPnetParams; q += kPnetThreads) s_p[q] = params[q];
        __syncthreads();
        if (i >= n) return;
#pragma unroll
        for (int q = 0; q < 9; ++q) s.a0[q] = in[9 * i + q];
        pnet_forward((const float*)s_p, s);
    } else {
        if (i >= n) return;
        load_pair(in + 9 * i, s.a0);
        pnet_forward((cfptr)params, s);
    }
    y[i] = s.y;
}

// Weight gradient of one layer over a wave's 64 pairs: acc[o][i] += sum over
// the pairs of d[o] a[i], o < NO, i < NI, and of d[o] in column NI (the
// bias), on v_mfma_f32_16x16x4_f32 (lane l supplies row or column l % 16 and
// contraction index l / 16, and receives rows 4 (l / 16) + r of column
// l % 16).  Each lane holds one pair; the operands pass through the wave's
// part of LDS, one row of 64 pairs per neuron.  Contraction step ks takes the
// pairs 16 g + ks of the lane groups g, so that a lane's sixteen operands are
// consecutive; rows 68 floats apart put the sixteen rows on different banks.
// Rows and columns past the layer's repeat its last one; what they give is
// not read.
constexpr int kPnetRow = 68;
constexpr int kPnetRows = 12;  // the widest layer
typedef float floatx4_p __attribute__((ext_vector_type(4)));

template <int NO, int NI>
__device__ __forceinline__ void outer_acc(floatx4_p& acc, float* sd, float* sa, const float (&d)[NO],
                                          const float (&a)[NI]) {
    static_assert(NO <= kPnetRows && NI <= kPnetRows, "LDS rows");
    const int lane = lane_id();
#pragma unroll
    for (int o = 0; o < NO; ++o) sd[o * kPnetRow + lane] = d[o];
#pragma unroll
    for (int i = 0; i < NI; ++i) sa[i * kPnetRow + lane] = a[i];
    wave_lds_sync();
    const int c = lane & 15, g = lane >> 4;
    const float* pd = sd + (c < NO ? c : NO - 1) * kPnetRow + 16 * g;
    const float* pa = sa + (c < NI ? c : NI - 1) * kPnetRow + 16 * g;
    float4 D[4], A[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        D[j] = *(const float4*)(pd + 4 * j);
        A[j] = *(const float4*)(pa + 4 * j);
        if (c == NI) A[j] = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
    }
    // two chains over half the pairs each: 2^22 pairs 188 us, with four chains
    // 200 us; the gradient's relative error against 64 bits at 1024 pairs is
    // 2.8e-8 with two, 2.6e-8 with four
    floatx4_p s[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) s[j] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        s[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(D[j].x, A[j].x, s[j & 1], 0, 0, 0);
        s[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(D[j].y, A[j].y, s[j & 1], 0, 0, 0);
        s[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(D[j].z, A[j].z, s[j & 1], 0, 0, 0);
        s[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(D[j].w, A[j].w, s[j & 1], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] += s[0][r] + s[1][r];
    wave_lds_sync();
}

// This lane's entries of a layer's accumulated tile into the wave's partial
// gradient: W at w0 (NO x NI row-major), bias at b0.
template <int NO, int NI>
__device__ __forceinline__ void put_tile(float* part, const floatx4_p& acc, int w0, int b0) {
    const int c = lane_id() & 15, g = lane_id() >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * g + r;
        if (o < NO && c < NI) part[w0 + o * NI + c] = acc[r];
        if (o < NO && c == NI) part[b0 + o] = acc[r];
    }
}

// v where the activation a is positive, else 0.  The value is made opaque so
// that it is selected, not computed in a branch of its own.
__device__ __forceinline__ float relu_delta(float a, float v) {
    asm("" : "+v"(v));
    return a > 0.0f ? v : 0.0f;
}

// Forward and backward of a workgroup's pairs (256 at a time, grid-strided),
// the next pairs' inputs read before the present ones are worked on.  The
// four weight gradients stay in MFMA accumulators until the end.  What bounds
// it: at a batch of 4096 (16 workgroups) the length of one pass through the
// layers: with the reduction 79.5 us per call with a butterfly sum over the
// wave per parameter (and one thread per parameter walking the partials),
// 11.5 us with this, most of it the two launches; at 2^22 pairs VALU issue
// and the matrix cores, 6509 and 188 us.
__global__ __launch_bounds__(kPnetThreads) void k_pnet_grad_block(const float* params, const float* in,
                                                                const float* target, int64_t n, int mae,
                                                                double* partials) {
    __shared__ __align__(16) float s_buf[kPnetThreads / 64][2 * kPnetRows * kPnetRow];
    __shared__ float s_part[kPnetThreads / 64][kPnetPart];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* sd = s_buf[wave];
    float* sa = sd + kPnetRows * kPnetRow;
    cfptr P = (cfptr)params;
    const int64_t stride = (int64_t)gridDim.x * kPnetThreads;
    floatx4_p g1 = {0.0f, 0.0f, 0.0f, 0.0f}, g2 = g1, g3 = g1, g4 = g1;
    int64_t base = (int64_t)blockIdx.x * kPnetThreads;
    float xn[9], tn;
    auto fetch = [&](int64_t b) {
        const int64_t i = b + tid < n ? b + tid : n - 1;
        load_pair(in + 9 * i, xn);
        tn = target[i];
    };
    fetch(base);
    for (; base < n; base += stride) {
        const bool act = base + tid < n;
        PnetActs s;  // (a lane past the end repeats the last pair, with delta 0)
#pragma unroll
        for (int q = 0; q < 9; ++q) s.a0[q] = xn[q];
        const float t = tn;
        if (base + stride < n) fetch(base + stride);
        // the parameter pointer is made opaque for each pass, so that the
        // scalar loads stay at their uses (hoisted out of the loop, 337
        // values do not fit the scalar registers)
        asm volatile("" : "+s"(P));
        pnet_forward(P, s);
        asm volatile("" : "+s"(P));
        const float e = act ? s.y - t : 0.0f;
        const float dy = mae ? (e > 0.0f ? 1.0f : (e < 0.0f ? -1.0f : 0.0f)) : e;
        // backward (per pair; the 1/n of the mean is applied by k_pnet_reduce);
        // ReLU' from the activation, which is positive exactly where z is
        float d4[2];
        d4[0] = dy * s.y * (1.0f - s.y);
        d4[1] = mae ? fabsf(e) : 0.5f * e * e;  // second row: the loss, in the bias column
        outer_acc<2, 9>(g4, sd, sa, d4, s.a3);
        float d3[9], d2[12], d1[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) d3[j] = relu_delta(s.a3[j], d4[0] * P[kW4 + j]);
        outer_acc<9, 12>(g3, sd, sa, d3, s.a2);
#pragma unroll
        for (int i2 = 0; i2 < 12; ++i2) {
            float v = P[kW3 + i2] * d3[0];
#pragma unroll
            for (int j = 1; j < 9; ++j) v = fmaf(P[kW3 + 12 * j + i2], d3[j], v);
            d2[i2] = relu_delta(s.a2[i2], v);
        }
        outer_acc<12, 9>(g2, sd, sa, d2, s.a1);
#pragma unroll
        for (int m = 0; m < 9; ++m) {
            float v = P[kW2 + m] * d2[0];
#pragma unroll
            for (int i2 = 1; i2 < 12; ++i2) v = fmaf(P[kW2 + 9 * i2 + m], d2[i2], v);
            d1[m] = relu_delta(s.a1[m], v);
        }
        outer_acc<9, 9>(g1, sd, sa, d1, s.a0);
    }
    float* part = s_part[wave];
    put_tile<9, 9>(part, g1, kW1, kB1);
    put_tile<12, 9>(part, g2, kW2, kB2);
    put_tile<9, 12>(part, g3, kW3, kB3);
    {
        // row 0: dW4, db4; row 1: the loss, in the bias column
        const int c = tid & 15, g = (tid >> 4) & 3;
        if (g == 0 && c < 9) part[kW4 + c] = g4[0];
        if (g == 0 && c == 9) {
            part[kB4] = g4[0];
            part[kPnetParams] = g4[1];
        }
    }
    __syncthreads();
    for (int q = tid; q < kPnetPart; q += kPnetThreads) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kPnetThreads / 64; ++w) t += (double)s_part[w][q];
        partials[(int64_t)blockIdx.x * kPnetPart + q] = t;
    }
}

// One workgroup of 16 waves per 64 entries: wave w sums the partials of the
// workgroups b = 16 c + w (c ascending, eight reads in flight), then wave 0
// adds the 16 wave sums in order.  The sums over waves and workgroups are in
// FP64, rounded once at the end: the gradient's relative error against 64 bits
// (mean of ten sets) at 4096, 40000 and 10^6 pairs is 2.5e-8, 2.5e-8 and
// 2.6e-7; with FP32 sums 6.1e-8, 6.3e-8 and 2.9e-7, at the same time per call;
// with butterfly sums over the lanes and one FP32 chain over the workgroups
// 6.3e-8, 1.9e-7 and 9.6e-7.
constexpr int kPnetReduceWaves = 16;

__global__ __launch_bounds__(64 * kPnetReduceWaves) void k_pnet_reduce(const double* partials, int64_t n_blocks,
                                                                      int64_t n, float* grad, float* loss) {
    __shared__ double s_q[kPnetReduceWaves][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int q = blockIdx.x * 64 + lane;
    const int qc = q < kPnetPart ? q : kPnetPart - 1;
    double t = 0.0;
    int64_t b = w;
    for (; b + 7 * kPnetReduceWaves < n_blocks; b += 8 * kPnetReduceWaves) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = partials[(b + kPnetReduceWaves * k) * kPnetPart + qc];
#pragma unroll
        for (int k = 0; k < 8; ++k) t += v[k];
    }
    for (; b < n_blocks; b += kPnetReduceWaves) t += partials[b * kPnetPart + qc];
    s_q[w][lane] = t;
    __syncthreads();
    if (w != 0 || q >= kPnetPart) return;
    t = s_q[0][lane];
#pragma unroll
    for (int k = 1; k < kPnetReduceWaves; ++k) t += s_q[k][lane];
    const float v = n > 0 ? (float)(t / (double)n) : 0.0f;
    if (q < kPnetParams)
        grad[q] = v;
    else if (loss)
        *loss = v;
}

__global__ __launch_bounds__(kPnetThreads) void k_pnet_adam(float* params, const float* grad, float* m_, float* v_,
                                                          float lr, float bc1, float bc2) {
    const int q = blockIdx.x * kPnetThreads + threadIdx.x;
    if (q >= kPnetParams) return;
    const float g = grad[q];
    const float m = 0.9f * m_[q] + 0.1f * g;
    const float v = 0.999f * v_[q] + 0.001f * g * g;
    m_[q] = m;
    v_[q] = v;
    params[q] -= lr * (m / bc1) / (sqrtf(v / bc2) + 1e-8f);
}

// workgroups of the gradient kernel: one per 256 pairs, at most four per
// compute unit (what its registers let be resident), which then take several
constexpr int64_t kPnetMaxBlocks = 1024;

static int64_t pnet_grad_blocks(int64_t n) {
    const int64_t nb = (n + kPnetThreads - 1) / kPnetThreads;
    return nb < kPnetMaxBlocks ? nb : kPnetMaxBlocks;
}

size_t pnet_workspace_bytes(int64_t n) {
    const int64_t nb = n > 0 ? pnet_grad_blocks(n) : 1;
    return sizeof(double) * (size_t)nb * kPnetPart;
}

hipError_t launch_pnet_target(const float* in, int64_t n, float* y, hipStream_t st) {
    if (n > 0) k_pnet_target<<<(unsigned)((n + kPnetThreads - 1) / kPnetThreads), kPnetThreads, 0, st>>>(in, n, y);
    return hipGetLastError();
}

hipError_t launch_pnet_forward(const float* params, const float* in, int64_t n, float* y, hipStream_t st) {
    if (n > 0)
        (n > kPnetLdsMin && n <= kPnetLdsMax ? k_pnet_fwd<true> : k_pnet_fwd<false>)
            <<<(unsigned)((n + kPnetThreads - 1) / kPnetThreads), kPnetThreads, 0, st>>>(params, in, n, y);
    return hipGetLastError();
}

hipError_t launch_pnet_grad(const float* params, const float* in, const float* target, int64_t n, int mae,
                            float* grad, float* loss, void* ws, hipStream_t st) {
    const int64_t nb = n > 0 ? pnet_grad_blocks(n) : 0;
    double* part = (double*)ws;
    if (nb > 0) k_pnet_grad_block<<<(unsigned)nb, kPnetThreads, 0, st>>>(params, in, target, n, mae, part);
    k_pnet_reduce<<<(kPnetPart + 63) / 64, 64 * kPnetReduceWaves, 0, st>>>(part, nb, n, grad, loss);
    return hipGetLastError();
}

hipError_t launch_pnet_adam(float* params, const float* grad, float* m, float* v, float lr, float bc1, float bc2,
                            hipStream_t st) {
    k_pnet_adam<<<(kPnetParams + kPnetThreads - 1) / kPnetThreads, kPnetThreads, 0, st>>>(params, grad, m, v, lr,
                                                                                        bc1, bc2);
    return hipGetLastError();
}

}  // namespace cs
