// infernet.hip -- the proposal network on one observed dataset, in one launch:
// data summaries, the three layers on one row and the decoded proposal.
//
// One 256-thread workgroup.  As five launches (summaries, a 64-row product per
// layer, decode) and a copy of the parameters this took 21 us more of a call
// (4096 particles x 1000 points: 74.5 us a call then, 53.4 with this kernel), most
// of it launches and the weights' latency layer by layer.  Here a wave owns 64 outputs of every layer, as in
// the fused training pass, and the weight fragments of all three layers (288
// registers per lane) are loaded while the summaries are finished, whose chain of
// reductions and Cholesky steps touches no global memory.  Bound: that chain, then
// three products of one row; 300 KB of weights through one CU take about as
// long as the summaries.
// The products use the instruction, fragments and order over K of
// gemm_nt_kernel, and the row's 16-row tile is filled with zeros, so every
// output has the bits of the 64-row products.
#include "device.h"
#include "fuse.h"
#include "host.h"
#include "proposal.h"
#include "summary.h"

namespace ppl {

// acc[j] (lanes 0..15, element 0) = sum over K of a[k] B[64 wave + 16 j + lane][k]
// for the row a in LDS.
template <int KD, int S>
__device__ __forceinline__ void row_mma(const uint16_t *a, const fbf16x8_t (&fb)[S][4], ffloatx4_t (&acc)[4]) {
    const int lane = threadIdx.x & 63;
    const bool row0 = (lane & 15) == 0;
    const int fk = (lane >> 4) * 8;
    fbf16x8_t zero;
#pragma unroll
    for (int e = 0; e < 8; ++e) zero[e] = (__bf16)0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = ffloatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KD / 32; ++s) {
        const fbf16x8_t v = *(const fbf16x8_t *)(a + 32 * s + fk);
        const fbf16x8_t fa = row0 ? v : zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[s][j], acc[j], 0, 0, 0);
    }
}

// exp(o[base + k] - max) summed over k < n in order, by the n first lanes of a
// group of eight; returns this lane's log-softmax entry.
__device__ __forceinline__ double log_softmax8(const float *o, int base, int n, int lane8) {
    double m = -INFINITY;
    for (int k = 0; k < n; ++k) m = fmax(m, (double)o[base + k]);
    const double v = (double)o[base + min(lane8, n - 1)];
    const double e = exp(v - m);
    double s = 0.0;
    for (int k = 0; k < n; ++k) s += __shfl(e, k, 8);
    return v - m - log(s);
}

// Summaries, network and decoded parameters:
//   POLY: {log-softmax of the degree logits [4], log-softmax of the mixture
//          logits [8], mean[4][8][5], lsd[4][8][5]} (slots j >= n zero).
//   GMM:  {log-softmax of the mixture logits [8], mean[8][d], lsd[8][d]}.
template <int MODEL>
__global__ __launch_bounds__(kSumThreads, 1) void infer_net_kernel(const void *__restrict__ xv,
                                                                 const void *__restrict__ yv, int64_t D, int K,
                                                                 MlpView w, double log_widen, double *__restrict__ q,
                                                                 double *__restrict__ q_copy,
                                                                 double *__restrict__ s64) {
#pragma clang fp contract(off)
    extern __shared__ float ysf[];
    __shared__ double wtot[kSumWaves][kPolyAcc];
    __shared__ double tot[kPolyAcc];
    __shared__ double s[kSummaryDim];
    __shared__ double red[kSumWaves];
    __shared__ int hist[32], nan_seen;
    __shared__ __align__(16) uint16_t row[3][kMlpHid];
    __shared__ float out[kMlpOut];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float bias[3][4];
    fbf16x8_t f1[kMlpIn / 32][4], f2[kMlpHid / 32][4], f3[kMlpHid / 32][4];
    auto load_weights = [&]() {
#pragma unroll
        for (int l = 0; l < 3; ++l)
#pragma unroll
            for (int j = 0; j < 4; ++j) bias[l][j] = w.master[MlpParams::b_off(l) + 64 * wave + 16 * j + (lane & 15)];
        fuse_load_w<kMlpIn>(w.wtf + MlpParams::bf16_w_off(0), f1);
        fuse_load_w<kMlpHid>(w.wtf + MlpParams::bf16_w_off(1), f2);
        fuse_load_w<kMlpHid>(w.wtf + MlpParams::bf16_w_off(2), f3);
    };
    if constexpr (MODEL == PPL_MODEL_POLY) {
        const double *X = (const double *)xv, *Y = (const double *)yv;
        double a[kPolyAcc];
#pragma unroll
        for (int k = 0; k < kPolyAcc; ++k) a[k] = 0.0;
        for (int64_t d = tid; d < D; d += kSumThreads) poly_acc_point(a, X[d], Y[d]);
        load_weights();
        poly_finish(a, D, wtot, tot, s);
    } else {
        const float *Y = (const float *)yv;
        if (tid < 32) hist[tid] = 0;
        if (tid == 0) nan_seen = 0;
        __syncthreads();
        double sum_y = 0.0;
        for (int64_t d = tid; d < D; d += kSumThreads) {
            const float yf = Y[d];
            ysf[d] = yf;
            sum_y += (double)yf;
            gmm_bin(hist, (double)yf);
            if (yf != yf) nan_seen = 1;
        }
        load_weights();
        __syncthreads();
        gmm_finish(ysf, D, hist, sum_y, red, s);
        if (nan_seen && tid < 16) s[tid] = NAN;      // a NaN has no rank: the order statistics are undefined
    }
    if (tid < kSummaryDim) {
        row[0][tid] = f32_to_bf16((float)s[tid]);
        if (s64) s64[tid] = s[tid];
    }
    __syncthreads();
    ffloatx4_t acc[4];
    row_mma<kMlpIn>(row[0], f1, acc);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (lane < 16) row[1][64 * wave + 16 * j + lane] = f32_to_bf16(fmaxf(acc[j][0] + bias[0][j], 0.0f));
    __syncthreads();
    row_mma<kMlpHid>(row[1], f2, acc);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (lane < 16) row[2][64 * wave + 16 * j + lane] = f32_to_bf16(fmaxf(acc[j][0] + bias[1][j], 0.0f));
    __syncthreads();
    row_mma<kMlpHid>(row[2], f3, acc);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (lane < 16) out[64 * wave + 16 * j + lane] = acc[j][0] + bias[2][j];
    __syncthreads();
    auto put = [&](int e, double v) {
        q[e] = v;
        if (q_copy) q_copy[e] = v;
    };
    auto O = [&](int k) { return (double)out[k]; };
    if constexpr (MODEL == PPL_MODEL_POLY) {
        if (tid < 160) {
            const int e = tid, n = 2 + e / 40, m = (e / 5) % 8, j = e % 5;
            const int off = poly_head_off(n);
            put(12 + e, j < n ? 10.0 * O(off + m * n + j) : 0.0);
            put(172 + e, j < n ? 5.0 * tanh(O(off + 8 * n + m * n + j) / 5.0) + log_widen : 0.0);
        } else if (wave == 3) {              // lanes 0..7 the degrees, 8..15 the components
            const bool deg = lane < 8;
            const double v = log_softmax8(out, deg ? 0 : 4, deg ? 4 : 8, lane & 7);
            if (lane < 4) put(lane, v);
            else if (lane >= 8 && lane < 16) put(4 + lane - 8, v);
        }
    } else {
        const int d = 2 * K - 1;
        if (tid < 8 * d) {
            put(8 + tid, 5.0 * O(8 + tid));
            put(8 + 8 * d + tid, 5.0 * tanh(O(8 + 8 * d + tid) / 5.0) + log_widen);
        } else if (wave == 3) {              // 8 d <= 120
            const double v = log_softmax8(out, 0, 8, lane & 7);
            if (lane < 8) put(lane, v);
        }
    }
}

int launch_infer_net(int model, int K, const void *x, const void *y, int64_t D, const MlpView &w, double log_widen,
                     double *q, double *q_copy, double *s64, hipStream_t st) {
    if (model == PPL_MODEL_POLY) {
        hipLaunchKernelGGL(infer_net_kernel<PPL_MODEL_POLY>, dim3(1), dim3(kSumThreads), 0, st, x, y, D, K, w, log_widen,
                           q, q_copy, s64);
    } else {
        if (D > kGmmSummaryMaxD) return fail(PPL_E_ARG, "mixture summaries take at most %d points", kGmmSummaryMaxD);
        const size_t lds = (size_t)(D > 0 ? D : 1) * sizeof(float);
        hipLaunchKernelGGL(infer_net_kernel<PPL_MODEL_GMM>, dim3(1), dim3(kSumThreads), lds, st, x, y, D, K, w, log_widen,
                           q, q_copy, s64);
    }
    PPL_LAUNCH_CHECK("infer_net_kernel");
    return PPL_OK;
}

}  // namespace ppl
