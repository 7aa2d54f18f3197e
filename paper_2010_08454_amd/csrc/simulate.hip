// simulate.hip -- training pairs drawn from the model's own prior and their 64
// data summaries, one 256-thread workgroup per dataset.
//
// Training pair of step t, pair i (Philox tag 4, counter (i, block, t, 4)):
//   POLY: block 0 word 0 -> degree n (uniform discrete); blocks 1, 2 -> eight
//         normals (two single-precision-stream Box-Muller pairs each), c_j =
//         sd z_j; block 8 + e -> points 2e, 2e + 1: x = 2u - 1 from words 0, 1
//         and the observation noise from a Box-Muller pair on words 2, 3;
//         y = poly_c(x) + noise_sd * eps.
//   GMM:  blocks 0, 1 -> Exp(1) draws E_k = -ln u_k, pi = E / sum E (a
//         Dirichlet(1) draw); blocks 2, 3 -> mu_k = mu_sd z_k; block 8 + e ->
//         the components of points 2e, 2e + 1 (inverse CDF on pi, words 0, 1)
//         and their noise (words 2, 3); latents returned in the ordered
//         unconstrained space (mu_(1), log gaps, log pi_(k) - log pi_(K)).
// Every step is in FP64 on uniforms that are exact in both precisions.
#include "adam.h"
#include "device.h"
#include "host.h"
#include "proposal.h"
#include "summary.h"

namespace ppl {

constexpr uint32_t kTagTrain = 4;

__device__ __forceinline__ double u01(uint32_t w) { return (double)unit_f32(w); }

// Index of the first cumulative probability above u (K - 1 if none).
__device__ __forceinline__ int categorical8(double u, const double (&p)[8], int K) {
    double c = 0.0;
    int r = K - 1;
    bool found = false;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (k < K && !found) {
            c += p[k];
            if (u < c) {
                r = k;
                found = true;
            }
        }
    }
    return r;
}

__device__ __forceinline__ double pick8(const double (&v)[8], int k) {
    double r = v[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) r = (k == j) ? v[j] : r;
    return r;
}

// -------------------------------------------------- training simulation --
// Dataset b of the batch (one workgroup).
template <int MODEL>
__device__ __forceinline__ void simulate_block(const SimSpec &sp, int B, Key key, const int64_t *__restrict__ step_ptr,
                                               uint16_t *__restrict__ x_row, uint16_t *__restrict__ x_col,
                                               double *__restrict__ theta, double *__restrict__ s64, int b) {
#pragma clang fp contract(off)
    extern __shared__ double ys[];
    __shared__ double wtot[kSumWaves][kPolyAcc];
    __shared__ double tot[kPolyAcc];
    __shared__ double s[kSummaryDim];
    __shared__ double red[kSumWaves];
    __shared__ int hist[32];
    const int tid = threadIdx.x;
    const uint32_t step = (uint32_t)*step_ptr;
    const uint32_t pair = (uint32_t)b;
    const int64_t D = sp.D;

    if constexpr (MODEL == PPL_MODEL_POLY) {
        const uint4 w0 = philox(pair, 0, step, kTagTrain, key);
        const int n = uniform_discrete(w0.x, (int)sp.hyper[1], (uint32_t)((int)sp.hyper[2] - (int)sp.hyper[1] + 1));
        // coefficient normals z_0..z_4: Box-Muller pairs 0..2 of blocks 1 and
        // 2 (pair q from words 2 (q % 2), 2 (q % 2) + 1 of block 1 + q / 2),
        // one pair per thread of the first three, shared through LDS
        __shared__ double s_z[6];
        if (tid < 3) {
            const uint4 w = philox(pair, 1 + (tid >> 1), step, kTagTrain, key);
            double za, zb;
            box_muller(u01((tid & 1) ? w.z : w.x), u01((tid & 1) ? w.w : w.y), za, zb);
            s_z[2 * tid] = za;
            s_z[2 * tid + 1] = zb;
        }
        __syncthreads();
        double c[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) c[j] = sp.hyper[0] * s_z[j];
        double a[kPolyAcc];
#pragma unroll
        for (int k = 0; k < kPolyAcc; ++k) a[k] = 0.0;
        for (int64_t e = tid; 2 * e < D; e += kSumThreads) {
            const uint4 w = philox(pair, (uint32_t)(8 + e), step, kTagTrain, key);
            double e0, e1;
            box_muller(u01(w.z), u01(w.w), e0, e1);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (2 * e + h < D) {
                    const double x = 2.0 * u01(h ? w.y : w.x) - 1.0;
                    double p = 0.0;
#pragma unroll
                    for (int j = 4; j >= 0; --j)
                        if (j < n) p = p * x + c[j];
                    const double y = p + sp.hyper[3] * (h ? e1 : e0);
                    poly_acc_point(a, x, y);
                }
            }
        }
        poly_finish(a, D, wtot, tot, s);
        if (tid < 6) theta[(size_t)b * kThetaStride + tid] = tid == 0 ? (double)n : (tid - 1 < n ? c[tid - 1] : 0.0);
    } else {
        const int K = sp.K;
        if (tid < 32) hist[tid] = 0;
        const uint4 wa = philox(pair, 0, step, kTagTrain, key), wb = philox(pair, 1, step, kTagTrain, key);
        const uint32_t ew[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
        double E[8], pi[8], mu[8], z[8], etot = 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            E[k] = k < K ? -log_unit(u01(ew[k])) : 0.0;
            if (k < K) etot += E[k];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) pi[k] = k < K ? E[k] / etot : 0.0;
        {
            const uint4 w2 = philox(pair, 2, step, kTagTrain, key), w3 = philox(pair, 3, step, kTagTrain, key);
            box_muller(u01(w2.x), u01(w2.y), z[0], z[1]);
            box_muller(u01(w2.z), u01(w2.w), z[2], z[3]);
            box_muller(u01(w3.x), u01(w3.y), z[4], z[5]);
            box_muller(u01(w3.z), u01(w3.w), z[6], z[7]);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) mu[k] = sp.hyper[0] * z[k];
        __syncthreads();
        double sum_y = 0.0;
        for (int64_t e = tid; 2 * e < D; e += kSumThreads) {
            const uint4 w = philox(pair, (uint32_t)(8 + e), step, kTagTrain, key);
            double e0, e1;
            box_muller(u01(w.z), u01(w.w), e0, e1);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (2 * e + h < D) {
                    const int k = categorical8(u01(h ? w.y : w.x), pi, K);
                    const double y = pick8(mu, k) + sp.hyper[1] * (h ? e1 : e0);
                    ys[2 * e + h] = y;
                    sum_y += y;
                    gmm_bin(hist, y);
                }
            }
        }
        __syncthreads();
        gmm_finish(ys, D, hist, sum_y, red, s);
        if (tid == 0) {
            // order the components by mean (insertion sort; ties keep index order)
            int ord[8] = {0, 1, 2, 3, 4, 5, 6, 7};
            for (int q = 1; q < K; ++q)
                for (int r = q; r > 0 && mu[ord[r]] < mu[ord[r - 1]]; --r) {
                    const int t = ord[r];
                    ord[r] = ord[r - 1];
                    ord[r - 1] = t;
                }
            double *u = theta + (size_t)b * kThetaStride;
            u[0] = mu[ord[0]];
            for (int q = 1; q < K; ++q) u[q] = log(mu[ord[q]] - mu[ord[q - 1]]);
            const double lk = log(pi[ord[K - 1]]);
            for (int q = 0; q < K - 1; ++q) u[K + q] = log(pi[ord[q]]) - lk;
        }
    }
    if (tid < kSummaryDim) {
        const double v = s[tid];
        const uint16_t h = f32_to_bf16((float)v);
        x_row[(size_t)b * kSummaryDim + tid] = h;
        x_col[(size_t)tid * B + b] = h;
        if (s64) s64[(size_t)b * kSummaryDim + tid] = v;
    }
}

template <int MODEL>
__global__ __launch_bounds__(kSumThreads) void simulate_kernel(SimSpec sp, int B, Key key,
                                                               const int64_t *__restrict__ step_ptr,
                                                               uint16_t *__restrict__ x_row,
                                                               uint16_t *__restrict__ x_col,
                                                               double *__restrict__ theta,
                                                               double *__restrict__ s64) {
    simulate_block<MODEL>(sp, B, key, step_ptr, x_row, x_col, theta, s64, (int)blockIdx.x);
}

// The simulation of the next step's batch (workgroups 0 .. B - 1, first, as
// the longer ones) and the Adam update of this step (the rest) in one launch:
// the simulation reads only the step count, which the step's bookkeeping has
// already advanced, and its buffers were last read by the launches before.
template <int MODEL>
__global__ __launch_bounds__(kSumThreads) void adam_simulate_kernel(MlpView w, SplitParts spl,
                                                                    const float *__restrict__ bgrad, AdamSpec ad,
                                                                    const float *__restrict__ coef, SimSpec sp, int B,
                                                                    Key key,
                                                                    const int64_t *__restrict__ step_ptr,
                                                                    uint16_t *__restrict__ x_row,
                                                                    uint16_t *__restrict__ x_col,
                                                                    double *__restrict__ theta) {
    if ((int)blockIdx.x >= B) {
        adam_unit(w, spl, bgrad, ad, coef, nullptr, (int64_t)((int)blockIdx.x - B) * kSumThreads + threadIdx.x);
        return;
    }
    simulate_block<MODEL>(sp, B, key, step_ptr, x_row, x_col, theta, nullptr, (int)blockIdx.x);
}

// ------------------------------------------------------------------ host --
int launch_simulate(const SimSpec &sp, int B, uint64_t seed, const int64_t *step, uint16_t *x_row, uint16_t *x_col,
                    double *theta, double *s64, hipStream_t st) {
    if (B <= 0) return fail(PPL_E_ARG, "simulation batch %d is not positive", B);
    const dim3 grid((unsigned)B), block(kSumThreads);
    if (sp.model == PPL_MODEL_POLY) {
        hipLaunchKernelGGL(simulate_kernel<PPL_MODEL_POLY>, grid, block, 0, st, sp, B, make_key(seed), step, x_row,
                           x_col, theta, s64);
        PPL_LAUNCH_CHECK("simulate_kernel<POLY>");
    } else {
        if (sp.D > kGmmTrainMaxD) return fail(PPL_E_ARG, "mixture training datasets hold at most %d points", kGmmTrainMaxD);
        const size_t lds = (size_t)(sp.D > 0 ? sp.D : 1) * sizeof(double);
        hipLaunchKernelGGL(simulate_kernel<PPL_MODEL_GMM>, grid, block, lds, st, sp, B, make_key(seed), step, x_row,
                           x_col, theta, s64);
        PPL_LAUNCH_CHECK("simulate_kernel<GMM>");
    }
    return PPL_OK;
}

int launch_update_simulate(const MlpView &w, const TrainBufs &b, const AdamSpec &ad, const SimSpec &sp, int B,
                           uint64_t seed, const int64_t *step, hipStream_t st) {
    if (B <= 0) return fail(PPL_E_ARG, "simulation batch %d is not positive", B);
    const int adam_blocks = (int)((MlpParams::count() + kSumThreads - 1) / kSumThreads);
    const dim3 grid((unsigned)(adam_blocks + B)), block(kSumThreads);
    const SplitParts spl = split_parts(b);
    if (sp.model == PPL_MODEL_POLY) {
        hipLaunchKernelGGL(adam_simulate_kernel<PPL_MODEL_POLY>, grid, block, 0, st, w, spl, (const float *)b.bgrad, ad,
                           (const float *)b.coef, sp, B, make_key(seed), step, b.x_row, b.x_col, b.theta);
    } else {
        if (sp.D > kGmmTrainMaxD) return fail(PPL_E_ARG, "mixture training datasets hold at most %d points", kGmmTrainMaxD);
        const size_t lds = (size_t)(sp.D > 0 ? sp.D : 1) * sizeof(double);
        hipLaunchKernelGGL(adam_simulate_kernel<PPL_MODEL_GMM>, grid, block, lds, st, w, spl, (const float *)b.bgrad, ad,
                           (const float *)b.coef, sp, B, make_key(seed), step, b.x_row, b.x_col, b.theta);
    }
    PPL_LAUNCH_CHECK("adam_simulate_kernel");
    return PPL_OK;
}

}  // namespace ppl
