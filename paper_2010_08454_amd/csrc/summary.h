// summary.h -- the 64 data summaries the proposal network reads, computed by one
// 256-thread workgroup per dataset: the threads stride over the data points,
// FP64 moment sums are combined by wave reductions and a fixed-order sum of the
// four wave totals, and the per-dataset finishing work (least-squares fits,
// order statistics) runs on the first wave.
#pragma once

#include "device.h"
#include "proposal.h"

namespace ppl {

constexpr int kSumThreads = 256;     // one dataset per workgroup
constexpr int kSumWaves = kSumThreads / 64;

// ------------------------------------------------------------- POLY --
// Moment accumulators: [0..7] sum x^j y, [8..22] sum x^k (k = 0..14), [23] sum y^2.
constexpr int kPolyAcc = 24;

__device__ __forceinline__ void poly_acc_point(double (&a)[kPolyAcc], double x, double y) {
#pragma clang fp contract(off)
    double p = 1.0;
#pragma unroll
    for (int k = 0; k <= 14; ++k) {
        if (k < 8) a[k] += p * y;
        a[8 + k] += p;
        p *= x;
    }
    a[23] += y * y;
}

// Least-squares fit with n coefficients from the normalised moments
// (normal equations G beta = m, G_ij = mean x^(i+j), m_i = mean x^i y) by a
// Cholesky factorisation and two triangular solves.
// The diagonal's reciprocals are formed once (one division per column, then
// products): the solve's chain of dependent FP64 divisions is its latency.
__device__ void poly_ls(int n, const double *gx, const double *mxy, double (&beta)[5]) {
#pragma clang fp contract(off)
    double L[5][5], z[5], rd[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            if (i < n) {
                double s = gx[i + j];
#pragma unroll
                for (int k = 0; k < j; ++k) s -= L[i][k] * L[j][k];
                if (i == j) {
                    L[i][i] = sqrt(s > 1e-300 ? s : 1e-300);
                    rd[i] = 1.0 / L[i][i];
                } else {
                    L[i][j] = s * rd[j];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        if (i < n) {
            double s = mxy[i];
#pragma unroll
            for (int k = 0; k < i; ++k) s -= L[i][k] * z[k];
            z[i] = s * rd[i];
        }
    }
#pragma unroll
    for (int i = 4; i >= 0; --i) {
        beta[i] = 0.0;
        if (i < n) {
            double s = z[i];
#pragma unroll
            for (int k = i + 1; k < 5; ++k)
                if (k < n) s -= L[k][i] * beta[k];
            beta[i] = s * rd[i];
        }
    }
}

// Sum of one double per thread over the workgroup, returned to every thread:
// wave butterflies, then the wave totals in a fixed order.  red holds
// kSumWaves doubles.
__device__ __forceinline__ double block_sum(double v, double *red) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// Reduce the thread accumulators and write the 64 POLY summaries to s[]:
//   [0..7] mean x^j y / 10; [8..21] mean x^k, k = 1..14; [22] mean y^2 / 100;
//   [23..36] least-squares coefficients for n = 2..5 / 10;
//   [37..40] log(1 + (RSS_n - RSS_5) / 2) / 10 (RSS_n the residual sum of
//   squares of the n-coefficient fit: the log-likelihood gap to the largest
//   fit, independent of the absolute noise level); [41] log D / 10; rest 0.
__device__ void poly_finish(double (&a)[kPolyAcc], int64_t D, double (*wtot)[kPolyAcc], double *tot, double *s) {
#pragma clang fp contract(off)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
#pragma unroll
    for (int k = 0; k < kPolyAcc; ++k) a[k] = wave_sum_dpp(a[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kPolyAcc; ++k) wtot[wv][k] = a[k];
    }
    __syncthreads();
    if (tid < kPolyAcc)
        tot[tid] = D > 0 ? ((wtot[0][tid] + wtot[1][tid]) + (wtot[2][tid] + wtot[3][tid])) / (double)D : 0.0;
    __syncthreads();
    if (wv == 0) {
        const double *mxy = tot, *gx = tot + 8;
        double v = 0.0;
        if (D > 0) {
            if (lane < 8) v = mxy[lane] / 10.0;
            else if (lane < 22) v = gx[lane - 7];
            else if (lane == 22) v = tot[23] / 100.0;
            else if (lane == 41) v = log((double)D) / 10.0;
        }
        if (lane < 23 || lane >= 41) s[lane] = v;
        double rss = 0.0;
        if (lane < 4) {
            const int n = 2 + lane;
            double beta[5];
            poly_ls(n, gx, mxy, beta);
            double fit = 0.0;
            const int o = 23 + (n - 2) * (n + 1) / 2;
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                if (j < n) {
                    s[o + j] = D > 0 ? beta[j] / 10.0 : 0.0;
                    fit += beta[j] * mxy[j];
                }
            }
            rss = tot[23] - fit;
            if (rss < 0.0) rss = 0.0;
        }
        const double rss5 = __shfl(rss, 3, 64);
        if (lane < 4) {
            double gap = (double)D * (rss - rss5) / 2.0;
            if (gap < 0.0) gap = 0.0;
            s[37 + lane] = D > 0 ? log1p(gap) / 10.0 : 0.0;
        }
    }
    __syncthreads();
}

// ------------------------------------------------------------- GMM --
// Summaries from the data in LDS ys[D] (FP64 simulated points, or the FP32
// observed values, compared and summed in FP64):
//   [0..15] order statistics y_(floor((q + 1/2) D / 16)) / 10;
//   [16..47] counts on the unit bins of [-16, 16) (ends clamped) / D;
//   [48] mean / 10, [49] sd / 10, [50] skewness, [51] excess kurtosis / 10,
//   [52] log D / 10; rest 0.  hist holds the workgroup's 32 bin counts,
//   already filled; sum_y is the thread's sum of its points.
template <typename T>
__device__ void gmm_finish(const T *ys, int64_t D, const int *hist, double sum_y, double *red, double *s) {
#pragma clang fp contract(off)
    const int tid = threadIdx.x;
    const double m1 = D > 0 ? block_sum(sum_y, red) / (double)D : 0.0;
    double c2 = 0.0, c3 = 0.0, c4 = 0.0;
    for (int64_t d = tid; d < D; d += kSumThreads) {
        const double y = (double)ys[d];
        int64_t r = 0;
        for (int64_t e = 0; e < D; ++e) {
            const double ye = (double)ys[e];
            r += (ye < y) || (ye == y && e < d);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (r == (int64_t)floor((q + 0.5) * (double)D / 16.0)) s[q] = y / 10.0;
        const double dv = y - m1;
        c2 += dv * dv;
        c3 += dv * dv * dv;
        c4 += dv * dv * dv * dv;
    }
    c2 = block_sum(c2, red);
    c3 = block_sum(c3, red);
    c4 = block_sum(c4, red);
    if (D <= 0 && tid < 16) s[tid] = 0.0;
    if (tid < 32) s[16 + tid] = D > 0 ? (double)hist[tid] / (double)D : 0.0;
    if (tid >= 53 && tid < kSummaryDim) s[tid] = 0.0;
    if (tid == 0) {
        double v2 = 0.0, v3 = 0.0, v4 = 0.0;
        if (D > 0) {
            v2 = c2 / (double)D;
            v3 = c3 / (double)D;
            v4 = c4 / (double)D;
        }
        const double sd = sqrt(v2);
        s[48] = m1 / 10.0;
        s[49] = sd / 10.0;
        s[50] = v2 > 0 ? v3 / (v2 * sd) : 0.0;
        s[51] = v2 > 0 ? (v4 / (v2 * v2) - 3.0) / 10.0 : 0.0;
        s[52] = D > 0 ? log((double)D) / 10.0 : 0.0;
    }
    __syncthreads();
}

__device__ __forceinline__ void gmm_bin(int *hist, double y) {
    int b = (int)floor(y + 16.0);
    b = b < 0 ? 0 : (b > 31 ? 31 : b);
    atomicAdd(&hist[b], 1);
}

}  // namespace ppl
