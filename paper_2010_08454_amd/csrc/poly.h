// poly.h -- the polynomial model of the paper's running example (Sec. 1.1):
// n ~ UniformDiscrete{n_lo..n_hi}, c_j ~ Normal(0, sd) for j < n,
// factor(-sum_d (y_d - sum_j c_j x_d^j)^2 / 2); shared by importance sampling
// and the Metropolis-Hastings chains (whose chains start from this draw).
#pragma once

#include "device.h"

namespace ppl {

// Prior draw of execution i (tag 0): block 0 word 0 picks n; blocks 1..3 give
// one double-precision Box-Muller pair each, c_0..c_5 (all drawn whatever n
// is, so the word table does not depend on the branch); c_j for j >= n are
// returned as they were drawn.
__device__ __forceinline__ void poly_prior_draw(uint32_t i, Key key, double sd, int n_lo, int n_hi, int &n,
                                                double c[5]) {
    const uint4 w0 = philox(i, 0, 0, kTagPrior, key);
    n = uniform_discrete(w0.x, n_lo, (uint32_t)(n_hi - n_lo + 1));
    double z[6];
#pragma unroll
    for (int b = 1; b <= 3; ++b) {
        const uint4 w = philox(i, b, 0, kTagPrior, key);
        box_muller(unit_f64(w.x, w.y), unit_f64(w.z, w.w), z[2 * (b - 1)], z[2 * (b - 1) + 1]);
    }
#pragma unroll
    for (int j = 0; j < 5; ++j) c[j] = sd * z[j];
}

// One point's contribution (y - p(x))^2 with p evaluated by Horner over the
// five coefficient slots, zero past the degree: 0 x + 0 = 0 exactly, so this
// equals n-term Horner and no lane branches on n.
__device__ __forceinline__ double poly_sq_residual(const double pc[5], double x, double y) {
    double v = pc[4];
    v = fma(v, x, pc[3]);
    v = fma(v, x, pc[2]);
    v = fma(v, x, pc[1]);
    v = fma(v, x, pc[0]);
    const double r = y - v;
    return r * r;
}

// ---------------------------------------------- a lane group per particle --
// Pieces of the kernels that give a particle L = 4 or 8 neighbouring lanes
// (calls too small to fill the chip with a lane each).

constexpr int kGroupPoints = 512;                // points in LDS at a time

// The workgroup's share of points d0 .. d0 + kGroupPoints - 1.
template <int THREADS>
__device__ __forceinline__ void poly_group_load(const double *__restrict__ X, const double *__restrict__ Y, int D,
                                                int d0, double2 (&v)[kGroupPoints / THREADS]) {
#pragma unroll
    for (int k = 0; k < kGroupPoints / THREADS; ++k) {
        const int d = d0 + (int)threadIdx.x + k * THREADS;
        v[k] = d < D ? make_double2(X[d], Y[d]) : make_double2(0.0, 0.0);
    }
}

// Lane b's share of sum_d (y_d - p(x_d))^2, the points d = b mod L; `first` holds
// the first points, already loaded.  Called by every thread of the workgroup.
template <int L, int THREADS>
__device__ __forceinline__ double poly_group_sq(const double (&pc)[5], const double *__restrict__ X,
                                                const double *__restrict__ Y, int D,
                                                double2 (&first)[kGroupPoints / THREADS], double2 *xy) {
    double acc = 0.0;
    for (int d0 = 0; d0 < D; d0 += kGroupPoints) {
        if (d0 > 0) {
            __syncthreads();
            poly_group_load<THREADS>(X, Y, D, d0, first);
        }
#pragma unroll
        for (int k = 0; k < kGroupPoints / THREADS; ++k) xy[threadIdx.x + k * THREADS] = first[k];
        __syncthreads();
        const int m = min(kGroupPoints, D - d0);
        int d = threadIdx.x % L;
        for (; d + 7 * L < m; d += 8 * L) {
            double2 p[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) p[k] = xy[d + L * k];
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += poly_sq_residual(pc, p[k].x, p[k].y);
        }
        for (; d < m; d += L) acc += poly_sq_residual(pc, xy[d].x, xy[d].y);
    }
    return acc;
}

// The workgroup's normaliser record from one log-weight per lane group (every
// lane of the group holds it, the degree and the coefficients, zero past the
// degree): lane b < 4 adds the sums of degree 2 + b.
template <int L, int NWAVES>
__device__ __forceinline__ void poly_group_record(double lw, bool live, int n, const double (&pc)[5],
                                                  double *__restrict__ part) {
    constexpr int kSums = 10;                    // degree slot: mass, 5 means; all: e, e^2, NaN, degree-1 c_0
    constexpr int kRows = 4 * NWAVES;            // rows of 16 lanes
    __shared__ double sums[kRows][4][kSums];
    const int tid = threadIdx.x, b = tid % L;
    const double M = block_max_f64<NWAVES>(isnan(lw) ? -INFINITY : lw);
    const double e = lw > -INFINITY ? exp_le0(lw - M) : 0.0;
    const double own = n - 2 == b ? e : 0.0, one = b == 0 ? e : 0.0;
    double v[kSums] = {own,
                       own * pc[0],
                       own * pc[1],
                       own * pc[2],
                       own * pc[3],
                       own * pc[4],
                       one,
                       one * one,
                       b == 0 && live && isnan(lw) ? 1.0 : 0.0,
                       n == 1 ? one * pc[0] : 0.0};
    // over the groups of a row of 16 lanes (rotations by 8 and, for quads, 4), then over the rows through LDS
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
        v[k] += dpp_f64<0x128, 0xF>(v[k]);
        if constexpr (L == 4) v[k] += dpp_f64<0x124, 0xF>(v[k]);
    }
    if ((tid & 15) < 4) {
#pragma unroll
        for (int k = 0; k < kSums; ++k) sums[tid >> 4][b][k] = v[k];
    }
    __syncthreads();
    double *rec = part + (size_t)blockIdx.x * (4 + kPolyNF);
    if (tid < 3 + kPolyNF) {
        // record slots after the maximum: s1, s2, nan, mass[4], c[4][5], degree-1 c_0
        int s = 0, k = 6 + tid;
        if (tid >= 3 && tid < 7) { s = tid - 3; k = 0; }
        else if (tid >= 7 && tid < 27) { s = (tid - 7) / 5; k = 1 + (tid - 7) % 5; }
        else if (tid == 27) k = 9;
        double t = 0.0;
#pragma unroll
        for (int r = 0; r < kRows; ++r) t += sums[r][s][k];
        rec[1 + tid] = t;
    }
    if (tid == 0) rec[0] = M;
}

}  // namespace ppl
