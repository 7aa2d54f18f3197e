// mcmc.hip -- lightweight Metropolis-Hastings (paper Sec. 3.6.3) on the GPU:
// many independent chains of the polynomial model, one chain per lane.
//
// A chain's trace holds the sites its execution reached: n and c_0..c_{n-1}.
// An iteration picks one site of the trace uniformly, resamples it from its
// prior and re-executes the model: when n changes, coefficients both
// executions reach keep their values, coefficients only the new execution
// reaches are drawn fresh from their prior, and those it no longer reaches
// are dropped.  With prior proposals every prior density cancels and
//     alpha = L(x') / L(x) * (n + 1) / (n' + 1)
// (likelihood ratio times the ratio of the traces' site counts).
//
// Words of iteration t of chain c (tag 8): block (c, 3t, 0) word 0 picks the
// site (uniform discrete over 0..n: 0 is n, j + 1 is c_j), word 1 the
// proposed n' (uniform discrete over n_lo..n_hi), word 2 the acceptance
// uniform v; blocks (c, 3t + 1, 0) and (c, 3t + 2, 0) give one
// double-precision Box-Muller pair each, z_0..z_3: a resampled c_j is sd z_0
// and fresh coefficients c_n, c_{n+1}, ... are sd z_1, sd z_2, sd z_3.  A
// chain starts from the importance sampler's prior draw of execution c.
// Accepted when log v < log alpha (FP64).
//
// Each lane keeps its chain's state and the post-burn-in sums in registers;
// the data points are the same for every lane and come through scalar loads.
// The sums fold into per-workgroup records in a fixed order, and one
// workgroup merges those.
#include <algorithm>

#include "device.h"
#include "host.h"
#include "mcmc.h"
#include "poly.h"
#include "timing.h"

namespace ppl {

constexpr int kMcThreads = 256;
constexpr int kMcWaves = kMcThreads / 64;
constexpr int kMcNF = 30;                   // per-chain sums: 29 summary fields + accepted count
constexpr uint32_t kTagMcmc = 8;

// Adds points d .. d + C - 1: one batch of scalar loads, all points' arithmetic.
template <int C>
__device__ __forceinline__ void mc_points(const double pc[5], const double *__restrict__ X,
                                          const double *__restrict__ Y, int d, double &acc) {
    double xs[C], ys[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        xs[k] = X[d + k];
        ys[k] = Y[d + k];
    }
#pragma unroll
    for (int k = 0; k < C; ++k) acc += poly_sq_residual(pc, xs[k], ys[k]);
}

// -1/2 sum_d (y_d - p(x_d))^2 in FP64.  At 2^16 chains each SIMD holds one wave,
// so every batch of scalar loads is waited for (about 180 cycles): points go in
// batches of sixteen (64 scalar registers), then four, then one.  Batches of eight
// and single points after them took 3.33 ms against 3.00 at 2^16 chains x 1000
// iterations over 100 points.  From LDS, eight points ahead, it was 3.83 ms:
// a broadcast of 16 bytes keeps the LDS busy for as long as four waves' arithmetic
// on the point.
__device__ __forceinline__ double mc_loglik(const double pc[5], const double *__restrict__ X,
                                            const double *__restrict__ Y, int D) {
    double acc = 0.0;
    int d = 0;
    for (; d + 16 <= D; d += 16) mc_points<16>(pc, X, Y, d, acc);
    for (; d + 4 <= D; d += 4) mc_points<4>(pc, X, Y, d, acc);
    for (; d < D; ++d) mc_points<1>(pc, X, Y, d, acc);
    return -0.5 * acc;
}

// log k for the trace-size ratio, k = n + 1 in [2, 6] (each literal the nearest
// double).  A chain of selects between literals; selects between the elements of a
// table are folded back into a load at a run-time index, which is an LDS table or
// scratch memory inside the iteration.
__device__ __forceinline__ double log_size(int k) {
    double r = 0x1.62e42fefa39efp-1;
    r = k == 3 ? 0x1.193ea7aad030bp+0 : r;
    r = k == 4 ? 0x1.62e42fefa39efp+0 : r;
    r = k == 5 ? 0x1.9c041f7ed8d33p+0 : r;
    r = k == 6 ? 0x1.cab0bfa2a2002p+0 : r;
    return r;
}

__global__ __launch_bounds__(kMcThreads) void mcmc_poly_kernel(
    const double *__restrict__ X, const double *__restrict__ Y, int D, int64_t C, int64_t T, int64_t burn,
    Key key, double sd, int n_lo, int n_hi, double *__restrict__ state_out, int64_t *__restrict__ acc_out,
    int8_t *__restrict__ n_tr, double *__restrict__ la_tr, double *__restrict__ part) {
    __shared__ double lds[kMcWaves][kMcNF];
    const int64_t c = (int64_t)blockIdx.x * kMcThreads + threadIdx.x;
    const bool valid = c < C;
    int n;
    double pc[5];
    poly_prior_draw((uint32_t)c, key, sd, n_lo, n_hi, n, pc);
#pragma unroll
    for (int j = 0; j < 5; ++j) pc[j] = j < n ? pc[j] : 0.0;
    double ll = mc_loglik(pc, X, Y, D);
    double sums[kMcNF];
#pragma unroll
    for (int k = 0; k < kMcNF; ++k) sums[k] = 0.0;
    const uint32_t range = (uint32_t)(n_hi - n_lo + 1);

    for (int64_t t = 0; t < T; ++t) {
        const uint4 w = philox((uint32_t)c, (uint32_t)(3 * t), 0, kTagMcmc, key);
        const int site = uniform_discrete(w.x, 0, (uint32_t)(n + 1));
        int n2 = n;
        double c2[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) c2[j] = pc[j];
        double z[4];
        {   // z_0 (a resampled coefficient) and z_1 (the first fresh one)
            const uint4 b1 = philox((uint32_t)c, (uint32_t)(3 * t + 1), 0, kTagMcmc, key);
            box_muller(unit_f64(b1.x, b1.y), unit_f64(b1.z, b1.w), z[0], z[1]);
        }
        if (site == 0) {
            n2 = uniform_discrete(w.y, n_lo, range);
            if (n2 > n + 1) {
                const uint4 b2 = philox((uint32_t)c, (uint32_t)(3 * t + 2), 0, kTagMcmc, key);
                box_muller(unit_f64(b2.x, b2.y), unit_f64(b2.z, b2.w), z[2], z[3]);
            } else {
                z[2] = z[3] = 0.0;
            }
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                // slot j: kept (j < n and j < n2), fresh (n <= j < n2, normal z_{1 + j - n}), dropped (j >= n2)
                const int f = j - n;                 // index of the fresh normal minus one
                const double fresh = sd * (f == 0 ? z[1] : (f == 1 ? z[2] : z[3]));
                c2[j] = j >= n2 ? 0.0 : (j < n ? pc[j] : fresh);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 5; ++j) c2[j] = (j == site - 1) ? sd * z[0] : pc[j];
        }
        const double ll2 = mc_loglik(c2, X, Y, D);
        const double la = (ll2 - ll) + (log_size(n + 1) - log_size(n2 + 1));
        const bool acc = log_unit((double)unit_f32(w.z)) < la;
        if (valid && la_tr) la_tr[t * C + c] = la;
        if (acc) {
            n = n2;
#pragma unroll
            for (int j = 0; j < 5; ++j) pc[j] = c2[j];
            ll = ll2;
            sums[29] += 1.0;
        }
        if (valid && n_tr) n_tr[t * C + c] = (int8_t)n;
        if (t >= burn) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const bool here = n == m + 2;
                sums[m] += here ? 1.0 : 0.0;
#pragma unroll
                for (int j = 0; j < 5; ++j) sums[4 + 5 * m + j] += here ? pc[j] : 0.0;
            }
#pragma unroll
            for (int j = 0; j < 5; ++j) sums[24 + j] += pc[j];
        }
    }
    if (valid) {
        if (state_out) {
            state_out[c] = (double)n;
#pragma unroll
            for (int j = 0; j < 5; ++j) state_out[(size_t)(1 + j) * C + c] = pc[j];
        }
        if (acc_out) acc_out[c] = (int64_t)sums[29];
    } else {
#pragma unroll
        for (int k = 0; k < kMcNF; ++k) sums[k] = 0.0;
    }
    // workgroup record: waves in order
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kMcNF; ++k) {
        const double v = wave_sum_dpp(sums[k]);
        if ((threadIdx.x & 63) == 0) lds[wave][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < kMcNF) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kMcWaves; ++w) v += lds[w][threadIdx.x];
        part[(size_t)blockIdx.x * kMcNF + threadIdx.x] = v;
    }
}

// Four lanes per chain, for calls of at most 2^14 chains (one wave per SIMD so), and
// up to 2^15 from 64 points on.  All four lanes hold the chain; lane b draws one
// of the iteration's three Philox blocks and its Box-Muller pair, takes every
// fourth point, from LDS, and keeps the sums of degree 2 + b.
// Bound: the latency of one iteration, with two waves per SIMD its issue.  us a call
// against a lane per chain: 1000 chains x 1000 iterations x 200 points 1889 and
// 4424, 10007 x 300 x 100 427 and 925, 2^15 x 300 x 200 920 and 1350 (1999, 460 and
// 947 with the trace-size logarithms in scratch memory; so too 20000 x 300 x 30
// 673 and about 610).
constexpr int kMcQuadChains = 32768;
constexpr int kMcQuadPoints = 2048;         // most points in LDS (32 KB)

__global__ __launch_bounds__(kMcThreads) void mcmc_poly_quad_kernel(
    const double *__restrict__ X, const double *__restrict__ Y, int D, int64_t C, int64_t T, int64_t burn,
    Key key, double sd, int n_lo, int n_hi, double *__restrict__ state_out, int64_t *__restrict__ acc_out,
    int8_t *__restrict__ n_tr, double *__restrict__ la_tr, double *__restrict__ part) {
    constexpr int kRows = kMcThreads / 16;
    constexpr int kSums = 8;                     // degree slot: count, 5 coefficients; lane 0: degree-1 c_0, accepted
    __shared__ double rows[kRows][4][kSums];
    extern __shared__ double2 xy[];              // D points
    for (int d = threadIdx.x; d < D; d += kMcThreads) xy[d] = make_double2(X[d], Y[d]);
    __syncthreads();
    const int b = threadIdx.x & 3;
    const int64_t c = (int64_t)blockIdx.x * (kMcThreads / 4) + (threadIdx.x >> 2);
    const bool valid = c < C;
    auto loglik = [&](const double (&pc)[5]) {
        double acc = 0.0;
        int d = b;
        for (; d + 28 < D; d += 32) {
            double2 p[8];
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) p[k] = xy[d + 4 * k];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = pc[4];
#pragma unroll
            for (int j = 3; j >= 0; --j)
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = fma(v[k], p[k].x, pc[j]);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const double r = p[k].y - v[k];
                acc = fma(r, r, acc);
            }
        }
        for (; d < D; d += 4) acc += poly_sq_residual(pc, xy[d].x, xy[d].y);
        acc += dpp_f64<0xB1, 0xF>(acc);
        acc += dpp_f64<0x4E, 0xF>(acc);
        return -0.5 * acc;
    };
    auto word0 = [](uint32_t v) {                // lane 0's word
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x00, 0xF, 0xF, false);
    };
    int n;
    double pc[5];
    poly_prior_draw((uint32_t)c, key, sd, n_lo, n_hi, n, pc);
#pragma unroll
    for (int j = 0; j < 5; ++j) pc[j] = j < n ? pc[j] : 0.0;
    double ll = loglik(pc);
    double sums[kSums];
#pragma unroll
    for (int k = 0; k < kSums; ++k) sums[k] = 0.0;
    const uint32_t range = (uint32_t)(n_hi - n_lo + 1);
    for (int64_t t = 0; t < T; ++t) {
        const uint4 w = philox((uint32_t)c, (uint32_t)(3 * t) + (uint32_t)min(b, 2), 0, kTagMcmc, key);
        const int site = uniform_discrete(word0(w.x), 0, (uint32_t)(n + 1));
        double za, zb;
        box_muller(unit_f64(w.x, w.y), unit_f64(w.z, w.w), za, zb);
        const double z0 = dpp_f64<0x55, 0xF>(za), z1 = dpp_f64<0x55, 0xF>(zb);
        const double z2 = dpp_f64<0xAA, 0xF>(za), z3 = dpp_f64<0xAA, 0xF>(zb);
        const int n2 = site == 0 ? uniform_discrete(word0(w.y), n_lo, range) : n;
        double c2[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            // site 0: slot j kept (j < n, j < n2), fresh (n <= j < n2) or dropped; else the chosen slot redrawn
            const int f = j - n;
            const double fresh = sd * (f == 0 ? z1 : (f == 1 ? z2 : z3));
            const double moved = j >= n2 ? 0.0 : (j < n ? pc[j] : fresh);
            c2[j] = site == 0 ? moved : (j == site - 1 ? sd * z0 : pc[j]);
        }
        const double ll2 = loglik(c2);
        const double la = (ll2 - ll) + (log_size(n + 1) - log_size(n2 + 1));
        const bool acc = log_unit((double)unit_f32(word0(w.z))) < la;
        if (valid && la_tr && b == 0) la_tr[t * C + c] = la;
        if (acc) {
            n = n2;
#pragma unroll
            for (int j = 0; j < 5; ++j) pc[j] = c2[j];
            ll = ll2;
            sums[7] += 1.0;
        }
        if (valid && n_tr && b == 0) n_tr[t * C + c] = (int8_t)n;
        if (t >= burn) {
            const bool here = n == b + 2;
            sums[0] += here ? 1.0 : 0.0;
#pragma unroll
            for (int j = 0; j < 5; ++j) sums[1 + j] += here ? pc[j] : 0.0;
            sums[6] += n == 1 ? pc[0] : 0.0;
        }
    }
    if (valid && b == 0) {
        if (state_out) {
            state_out[c] = (double)n;
#pragma unroll
            for (int j = 0; j < 5; ++j) state_out[(size_t)(1 + j) * C + c] = pc[j];
        }
        if (acc_out) acc_out[c] = (int64_t)sums[7];
    }
    // workgroup record: the four chains of a row of 16 lanes, then the rows in order
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
        double v = valid ? sums[k] : 0.0;
        v += dpp_f64<0x128, 0xF>(v);
        v += dpp_f64<0x124, 0xF>(v);
        if ((threadIdx.x & 15) < 4) rows[threadIdx.x >> 4][b][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < kMcNF) {
        // fields: count[4], c[4][5], overall c[5] (all degrees, with degree 1's c_0), accepted
        const int k = threadIdx.x;
        double v = 0.0;
        for (int r = 0; r < kRows; ++r) {
            if (k < 4) v += rows[r][k][0];
            else if (k < 24) v += rows[r][(k - 4) / 5][1 + (k - 4) % 5];
            else if (k < 29) {
                const int j = k - 24;
                v += (rows[r][0][1 + j] + rows[r][1][1 + j]) + (rows[r][2][1 + j] + rows[r][3][1 + j]);
                if (j == 0) v += rows[r][0][6];
            } else v += rows[r][0][7];
        }
        part[(size_t)blockIdx.x * kMcNF + threadIdx.x] = v;
    }
}

// One workgroup: the records summed in a fixed order (a half-wave per record,
// a field per lane, eight records in flight; one thread per field adding 256
// records in turn took 62 us), then the summaries (as importance sampling lays
// them out) and {acceptance rate, kept samples, chains, status}.
__global__ __launch_bounds__(1024) void mcmc_finalize_kernel(const double *__restrict__ part, int64_t nblocks,
                                                             int64_t C, int64_t T, double *__restrict__ scalars,
                                                             double *__restrict__ summaries) {
    __shared__ double sums[32][32];
    __shared__ double tot[kMcNF];
    const int f = threadIdx.x & 31, half = threadIdx.x >> 5;
    double v = 0.0;
    for (int64_t b0 = half; b0 < nblocks; b0 += 8 * 32) {
        double r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = b0 + 32 * u < nblocks && f < kMcNF ? part[(size_t)(b0 + 32 * u) * kMcNF + f] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) v += r[u];
    }
    sums[half][f] = v;
    __syncthreads();
    if (threadIdx.x < kMcNF) {
        double t = sums[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < 32; ++w) t += sums[w][threadIdx.x];
        tot[threadIdx.x] = t;
    }
    __syncthreads();
    const double all = tot[0] + tot[1] + tot[2] + tot[3];
    if (summaries && threadIdx.x < 29) {
        const int k = threadIdx.x, m = (k - 4) / 5;
        double r;
        if (k < 4) r = all > 0 ? tot[k] / all : 0.0;
        else if (k < 24) r = tot[m] > 0 ? tot[k] / tot[m] : 0.0;
        else r = all > 0 ? tot[k] / all : 0.0;
        summaries[k] = r;
    }
    if (threadIdx.x != 0) return;
    scalars[0] = T > 0 ? tot[29] / ((double)C * (double)T) : 0.0;
    scalars[1] = all;
    scalars[2] = (double)C;
    scalars[3] = 0.0;
}

static size_t mcmc_bytes(int64_t records) { return 256 + align_up((size_t)records * kMcNF * sizeof(double), 256); }

size_t mcmc_ws_min_bytes(int64_t chains) { return mcmc_bytes((chains + kMcThreads - 1) / kMcThreads); }

// Room for the quad kernel's records at every chain count it may take, so that
// the size never falls as the chains grow.
size_t mcmc_ws_bytes(int64_t chains) {
    const int64_t quads = (std::min<int64_t>(chains, kMcQuadChains) + kMcThreads / 4 - 1) / (kMcThreads / 4);
    return std::max(mcmc_ws_min_bytes(chains), mcmc_bytes(quads));
}

// A workspace too small for the quad kernel's records takes a lane per chain (four
// times fewer records), which is also faster there than quads in workgroups of 1024
// threads with as few records (1000 chains x 1000 iterations x 200 points: 6.0 ms).
int run_mcmc_poly(const McmcArgs &a, hipStream_t st) {
    const bool quad = a.C <= (a.D < 64 ? kMcQuadChains / 2 : kMcQuadChains) && a.D <= kMcQuadPoints &&
                      a.ws_bytes >= mcmc_ws_bytes(a.C);
    const int64_t per = quad ? kMcThreads / 4 : kMcThreads;
    const int64_t blocks = (a.C + per - 1) / per;
    if (int rc = check_grid("mcmc_poly_kernel", blocks, kMcThreads)) return rc;
    double *part = (double *)((char *)a.ws + 256);
    {
        KernelTimer timer("mcmc_poly_kernel", st);
        hipLaunchKernelGGL(quad ? mcmc_poly_quad_kernel : mcmc_poly_kernel, dim3((unsigned)blocks), dim3(kMcThreads),
                           quad ? (size_t)a.D * sizeof(double2) : 0, st, a.x, a.y, (int)a.D, a.C,
                           a.T, a.burn, make_key(a.seed), a.hyper[0], (int)a.hyper[1], (int)a.hyper[2], a.state_out,
                           a.acc_out, a.n_trace, a.la_trace, part);
        timer.stop();
    }
    PPL_LAUNCH_CHECK("mcmc_poly_kernel");
    hipLaunchKernelGGL(mcmc_finalize_kernel, dim3(1), dim3(1024), 0, st, part, blocks, a.C, a.T, a.scalars,
                       a.summaries);
    PPL_LAUNCH_CHECK("mcmc_finalize_kernel");
    return PPL_OK;
}

}  // namespace ppl
