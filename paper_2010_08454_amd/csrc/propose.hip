// propose.hip -- importance sampling (paper Sec. 3.6.2) with a diagonal
// Gaussian-mixture proposal q -- the decoded output of the proposal network --
// in place of the prior, and prior importance sampling of the mixture model.
// Each particle draws its latents from q (Philox tag 1), and its log-weight is
// log p(latents) + log L(latents) - log q(latents); the block partials and the
// finalize step are those of the prior importance sampler.  FP64 throughout,
// except the mixture model's likelihood: FP32 per datum (hardware exp and
// log), summed in FP32 within 16-datum blocks and in FP64 across them.
//
// Proposal parameter blocks (FP64, device):
//   POLY (degrees 2..5): lognl[4], logmix[8], mean[4][8][5], lsd[4][8][5];
//        block 0 word 0 picks the degree, word 1 the component (inverse CDF),
//        blocks 1, 2 give eight normals, c_j = mean + exp(lsd) z_j for j < n.
//   GMM (K components, d = 2K - 1): logmix[8], mean[8][d], lsd[8][d]; block 0
//        word 0 picks the component, blocks 1..4 give sixteen normals, u_k =
//        mean + exp(lsd) z_k over the ordered unconstrained latents
//        u = (mu_(1), log(mu_(k) - mu_(k-1)), log pi_(k) - log pi_(K)); its
//        prior density carries the Dirichlet(1) normaliser (K-1)!, the K!
//        orderings (p and L are invariant under relabelling) and the
//        Jacobians of the gap and softmax maps.
#include "device.h"
#include "host.h"
#include "kernels.h"
#include "poly.h"
#include "proposal.h"
#include "timing.h"

namespace ppl {

constexpr int kPropThreads = 256;
constexpr int kGmmNF = 8;
constexpr double kHalfLog2PiD = 0.91893853320467274178;

__device__ __forceinline__ double u01d(uint32_t w) { return (double)unit_f32(w); }

__device__ __forceinline__ void normals4_d(uint4 w, double *z) {
    box_muller(u01d(w.x), u01d(w.y), z[0], z[1]);
    box_muller(u01d(w.z), u01d(w.w), z[2], z[3]);
}

// log Normal(v; m, exp(lsd)) given isd = exp(-lsd).
__device__ __forceinline__ double log_normal(double v, double m, double lsd, double isd) {
    const double r = (v - m) * isd;
    return -0.5 * r * r - lsd - kHalfLog2PiD;
}

// exp(lsd) and exp(-lsd) of the proposal's ns log-scales, computed once per
// workgroup into LDS (every particle of the workgroup uses the same table).
// Every thread of the workgroup must call it.
__device__ __forceinline__ void stage_scales(const double *__restrict__ lsdv, int ns, double *sdv, double *isdv) {
    for (int t = threadIdx.x; t < ns; t += kPropThreads) {
        sdv[t] = exp(lsdv[t]);
        isdv[t] = exp(-lsdv[t]);
    }
    __syncthreads();
}

// The first k whose running sum of probabilities exceeds u (K - 1 if none);
// p[k] = exp(logp[k]), formed once per workgroup.
template <int K>
__device__ __forceinline__ int categorical_cdf(double u, const double *p) {
    double c = 0.0;
    int r = K - 1;
    bool found = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        c += p[k];
        if (!found && u < c) {
            r = k;
            found = true;
        }
    }
    return r;
}

// -------------------------------------------------------------- POLY --
__global__ __launch_bounds__(kPropThreads) void poly_mix_is_kernel(
    const double *__restrict__ X, const double *__restrict__ Y, int D, int64_t N, Key key, double lsd0, double isd0,
    const double *__restrict__ q, double *__restrict__ lw_out, double *__restrict__ lat_out, double *__restrict__ part) {
    const int64_t i = (int64_t)blockIdx.x * kPropThreads + threadIdx.x;
    const bool live = i < N;
    const uint32_t ii = (uint32_t)i;
    const double *lnl = q, *lmix = q + 4, *mean = q + 12, *lsdv = q + 172;
    __shared__ double sdv[160], isdv[160], prob[12];
    if (threadIdx.x < 12) prob[threadIdx.x] = exp(q[threadIdx.x]);
    stage_scales(lsdv, 160, sdv, isdv);
    const uint4 w0 = philox(ii, 0, 0, kTagProposal, key);
    const int n = 2 + categorical_cdf<4>(u01d(w0.x), prob);
    const int comp = categorical_cdf<8>(u01d(w0.y), prob + 4);
    double z[8];
    normals4_d(philox(ii, 1, 0, kTagProposal, key), z);
    normals4_d(philox(ii, 2, 0, kTagProposal, key), z + 4);
    double c[5];
    double lp = -log(4.0);
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const int o = ((n - 2) * 8 + comp) * 5 + j;
        c[j] = j < n ? mean[o] + sdv[o] * z[j] : 0.0;
        if (j < n) lp += log_normal(c[j], 0.0, lsd0, isd0);
    }
    // log q(n, c): degree term plus the mixture over components.
    double t[8], tm = -INFINITY;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        double a = lmix[m];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const int o = ((n - 2) * 8 + m) * 5 + j;
            if (j < n) a += log_normal(c[j], mean[o], lsdv[o], isdv[o]);
        }
        t[m] = a;
        tm = fmax(tm, a);
    }
    double ts = 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) ts += exp_le0(t[m] - tm);
    const double lq = lnl[n - 2] + tm + log(ts);
    // Points in chunks of eight (one batch of scalar loads per chunk); the
    // sum order is unchanged.
    double acc = 0.0;
    int d = 0;
    for (; d + 8 <= D; d += 8) {
        double xs[8], ys[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            xs[k] = X[d + k];
            ys[k] = Y[d + k];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            double v = c[4];
            v = fma(v, xs[k], c[3]);
            v = fma(v, xs[k], c[2]);
            v = fma(v, xs[k], c[1]);
            v = fma(v, xs[k], c[0]);
            const double r = ys[k] - v;
            acc = fma(r, r, acc);
        }
    }
    for (; d < D; ++d) {
        const double xv = X[d], yv = Y[d];
        double v = c[4];
        v = fma(v, xv, c[3]);
        v = fma(v, xv, c[2]);
        v = fma(v, xv, c[1]);
        v = fma(v, xv, c[0]);
        const double r = yv - v;
        acc = fma(r, r, acc);
    }
    const double lw = live ? lp - 0.5 * acc - lq : -INFINITY;
    if (live) {
        if (lw_out) lw_out[i] = lw;
        if (lat_out) {
            lat_out[i] = (double)n;
#pragma unroll
            for (int j = 0; j < 5; ++j) lat_out[(size_t)(1 + j) * N + i] = c[j];
        }
    }
    Partial<kPolyNF> pp = partial_empty<kPolyNF>();
    if (live && isnan(lw)) pp.nan = 1.0;
    pp.m = lw;
    if (lw > -INFINITY) {
        pp.s1 = 1.0;
        pp.s2 = 1.0;
        const int k = n - 2;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double sel = s == k ? 1.0 : 0.0;
            pp.f[s] = sel;
#pragma unroll
            for (int j = 0; j < 5; ++j) pp.f[4 + 5 * s + j] = sel * c[j];
        }
    } else {
        pp.m = -INFINITY;
    }
    partial_block_reduce_store<kPolyNF, kPropThreads / 64>(pp, part + (size_t)blockIdx.x * (4 + kPolyNF));
}

// Eight lanes per particle, for calls too small to fill the chip: lane b draws
// one Box-Muller pair (b < 3), owns mixture component b of log q and takes every
// eighth point.  Bound: the latency of the chain.  us a call against a lane per
// particle: 4096 x 1000 points 23.8 and 52.4, 2^14 x 1000 28.2 and 51.6, 1000 x 50
// 20.0 and 25.0.
constexpr int kMixParticles = kPropThreads / 8;      // particles per workgroup

__global__ __launch_bounds__(kPropThreads) void poly_mix_group_is_kernel(
    const double *__restrict__ X, const double *__restrict__ Y, int D, int64_t N, Key key, double lsd0, double isd0,
    const double *__restrict__ q, double *__restrict__ lw_out, double *__restrict__ lat_out, double *__restrict__ part) {
    __shared__ double sdv[160], isdv[160], prob[12];
    __shared__ double2 xy[kGroupPoints];
    const int tid = threadIdx.x, b = tid & 7;
    const int64_t i = (int64_t)blockIdx.x * kMixParticles + (tid >> 3);
    const bool live = i < N;
    const uint32_t ii = (uint32_t)i;
    double2 first[kGroupPoints / kPropThreads];
    poly_group_load<kPropThreads>(X, Y, D, 0, first);
    const double *lnl = q, *lmix = q + 4, *mean = q + 12, *lsdv = q + 172;
    if (tid >= 192 && tid < 204) prob[tid - 192] = exp(q[tid - 192]);
    stage_scales(lsdv, 160, sdv, isdv);
    const uint4 w0 = philox(ii, 0, 0, kTagProposal, key);
    const int n = 2 + categorical_cdf<4>(u01d(w0.x), prob);
    const int comp = categorical_cdf<8>(u01d(w0.y), prob + 4);
    const uint4 w = philox(ii, 1 + ((b >> 1) & 1), 0, kTagProposal, key);
    double za, zb;
    box_muller(u01d((b & 1) ? w.z : w.x), u01d((b & 1) ? w.w : w.y), za, zb);
    const double z[5] = {__shfl(za, 0, 8), __shfl(zb, 0, 8), __shfl(za, 1, 8), __shfl(zb, 1, 8), __shfl(za, 2, 8)};
    double c[5];
    double lp = -log(4.0), t = lmix[b];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const int o = ((n - 2) * 8 + comp) * 5 + j, ob = ((n - 2) * 8 + b) * 5 + j;
        c[j] = j < n ? mean[o] + sdv[o] * z[j] : 0.0;
        if (j < n) {
            lp += log_normal(c[j], 0.0, lsd0, isd0);
            t += log_normal(c[j], mean[ob], lsdv[ob], isdv[ob]);
        }
    }
    // log q(n, c): degree term plus the mixture over the components, one per lane
    double tm = fmax(t, dpp_keep_f64<0xB1, 0xF>(t));
    tm = fmax(tm, dpp_keep_f64<0x4E, 0xF>(tm));
    tm = fmax(tm, dpp_keep_f64<0x141, 0xF>(tm));
    double ts = exp_le0(t - tm);
    ts += dpp_f64<0xB1, 0xF>(ts);
    ts += dpp_f64<0x4E, 0xF>(ts);
    ts += dpp_f64<0x141, 0xF>(ts);
    const double lq = lnl[n - 2] + tm + log(ts);
    double acc = poly_group_sq<8, kPropThreads>(c, X, Y, D, first, xy);
    acc += dpp_f64<0xB1, 0xF>(acc);
    acc += dpp_f64<0x4E, 0xF>(acc);
    acc += dpp_f64<0x141, 0xF>(acc);
    const double lw = live ? lp - 0.5 * acc - lq : -INFINITY;
    if (live) {
        if (lw_out && b == 6) lw_out[i] = lw;
        if (lat_out && b < 6) {
            double v = (double)n;
#pragma unroll
            for (int j = 0; j < 5; ++j) v = b == j + 1 ? c[j] : v;
            lat_out[(size_t)b * N + i] = v;
        }
    }
    poly_group_record<8, kPropThreads / 64>(lw, live, n, c, part);
}

// --------------------------------------------------------------- GMM --
// One datum's log-factor, log sum_k pi_k Normal(y; mu_k, sd), in FP32 with the
// max shift and the hardware exp and log, as in the batched mixture SMC;
// hc[k] = (log pi_k - log(sd sqrt(2 pi))) / 2, hisd = 1 / (2 sd).  The terms are
// kept halved: t / 2 = c / 2 - (r / 2)^2 takes one instruction fewer than
// t = c - r^2 / 2 and, all scalings being powers of two, the same roundings.
// KK components, fully unrolled.
template <int KK>
__device__ __forceinline__ float gmm_point(float y, const float (&hc)[KK], const float (&mu)[KK], float hisd) {
    float t[KK];
#pragma unroll
    for (int k = 0; k < KK; ++k) {
        const float h = (y - mu[k]) * hisd;
        t[k] = fmaf(-h, h, hc[k]);
    }
    float mx = t[0];
#pragma unroll
    for (int k = 1; k < KK; ++k) mx = fmaxf(mx, t[k]);
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < KK; ++k) s += __builtin_amdgcn_exp2f((t[k] - mx) * 0x1.715476p+1f);   // 2 log2 e
    return fmaf(2.0f, mx, __logf(s));
}

// Sum of the log-factors over the data: FP32 within blocks of 16 points (one
// batch of scalar loads each), FP64 across blocks.
template <int KK>
__device__ __forceinline__ double gmm_loglik(const float *__restrict__ Y, int D, const float (&hc)[KK],
                                             const float (&mu)[KK], float hisd) {
    double ll = 0.0;
    int d = 0;
    for (; d + 16 <= D; d += 16) {
        float ys[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) ys[k] = Y[d + k];
        float sb = 0.0f;
#pragma unroll 4
        for (int k = 0; k < 16; ++k) sb += gmm_point<KK>(ys[k], hc, mu, hisd);
        ll += (double)sb;
    }
    if (d < D) {
        float sb = 0.0f;
        for (; d < D; ++d) sb += gmm_point<KK>(Y[d], hc, mu, hisd);
        ll += (double)sb;
    }
    return ll;
}

// Model constants, formed on the host: log((K-1)!) + log(K!), log mu_sd,
// 1 / mu_sd, -log(sd sqrt(2 pi)).
struct GmmConst {
    double mu_sd, lfact, lmu, imu, cst;
    float hisd;
};

// K components: a kernel per K, so that the latents, their densities and the
// sort unroll to exactly K (2 K - 1) slots and only the Box-Muller pairs that are
// used are drawn.  Bound: vector issue, the FP32 likelihood (100 points of 5
// components: 3900 slots with the hardware exp and log at half rate) ahead of
// the FP64 draw and densities (about 2000).  2^20 particles x 100 points, K = 5:
// 193 us a call against 249 with one kernel for all K, whose densities also took
// two lgamma, the model's logs and eight exps of the mixture weights per particle.
template <bool PROP, int K>
__global__ __launch_bounds__(kPropThreads) void gmm_is_kernel(const float *__restrict__ Y, int D, int64_t N,
                                                              Key key, GmmConst g,
                                                              const double *__restrict__ q, double *__restrict__ lw_out,
                                                              double *__restrict__ lat_out, double *__restrict__ part) {
    const int64_t i = (int64_t)blockIdx.x * kPropThreads + threadIdx.x;
    const bool live = i < N;
    const uint32_t ii = (uint32_t)i;
    constexpr int d = 2 * K - 1;
    double lpi[K], mu[K], extra = 0.0;
    __shared__ double sdv[PROP ? 8 * d : 1], isdv[PROP ? 8 * d : 1], prob[8];
    if constexpr (PROP) {
        if (threadIdx.x < 8) prob[threadIdx.x] = exp(q[threadIdx.x]);
        stage_scales(q + 8 + 8 * d, 8 * d, sdv, isdv);
    }
    if constexpr (!PROP) {
        // Prior draws (the SMC initial particles): Dirichlet(1) weights as
        // normalised Exp(1) draws, means mu_sd z.
        double E[K], tot = 0.0, z[(K + 3) / 4 * 4];
#pragma unroll
        for (int b = 0; b < (K + 3) / 4; ++b) {
            const uint4 we = philox(ii, b, 0, kTagPrior, key);
            const uint32_t ew[4] = {we.x, we.y, we.z, we.w};
#pragma unroll
            for (int k = 4 * b; k < 4 * b + 4; ++k) {
                if (k < K) {
                    E[k] = -log_unit(u01d(ew[k - 4 * b]));
                    tot += E[k];
                }
            }
            normals4_d(philox(ii, 2 + b, 0, kTagPrior, key), z + 4 * b);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            lpi[k] = log(E[k] / tot);
            mu[k] = g.mu_sd * z[k];
        }
    } else {
        const double *lmix = q, *mean = q + 8, *lsdv = q + 8 + 8 * d;
        const uint4 w0 = philox(ii, 0, 0, kTagProposal, key);
        const int comp = categorical_cdf<8>(u01d(w0.x), prob);
        double z[(d + 3) / 4 * 4], u[d];
#pragma unroll
        for (int b = 0; b < (d + 3) / 4; ++b) normals4_d(philox(ii, 1 + b, 0, kTagProposal, key), z + 4 * b);
#pragma unroll
        for (int k = 0; k < d; ++k) u[k] = mean[comp * d + k] + sdv[comp * d + k] * z[k];
        // prior density of u and the map to (log pi, mu)
        double lgm = 0.0, lgs = 0.0;
#pragma unroll
        for (int k = 0; k < K - 1; ++k) lgm = fmax(lgm, u[K + k]);
#pragma unroll
        for (int k = 0; k < K - 1; ++k) lgs += exp_le0(u[K + k] - lgm);
        lgs += exp_le0(-lgm);
        const double lz = lgm + log(lgs);
        double lp = g.lfact;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            mu[k] = k == 0 ? u[0] : mu[k > 0 ? k - 1 : 0] + exp(u[k]);
            lpi[k] = (k < K - 1 ? u[K + k < d ? K + k : 0] : 0.0) - lz;
            lp += log_normal(mu[k], 0.0, g.lmu, g.imu) + lpi[k];
            if (k >= 1) lp += u[k];
        }
        // log q(u): a running log-sum-exp over the components, not unrolled (the
        // proposal's 16 d scalars at once would spill)
        double tm = -1e300, ts = 0.0;
#pragma unroll 1
        for (int m = 0; m < 8; ++m) {
            double a = lmix[m];
#pragma unroll
            for (int k = 0; k < d; ++k) a += log_normal(u[k], mean[m * d + k], lsdv[m * d + k], isdv[m * d + k]);
            const double e = exp_le0(-fabs(a - tm));
            ts = a > tm ? fma(ts, e, 1.0) : ts + e;
            tm = a > tm ? a : tm;
        }
        extra = lp - (ts > 0.0 ? tm + log(ts) : NAN);
    }
    float hc[K], muf[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        hc[k] = 0.5f * (float)(lpi[k] + g.cst);
        muf[k] = (float)mu[k];
    }
    const double ll = gmm_loglik<K>(Y, D, hc, muf, g.hisd);
    const double lw = live ? ll + extra : -INFINITY;
    if (live) {
        if (lw_out) lw_out[i] = lw;
        if (lat_out) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                lat_out[(size_t)k * N + i] = lpi[k];
                lat_out[(size_t)(K + k) * N + i] = mu[k];
            }
        }
    }
    // summaries: E[mu_(k)] over the means in increasing order
#pragma unroll
    for (int a = 1; a < K; ++a)
#pragma unroll
        for (int b = a; b > 0; --b) {
            const double lo = fmin(mu[b - 1], mu[b]), hi = fmax(mu[b - 1], mu[b]);
            mu[b - 1] = lo;
            mu[b] = hi;
        }
    Partial<kGmmNF> pp = partial_empty<kGmmNF>();
    if (live && isnan(lw)) pp.nan = 1.0;
    if (lw > -INFINITY) {
        pp.m = lw;
        pp.s1 = 1.0;
        pp.s2 = 1.0;
#pragma unroll
        for (int k = 0; k < K; ++k) pp.f[k] = mu[k];
    }
    partial_block_reduce_store<kGmmNF, kPropThreads / 64>(pp, part + (size_t)blockIdx.x * (4 + kGmmNF));
}

// ---------------------------------------------------------------- host --
size_t prop_partial_bytes(int model, int64_t N) {
    const int64_t blocks = (N + kPropThreads - 1) / kPropThreads;
    const int nf = model == PPL_MODEL_POLY ? kPolyWsFields : kGmmNF;
    return (size_t)blocks * (4 + nf) * sizeof(double) + merge_scratch_bytes(nf);
}

template <int K>
static void launch_gmm_is(const IsArgs &a, int64_t blocks, const GmmConst &g, hipStream_t st) {
    auto kern = a.q_params ? gmm_is_kernel<true, K> : gmm_is_kernel<false, K>;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kPropThreads), 0, st, (const float *)a.y, (int)a.D, a.N,
                       make_key(a.seed), g, (const double *)a.q_params, (double *)a.lw_out, (double *)a.lat_out, a.part);
}

// Up to 2^14 particles (two waves per SIMD so) the polynomial model takes eight
// lanes per particle; the records of 32 particles fit the workspace beside one
// of 256, since up to kMergeDirect records the second merge level's room is free.
int run_importance_q(const IsArgs &a, hipStream_t st) {
    const bool group = a.model == PPL_MODEL_POLY && a.N <= 16384;
    const int64_t per = group ? kMixParticles : kPropThreads;
    const int64_t blocks = (a.N + per - 1) / per;
    const char *name = a.model == PPL_MODEL_POLY ? "poly_mix_is_kernel" : (a.q_params ? "gmm_mix_is_kernel" : "gmm_is_kernel");
    if (int rc = check_grid(name, blocks, kPropThreads)) return rc;
    {
        KernelTimer timer(name, st);
        if (a.model == PPL_MODEL_POLY) {
            const double lsd0 = log(a.hyper[0]);
            hipLaunchKernelGGL(group ? poly_mix_group_is_kernel : poly_mix_is_kernel, dim3((unsigned)blocks), dim3(kPropThreads), 0, st,
                               (const double *)a.x, (const double *)a.y, (int)a.D, a.N, make_key(a.seed), lsd0,
                               exp(-lsd0), (const double *)a.q_params, (double *)a.lw_out, (double *)a.lat_out, a.part);
        } else {
            GmmConst g;
            double f = 1.0;                      // (K - 1)!
            for (int k = 2; k < a.dim; ++k) f *= k;
            g.mu_sd = a.hyper[0];
            g.lfact = log(f) + log(f * a.dim);
            g.lmu = log(a.hyper[0]);
            g.imu = exp(-g.lmu);
            g.cst = -kHalfLog2PiD - log(a.hyper[1]);
            g.hisd = 0.5f * (float)(1.0 / a.hyper[1]);
            switch (a.dim) {
                case 1: launch_gmm_is<1>(a, blocks, g, st); break;
                case 2: launch_gmm_is<2>(a, blocks, g, st); break;
                case 3: launch_gmm_is<3>(a, blocks, g, st); break;
                case 4: launch_gmm_is<4>(a, blocks, g, st); break;
                case 5: launch_gmm_is<5>(a, blocks, g, st); break;
                case 6: launch_gmm_is<6>(a, blocks, g, st); break;
                case 7: launch_gmm_is<7>(a, blocks, g, st); break;
                default: launch_gmm_is<8>(a, blocks, g, st); break;
            }
        }
        timer.stop();
        PPL_LAUNCH_CHECK(name);
    }
    if (a.model == PPL_MODEL_POLY)
        return finalize_weights<kPolyNF>(a.part, blocks, a.part + (size_t)blocks * (4 + kPolyNF), a.N, a.model, a.scalars,
                                         a.summaries, st);
    return finalize_weights<kGmmNF>(a.part, blocks, a.part + (size_t)blocks * (4 + kGmmNF), a.N, a.model, a.scalars,
                                    a.summaries, st);
}

}  // namespace ppl
