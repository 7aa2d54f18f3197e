// importance.hip -- importance-sampling kernels (paper Sec. 3.6.2).
//
// Each thread owns P particles.  A particle draws its latents at the model's
// sample sites, accumulates its factors over the data, and its log-weight is
// folded into a per-block FP64 partial {max, sum e, sum e^2, sum e f}; one
// workgroup (weights_finalize_kernel) merges the block partials in a fixed order
// and writes log Z-hat = LSE - log N, the ESS and the posterior summaries.
//
// Data are the same for every lane of a wave (all lanes process the same datum
// for different particles): scalar loads bring them into SGPRs, and the rows of
// the linear regression into the matrix operand; per-particle state stays in
// VGPRs for the whole data loop.
#include "blr.h"
#include "device.h"
#include "host.h"
#include "kernels.h"
#include "poly.h"
#include "timing.h"

namespace ppl {

constexpr int kIsThreads = 256;
constexpr int kIsWaves = kIsThreads / 64;

// ------------------------------------------------------------------ BLR --
// The residuals r = y_d - x_d . w of a particle set are a matrix product, and
// run on the matrix cores: v_mfma_f32_4x4x1_16b_f32 multiplies, in each of its
// 16 blocks, 4 rows of A by 4 columns of B with one term of the sum, so lane l
// holds one particle (column) and gets four data rows in its four results.
// A's values of one block are broadcast to all blocks (CBSZ = 4, ABID = block),
// so one register per column k holds the k-th entry of 64 data rows, one row
// per lane, loaded once per 64 rows with whole cache lines.
// Why this shape: one term per instruction makes each result the chain
// fma(-x_k, w_k, r), k in order, that a lane would compute by itself, in the
// same FP32 rounding (checked bit for bit, subnormals, infinities and NaN
// included), and all rows of a particle stay in its lane, so the FP32 sums of
// squares within 32 rows keep their order too.  The matrix cores take FP32 at
// 256 FLOP per cycle and CU, the vector units at 128 without packed FP32.
// Measured at 2^20 particles x 10^4 rows, d = 16: 2.67 ms a call against 4.89 for
// the same chain on the vector units (0.95 of their rate): 32 FLOP per particle
// and row on the matrix cores, 126 of their 157 TFLOP/s.  Bound: matrix-core issue;
// the squares run beside it on the vector units.
typedef float blr_f32x4 __attribute__((ext_vector_type(4)));
typedef float blr_row4 __attribute__((ext_vector_type(4), aligned(4)));   // data rows are 4-byte aligned

// Adds the squared residuals of row groups B .. E - 1 (four rows each) of the
// rows in a to s, G groups at a time: G P independent chains hide the latency
// of the dependent products.
template <int P, int DIM, int G, int B, int E>
__device__ __forceinline__ void blr_row_groups(const float (&a)[DIM], const float *__restrict__ Y,
                                               const float (&w)[P][DIM], float (&s)[P]) {
    if constexpr (B < E) {
        static_assert(G == 1 || G == 4, "row groups per step");
        blr_f32x4 r[G][P];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int p = 0; p < P; ++p)
                r[g][p] = blr_f32x4{Y[4 * (B + g)], Y[4 * (B + g) + 1], Y[4 * (B + g) + 2], Y[4 * (B + g) + 3]};
#pragma unroll
        for (int k = 0; k < DIM; ++k)
#pragma unroll
            for (int p = 0; p < P; ++p) {
                r[0][p] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k], w[p][k], r[0][p], 4, B, 0);
                if constexpr (G == 4) {
                    r[1][p] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k], w[p][k], r[1][p], 4, B + 1, 0);
                    r[2][p] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k], w[p][k], r[2][p], 4, B + 2, 0);
                    r[3][p] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k], w[p][k], r[3][p], 4, B + 3, 0);
                }
            }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int p = 0; p < P; ++p) s[p] = fmaf(r[g][p][i], r[g][p][i], s[p]);
        blr_row_groups<P, DIM, G, B + G, E>(a, Y, w, s);
    }
}

// Lane l's row d + l (rows past the last are not used: the last one is read
// again), negated.
template <int DIM>
__device__ __forceinline__ void blr_load_rows(const float *__restrict__ X, int d, int last, float (&a)[DIM]) {
    const blr_row4 *row = (const blr_row4 *)(X + (size_t)min(d + (int)(threadIdx.x & 63), last) * DIM);
#pragma unroll
    for (int q = 0; q < DIM / 4; ++q) {
        const blr_row4 v = row[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * q + e] = -v[e];
    }
}

// Likelihood of one particle set: FP32 residuals r = y_d - x_d . w and squared
// sums in FP32 within consecutive 32-row blocks; block sums accumulate in FP64.
// The workgroup's 64 NW threads are S slices of NW / S waves: every slice holds
// the same particles, P per lane, and takes one contiguous share of the rows
// (in units of 64); the slices' FP64 sums are added in order through LDS.
template <int P, int DIM, bool PROP, int S, int NW>
__global__ __launch_bounds__(64 * NW, NW == 16 ? 4 : (PROP ? 2 : 3)) void blr_is_kernel(
    const float *__restrict__ X, const float *__restrict__ Y, int D, int64_t N, Key key,
    float prior_sd, double noise_sd, const float *__restrict__ qp, double *__restrict__ lw_out,
    float *__restrict__ lat_out, double *__restrict__ part) {
    constexpr int kLanes = 64 * NW / S;      // particles of one index p
    const int tid = threadIdx.x % kLanes;
    const int slice = S == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLanes);
    const int64_t base = (int64_t)blockIdx.x * (kLanes * P);

    float w[P][DIM];
    double extra[P];
    blr_draw<P, DIM, PROP, kLanes>(base, tid, key, prior_sd, qp, w, extra);

    double acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] = 0.0;
    constexpr int G = P == 1 ? 4 : 1;
    const int tiles = D / 64;
    const int per = (tiles + S - 1) / S;
    const int d1 = 64 * min(tiles, (slice + 1) * per);
    int d = 64 * min(tiles, slice * per);
    for (; d < d1; d += 64) {
        float a[DIM];
        blr_load_rows<DIM>(X, d, D - 1, a);
        float s0[P], s1[P];
#pragma unroll
        for (int p = 0; p < P; ++p) s0[p] = s1[p] = 0.0f;
        blr_row_groups<P, DIM, G, 0, 8>(a, Y + d, w, s0);
        blr_row_groups<P, DIM, G, 8, 16>(a, Y + d, w, s1);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            acc[p] += (double)s0[p];
            acc[p] += (double)s1[p];
        }
    }
    if (slice == S - 1) {                    // the rows after the last 64
        d = 64 * tiles;
        if (d + 32 <= D) {
            float a[DIM], s[P];
            blr_load_rows<DIM>(X, d, D - 1, a);
#pragma unroll
            for (int p = 0; p < P; ++p) s[p] = 0.0f;
            blr_row_groups<P, DIM, G, 0, 8>(a, Y + d, w, s);
#pragma unroll
            for (int p = 0; p < P; ++p) acc[p] += (double)s[p];
            d += 32;
        }
        if (d < D) {
            float s[P];
#pragma unroll
            for (int p = 0; p < P; ++p) s[p] = 0.0f;
            for (; d < D; ++d) {
                const float *row = X + (size_t)d * DIM;
                const float yv = Y[d];
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    float r = yv;
#pragma unroll
                    for (int k = 0; k < DIM; ++k) r = fmaf(-row[k], w[p][k], r);
                    s[p] = fmaf(r, r, s[p]);
                }
            }
#pragma unroll
            for (int p = 0; p < P; ++p) acc[p] += (double)s[p];
        }
    }
    if constexpr (S > 1) {
        __shared__ double sums[S - 1][kLanes * P];
        if (slice > 0) {
#pragma unroll
            for (int p = 0; p < P; ++p) sums[slice - 1][p * kLanes + tid] = acc[p];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < S - 1; ++q)
#pragma unroll
            for (int p = 0; p < P; ++p) acc[p] += sums[q][p * kLanes + tid];
    }

    const double var = noise_sd * noise_sd;
    const double cterm = (double)D * (-0.5 * log(2.0 * M_PI * var));
    double lw[P];
#pragma unroll
    for (int p = 0; p < P; ++p) lw[p] = cterm - acc[p] / (2.0 * var) + extra[p];
    // slice 0 holds the particles; the others add nothing to the record
    blr_finish<P, DIM, kLanes, NW>(base, tid, slice == 0 ? N : 0, w, lw, lw_out, lat_out, part);
}

// ----------------------------------------------------------------- POLY --
// FP64 polynomial model.  Horner over the five coefficient slots with slots
// j >= n set to zero: 0 * x + 0 = 0 exactly, so this equals n-term Horner and
// no lane branches on the sampled degree.
// Bound: FP64 and integer vector issue, about as much in the draws as in 100
// points; 2 x 10^6 x 100 points in 97 us a call (114.6 with the library's log and
// sincospi, one particle per lane and 29 fields).
template <int P>
__global__ __launch_bounds__(kIsThreads) void poly_is_kernel(
    const double *__restrict__ X, const double *__restrict__ Y, int D, int64_t N, Key key, double sd,
    int n_lo, int n_hi, double *__restrict__ lw_out, double *__restrict__ lat_out, double *__restrict__ part) {
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * (kIsThreads * P);
    double c[P][5];
    int nn[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        poly_prior_draw((uint32_t)(base + p * kIsThreads + tid), key, sd, n_lo, n_hi, nn[p], c[p]);
    }
    double pc[P][5];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int j = 0; j < 5; ++j) pc[p][j] = j < nn[p] ? c[p][j] : 0.0;

    double acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] = 0.0;
    // Points in chunks of eight: one batch of scalar loads per chunk instead
    // of a scalar-memory round trip per point; the sum order is unchanged.
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
#pragma unroll
            for (int p = 0; p < P; ++p) {
                double v = pc[p][4];
                v = fma(v, xs[k], pc[p][3]);
                v = fma(v, xs[k], pc[p][2]);
                v = fma(v, xs[k], pc[p][1]);
                v = fma(v, xs[k], pc[p][0]);
                const double r = ys[k] - v;
                acc[p] = fma(r, r, acc[p]);
            }
        }
    }
    for (; d < D; ++d) {
        const double xv = X[d], yv = Y[d];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            double v = pc[p][4];
            v = fma(v, xv, pc[p][3]);
            v = fma(v, xv, pc[p][2]);
            v = fma(v, xv, pc[p][1]);
            v = fma(v, xv, pc[p][0]);
            const double r = yv - v;
            acc[p] = fma(r, r, acc[p]);
        }
    }

    double lw[P];
    Partial<kPolyNF> pp = partial_empty<kPolyNF>();
    double mloc = -INFINITY;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int64_t i = base + p * kIsThreads + tid;
        lw[p] = (i < N) ? -0.5 * acc[p] : -INFINITY;
        if (i < N && isnan(lw[p])) pp.nan += 1.0;
        if (lw[p] > mloc) mloc = lw[p];
        if (i < N) {
            if (lw_out) lw_out[i] = lw[p];
            if (lat_out) {
                lat_out[i] = (double)nn[p];
#pragma unroll
                for (int j = 0; j < 5; ++j) lat_out[(size_t)(1 + j) * N + i] = c[p][j];
            }
        }
    }
    pp.m = mloc;
    if (mloc > -INFINITY) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const double e = exp(lw[p] - mloc);
            pp.s1 += e;
            pp.s2 += e * e;
            const int k = nn[p] - 2;  // degree slot (n in 2..5)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double sel = (s == k) ? e : 0.0;
                pp.f[s] += sel;
#pragma unroll
                for (int j = 0; j < 5; ++j) pp.f[4 + 5 * s + j] += sel * pc[p][j];
            }
            pp.f[24] += k < 0 ? e * pc[p][0] : 0.0;
        }
    }
    partial_block_reduce_store<kPolyNF, kIsWaves>(pp, part + (size_t)blockIdx.x * (4 + kPolyNF));
}

// Four lanes per particle, for calls too small to fill the chip with a particle
// per lane: lane b of a quad draws Philox block b (the degree, or one
// Box-Muller pair), takes every fourth point, and adds the summaries of degree
// 2 + b.  Bound: the latency of this chain (10^4 particles are 157 workgroups).
// us a call against a lane per particle: 10^4 particles x 1000 points 14.1 and
// 36.6, x 100 points 11.0 and 11.5, 2^15 x 1000 18.8 and 36.9.
constexpr int kQuadParticles = kIsThreads / 4;   // particles per workgroup

__global__ __launch_bounds__(kIsThreads) void poly_quad_is_kernel(
    const double *__restrict__ X, const double *__restrict__ Y, int D, int64_t N, Key key, double sd,
    int n_lo, int n_hi, double *__restrict__ lw_out, double *__restrict__ lat_out, double *__restrict__ part) {
    __shared__ double2 xy[kGroupPoints];
    const int tid = threadIdx.x, b = tid & 3;
    const int64_t i = (int64_t)blockIdx.x * kQuadParticles + (tid >> 2);
    const bool live = i < N;
    // the first points are on their way while the particle is drawn
    double2 first[kGroupPoints / kIsThreads];
    poly_group_load<kIsThreads>(X, Y, D, 0, first);
    const uint4 w = philox((uint32_t)i, b, 0, kTagPrior, key);
    const int n = __builtin_amdgcn_update_dpp(0, uniform_discrete(w.x, n_lo, (uint32_t)(n_hi - n_lo + 1)), 0x00, 0xF,
                                              0xF, false);
    double z0, z1;
    box_muller(unit_f64(w.x, w.y), unit_f64(w.z, w.w), z0, z1);
    z0 *= sd;
    z1 *= sd;
    double pc[5] = {dpp_f64<0x55, 0xF>(z0), dpp_f64<0x55, 0xF>(z1), dpp_f64<0xAA, 0xF>(z0), dpp_f64<0xAA, 0xF>(z1),
                    dpp_f64<0xFF, 0xF>(z0)};
#pragma unroll
    for (int j = 0; j < 5; ++j) pc[j] = j < n ? pc[j] : 0.0;

    double acc = poly_group_sq<4, kIsThreads>(pc, X, Y, D, first, xy);
    acc += dpp_f64<0xB1, 0xF>(acc);
    acc += dpp_f64<0x4E, 0xF>(acc);

    const double lw = live ? -0.5 * acc : -INFINITY;
    if (live) {
        if (lw_out && b == 0) lw_out[i] = lw;
        if (lat_out) {                           // the lane's own pair; n beside the first
            double *o = lat_out + (size_t)(2 * b) * N + i;
            if (b > 0) o[-(int64_t)N] = z0;
            if (b < 3) o[0] = b == 0 ? (double)n : z1;
        }
    }
    poly_group_record<4, kIsWaves>(lw, live, n, pc, part);
}

// ---------------------------------------------------------------- host --
size_t is_partial_bytes(int model, int dim, int64_t N) {
    const int P = model == PPL_MODEL_POLY ? 1 : 4;
    const int64_t blocks = (N + (int64_t)kIsThreads * P - 1) / ((int64_t)kIsThreads * P);
    const int nf = model == PPL_MODEL_POLY ? kPolyWsFields : dim;
    return (size_t)blocks * (4 + nf) * sizeof(double) + merge_scratch_bytes(nf);
}

// Launch shape of blr_is_kernel.  The largest calls fill the chip with four
// particles per lane and no split; below that the rows are split over the waves
// of a workgroup, and at the smallest N a lane holds one particle, so that
// 1000 waves or more share the work (n = 10^4 rows, d = 16, us a call before and
// now: 1664 and 67 at 1000 particles, 1687 and 346 at 10^5; 768 and 354 at
// 262144 x 5000 rows).  Splitting repeats the draw of the latents
// in every slice, so it needs rows enough to pay for that (5000 x 200 rows
// without it: 50 and 16 us).
// A shape's workgroups never exceed those of (P = 4, S = 1) by more than
// kMergeGroups, so its records fit where the second merge level's would be
// (is_partial_bytes), which up to kMergeDirect records are not used.
struct BlrShape {
    int P, S, NW;
};
static BlrShape blr_shape(int64_t N, int64_t D) {
    if (N <= 8192 && D >= 1024) return {1, 16, 16};
    if (N <= 32768 && D >= 512) return {1, 4, 4};
    if (N <= 131072) return D >= 512 ? BlrShape{4, 4, 4} : BlrShape{1, 1, 4};
    if (N <= 524288 && D >= 512) return {4, 2, 4};
    return {4, 1, 4};
}

template <int DIM, int P, int S, int NW>
static int launch_blr_shape(const IsArgs &a, double *part, hipStream_t st) {
    constexpr int64_t kPer = (int64_t)64 * NW / S * P;
    const int64_t blocks = (a.N + kPer - 1) / kPer;
    if (int rc = check_grid("blr_is_kernel", blocks, 64 * NW)) return rc;
    KernelTimer timer("blr_is_kernel", st);
    if (a.q_params)
        hipLaunchKernelGGL((blr_is_kernel<P, DIM, true, S, NW>), dim3((unsigned)blocks), dim3(64 * NW), 0, st,
                           (const float *)a.x, (const float *)a.y, (int)a.D, a.N, make_key(a.seed),
                           (float)a.hyper[0], a.hyper[1], (const float *)a.q_params, (double *)a.lw_out,
                           (float *)a.lat_out, part);
    else
        hipLaunchKernelGGL((blr_is_kernel<P, DIM, false, S, NW>), dim3((unsigned)blocks), dim3(64 * NW), 0, st,
                           (const float *)a.x, (const float *)a.y, (int)a.D, a.N, make_key(a.seed),
                           (float)a.hyper[0], a.hyper[1], nullptr, (double *)a.lw_out, (float *)a.lat_out, part);
    timer.stop();
    PPL_LAUNCH_CHECK("blr_is_kernel");
    return finalize_weights<DIM>(part, blocks, part + (size_t)blocks * (4 + DIM), a.N, (int)PPL_MODEL_BLR, a.scalars,
                                a.summaries, st);
}

template <int DIM>
static int launch_blr(const IsArgs &a, hipStream_t st) {
    const BlrShape s = blr_shape(a.N, a.D);
    if (s.S == 16) return launch_blr_shape<DIM, 1, 16, 16>(a, a.part, st);
    if (s.P == 1) return s.S == 4 ? launch_blr_shape<DIM, 1, 4, 4>(a, a.part, st) : launch_blr_shape<DIM, 1, 1, 4>(a, a.part, st);
    if (s.S == 4) return launch_blr_shape<DIM, 4, 4, 4>(a, a.part, st);
    if (s.S == 2) return launch_blr_shape<DIM, 4, 2, 4>(a, a.part, st);
    return launch_blr_shape<DIM, 4, 1, 4>(a, a.part, st);
}

// Launch shape of the polynomial model.  Up to 2^15 particles a quad of lanes
// per particle (at most two waves per SIMD so; the records of 64 particles fit
// the workspace beside one of 256 by the same count as in blr_shape); above, a
// lane per particle, and from 2^18 on four, which share the point loads and the
// workgroup's reduction.
static int launch_poly(const IsArgs &a, hipStream_t st) {
    const int64_t per = a.N <= 32768 ? kQuadParticles : a.N < 262144 ? kIsThreads : 4 * kIsThreads;
    const int64_t blocks = (a.N + per - 1) / per;
    if (int rc = check_grid("poly_is_kernel", blocks, kIsThreads)) return rc;
    auto kern = per == kQuadParticles ? poly_quad_is_kernel : per == kIsThreads ? poly_is_kernel<1> : poly_is_kernel<4>;
    KernelTimer timer("poly_is_kernel", st);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kIsThreads), 0, st, (const double *)a.x,
                       (const double *)a.y, (int)a.D, a.N, make_key(a.seed), a.hyper[0], (int)a.hyper[1],
                       (int)a.hyper[2], (double *)a.lw_out, (double *)a.lat_out, a.part);
    timer.stop();
    PPL_LAUNCH_CHECK("poly_is_kernel");
    return finalize_weights<kPolyNF>(a.part, blocks, a.part + (size_t)blocks * (4 + kPolyNF), a.N,
                                     (int)PPL_MODEL_POLY, a.scalars, a.summaries, st);
}

int run_importance(const IsArgs &a, hipStream_t st) {
    if (a.model == PPL_MODEL_POLY) {
        return launch_poly(a, st);
    }
    switch (a.dim) {
        case 4: return launch_blr<4>(a, st);
        case 8: return launch_blr<8>(a, st);
        case 12: return launch_blr<12>(a, st);
        case 16: return launch_blr<16>(a, st);
    }
    return fail(PPL_E_ARG, "BLR dim must be 4, 8, 12 or 16 (got %d)", a.dim);
}

}  // namespace ppl
