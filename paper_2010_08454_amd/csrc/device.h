// device.h -- device primitives shared by the libppl kernels (gfx950 only).
//
// Random stream: Philox4x32-10 as described by Salmon, Moraes, Dror and Shaw,
// "Parallel Random Numbers: As Easy as 1, 2, 3" (SC'11).  Counter words are
// (particle or slot index, block index, step, instance << 8 | tag); the key is
// the 64-bit seed split into two 32-bit words.  Sampling and scoring of the
// built-in distributions is what the paper's runtime library provides on each
// target (Sec. 4.2.3); here it is a set of inline device functions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "host.h"
#include "ppl.h"

namespace ppl {

// Philox S-box multipliers and Weyl key increments (SC'11).
constexpr uint32_t kPhiloxMulA = 0xD2511F53u;
constexpr uint32_t kPhiloxMulB = 0xCD9E8D57u;
constexpr uint32_t kPhiloxWeylA = 0x9E3779B9u;
constexpr uint32_t kPhiloxWeylB = 0xBB67AE85u;

enum : uint32_t { kTagPrior = 0, kTagProposal = 1, kTagResample = 2, kTagMove = 7 };

// Compensated (Kahan) FP32 accumulation: sum += v with the running rounding
// error kept in c.  The error of the sum stays near 2 ulp of sum |v| however
// many terms are added, where a plain FP32 running sum loses up to a
// relative L 2^-24 over L terms (the SMC log-weights add one term per factor
// for as long as an epoch lasts).
__device__ __forceinline__ void kahan_add(float &sum, float &c, float v) {
    const float y = v - c;
    const float t = sum + y;
    c = (t - sum) - y;
    sum = t;
}

struct Key {
    uint32_t k0, k1;
};

__host__ __device__ inline Key make_key(uint64_t seed) { return Key{(uint32_t)seed, (uint32_t)(seed >> 32)}; }

// Ten Philox rounds on one 128-bit counter block.
__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, Key key) {
    uint32_t k0 = key.k0, k1 = key.k1;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += kPhiloxWeylA;
            k1 += kPhiloxWeylB;
        }
        const uint32_t hi_a = __umulhi(kPhiloxMulA, c0), lo_a = kPhiloxMulA * c0;
        const uint32_t hi_b = __umulhi(kPhiloxMulB, c2), lo_b = kPhiloxMulB * c2;
        const uint32_t n0 = hi_b ^ c1 ^ k0;
        const uint32_t n2 = hi_a ^ c3 ^ k1;
        c0 = n0;
        c1 = lo_b;
        c2 = n2;
        c3 = lo_a;
    }
    return make_uint4(c0, c1, c2, c3);
}

// Uniform on (0,1) from one word: the 23 high bits plus one half, times 2^-23.
// Every step is exact in FP32, so both precisions see the same value.
__device__ __forceinline__ float unit_f32(uint32_t w) { return ((float)(w >> 9) + 0.5f) * 0x1p-23f; }

// Uniform on (0,1) from two words (lo first): 52 bits plus one half, times 2^-52.
__device__ __forceinline__ double unit_f64(uint32_t lo, uint32_t hi) {
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    return ((double)(v >> 12) + 0.5) * 0x1p-52;
}

// Box-Muller pair: radius sqrt(-2 ln u1), angle 2 pi u2 (sincospi avoids rounding 2 pi).
__device__ __forceinline__ void box_muller(float u1, float u2, float &z0, float &z1) {
    const float r = sqrtf(-2.0f * logf(u1));
    float s, c;
    sincospif(2.0f * u2, &s, &c);
    z0 = r * c;
    z1 = r * s;
}

// FP64 log, square root and sine / cosine for what the samplers hand them: u in
// (0, 1) and no smaller than 2^-53, -2 ln u in [2^-53, 74].  The general library
// functions spend many of their instructions on the rest of the number line
// (subnormals, infinities, huge angles): a Box-Muller pair takes 191 vector
// instructions with them, 129 with these, and the draws are most of what the
// small-data polynomial kernels do (2 x 10^6 particles x 100 points 109.6 ->
// 100.6 us, 2^16 chains x 1000 Metropolis-Hastings steps 3.45 -> 3.33 ms).
// Largest error against 80-bit values over 2 x 10^7 uniforms of both widths and
// the ends of the range, in units in the last place: log 0.97, sqrt 0.50, sin
// and cos 0.91; the pair's relative root-mean-square error is 8.12e-17, as with
// the library functions.

// ln u.  u = m 2^k with m in [sqrt(1/2), sqrt 2), f = m - 1, s = f / (2 + f):
// ln m = 2 atanh s = f - s (f - P(s^2)), P(z) = 2 z / 3 + 2 z^2 / 5 + ... as a
// degree-7 polynomial (interpolated at Chebyshev nodes on z <= 0.0295, error 1e-17).
__device__ __forceinline__ double log_unit(double u) {
    double m = __builtin_amdgcn_frexp_mant(u);
    int k = __builtin_amdgcn_frexp_exp(u);
    const bool low = m < 0x1.6a09e667f3bcdp-1;
    m = low ? m + m : m;
    k = low ? k - 1 : k;
    const double f = m - 1.0, d = 2.0 + f;
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    y = fma(fma(-d, y, 1.0), y, y);
    double s = f * y;
    s = fma(fma(-d, s, f), y, s);
    const double z = s * s;
    double q = 0x1.2b5900de57b3bp-3;
    q = fma(q, z, 0x1.39fe51a7c12d9p-3);
    q = fma(q, z, 0x1.7462b51cb66eap-3);
    q = fma(q, z, 0x1.c71c62e3f11e5p-3);
    q = fma(q, z, 0x1.2492492df281ap-2);
    q = fma(q, z, 0x1.99999999952d7p-2);
    q = fma(q, z, 0x1.5555555555558p-1);
    // k ln 2 in two parts, the first with 21 trailing zero bits (exact for
    // |k| <= 53); its sum with f keeps the rounding error e
    const double kl = (double)k * 0x1.62e42p-1, h = kl + f, e = f - (h - kl);
    return h + fma((double)k, 0x1.fdf473de6af28p-22, fma(-s, fma(-q, z, f), e));
}

// exp x for x <= 0 (-inf and NaN included): x = k ln 2 + r with |r| <= ln 2 / 2,
// exp r = 1 + r + r^2 q(r) (degree 12 in r, interpolated at Chebyshev nodes,
// error 4e-19), scaled by 2^k; e is the rounding error of r.  27 vector
// instructions against 42 of the library's exp, which also covers overflow;
// largest error 0.83 units in the last place (the library's: 0.86).
__device__ __forceinline__ double exp_le0(double x) {
    x = x < -800.0 ? -800.0 : x;         // NaN stays
    const double k = __builtin_rint(x * 0x1.71547652b82fep+0);
    const double a = fma(k, -0x1.62e42p-1, x);                     // exact
    const double r = fma(k, -0x1.fdf473de6af28p-22, a), e = fma(k, -0x1.fdf473de6af28p-22, a - r);
    double q = 0x1.1f730a202ec17p-29;
    q = fma(q, r, 0x1.af4df5750ec30p-26);
    q = fma(q, r, 0x1.27e4db6121beep-22);
    q = fma(q, r, 0x1.71de022bd5558p-19);
    q = fma(q, r, 0x1.a01a01a6d9931p-16);
    q = fma(q, r, 0x1.a01a01abe9ce8p-13);
    q = fma(q, r, 0x1.6c16c16c162d2p-10);
    q = fma(q, r, 0x1.11111111100d8p-7);
    q = fma(q, r, 0x1.5555555555556p-5);
    q = fma(q, r, 0x1.5555555555557p-3);
    q = fma(q, r, 0x1.0000000000000p-1);
    return __builtin_ldexp(1.0 + (r + fma(r * r, q, e)), (int)k);
}

// sqrt x for x in [2^-53, 74]: the reciprocal root estimate refined twice, then
// one correction of the root itself.
__device__ __forceinline__ double sqrt_unit(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}

// sin and cos of 2 pi u for u in [0, 1]: r = 2 u - q / 2 in [-1/4, 1/4] with q
// the nearest integer to 4 u (both exact), sin pi r and cos pi r from their
// polynomials in r^2 (interpolated at Chebyshev nodes, errors below 5e-18),
// swapped and negated by the quadrant q.
__device__ __forceinline__ void sincos_turn(double u, double &sn, double &cs) {
    const double q = __builtin_rint(4.0 * u);
    const double r = fma(q, -0.5, u + u), z = r * r;
    double a = -0x1.6cc564dff874ap-16;
    a = fma(a, z, 0x1.e8f036889ff5ep-12);
    a = fma(a, z, -0x1.e3074d25df4e9p-8);
    a = fma(a, z, 0x1.50783486fab1cp-4);
    a = fma(a, z, -0x1.32d2cce62b872p-1);
    a = fma(a, z, 0x1.466bc6775aae1p+1);
    a = fma(a, z, -0x1.4abbce625be53p+2);
    const double s = fma(r, 0x1.921fb54442d18p+1, r * fma(a, z, 0x1.1a62633145c07p-53));
    // 1 - (pi^2 / 2) z + z^2 b with the errors of the product and of the sum
    double b = -0x1.b3832af1bdeebp-14;
    b = fma(b, z, 0x1.f9cfc045ae085p-10);
    b = fma(b, z, -0x1.a6d1f0ab527c3p-6);
    b = fma(b, z, 0x1.e1f5068830144p-3);
    b = fma(b, z, -0x1.55d3c7e3cbd74p+0);
    b = fma(b, z, 0x1.03c1f081b5ac4p+2);
    const double p2 = z * -0x1.3bd3cc9be45dep+2, h = 1.0 + p2;
    const double l = fma(z, -0x1.3bd3cc9be45dep+2, -p2) + z * -0x1.692b71366cc04p-52;
    const double c = h + (((1.0 - h) + p2) + fma(z * z, b, l));
    const int n = (int)q;
    const double p = (n & 1) ? c : s, w = (n & 1) ? s : c;
    sn = (n & 2) ? -p : p;
    cs = ((n + 1) & 2) ? -w : w;
}

__device__ __forceinline__ void box_muller(double u1, double u2, double &z0, double &z1) {
    const double r = sqrt_unit(-2.0 * log_unit(u1));
    double s, c;
    sincos_turn(u2, s, c);
    z0 = r * c;
    z1 = r * s;
}

// Four standard normals from one Philox block (two single-precision pairs).
__device__ __forceinline__ void normals4(uint4 w, float z[4]) {
    box_muller(unit_f32(w.x), unit_f32(w.y), z[0], z[1]);
    box_muller(unit_f32(w.z), unit_f32(w.w), z[2], z[3]);
}

// Uniform-discrete on {lo .. lo + range - 1}: lo + floor(w * range / 2^32).
__device__ __forceinline__ int uniform_discrete(uint32_t w, int lo, uint32_t range) {
    return lo + (int)__umulhi(w, range);
}

// ------------------------------------------------------- wave reductions --
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
// Wave-wide FP32 reductions through DPP row operations (full-rate VALU
// moves, no LDS permute): two quad permutations, the half-row and row
// mirrors, then the row-15 and row-31 broadcasts (rows left out of a
// broadcast keep the identity), which leave the total in lane 63; one
// v_readlane returns it to every lane.  All 64 lanes must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_f32(float v, float identity) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, identity),
                                                                 __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
    const float id = -INFINITY;
    v = fmaxf(v, dpp_f32<0xB1, 0xF>(v, id));    // quad_perm [1,0,3,2]
    v = fmaxf(v, dpp_f32<0x4E, 0xF>(v, id));    // quad_perm [2,3,0,1]
    v = fmaxf(v, dpp_f32<0x141, 0xF>(v, id));   // row_half_mirror
    v = fmaxf(v, dpp_f32<0x140, 0xF>(v, id));   // row_mirror
    v = fmaxf(v, dpp_f32<0x142, 0xA>(v, id));   // row_bcast15 into rows 1, 3
    v = fmaxf(v, dpp_f32<0x143, 0xC>(v, id));   // row_bcast31 into rows 2, 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
    v += dpp_f32<0xB1, 0xF>(v, 0.0f);
    v += dpp_f32<0x4E, 0xF>(v, 0.0f);
    v += dpp_f32<0x141, 0xF>(v, 0.0f);
    v += dpp_f32<0x140, 0xF>(v, 0.0f);
    v += dpp_f32<0x142, 0xA>(v, 0.0f);
    v += dpp_f32<0x143, 0xC>(v, 0.0f);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
// FP64 sum with the same DPP steps: both 32-bit halves move with the same
// pattern and the add is FP64.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ double wave_sum_dpp(double v) {
    v += dpp_f64<0xB1, 0xF>(v);
    v += dpp_f64<0x4E, 0xF>(v);
    v += dpp_f64<0x141, 0xF>(v);
    v += dpp_f64<0x140, 0xF>(v);
    v += dpp_f64<0x142, 0xA>(v);
    v += dpp_f64<0x143, 0xC>(v);
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// FP64 maximum with the same DPP steps; a row left out of a broadcast keeps its
// own value.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_keep_f64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
    const int nlo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
    const int nhi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)nhi << 32) | (uint32_t)nlo);
}
__device__ __forceinline__ double wave_max_dpp(double v) {
    v = fmax(v, dpp_keep_f64<0xB1, 0xF>(v));
    v = fmax(v, dpp_keep_f64<0x4E, 0xF>(v));
    v = fmax(v, dpp_keep_f64<0x141, 0xF>(v));
    v = fmax(v, dpp_keep_f64<0x140, 0xF>(v));
    v = fmax(v, dpp_keep_f64<0x142, 0xA>(v));
    v = fmax(v, dpp_keep_f64<0x143, 0xC>(v));
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// ------------------------------------------- weighted-sum partial records --
// A partial over a set of particles: {m = max lw, s1 = sum e, s2 = sum e^2,
// nan = number of NaN log-weights, f[k] = sum e * f_k}, with e = exp(lw - m).
// Partials merge by rescaling their sums to the largest maximum.
template <int NF>
struct Partial {
    double m, s1, s2, nan;
    double f[NF];
};

template <int NF>
__device__ __forceinline__ Partial<NF> partial_load(const double *src) {
    Partial<NF> p;
    p.m = src[0];
    p.s1 = src[1];
    p.s2 = src[2];
    p.nan = src[3];
#pragma unroll
    for (int k = 0; k < NF; ++k) p.f[k] = src[4 + k];
    return p;
}

template <int NF>
__device__ __forceinline__ Partial<NF> partial_empty() {
    Partial<NF> p;
    p.m = -INFINITY;
    p.s1 = 0.0;
    p.s2 = 0.0;
    p.nan = 0.0;
#pragma unroll
    for (int k = 0; k < NF; ++k) p.f[k] = 0.0;
    return p;
}

// Reduce-scatter of F doubles across the 64 lanes of a wave by recursive
// halving.  At each level a lane and its partner (lane ^ O) hold the same N
// slots; the lane with bit O clear keeps the first ceil(N/2) slots, the other
// the last ceil(N/2) (for odd N both keep the middle one), and each adds the
// partner's copy of what it keeps.  Every add is a + b on one side and b + a on
// the other, so a slot held by several lanes holds bitwise the same total.
// A level costs ceil(N/2) shuffles instead of N, about 2F shuffles in all
// instead of 6F for a butterfly.  On return slot j of the lane holds the
// wave total of field lo + j (j < the final slot count).
template <int F, int N, int O>
struct WaveReduceScatter {
    static constexpr int kFinal = WaveReduceScatter<F, N - N / 2, O / 2>::kFinal;
    __device__ __forceinline__ static void run(double (&v)[F], int lane, int &lo) {
        constexpr int H = N / 2, C = N - H;
        const bool up = (lane & O) != 0;
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const double keep = up ? v[H + j] : v[j];
            const double send = up ? v[j] : v[H + j];
            v[j] = keep + __shfl_xor(send, O, 64);
        }
        if (up) lo += H;
        WaveReduceScatter<F, C, O / 2>::run(v, lane, lo);
    }
};
template <int F, int N>
struct WaveReduceScatter<F, N, 0> {
    static constexpr int kFinal = N;
    __device__ __forceinline__ static void run(double (&)[F], int, int &) {}
};

// Block-wide maximum of one double per thread; every thread receives it.
template <int NWAVES>
__device__ __forceinline__ double block_max_f64(double v) {
    __shared__ double lds_m[NWAVES];
    v = wave_max_dpp(v);
    if ((threadIdx.x & 63) == 0) lds_m[threadIdx.x >> 6] = v;
    __syncthreads();
    double m = lds_m[0];
#pragma unroll
    for (int w = 1; w < NWAVES; ++w) m = fmax(m, lds_m[w]);
    return m;
}

// Sum of F doubles per thread across the block (blockDim = 64 * NWAVES):
// a reduce-scatter within each wave, then a fixed-order sum over the waves;
// dst[t] receives the total of field t.  Called at most once per kernel.
template <int F, int NWAVES>
__device__ __forceinline__ void block_sum_store(double (&v)[F], double *dst) {
    __shared__ double lds[NWAVES][F];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int lo = 0;
    WaveReduceScatter<F, F, 32>::run(v, lane, lo);
#pragma unroll
    for (int j = 0; j < WaveReduceScatter<F, F, 32>::kFinal; ++j)
        if (lo + j < F) lds[wv][lo + j] = v[j];
    __syncthreads();
    for (int t = threadIdx.x; t < F; t += 64 * NWAVES) {
        double s = lds[0][t];
#pragma unroll
        for (int w = 1; w < NWAVES; ++w) s += lds[w][t];
        dst[t] = s;
    }
}

// Block-level reduction of per-thread partials (blockDim = 64 * nwaves) into
// one record at dst.  The block maximum M comes first; each thread rescales
// its sums to M (one exp), and the sums then reduce with plain adds: a
// reduce-scatter within each wave and a fixed-order sum over the waves.  The
// result does not depend on timing.
template <int NF, int NWAVES>
__device__ __forceinline__ void partial_block_reduce_store(Partial<NF> &p, double *dst) {
    constexpr int F = 3 + NF;  // s1, s2, nan, f[NF]
    const double M = block_max_f64<NWAVES>(p.m);
    const double c = (p.m > -INFINITY) ? exp(p.m - M) : 0.0;
    double v[F];
    v[0] = p.s1 * c;
    v[1] = p.s2 * (c * c);
    v[2] = p.nan;
#pragma unroll
    for (int k = 0; k < NF; ++k) v[3 + k] = p.f[k] * c;
    block_sum_store<F, NWAVES>(v, dst + 1);
    if (threadIdx.x == 0) dst[0] = M;
}

// Block-level merge of the records in[r], r in [lo, hi), each {m, s1, s2, nan,
// f[NF]}, into one record at dst.  A first pass takes the maximum M of the
// record maxima; then every record is scaled by exp(m - M) and added, in a fixed
// order.  Called at most once per kernel.  One workgroup merges, so its time is
// the latency of its loads and of the exponentials:
//   up to 13 fields a thread takes whole records, all their words in flight;
//   above, one thread per record forms its scale in LDS and each half-wave adds
//   whole records, one field per lane (consecutive words: a thread per record
//   would touch a line per lane and field), kUnroll of them in flight.
// Importance sampling of the polynomial model, us a call with a thread per
// record and with half-waves: 14.6 and 12.2 at 10^4 particles (40 records), 62.1
// and 54.2 at 5 x 10^5 (1954); with 8 fields and 1024 records half-waves took
// 3 us longer (37.1 against 33.7).
template <int NF, int NWAVES>
__device__ __forceinline__ void records_block_reduce_store(const double *__restrict__ in, int64_t lo, int64_t hi,
                                                           double *dst) {
    constexpr int F = 3 + NF;
    constexpr int R = 4 + NF;
    constexpr int kThreads = 64 * NWAVES;
    const int64_t first = lo + threadIdx.x;
    if constexpr (F <= 16) {
        double m = -INFINITY;
        for (int64_t r = first; r < hi; r += kThreads) m = fmax(m, in[(size_t)r * R]);
        const double M = block_max_f64<NWAVES>(m);
        double v[F];
#pragma unroll
        for (int k = 0; k < F; ++k) v[k] = 0.0;
        for (int64_t r = first; r < hi; r += kThreads) {
            const double *rec = in + (size_t)r * R;
            const double mr = rec[0];
            v[2] += rec[3];
            if (mr > -INFINITY) {
                const double c = exp(mr - M);
                v[0] += rec[1] * c;
                v[1] += rec[2] * (c * c);
#pragma unroll
                for (int k = 0; k < NF; ++k) v[3 + k] += rec[4 + k] * c;
            }
        }
        block_sum_store<F, NWAVES>(v, dst + 1);
        if (threadIdx.x == 0) dst[0] = M;
    } else {
        constexpr int kGroups = 2 * NWAVES, kChunk = 2048, kUnroll = 16;
        static_assert(F <= 32, "a half-wave holds one record's sums");
        __shared__ double scale[kChunk];
        __shared__ double sums[NWAVES][32];
        const int f = threadIdx.x & 31, group = threadIdx.x >> 5;
        double m = -INFINITY;
        for (int64_t r = first; r < hi; r += kThreads) m = fmax(m, in[(size_t)r * R]);
        const double M = block_max_f64<NWAVES>(m);
        double acc = 0.0;
        for (int64_t c0 = lo; c0 < hi; c0 += kChunk) {
            const int n = (int)(hi - c0 < kChunk ? hi - c0 : kChunk);
            const double *rec = in + (size_t)c0 * R;
            if (c0 > lo) __syncthreads();
            for (int r = threadIdx.x; r < n; r += kThreads) {
                const double mr = rec[(size_t)r * R];
                scale[r] = mr > -INFINITY ? exp(mr - M) : 0.0;
            }
            __syncthreads();
            for (int r0 = group; r0 < n; r0 += kUnroll * kGroups) {
                double v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int r = r0 + u * kGroups;
                    v[u] = r < n && f < F ? rec[(size_t)r * R + 1 + f] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int r = r0 + u * kGroups;
                    const double c = r < n ? scale[r] : 0.0;
                    acc += f == 2 ? v[u] : v[u] * (f == 1 ? c * c : c);
                }
            }
        }
        acc += __shfl_xor(acc, 32, 64);
        if ((threadIdx.x & 63) < F) sums[threadIdx.x >> 6][f] = acc;
        __syncthreads();
        if (threadIdx.x < F) {
            double t = sums[0][f];
#pragma unroll
            for (int w = 1; w < NWAVES; ++w) t += sums[w][f];
            dst[1 + f] = t;
        }
        if (threadIdx.x == 0) dst[0] = M;
    }
}

// ------------------------------------------------ two-level partial merge --
// Up to kMergeDirect block partials are merged by the one workgroup of the
// finalize kernel; beyond that a first pass of at most kMergeGroups workgroups
// merges fixed contiguous ranges (a fixed order, so the result does not depend
// on timing) and the finalize workgroup merges those records.
constexpr int kMergeGroups = 512;
constexpr int64_t kMergeDirect = 2048;

template <int NF>
__global__ __launch_bounds__(256) void partial_merge_kernel(const double *__restrict__ in, int64_t n, int64_t per,
                                                            double *__restrict__ out) {
    const int64_t lo = (int64_t)blockIdx.x * per;
    const int64_t hi = lo + per < n ? lo + per : n;
    records_block_reduce_store<NF, 4>(in, lo, hi, out + (size_t)blockIdx.x * (4 + NF));
}

// Bytes of second-level records a merge of NF-field partials may need.
inline size_t merge_scratch_bytes(int nf) { return (size_t)kMergeGroups * (4 + nf) * sizeof(double); }

// Runs the first pass when nblocks is large; returns the records the final
// wave merges and their count in *nrec.  scratch holds merge_scratch_bytes(NF).
template <int NF>
inline const double *merge_partials_first(const double *part, int64_t nblocks, double *scratch, int *nrec,
                                          hipStream_t st) {
    if (nblocks <= kMergeDirect) {
        *nrec = (int)nblocks;
        return part;
    }
    const int64_t per = (nblocks + kMergeGroups - 1) / kMergeGroups;
    const int groups = (int)((nblocks + per - 1) / per);
    hipLaunchKernelGGL(partial_merge_kernel<NF>, dim3(groups), dim3(256), 0, st, part, nblocks, per, scratch);
    *nrec = groups;
    return scratch;
}


// ------------------------------------------------ importance finalize --
// Summary fields of the polynomial model: [s] sum of e, [4 + 5 s + j] sum of
// e c_j over the executions of degree n = 2 + s (s < 4, j < 5), and [24] sum of
// e c_0 over those of degree 1.
constexpr int kPolyNF = 25;
// Workspaces keep the room of 29 fields, the number of summaries.
constexpr int kPolyWsFields = 29;

// One workgroup merges the block partials and writes scalars[8] = {log Z-hat,
// ESS, 0, status, M, s1, s2, N} and the model summaries, one per thread: for
// the polynomial model P(n | y) for n = 2..5, coefficient means per degree and
// overall (29 values); for the others the weighted mean of each field.
template <int NF, int NWAVES>
__global__ __launch_bounds__(64 * NWAVES) void weights_finalize_kernel(const double *__restrict__ part,
                                                                          int nrec, int64_t N, int model,
                                                                          double *__restrict__ scalars,
                                                                          double *__restrict__ summaries) {
    __shared__ double rec[4 + NF];
    records_block_reduce_store<NF, NWAVES>(part, 0, nrec, rec);
    __syncthreads();
    const int t = threadIdx.x;
    const double m = rec[0], s1 = rec[1], s2 = rec[2], nan = rec[3], *f = rec + 4;
    int status = 0;
    if (nan > 0) status = PPL_E_NONFINITE;
    else if (!(m > -INFINITY)) status = PPL_E_ZERO_WEIGHT;
    if (t == 0) {
        scalars[0] = status ? (nan > 0 ? NAN : -INFINITY) : m + log(s1) - log((double)N);
        scalars[1] = status ? 0.0 : s1 * s1 / s2;
        scalars[2] = 0.0;
        scalars[3] = (double)status;
        scalars[4] = m;
        scalars[5] = s1;
        scalars[6] = s2;
        scalars[7] = (double)N;
    }
    if (!summaries) return;
    if constexpr (NF == kPolyNF) {
        if (model == PPL_MODEL_POLY) {
            if (t >= 64 && t < 64 + 29) {        // the second wave: the first has the scalars
                const int k = t - 64, s = (k - 4) / 5, j = (k - 4) % 5;
                double v = 0.0;
                if (k < 4) v = f[k] / s1;
                else if (k < 24) v = f[s] > 0 ? f[k] / f[s] : 0.0;
                else v = (((f[4 + j] + f[9 + j]) + (f[14 + j] + f[19 + j])) + (j == 0 ? f[24] : 0.0)) / s1;
                summaries[k] = status ? 0.0 : v;
            }
            return;
        }
    }
    if (t >= 64 && t < 64 + NF) summaries[t - 64] = status ? 0.0 : f[t - 64] / s1;
}

// Merges the block partials part[0 .. nblocks) (scratch: merge_scratch_bytes)
// and writes the scalars and summaries.  The finalize workgroup has 16 waves
// where their loads overlap more records than four would hold in one round;
// with fewer records the four start and meet sooner (98 records of 8 fields:
// 22.4 us a call against 23.2).
template <int NF>
inline int finalize_weights(const double *part, int64_t nblocks, double *scratch, int64_t N, int model,
                            double *scalars, double *summaries, hipStream_t st) {
    int nrec = 0;
    const double *rec = merge_partials_first<NF>(part, nblocks, scratch, &nrec, st);
    PPL_LAUNCH_CHECK("partial_merge_kernel");
    if (nrec <= 256)
        hipLaunchKernelGGL((weights_finalize_kernel<NF, 4>), dim3(1), dim3(256), 0, st, rec, nrec, N, model, scalars,
                           summaries);
    else
        hipLaunchKernelGGL((weights_finalize_kernel<NF, 16>), dim3(1), dim3(1024), 0, st, rec, nrec, N, model, scalars,
                           summaries);
    PPL_LAUNCH_CHECK("weights_finalize_kernel");
    return PPL_OK;
}

}  // namespace ppl
