// enumerate.hip -- exact inference by enumeration (paper Sec. 3.6.1) on the
// GPU: every execution of a model whose sample sites all have finite support,
// weighted by its sample probabilities and factors.
//
// Model: a hidden Markov chain of K states over T steps, z_0 ~ Cat(pi0),
// z_t ~ Cat(A[z_{t-1}]), observe(Normal(mu[z_t], sigma), y_t).  An execution
// is a path; the paths form the support product {0..K-1}^T, indexed by
// sum_t z_t K^(T-1-t).  A path's log-weight is the sum over sites of
// c_t(z_{t-1}, z_t) = log A[z_{t-1}][z_t] + log N(y_t; mu[z_t], sigma) (site 0:
// log pi0[z_0] + its emission).
//
// The paper enumerates breadth first, resuming an execution at a sample site
// once for every value of its support.  Here the first T - Ts sites (the
// prefix) are fanned out over threads, a prefix per thread and 128 prefixes
// per tile, workgroups striding over the tiles; a thread resumes its prefix
// for every value of the last Ts sites in nested loops fixed at compile time.
// One pass over the paths sums exp(lw - R) in total and per (t, z_t), R a scale
// near the largest log-weight (enum_emission_kernel), and finds the prefix that
// holds the heaviest path: the nested sites' sums in registers, the prefix
// sites' per tile through LDS into one owner thread per (t, k).  Records are
// merged in a fixed order, so results do not depend on timing.
//
// The pass runs in the linear domain from one exp per prefix: each node carries
// the weight, relative to R, of the best path below it, w = exp(lw_node +
// V_L[z] - R), where V_L[j] is the largest log-weight any completion from state
// j at nested level L can add (a max over the suffix, tabulated per state).  A
// child's weight is the parent's times F_L[j][k] = exp(c + V_{L+1}[k] - V_L[j])
// <= 1, so no product overflows, and a product that underflows belongs to a
// subtree whose every path is below e^-745 of the best.  The references set the
// scale only: every path's weight is still formed and added, and every last
// parent's weight (its heaviest path's) compared.
//
// The most probable path and its log joint are those of the log domain: lw
// summed site by site, the largest, the lowest index among equals.  The linear
// weights differ from exp of those sums by rounding, so they only select: if
// one prefix's heaviest weight beats every other prefix's by more than all
// rounding can account for, that prefix alone is walked in the log domain
// (enum_pick_kernel); otherwise every path is (enum_max_kernel, which returns
// at once in the first case).  Near-ties between prefixes, observations that
// make every path impossible and NaN take the second way.
#include "device.h"
#include "host.h"
#include "kernels.h"
#include "timing.h"

namespace ppl {

constexpr int kEnThreads = 128;
constexpr int kEnMaxT = 40;
constexpr int kEnMaxGrid = 2048;
constexpr int kEnMaxC = 1024;            // T K^2 at the path limit (K = 8, T = 16)
constexpr int kEnMaxTS = 12;             // nested sites
constexpr int kEnMaxF = 256;             // TS K^2 factors

__host__ __device__ constexpr uint64_t ipow(uint64_t b, int e) { return e == 0 ? 1 : b * ipow(b, e - 1); }

struct EnumDev {
    int T, tail;                 // sites, prefix sites (T - Ts)
    uint64_t n_prefix;           // K^tail
    uint64_t n_tiles;            // ceil(n_prefix / kEnThreads)
    const double *le;            // [T][K] log emission densities
    double lpi[8], lA[64];
    double *rec1;                // [grid][2] {heaviest weight, negated beside a near-tie; its prefix (bits)}, then
                                 // from enum_max_kernel {best lw, best index (bits)}
    double *glob;                // [6] {scale R, near-tie margin, non-finite, 1 if the path is found, M, best index (bits)}
    double *rec2;                // [grid][1 + T K] records {total, per-site sums}
};

struct EnLds {
    double c[kEnMaxC];           // c[t][j][k], t >= 1
    double c0[8];                // site 0: log pi0[k] + le[0][k]
    double cn[kEnMaxF];          // cn[L][j][k] = c[tail + L][j][k], nested level L (compile-time offsets)
    double F[kEnMaxF];           // F[L][j][k], nested level L (site tail + L)
    double V[(kEnMaxTS + 1) * 8];// V[L][j], V[TS][j] = 0
    double G[kEnMaxTS * 8];      // G[L][j] = sum_k F[L][j][k] (k in order)
    double cm[8];                // cm[j] = max_k cn[TS - 1][j][k] (k in order)
};

// Stages the tables: c for every site, and for the TS nested sites the
// suffix maxima V and the linear-domain factors F (pass 2 only).
template <int K, int TS>
__device__ void en_stage(EnLds &s, const EnumDev &a, bool factors) {
    const int T = a.T, tail = a.tail;
    for (int i = threadIdx.x; i < T * K * K; i += kEnThreads) {
        const int t = i / (K * K), j = (i / K) % K, k = i % K;
        s.c[i] = t == 0 ? 0.0 : a.lA[j * K + k] + a.le[t * K + k];
    }
    if (threadIdx.x < K) s.c0[threadIdx.x] = a.lpi[threadIdx.x] + a.le[threadIdx.x];
    __syncthreads();
    for (int i = threadIdx.x; i < TS * K * K; i += kEnThreads) s.cn[i] = s.c[tail * K * K + i];
    if constexpr (TS > 0)
        if (threadIdx.x < K) {
            const double *row = s.c + ((tail + TS - 1) * K + threadIdx.x) * K;
            double v = row[0];
            for (int k = 1; k < K; ++k) v = fmax(v, row[k]);
            s.cm[threadIdx.x] = v;
        }
    __syncthreads();
    if (!factors) return;
    if (threadIdx.x == 0) {
        for (int j = 0; j < K; ++j) s.V[TS * K + j] = 0.0;
        for (int L = TS - 1; L >= 0; --L)
            for (int j = 0; j < K; ++j) {
                double v = -INFINITY;
                for (int k = 0; k < K; ++k) v = fmax(v, s.c[((tail + L) * K + j) * K + k] + s.V[(L + 1) * K + k]);
                s.V[L * K + j] = v;
            }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < TS * K * K; i += kEnThreads) {
        const int L = i / (K * K), j = (i / K) % K, k = i % K;
        const double vj = s.V[L * K + j];
        s.F[i] = vj > -INFINITY ? exp(s.c[((tail + L) * K + j) * K + k] + s.V[(L + 1) * K + k] - vj) : 0.0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < TS * K; i += kEnThreads) {
        double g = 0.0;
        for (int k = 0; k < K; ++k) g += s.F[i * K + k];
        s.G[i] = g;
    }
    __syncthreads();
}

// Innermost unrolled levels per state count (K^UL paths below the node the
// runtime loops hand over: 64, 81, 64, then K^2).
constexpr int en_ul_max(int K) { return K == 2 ? 6 : K == 3 ? 4 : K == 4 ? 3 : 2; }

// Log-weight of prefix p (its digits are sites 0..tail-1) and its last state.
template <int K>
__device__ __forceinline__ double en_prefix(const EnLds &s, int tail, uint64_t p, int &last) {
    int z[kEnMaxT];
    for (int t = tail - 1; t >= 0; --t) {
        z[t] = (int)(p % K);
        p /= K;
    }
    double lw = s.c0[z[0]];
    for (int t = 1; t < tail; ++t) lw += s.c[(t * K + z[t - 1]) * K + z[t]];
    last = z[tail - 1];
    return lw;
}

// ---- log domain.  Levels above TS - UL are runtime loops; the last
// UL levels are unrolled, so their table rows are compile-time indices.
template <int K, int L, int TS, int UL>
struct WalkMax {
    // largest log-weight below a node of an unrolled level
    __device__ static double leafmax(const EnLds &s, int prev, double lw) {
        // Round-to-nearest addition is monotone, so the largest of lw + c_k
        // over the last site's K states is lw plus the largest c_k: the same
        // double as taking the K sums and their maximum.
        if constexpr (L == TS - 1) {
            return lw + s.cm[prev];
        } else {
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double x = WalkMax<K, L + 1, TS, UL>::leafmax(s, k, lw + s.cn[(L * K + prev) * K + k]);
                v = k == 0 ? x : fmax(v, x);
            }
            return v;
        }
    }
    // Raises best to the largest log-weight below the node and, when it does,
    // records the index of the node at level TS - UL that holds it.
    __device__ static void run(const EnLds &s, int prev, double lw, uint64_t idx, double &best, uint64_t &bnode) {
        if constexpr (L < TS - UL) {
#pragma unroll 1
            for (int k = 0; k < K; ++k)
                WalkMax<K, L + 1, TS, UL>::run(s, k, lw + s.cn[(L * K + prev) * K + k], idx * K + k, best, bnode);
        } else {
            const double v = leafmax(s, prev, lw);
            if (v > best) {
                best = v;
                bnode = idx;
            }
        }
    }
};

// The path index of the largest log-weight v below node `node` (at level
// TS - UL) of prefix p: the node's log-weight is re-summed in the walk's
// order, then the first of its K^UL completions that reaches v is found.
template <int K, int TS, int UL>
__device__ uint64_t en_locate(const EnLds &s, int tail, uint64_t p, uint64_t node, double v) {
    constexpr int NL = TS - UL;                  // runtime levels above the node
    constexpr int n = (int)ipow(K, UL);
    int prev;
    double lw = en_prefix<K>(s, tail, p, prev);
    uint64_t div = ipow(K, NL) / K;
    for (int L = 0; L < NL; ++L, div /= K) {
        const int k = (int)((node / div) % K);
        lw = lw + s.cn[(L * K + prev) * K + k];
        prev = k;
    }
    int m = 0;
    for (; m < n - 1; ++m) {
        double x = lw;
        int pv = prev, r = m;
        for (int d = 0, dv = n / K; d < UL; ++d, dv /= K) {
            const int k = r / dv;
            r -= k * dv;
            x = x + s.cn[((NL + d) * K + pv) * K + k];
            pv = k;
        }
        if (x == v) break;
    }
    return (p * ipow(K, NL) + node) * n + m;
}

// ---- linear domain.  Factors of the last levels (those whose parent state is
// a compile-time index) in scalar registers, as far as 36 values go: a
// v_fma_f64 with a scalar operand reads two vector register pairs instead of
// three, and 72 fewer vector registers leave room for a third wave per SIMD.
// Bound: FP64 issue, 2.45 vector instructions per path (4 states: the FMA, a
// quarter each of the parent's weight, its subtotal twice and its maximum, and
// the levels above), 0.72 of the rate at 4 states x 20 steps: 95 ms a call for
// 2^40 paths; 146 ms with a maximum pass of its own, factors in vector registers
// and records added one by one.
template <int K, int TS, int UL>
struct ScalarF {
    static constexpr int kRoom = (36 - K) / (K * K);
    static constexpr int NS = kRoom < UL - 1 ? (kRoom > 0 ? kRoom : 0) : (UL > 1 ? UL - 1 : 0);   // levels held
    double f[NS > 0 ? NS * K * K : 1], g[K];
    __device__ __forceinline__ void load(const EnLds &s) {
        if constexpr (NS > 0) {
#pragma unroll
            for (int i = 0; i < NS * K * K; ++i) f[i] = uniform(s.F[(TS - NS) * K * K + i]);
#pragma unroll
            for (int k = 0; k < K; ++k) g[k] = uniform(s.G[(TS - 1) * K + k]);
        }
    }
    __device__ __forceinline__ static double uniform(double v) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    }
};

// Returns the sum of the path weights below the node, adds each nested site's
// share to marg and raises wm to the heaviest path's weight.
template <int K, int L, int TS, int UL>
struct WalkSum {
    using SF = ScalarF<K, TS, UL>;
    __device__ static double run(const EnLds &s, const SF &sf, int prev, double w, double (&marg)[TS][K], double &wm) {
        constexpr bool scalar = L >= TS - SF::NS;
        auto F = [&](int k) {
            if constexpr (scalar) return sf.f[((L - (TS - SF::NS)) * K + prev) * K + k];
            else return s.F[(L * K + prev) * K + k];
        };
        double tot = 0.0;
        if constexpr (L < TS - UL) {
#pragma unroll 1
            for (int k = 0; k < K; ++k) {
                const double sub = WalkSum<K, L + 1, TS, UL>::run(s, sf, k, w * F(k), marg, wm);
#pragma unroll
                for (int kk = 0; kk < K; ++kk) marg[L][kk] += (k == kk) ? sub : 0.0;
                tot += sub;
            }
        } else if constexpr (L == TS - 1) {
            // each path's weight w F[k] goes into its site sum; the node's
            // subtotal, their sum, is w times the row sum G (one product for
            // the K paths); the heaviest of them is w itself (the largest F of
            // a row is 1)
#pragma unroll
            for (int k = 0; k < K; ++k) marg[L][k] = fma(w, F(k), marg[L][k]);
            wm = fmax(wm, w);
            if constexpr (scalar) tot = w * sf.g[prev];
            else tot = w * s.G[L * K + prev];
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double sub = WalkSum<K, L + 1, TS, UL>::run(s, sf, k, w * F(k), marg, wm);
                marg[L][k] += sub;
                tot += sub;
            }
        }
        return tot;
    }
};

// Every path in the log domain: the largest log-weight and its path.  Only if
// enum_pick_kernel could not tell the prefix from the weights.
template <int K, int TS, int UL>
__global__ __launch_bounds__(kEnThreads) void enum_max_kernel(EnumDev a) {
    __shared__ EnLds s;
    __shared__ double s_best[kEnThreads];
    __shared__ uint64_t s_idx[kEnThreads];
    if (a.glob[3] != 0.0) return;
    en_stage<K, TS>(s, a, false);
    double best = -INFINITY;
    uint64_t bidx = 0, bp = 0, bnode = 0;
    for (uint64_t tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
        const uint64_t p = tile * kEnThreads + threadIdx.x;
        if (p >= a.n_prefix) continue;
        int last;
        const double lw = en_prefix<K>(s, a.tail, p, last);
        if constexpr (TS == 0) {
            if (lw > best) { best = lw; bidx = p; }
        } else {
            const double before = best;
            uint64_t node = 0;
            WalkMax<K, 0, TS, UL>::run(s, last, lw, 0, best, node);
            if (best > before) {
                bp = p;
                bnode = node;
            }
        }
    }
    if constexpr (TS > 0)
        if (best > -INFINITY) bidx = en_locate<K, TS, UL>(s, a.tail, bp, bnode, best);
    s_best[threadIdx.x] = best;
    s_idx[threadIdx.x] = bidx;
    __syncthreads();
    if (threadIdx.x == 0) {
        double bl = -INFINITY;
        uint64_t bi = 0;
        for (int i = 0; i < kEnThreads; ++i)
            if (s_best[i] > bl || (s_best[i] == bl && s_idx[i] < bi)) { bl = s_best[i]; bi = s_idx[i]; }
        double *r = a.rec1 + 2 * (size_t)blockIdx.x;
        r[0] = bl;
        r[1] = __longlong_as_double((long long)bi);
    }
}

// The prefix of the heaviest path, if the weights tell it apart (no other
// prefix within the margin), walked in the log domain: the largest of its
// log-weights and the lowest index that reaches it.  One workgroup; a thread
// takes whole last parents, whose log-weights are summed in the walk's order.
template <int K, int TS>
__global__ __launch_bounds__(256) void enum_pick_kernel(EnumDev a, int nrec) {
    __shared__ EnLds s;
    __shared__ double s_best[256];
    __shared__ uint64_t s_idx[256];
    __shared__ int s_near;
    // the heaviest record, and how many are within the margin of it
    double wb = 0.0;
    uint64_t p = 0;
    for (int r = threadIdx.x; r < nrec; r += 256) {
        const double w = fabs(a.rec1[2 * (size_t)r]);
        if (w > wb) {
            wb = w;
            p = (uint64_t)__double_as_longlong(a.rec1[2 * (size_t)r + 1]);
        }
    }
    if (threadIdx.x == 0) s_near = 0;
    s_best[threadIdx.x] = wb;
    s_idx[threadIdx.x] = p;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o && s_best[threadIdx.x + o] > s_best[threadIdx.x]) {
            s_best[threadIdx.x] = s_best[threadIdx.x + o];
            s_idx[threadIdx.x] = s_idx[threadIdx.x + o];
        }
        __syncthreads();
    }
    wb = s_best[0];
    p = s_idx[0];
    const double margin = a.glob[1], least = wb * (1.0 - margin);
    int near = 0;
    for (int r = threadIdx.x; r < nrec; r += 256) {
        const double w = a.rec1[2 * (size_t)r];
        if (fabs(w) >= least) near += w < 0.0 ? 2 : 1;
    }
    if (near) atomicAdd(&s_near, near);
    __syncthreads();
    const bool found = wb > 0.0 && wb < INFINITY && margin < 0.5 && s_near == 1 && a.glob[2] == 0.0;
    if (threadIdx.x == 0) a.glob[3] = found ? 1.0 : 0.0;
    if (!found) return;
    en_stage<K, TS>(s, a, false);
    double best = -INFINITY;
    uint64_t bidx = 0;
    if constexpr (TS == 0) {
        int last;
        best = en_prefix<K>(s, a.tail, p, last);
        bidx = p;
    } else {
        constexpr int n = (int)ipow(K, TS - 1);      // last parents of the prefix
        int last;
        const double lw0 = en_prefix<K>(s, a.tail, p, last);
        for (int m = threadIdx.x; m < n; m += 256) {
            double x = lw0;
            int pv = last, r = m;
#pragma unroll
            for (int L = 0, dv = n / K; L < TS - 1; ++L, dv /= K) {
                const int k = r / dv;
                r -= k * dv;
                x = x + s.cn[(L * K + pv) * K + k];
                pv = k;
            }
            const double v = x + s.cm[pv];
            if (v > best) {
                int k = 0;
                for (; k < K - 1; ++k)
                    if (x + s.cn[((TS - 1) * K + pv) * K + k] == v) break;
                best = v;
                bidx = (p * n + m) * K + k;
            }
        }
    }
    s_best[threadIdx.x] = best;
    s_idx[threadIdx.x] = bidx;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            const double v = s_best[threadIdx.x + o];
            const uint64_t i = s_idx[threadIdx.x + o];
            if (v > s_best[threadIdx.x] || (v == s_best[threadIdx.x] && i < s_idx[threadIdx.x])) {
                s_best[threadIdx.x] = v;
                s_idx[threadIdx.x] = i;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.glob[4] = s_best[0];
        a.glob[5] = __longlong_as_double((long long)s_idx[0]);
    }
}

// Sums of exp(lw - R) in total and per (t, z_t), and the heaviest path's prefix.
template <int K, int TS, int UL>
__global__ __launch_bounds__(kEnThreads, 2) void enum_sum_kernel(EnumDev a) {
    constexpr int TSA = TS > 0 ? TS : 1;
    constexpr int kWaves = kEnThreads / 64;
    __shared__ EnLds s;
    __shared__ double s_sub[kEnThreads];
    __shared__ double s_wsum[kWaves];
    en_stage<K, TS>(s, a, true);
    const double R = a.glob[0];
    const bool skip = !(R > -INFINITY) || a.glob[2] != 0.0;
    const int tail = a.tail, T = a.T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double *rec = a.rec2 + (size_t)blockIdx.x * (1 + T * K);
    // owner entries e = t K + k of the prefix sites: this thread owns e = threadIdx.x + j kEnThreads
    constexpr int kOwn = (kEnMaxT * 8 + kEnThreads - 1) / kEnThreads;
    double own[kOwn];
#pragma unroll
    for (int j = 0; j < kOwn; ++j) own[j] = 0.0;
    double marg[TSA][K];
#pragma unroll
    for (int l = 0; l < TSA; ++l)
#pragma unroll
        for (int k = 0; k < K; ++k) marg[l][k] = 0.0;
    ScalarF<K, TSA, UL> sf;
    if constexpr (TS > 0) sf.load(s);
    double tot = 0.0;
    double best = 0.0, second = 0.0;             // heaviest weights of two prefixes of this thread
    uint64_t best_p = 0;
    for (uint64_t tile = blockIdx.x; !skip && tile < a.n_tiles; tile += gridDim.x) {
        const uint64_t base = tile * kEnThreads;
        const uint64_t p = base + threadIdx.x;
        double sub = 0.0;
        if (p < a.n_prefix) {
            int last;
            const double lw = en_prefix<K>(s, tail, p, last);
            double wm = 0.0;
            if constexpr (TS == 0) {
                sub = wm = exp(lw - R);
            } else {
                const double w = exp(lw + s.V[last] - R);      // the best path below the prefix, near 1 at most
                sub = WalkSum<K, 0, TS, UL>::run(s, sf, last, w, marg, wm);
            }
            if (wm > best) {
                second = best;
                best = wm;
                best_p = p;
            } else {
                second = fmax(second, wm);
            }
        }
        tot += sub;
        // the tile's total, the same bits in every lane (butterfly of commutative adds)
        double ws = sub;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) ws += __shfl_xor(ws, o);
        s_sub[threadIdx.x] = sub;
        if (lane == 0) s_wsum[wave] = ws;
        __syncthreads();
        double tile_tot = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) tile_tot += s_wsum[w];
        // prefix site t of prefix base + i has digit (q + (r + i) div pw) mod K, q and r from base = q pw + r
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
            const int e = threadIdx.x + j * kEnThreads;
            if (e < tail * K) {
                const int t = e / K, k = e - t * K;
                uint64_t pw = 1;
                for (int u = t + 1; u < tail; ++u) pw *= K;
                const uint64_t q = base / pw, r = base - q * pw;
                const int qm = (int)(q % K);
                double acc = 0.0;
                if (pw - r >= (uint64_t)kEnThreads) {
                    acc = qm == k ? tile_tot : 0.0;          // one digit over the whole tile
                } else if (pw >= (uint64_t)kEnThreads) {
                    // the digit steps once, at c = pw - r
                    const int c = (int)(pw - r);
                    if (qm == k)
                        for (int i = 0; i < c; ++i) acc += s_sub[i];
                    if ((qm + 1) % K == k)
                        for (int i = c; i < kEnThreads; ++i) acc += s_sub[i];
                } else {
                    // runs of pw prefixes per digit: those of digit k start at n pw - r, n = (k - qm) mod K + K i
                    const int pw32 = (int)pw, r32 = (int)r;
                    for (int n = (k - qm + K) % K; n * pw32 - r32 < kEnThreads; n += K) {
                        const int lo = max(0, n * pw32 - r32), hi = min(kEnThreads, (n + 1) * pw32 - r32);
                        for (int i = lo; i < hi; ++i) acc += s_sub[i];
                    }
                }
                own[j] += acc;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < kOwn; ++j) {
        const int e = threadIdx.x + j * kEnThreads;
        if (e < tail * K) rec[1 + e] = own[j];
    }
    // the total and the nested sites: wave sums, then the waves in order
    __shared__ double s_tot[kWaves][1 + TSA * K];
    {
        const double v = wave_sum_dpp(tot);
        if (lane == 0) s_tot[wave][0] = v;
    }
#pragma unroll
    for (int l = 0; l < TS; ++l)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double v = wave_sum_dpp(marg[l][k]);
            if (lane == 0) s_tot[wave][1 + l * K + k] = v;
        }
    // the heaviest prefix of the workgroup; negated where another is within the margin
    __shared__ double s_best[kEnThreads], s_second[kEnThreads];
    __shared__ uint64_t s_p[kEnThreads];
    s_best[threadIdx.x] = best;
    s_second[threadIdx.x] = second;
    s_p[threadIdx.x] = best_p;
    __syncthreads();
    for (int o = kEnThreads / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            const double b = s_best[threadIdx.x + o];
            s_second[threadIdx.x] = fmax(fmax(s_second[threadIdx.x], s_second[threadIdx.x + o]), fmin(s_best[threadIdx.x], b));
            if (b > s_best[threadIdx.x]) {
                s_best[threadIdx.x] = b;
                s_p[threadIdx.x] = s_p[threadIdx.x + o];
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const bool near = s_second[0] >= s_best[0] * (1.0 - a.glob[1]);
        a.rec1[2 * (size_t)blockIdx.x] = near ? -s_best[0] : s_best[0];
        a.rec1[2 * (size_t)blockIdx.x + 1] = __longlong_as_double((long long)s_p[0]);
    }
    for (int e = threadIdx.x; e < 1 + TS * K; e += kEnThreads) {
        double v = s_tot[0][e];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += s_tot[w][e];
        rec[e == 0 ? 0 : tail * K + e] = v;
    }
}

// Merges the records: scal[4] = {log Z, paths, log joint of the most probable
// path, status}, marg[T][K] = P(z_t = k | y), map[T] the most probable path.
// Workgroup f merges value f of the records (and all of them the total, 0),
// thread t adding records t, t + 256, ... and the threads in a fixed order: one
// workgroup adding them all in turn took 0.87 ms.
__global__ __launch_bounds__(256) void enum_finalize_kernel(const double *__restrict__ rec2, int nrec, int K, int T,
                                                            double paths, const double *__restrict__ rec1,
                                                            const double *__restrict__ glob,
                                                            double *__restrict__ scal, double *__restrict__ marg,
                                                            int32_t *__restrict__ map) {
    __shared__ double s_sum[2][4], s_best[256];
    __shared__ uint64_t s_idx[256];
    const int rl = 1 + T * K, f = blockIdx.x;
    double tot = 0.0, acc = 0.0, M = -INFINITY;
    uint64_t bi = 0;
    const bool found = glob[3] != 0.0;
    for (int r = threadIdx.x; r < nrec; r += 256) {
        const double *rec = rec2 + (size_t)r * rl;
        tot += rec[0];
        acc += rec[f];
        if (!found) {
            const double b = rec1[2 * (size_t)r];
            const uint64_t i = (uint64_t)__double_as_longlong(rec1[2 * (size_t)r + 1]);
            if (b > M || (b == M && i < bi)) { M = b; bi = i; }
        }
    }
    tot = wave_sum_dpp(tot);
    acc = wave_sum_dpp(acc);
    if ((threadIdx.x & 63) == 0) {
        s_sum[0][threadIdx.x >> 6] = tot;
        s_sum[1][threadIdx.x >> 6] = acc;
    }
    s_best[threadIdx.x] = M;
    s_idx[threadIdx.x] = bi;
    __syncthreads();
    if (found) {
        M = glob[4];
        bi = (uint64_t)__double_as_longlong(glob[5]);
    } else {
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) {
                const double b = s_best[threadIdx.x + o];
                const uint64_t i = s_idx[threadIdx.x + o];
                if (b > s_best[threadIdx.x] || (b == s_best[threadIdx.x] && i < s_idx[threadIdx.x])) {
                    s_best[threadIdx.x] = b;
                    s_idx[threadIdx.x] = i;
                }
            }
            __syncthreads();
        }
        M = s_best[0];
        bi = s_idx[0];
    }
    if (threadIdx.x != 0) return;
    tot = (s_sum[0][0] + s_sum[0][1]) + (s_sum[0][2] + s_sum[0][3]);
    acc = (s_sum[1][0] + s_sum[1][1]) + (s_sum[1][2] + s_sum[1][3]);
    const int status = glob[2] != 0.0 ? PPL_E_NONFINITE : M > -INFINITY ? PPL_OK : PPL_E_ZERO_WEIGHT;
    if (f > 0) {
        if (marg) marg[f - 1] = status == PPL_OK ? acc / tot : 0.0;
        return;
    }
    scal[0] = status == PPL_OK ? glob[0] + log(tot) : status == PPL_E_NONFINITE ? NAN : -INFINITY;
    scal[1] = paths;
    scal[2] = status == PPL_OK ? M : scal[0];
    scal[3] = (double)status;
    if (map) {
        for (int t = T - 1; t >= 0; --t) { map[t] = (int32_t)(bi % (uint64_t)K); bi /= (uint64_t)K; }
    }
}

struct EnEmission {
    double mu[8];
    double sigma;
};

// log emission densities le[t][k] = log Normal(y_t; mu_k, sigma), and what the
// walk needs of the whole chain: the scale R, the largest log-weight up to
// rounding (a max per site and state), a flag for a NaN emission (it makes every
// path's log-weight NaN) and the near-tie margin, a bound of the rounding error
// that the linear weights and the log-domain sums can differ by: 2^-44 (T adds
// and as many factors, each within 2^-52 of partial sums below S) times S, the
// sum over the sites of their largest finite |c_t|, and 1e-9.  One workgroup.
__global__ __launch_bounds__(256) void enum_emission_kernel(const double *__restrict__ y, EnumDev a, int K,
                                                            EnEmission e, double *__restrict__ le,
                                                            double *__restrict__ glob) {
    __shared__ double s_le[kEnMaxC], s_v[2][8], s_size[256];
    __shared__ int s_bad;
    const int n = a.T * K;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    int bad = 0;
    for (int i = threadIdx.x; i < n; i += 256) {
        const int t = i / K, k = i % K;
        const double r = (y[t] - e.mu[k]) / e.sigma;
        const double v = -0.5 * log(2.0 * M_PI) - log(e.sigma) - 0.5 * r * r;
        le[i] = v;
        s_le[i] = v;
        bad |= v != v;
    }
    if (bad) atomicOr(&s_bad, 1);
    __syncthreads();
    double size = 0.0;
    for (int t = threadIdx.x; t < a.T; t += 256) {
        double m = 0.0;
        for (int j = 0; j < (t == 0 ? 1 : K); ++j)
            for (int k = 0; k < K; ++k) {
                const double c = fabs((t == 0 ? a.lpi[k] : a.lA[j * K + k]) + s_le[t * K + k]);
                if (c < INFINITY) m = fmax(m, c);
            }
        size += m;
    }
    s_size[threadIdx.x] = size;
    if ((int)threadIdx.x < K) s_v[0][threadIdx.x] = a.lpi[threadIdx.x] + s_le[threadIdx.x];
    for (int t = 1; t < a.T; ++t) {
        __syncthreads();
        if ((int)threadIdx.x < K) {
            double v = -INFINITY;
            for (int j = 0; j < K; ++j) v = fmax(v, s_v[(t - 1) & 1][j] + a.lA[j * K + threadIdx.x]);
            s_v[t & 1][threadIdx.x] = v + s_le[t * K + threadIdx.x];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double R = -INFINITY, S = 0.0;
        for (int k = 0; k < K; ++k) R = fmax(R, s_v[(a.T - 1) & 1][k]);
        for (int i = 0; i < a.T; ++i) S += s_size[i];
        glob[0] = R;
        glob[1] = 1e-9 + 0x1p-44 * S;
        glob[2] = s_bad ? 1.0 : 0.0;
    }
}

// ---------------------------------------------------------------- host --
// Nested sites per state count (the paths below a prefix: 2^12, 3^7, 4^6,
// 5^5, 6^5, 7^4, 8^4).
constexpr int en_ts_max(int K) { return K == 2 ? 12 : K == 3 ? 7 : K == 4 ? 6 : K <= 6 ? 5 : 4; }
constexpr int en_ul(int K, int ts) { return std::min(en_ul_max(K), ts); }

struct EnPlan {
    int Ts, tail, grid;
    uint64_t n_prefix, n_tiles;
};

static int en_plan(int K, int T, EnPlan &p) {
    if (K < 1 || K > 8 || T < 1 || T > kEnMaxT || T * K * K > kEnMaxC)
        return fail(PPL_E_UNSUPPORTED, "no enumeration plan for %d states over %d steps", K, T);
    p.Ts = K == 1 ? 0 : std::min(en_ts_max(K), T - 1);   // site 0 is always a prefix site
    p.tail = T - p.Ts;
    p.n_prefix = ipow((uint64_t)K, p.tail);
    p.n_tiles = (p.n_prefix + kEnThreads - 1) / kEnThreads;
    p.grid = (int)std::min<uint64_t>(p.n_tiles, kEnMaxGrid);
    return PPL_OK;
}

// Workgroups of the sum kernel that a CU holds: 18 KB of LDS leave room for eight,
// more than 128 vector registers for six (three waves per SIMD), more than 168 for four.
constexpr int en_resident(int K, int ts) {
    if (K >= 6) return ts >= 3 ? 4 : K == 7 && ts == 2 ? 6 : 8;
    return ts * K > (K == 5 ? 19 : 20) ? 6 : 8;
}

// Workgroups of the walk, each with a record.  Every workgroup takes an equal share of
// the tiles, so one more round of a few workgroups would leave most SIMDs idle (2048
// workgroups where 1536 fit took 113 ms instead of 95 for 4 states x 20 steps): as
// many as an MI355X's 256 CUs hold.  A constant and not the number that the device at
// hand holds: the records decide how the FP64 sums are grouped, and the results
// depend on the inputs only.
constexpr int kEnCus = 256;
static int en_records(const EnPlan &p, int K) { return std::min(p.grid, kEnCus * en_resident(K, p.Ts)); }

int enum_records(int K, int T) {
    EnPlan p;
    return en_plan(K, T, p) ? 0 : en_records(p, K);
}

// Workspace: [256 scalars][le T K][glob 6][rec1 grid 2][rec2 grid (1 + T K)], each 256-byte aligned.
size_t enum_ws_bytes(int K, int T) {
    EnPlan p;
    if (en_plan(K, T, p)) return 0;
    return 256 + align_up((size_t)T * K * 8, 256) + 256 + align_up((size_t)p.grid * 2 * 8, 256) +
           align_up((size_t)p.grid * (1 + T * K) * 8, 256);
}

template <int K, int TS>
static int en_launch(const EnumDev &d, int nrec, hipStream_t st) {
    constexpr int UL = en_ul(K, TS);
    static_assert(TS <= kEnMaxTS && TS * K * K <= kEnMaxF, "nested tables exceed their LDS slots");
    {
        KernelTimer timer("enum_sum_kernel", st);
        hipLaunchKernelGGL((enum_sum_kernel<K, TS, UL>), dim3((unsigned)nrec), dim3(kEnThreads), 0, st, d);
        timer.stop();
    }
    PPL_LAUNCH_CHECK("enum_sum_kernel");
    hipLaunchKernelGGL((enum_pick_kernel<K, TS>), dim3(1), dim3(256), 0, st, d, nrec);
    PPL_LAUNCH_CHECK("enum_pick_kernel");
    {
        KernelTimer timer("enum_max_kernel", st);
        hipLaunchKernelGGL((enum_max_kernel<K, TS, UL>), dim3((unsigned)nrec), dim3(kEnThreads), 0, st, d);
        timer.stop();
    }
    PPL_LAUNCH_CHECK("enum_max_kernel");
    return PPL_OK;
}

template <int K, int TS = en_ts_max(K)>
static int en_dispatch(const EnumDev &d, const EnPlan &p, int nrec, hipStream_t st) {
    if (p.Ts == TS) return en_launch<K, TS>(d, nrec, st);
    if constexpr (TS > 0) return en_dispatch<K, TS - 1>(d, p, nrec, st);
    return fail(PPL_E_UNSUPPORTED, "no enumeration kernel for %d states with %d nested sites", K, p.Ts);
}

int run_enumerate_hmm(const EnumArgs &a, hipStream_t st) {
    const int K = a.K, T = a.T;
    EnPlan p;
    if (int rc = en_plan(K, T, p)) return rc;
    char *w = (char *)a.ws + 256;             // the first 256 bytes hold the scalars when the caller passes none
    double *le = (double *)w;
    w += align_up((size_t)T * K * 8, 256);
    double *glob = (double *)w;
    w += 256;
    double *rec1 = (double *)w;
    w += align_up((size_t)p.grid * 2 * 8, 256);
    double *rec2 = (double *)w;
    EnEmission em{};
    for (int k = 0; k < K; ++k) em.mu[k] = a.mu[k];
    em.sigma = a.sigma;
    EnumDev d{};
    d.T = T;
    d.tail = p.tail;
    d.n_prefix = p.n_prefix;
    d.n_tiles = p.n_tiles;
    d.le = le;
    d.rec1 = rec1;
    d.glob = glob;
    d.rec2 = rec2;
    for (int k = 0; k < K; ++k) d.lpi[k] = log(a.pi0[k]);
    for (int k = 0; k < K * K; ++k) d.lA[k] = log(a.A[k]);
    hipLaunchKernelGGL(enum_emission_kernel, dim3(1), dim3(256), 0, st, a.y, d, K, em, le, glob);
    PPL_LAUNCH_CHECK("enum_emission_kernel");
    int rc = PPL_E_ARG;
    const int nrec = en_records(p, K);
    switch (K) {
        case 1: rc = en_launch<1, 0>(d, nrec, st); break;
        case 2: rc = en_dispatch<2>(d, p, nrec, st); break;
        case 3: rc = en_dispatch<3>(d, p, nrec, st); break;
        case 4: rc = en_dispatch<4>(d, p, nrec, st); break;
        case 5: rc = en_dispatch<5>(d, p, nrec, st); break;
        case 6: rc = en_dispatch<6>(d, p, nrec, st); break;
        case 7: rc = en_dispatch<7>(d, p, nrec, st); break;
        case 8: rc = en_dispatch<8>(d, p, nrec, st); break;
    }
    if (rc) return rc;
    hipLaunchKernelGGL(enum_finalize_kernel, dim3((unsigned)(1 + T * K)), dim3(256), 0, st, rec2, nrec, K, T,
                       (double)ipow((uint64_t)K, T), rec1, glob, a.scalars, a.marginals, a.map);
    PPL_LAUNCH_CHECK("enum_finalize_kernel");
    return PPL_OK;
}

}  // namespace ppl
