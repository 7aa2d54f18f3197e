// smc.hip -- sequential Monte Carlo in one persistent cooperative launch.
//
// The paper suspends a model at each factor with a delimited continuation
// (Sec. 3.4, 4.3) and names particle-based inference on the GPU as future work
// (Sec. 6).  Here a suspended particle is its resume point (the factor index s,
// shared by all particles) plus fixed-size state held in registers across the
// whole run; only resampling moves state through device memory.
//
// One workgroup of 512 threads per CU, P particles per thread (slots
// j = block * 512 P + thread * P + p; a block's slots form one "tile").
// 512 threads leave each wave 256 registers, so the particle state, the
// resampling variables and the FP64 normaliser calls fit without spilling
// (spilled registers would be written back and refetched through HBM at
// every grid barrier).
//
// What bounds it is the chain of a factor, not arithmetic: at N = 2^20 (256 blocks
// of 8 particles per thread) the 1000 factors and 715 events of the state-space
// model hold 1715 exchanges of about 4 us, each a store that has to reach the
// others' caches and a poll that has to come back, and the rest is work of the
// two waves per SIMD between exchanges.  So the chain is kept short: records are
// merged from LDS by all waves with one workgroup barrier, a tile's totals leave
// before its prefix sums and state do, noise and log Z-hat are worked on while
// records travel, and a particle marks its slots instead of every slot searching
// (8 slots per thread: 6.6 us of search and 1.3 us of staging per event).
// Measured against merging by one wave, serial polls and a search per slot:
// 1000 x 2^20 30.0 -> 20.1 ms, 300 x 1000 3.45 -> 2.11 ms, 300 x 100003 4.57 ->
// 2.94 ms, mixtures with K = 4 300 x 20011 1.28 -> 1.19 ms, 300 x 131072 2.27 -> 1.69 ms.
// Per factor s:
//   1. every particle advances to factor s and adds its log-factor (FP32,
//      compensated summation);
//   2. block partial {max lw, sum e, sum e^2}, e = exp(lw - max) -> memory;
//      grid barrier; every block merges the partials in the same order, so
//      every block takes the same ESS decision;
//   3. if ESS < ess_frac N (and s is not the last factor): FP64 weights
//      e = exp(lw - max) give the epoch normaliser and the quantised integer
//      weights q; each block scans its q and publishes its tile total, its
//      tile-local exclusive prefix sums and its particles' state; grid barrier; every
//      particle of the few tiles that hold a block's ancestors marks the first slot
//      it is the ancestor of, a running maximum fills the other slots, and every
//      slot gathers its ancestor's state; lw = 0.
// Blocks meet at a record barrier: each block stores its record (the partial
// of step 2, the tile total of step 3, the final sums) on its own cache line
// and thread t of every block polls line t, so every block holds every record
// when it leaves, with no shared counter.  Every word a block publishes for
// others (record words, the prefix sums and state of step 3) carries the tag
// of its epoch or event, so a reader knows it has the current value without
// any release or acquire, and a reader that is early polls again.  The spin
// is bounded: if a wait exceeds the limit, the block raises the abort flag
// and every block leaves its loop at its next barrier, so the grid always
// drains.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>

#include "device.h"
#include "host.h"
#include "smc.h"
#include "timing.h"

namespace ppl {

constexpr int kSmcThreads = 512;
constexpr int kSmcWaves = kSmcThreads / 64;
constexpr int kSmcMaxBlocks = 1024;
constexpr int kBarLine = 32;                  // unsigned per 128-byte line
constexpr int kBarWords = kBarLine;           // word 1: abort flag
constexpr int kRecWords = 16;                 // 64-bit words per 128-byte record line
constexpr uint32_t kSpinLimit = 1u << 24;     // polls before a wait is declared hung (seconds)
constexpr int kPollAtOnce = 64;               // most blocks that poll for records at once (see tagged_wait)
constexpr int kYChunk = 2048;                 // observations staged in LDS at a time
// Most tiles whose particles mark a block's slots.  At even weights a block's ancestors
// lie in its own and one or two neighbouring tiles; ancestors that are strewn wider are
// left to a search in memory per slot.  The line is a number of tiles at every tile
// size: us for 60 factors and 59 events of the state-space model with observations so
// sharp that few particles keep weight, for at most 3, 5 and 16 tiles: 131072
// particles (tiles of 512) 923, 915 and 1116; 262144 (1024) 1207, 1185 and (8) 1125;
// 2^20 (4096) 2995, 2135 (3 and 5).  Staging up to 8192 prefix sums in LDS and searching
// them took 1240, 1480 and 3550.
constexpr int kScatterTiles = 5;
constexpr int kBatchTries = 64;               // reloads of a batch of tagged words before polling them one by one

struct SmcDev {
    const float *y;
    int64_t T, N;
    int K;
    Key key;
    uint32_t inst;
    float ess_frac;
    float hyp[5];            // model constants (FP32)
    double lconst;           // LGSSM: -1/2 log(2 pi r^2) ; GMM: -1/2 log(2 pi) - log(sd)
    int kbits;               // quantisation exponent
    uint64_t inv_n;          // floor((2^64 - 1) / N)
    // outputs (may be null)
    double *scalars;
    float *lw_out, *lat_out;
    double *ess_trace;
    uint8_t *resampled;
    int32_t *anc_out;
    float *elw_out;          // [max_events][N] log-weights each event resampled from
    double *logz_tr;         // [T] normaliser increment added after factor s
    double *alpha_out;       // [max_events][move_steps][N] log acceptance ratios of the moves
    int64_t max_events;
    int64_t t0, t1;          // factors of this launch [t0, t1)
    char *ckpt;              // checkpoint: header then [NF][N] state, [N] lw, [N] compensation
    int move_steps;          // resample-move steps per particle after each resampling
    double move_lam;         // random-walk scale factor
    double hyp64[2];         // GMM {mu_sd, comp_sd} in FP64 (move scales)
    int poll_all;            // 1: every tagged read takes the polling path (a checking aid)
    // workspace
    unsigned *bar;           // [1] abort flag
    uint64_t *rec;           // [2][nb][16] record lines: word 0 the epoch, words 1..3 the record
    uint64_t *qtag;          // [N] tagged tile-local exclusive prefix sums of q
    uint64_t *xtag;          // [NF][N] tagged particle state
    float *xbuf2;            // [NF][N] gathered particles while they move (resample-move)
};

// Checkpoint header (the first 256 bytes of a checkpoint).
struct SmcCkpt {
    int64_t t;               // next factor
    int64_t N;
    int64_t nres;
    int32_t nf;
    int32_t status;
    double logz;
    float mlast;
};
constexpr size_t kCkptHeader = 256;

// ------------------------------------------------------------- barrier --
// Record exchange for epoch e (a grid barrier that also hands every block
// every block's record): thread 0 stores NW words on its line of buffer
// e mod 2 with relaxed device-scope stores, each word holding e in its high
// half and 32 bits of the record in its low half; thread t < nb polls line t
// until every word of the line holds e, and leaves the words in LDS.  Each word
// validates itself, so the exchange needs no release and no acquire (a
// device-scope release writes back the L2 of the issuing XCD, which at 256
// workgroups costs more than the exchange itself).  Two buffers suffice: a
// block cannot store record e + 2 before every block has stored record e + 1,
// which each does only after reading all records e.  In two parts: what
// runs between them overlaps the records' way to the other blocks.
template <int NW>
__device__ __forceinline__ void tagged_post(uint64_t *rec, unsigned epoch, int nb, const uint32_t (&w)[NW]) {
    static_assert(NW <= kRecWords, "record line overflow");
    if (threadIdx.x == 0) {
        uint64_t *mine = rec + ((size_t)(epoch & 1u) * nb + blockIdx.x) * kRecWords;
        const uint64_t tag = (uint64_t)epoch << 32;
#pragma unroll
        for (int k = 0; k < NW; ++k) __hip_atomic_store(mine + k, tag | w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Every block's record words, by word and block, after tagged_wait.
struct RecLds {
    uint32_t w[5][kSmcThreads];
    int bad;                          // set (never reset) once a wait or a tagged read gave up
};

// Leaves word k of block t's record in L.w[k][t].  Returns false (uniformly in the
// block) once any block has aborted.  L.w is free for the next wait after the
// workgroup barrier that every caller passes in between.
// The nb^2 polls of the grid share the memory system with the records that they wait
// for: with many blocks, polls before the records can be there hold those up, and the
// first poll comes 1024 cycles late.  us for 300 factors of a 3-component mixture
// without an event, with and without: 131072 particles (256 blocks) 1351 and 2500,
// 50000 (98 blocks) 1058 and 1310; of the state-space model 1350 and 1910, 1048 and
// 1120.  Up to kPollAtOnce blocks the wait costs about what it gains (32768
// particles, 64 blocks: 1040 .. 1120 and 1155, 1000 .. 1010 and 990).
template <int NW>
__device__ __forceinline__ bool tagged_wait(uint64_t *rec, unsigned *bar, unsigned epoch, int nb, RecLds &L) {
    static_assert(NW <= 5, "record words in LDS");
    unsigned *abort_flag = bar + 1;
    if (nb > kPollAtOnce) __builtin_amdgcn_s_sleep(16);
    if (threadIdx.x < nb) {          // nb <= kSmcThreads
        uint64_t *line = rec + ((size_t)(epoch & 1u) * nb + threadIdx.x) * kRecWords;
        uint32_t spins = 0;
        while (true) {
            uint64_t v[NW];
            bool all = true;
#pragma unroll
            for (int k = 0; k < NW; ++k) v[k] = __hip_atomic_load(line + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int k = 0; k < NW; ++k) all = all && (v[k] >> 32) == (uint64_t)epoch;
            if (all) {
#pragma unroll
                for (int k = 0; k < NW; ++k) L.w[k][threadIdx.x] = (uint32_t)v[k];
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            if ((++spins & 63) == 0) {
                if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) { L.bad = 1; break; }
                if (spins > kSpinLimit) {
                    __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    L.bad = 1;
                    break;
                }
            }
        }
    }
    __syncthreads();
    return L.bad == 0;
}

__device__ __forceinline__ uint32_t hi32(double v) { return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32); }
__device__ __forceinline__ uint32_t lo32(double v) { return (uint32_t)(uint64_t)__double_as_longlong(v); }
__device__ __forceinline__ double from32(uint32_t hi, uint32_t lo) {
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}


// --------------------------------------------------------------- models --
struct Lgssm {
    static constexpr int NF = 1;
    // hyp = {a, q_sd, r_sd, m0, p0_sd}
    __device__ static void init(const SmcDev &a, uint32_t j, float st[NF]) {
        float x = a.hyp[3];
        if (a.hyp[4] != 0.0f) {
            float z[4];
            normals4(philox(j, 1, 0, (a.inst << 8) | kTagPrior, a.key), z);
            x = fmaf(a.hyp[4], z[0], x);
        }
        st[0] = x;
    }
    static constexpr bool kNoise = true;
    // Noise of slot j at factor s is normal (s mod 4) of block (j, 0, s div 4):
    // for an even s, z0 is factor s's and z1 factor s + 1's (one Box-Muller pair).
    // It depends on nothing else, so it is drawn every other factor while the
    // factor's records are on their way between the blocks.
    __device__ static void noise(const SmcDev &a, int64_t s, uint32_t j, float &z0, float &z1) {
        const uint4 w = philox(j, 0, (uint32_t)(s >> 2), (a.inst << 8) | kTagPrior, a.key);
        box_muller(unit_f32((s & 2) ? w.z : w.x), unit_f32((s & 2) ? w.w : w.y), z0, z1);
    }
    __device__ static float step(const SmcDev &a, float z, float st[NF], float ys) {
        const float x = fmaf(a.hyp[0], st[0], a.hyp[1] * z);
        st[0] = x;
        const float r = (ys - x) / a.hyp[2];
        return (float)a.lconst - 0.5f * r * r;
    }
};

template <int K>
struct Gmm {
    static constexpr int NF = 2 * K;
    static constexpr bool kNoise = false;
    __device__ static void noise(const SmcDev &, int64_t, uint32_t, float &, float &) {}
    // hyp = {mu_sd, comp_sd}; state = {log pi_0..K-1, mu_0..K-1}
    __device__ static void init(const SmcDev &a, uint32_t j, float st[NF]) {
        const uint32_t c3 = (a.inst << 8) | kTagPrior;
        const uint4 w0 = philox(j, 0, 0, c3, a.key), w1 = philox(j, 1, 0, c3, a.key);
        const uint32_t w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
        float E[K], tot = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            E[k] = -logf(unit_f32(w[k]));
            tot += E[k];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) st[k] = logf(E[k] / tot);
        float z[8];
        normals4(philox(j, 2, 0, c3, a.key), z);
        normals4(philox(j, 3, 0, c3, a.key), z + 4);
#pragma unroll
        for (int k = 0; k < K; ++k) st[K + k] = a.hyp[0] * z[k];
    }
    __device__ static float step(const SmcDev &a, float, float st[NF], float ys) {
        const float inv = 1.0f / a.hyp[1];
        float t[K], mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float r = (ys - st[K + k]) * inv;
            t[k] = fmaf(-0.5f * r, r, st[k]);
            mx = fmaxf(mx, t[k]);
        }
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) s += expf(t[k] - mx);
        return (float)a.lconst + mx + logf(s);
    }
};

// ------------------------------------------------------- resample-move --
// After each resampling at factor s a mixture particle takes move_steps
// Metropolis-Hastings steps whose target is the posterior given y_0..y_s
// (particle inference of Sec. 6 with the acceptance rule of the paper's
// Metropolis-Hastings method, Sec. 3.6.3).  Coordinates u = (log pi_k -
// log pi_K for k < K, mu_k); prior density Dirichlet(1) (the softmax
// Jacobian sum_k log pi_k) times Normal(0, mu_sd) per mean; symmetric Gaussian
// random walk u' = u + h z with
//   h_mu = lam / sqrt(1/mu_sd^2 + (s+1)/(K comp_sd^2)),
//   h_b  = lam / sqrt(3/pi^2 + (s+1)/(2K)),
// accepted when log v < log alpha (FP64).  Move m of slot j draws sixteen
// normals from Philox blocks (j, 8m + b, s, inst << 8 | 7), b < 4, and v
// from word 0 of block 8m + 4.  The log-likelihood of y_0..y_s sums the
// model's FP32 factor within blocks of 16 data and in FP64 across blocks.
template <int K>
__device__ double gmm_loglik_upto(const SmcDev &a, int64_t s, const float st[2 * K]) {
    double tot = 0.0;
    float blk = 0.0f;
    int64_t d = 0;
    // kSide data side by side, then added in order: one after the other, a
    // factor's chain of exp, log and adds left the SIMD idle (500 x 20011, K = 4,
    // one move per event: 4.59 -> 4.19 ms)
    constexpr int kSide = 4;
    for (; d + kSide <= s + 1; d += kSide) {
        float f[kSide];
#pragma unroll
        for (int i = 0; i < kSide; ++i) f[i] = Gmm<K>::step(a, 0.0f, const_cast<float *>(st), a.y[d + i]);
#pragma unroll
        for (int i = 0; i < kSide; ++i) blk += f[i];
        if (((d + kSide) & 15) == 0) {
            tot += (double)blk;
            blk = 0.0f;
        }
    }
    for (; d <= s; ++d) blk += Gmm<K>::step(a, 0.0f, const_cast<float *>(st), a.y[d]);
    return tot + (double)blk;
}

template <int K>
__device__ __forceinline__ double gmm_log_prior(const float st[2 * K], float inv_mu_sd) {
    double l = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float r = st[K + k] * inv_mu_sd;
        l += (double)st[k] - 0.5 * (double)(r * r);
    }
    return l;
}

// One particle's moves; its state is read from and written back to g[f * stride].
template <int K>
__device__ void gmm_move(const SmcDev &a, int64_t s, uint32_t j, float *g, size_t stride,
                                      double *alpha_row, int64_t N) {
    float st[2 * K];
#pragma unroll
    for (int f = 0; f < 2 * K; ++f) st[f] = g[f * stride];
    const double n = (double)(s + 1);
    const float h_mu = (float)(a.move_lam / sqrt(1.0 / (a.hyp64[0] * a.hyp64[0]) +
                                                n / ((double)K * a.hyp64[1] * a.hyp64[1])));
    const float h_b = (float)(a.move_lam / sqrt(3.0 / (M_PI * M_PI) + n / (2.0 * K)));
    const float inv_mu_sd = 1.0f / a.hyp[0];
    const uint32_t c3 = (a.inst << 8) | kTagMove;
    double ll = gmm_loglik_upto<K>(a, s, st);
    double lp = gmm_log_prior<K>(st, inv_mu_sd);
    for (int m = 0; m < a.move_steps; ++m) {
        float z[16];
#pragma unroll
        for (int b = 0; b < 4; ++b) normals4(philox(j, (uint32_t)(8 * m + b), (uint32_t)s, c3, a.key), z + 4 * b);
        const float v = unit_f32(philox(j, (uint32_t)(8 * m + 4), (uint32_t)s, c3, a.key).x);
        float st2[2 * K];
        float mx = 0.0f;
#pragma unroll
        for (int k = 0; k < K - 1; ++k) {
            st2[k] = fmaf(h_b, z[k], st[k] - st[K - 1]);
            mx = fmaxf(mx, st2[k]);
        }
        float se = expf(-mx);
#pragma unroll
        for (int k = 0; k < K - 1; ++k) se += expf(st2[k] - mx);
        const float lse = mx + logf(se);
#pragma unroll
        for (int k = 0; k < K - 1; ++k) st2[k] -= lse;
        st2[K - 1] = -lse;
#pragma unroll
        for (int k = 0; k < K; ++k) st2[K + k] = fmaf(h_mu, z[K - 1 + k], st[K + k]);
        const double ll2 = gmm_loglik_upto<K>(a, s, st2);
        const double lp2 = gmm_log_prior<K>(st2, inv_mu_sd);
        const double la = (ll2 + lp2) - (ll + lp);
        if (alpha_row) alpha_row[(size_t)m * N + j] = la;
        if (log((double)v) < la) {
#pragma unroll
            for (int k = 0; k < 2 * K; ++k) st[k] = st2[k];
            ll = ll2;
            lp = lp2;
        }
    }
#pragma unroll
    for (int f = 0; f < 2 * K; ++f) g[f * stride] = st[f];
}

template <class M>
struct MoveOf {
    __device__ static void run(const SmcDev &, int64_t, uint32_t, float *, size_t, double *, int64_t) {}
};
template <int K>
struct MoveOf<Gmm<K>> {
    __device__ static void run(const SmcDev &a, int64_t s, uint32_t j, float *g, size_t stride, double *alpha_row,
                               int64_t N) {
        gmm_move<K>(a, s, j, g, stride, alpha_row, N);
    }
};

// FP64 log/exp kept out of line: inlined, their polynomial constants get hoisted
// out of the factor loop and occupy registers for the whole run.
__device__ __noinline__ double log_f64(double v) { return log(v); }
__device__ __noinline__ double exp_f64(double v) { return exp(v); }

// ------------------------------------------------------ block helpers --
// Two sums in one pass (lds holds 2 * kSmcWaves doubles).
__device__ __forceinline__ void block_sum2_f64(double &u, double &v, double *lds) {
    u = wave_sum_dpp(u);
    v = wave_sum_dpp(v);
    if ((threadIdx.x & 63) == 0) {
        lds[threadIdx.x >> 6] = u;
        lds[kSmcWaves + (threadIdx.x >> 6)] = v;
    }
    __syncthreads();
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int w = 0; w < kSmcWaves; ++w) {
        a += lds[w];
        b += lds[kSmcWaves + w];
    }
    __syncthreads();
    u = a;
    v = b;
}

// Inclusive scan of one u64 per lane: four row shifts and two row broadcasts
// (DPP; lanes that a step leaves out add 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_scan_u64(uint64_t v) {
    v += dpp_u64<0x111, 0xF>(v);     // row_shr 1, 2, 4, 8: inclusive within each row of 16
    v += dpp_u64<0x112, 0xF>(v);
    v += dpp_u64<0x114, 0xF>(v);
    v += dpp_u64<0x118, 0xF>(v);
    v += dpp_u64<0x142, 0xA>(v);     // row 0's total into row 1, row 2's into row 3
    v += dpp_u64<0x143, 0xC>(v);     // rows 0 and 1's total into rows 2 and 3
    return v;
}

// Maximum and inclusive running maximum of one u32 per lane, the same steps.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan_max_u32(uint32_t v) {
    v = max(v, dpp_u32<0x111, 0xF>(v));
    v = max(v, dpp_u32<0x112, 0xF>(v));
    v = max(v, dpp_u32<0x114, 0xF>(v));
    v = max(v, dpp_u32<0x118, 0xF>(v));
    v = max(v, dpp_u32<0x142, 0xA>(v));
    v = max(v, dpp_u32<0x143, 0xC>(v));
    return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_max_u32(v), 63);
}

// Position of entry i in the LDS arrays that a thread reads or writes P = 8
// consecutive entries of: one word of padding per eight, so that the lanes'
// eight-word strides fall on different banks.
__device__ __forceinline__ int padded(int i) { return i + (i >> 3); }
constexpr int64_t padded_size(int64_t n) { return n + (n + 7) / 8; }

constexpr int kRecGroups = kSmcThreads / 64;     // groups of 64 records, at most one per wave

// Merges the per-block partials {max, s1, s2} (FP32 rescale factors: this feeds the
// resampling trigger only), in the same order in every block: every wave takes
// the maximum over all records for itself, wave g sums records 64 g .. 64 g + 63,
// and after one workgroup barrier every thread adds the groups in order.
__device__ __forceinline__ void merge_partials(const RecLds &L, int nb, double *lds, float &M, double &S1, double &S2) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float mx = -INFINITY;
#pragma unroll
    for (int g = 0; g < kRecGroups; ++g)
        if (64 * g < nb && 64 * g + lane < nb) mx = fmaxf(mx, __uint_as_float(L.w[0][64 * g + lane]));
    M = wave_max_dpp(mx);
    if (64 * wv < nb) {
        const int t = 64 * wv + lane;
        const float mb = t < nb ? __uint_as_float(L.w[0][t]) : -INFINITY;
        double s1 = 0.0, s2 = 0.0;
        if (M > -INFINITY && mb > -INFINITY) {
            const float c = expf(mb - M);
            s1 = from32(L.w[1][t], L.w[2][t]) * (double)c;
            s2 = from32(L.w[3][t], L.w[4][t]) * (double)(c * c);
        }
        s1 = wave_sum_dpp(s1);
        s2 = wave_sum_dpp(s2);
        if (lane == 0) {
            lds[wv] = s1;
            lds[kRecGroups + wv] = s2;
        }
    }
    __syncthreads();
    S1 = 0.0;
    S2 = 0.0;
#pragma unroll
    for (int g = 0; g < kRecGroups; ++g) {
        if (64 * g < nb) {
            S1 += lds[g];
            S2 += lds[kRecGroups + g];
        }
    }
}

// Slot thresholds.  For integers, N Q_a > j S + U  <=>  Q_a > floor((j S + U) / N),
// and with S = N Sq + Sr (Sr < N < 2^31):
//   tau_j = floor((j S + U) / N) = j Sq + floor((j Sr + U) / N),
// where j Sr + U < 2^63, so tau_j needs only 64-bit arithmetic.  Consecutive
// slots update the quotient and remainder incrementally.
struct SlotThreshold {
    uint64_t quo, rem;   // of (j Sr + U) / N
};

// num / N and the remainder with inv = floor((2^64 - 1) / N): the high half of
// num inv is at most two short of the quotient.
__device__ __forceinline__ SlotThreshold divide_n(uint64_t num, uint64_t N, uint64_t inv) {
    SlotThreshold t;
    t.quo = __umul64hi(num, inv);
    t.rem = num - t.quo * N;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const bool more = t.rem >= N;
        t.rem = more ? t.rem - N : t.rem;
        t.quo = more ? t.quo + 1 : t.quo;
    }
    return t;
}

__device__ __forceinline__ SlotThreshold slot_threshold(uint32_t j, uint64_t Sr, uint64_t U, uint64_t N, uint64_t inv) {
    return divide_n((uint64_t)j * Sr + U, N, inv);
}

__device__ __forceinline__ void slot_threshold_next(SlotThreshold &t, uint64_t Sr, uint64_t N) {
    t.rem += Sr;
    if (t.rem >= N) {
        t.rem -= N;
        t.quo += 1;
    }
}

// Resampling data carry their event's tag, so the readers need no acquire
// (and the writers no release).  A prefix word holds the tag in its top two
// bits (1 + r mod 3 for the (r + 1)-th event of the call: never 0, the value
// the words are cleared to before the launch, and never the previous
// event's) and the tile-local exclusive prefix (< 2^62) below; a state word
// holds r + 1 in its high half and the FP32 bits in its low half.  A reader
// that finds another tag (the store has not reached it yet) polls the word
// again; after kSpinLimit polls, or once another block has aborted, it sets
// `bad` and returns 0 (an in-range value, so every index derived from it
// stays in bounds).
constexpr int kQTagShift = 62;
constexpr uint64_t kQMask = (1ull << kQTagShift) - 1;

__device__ __forceinline__ uint64_t qtag_of(int64_t r) { return (uint64_t)(1 + r % 3) << kQTagShift; }

__device__ __forceinline__ uint64_t read_q(const uint64_t *w, uint64_t tag, unsigned *abort_flag, bool &bad) {
    uint64_t v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t spins = 0;
    while ((v & ~kQMask) != tag) {
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 63) == 0 &&
            (spins > kSpinLimit || __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bad = true;
            return 0;
        }
        v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return v & kQMask;
}

__device__ __forceinline__ float read_x(const uint64_t *w, uint32_t tag, unsigned *abort_flag, bool &bad) {
    uint64_t v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t spins = 0;
    while ((uint32_t)(v >> 32) != tag) {
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 63) == 0 &&
            (spins > kSpinLimit || __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bad = true;
            return 0.0f;
        }
        v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return __uint_as_float((uint32_t)v);
}

// Ancestor of the slot with threshold tau over the whole population: the
// last a with X_a <= tau, where X_a = tile_pre[b] + x_a is the exclusive
// prefix of q before a (x_a tile-local, tagged in device memory; tile ends
// and exclusive tile prefixes are in LDS).  This is min{a : Q_a > tau} for the
// inclusive prefix Q: a particle of zero weight shares its prefix with the
// next one.  lo_bound (the previous slot's ancestor, or -1) has X <= tau.
__device__ __forceinline__ int find_ancestor_global(uint64_t tau, int64_t N, int nb, int tile, const uint64_t *tile_end,
                                                    const uint64_t *tile_pre, const uint64_t *qt, uint64_t tag,
                                                    int lo_bound, unsigned *abort_flag, bool &bad) {
    int lo = lo_bound < 0 ? 0 : lo_bound / tile, hi = nb - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tile_end[mid] > tau) hi = mid; else lo = mid + 1;
    }
    const uint64_t pre = tile_pre[lo];
    // X of the tile's first particle is tile_pre[lo] <= tau (tile lo is the first
    // whose end exceeds tau), so the answer is in [a0, a1): search for the first
    // index after a0 whose prefix exceeds tau
    int a0 = lo * tile;
    const int a1 = (int)min((int64_t)a0 + tile, N);
    if (lo_bound > a0) a0 = lo_bound;
    int l = a0 + 1, h = a1;
    while (l < h) {
        const int mid = (l + h) >> 1;
        if (pre + read_q(qt + mid, tag, abort_flag, bad) > tau) h = mid; else l = mid + 1;
    }
    return l - 1;
}

// ---------------------------------------------------------------- kernel --
// MOVES: the resample-move instantiation (a separate kernel, so the moves'
// registers never add to the plain filter's).
template <class M, int P, bool MOVES>
__global__ __launch_bounds__(kSmcThreads) void smc_persistent_kernel(SmcDev a) {
    __shared__ float s_max[kSmcWaves];
    __shared__ double ldsd[2 * kSmcWaves];
    __shared__ uint64_t s_scan[kSmcWaves];
    __shared__ double s_esum[kSmcWaves];
    __shared__ float ybuf[kYChunk];
    __shared__ uint32_t s_cnt[kSmcWaves];
    __shared__ double s_merge[2 * kRecGroups];
    __shared__ RecLds L;
    // dynamic LDS: tile_end[nb] | tile_pre[nb] | own_q[kTile] (u64) | s_slot[kTile] (i32) |
    // own_x[kTile] (FP32, one-field models only); the last three with padded() positions
    constexpr int kTile = kSmcThreads * P;
    constexpr int kTilePad = (int)padded_size(kTile);
    constexpr bool kOwnX = M::NF == 1;
    extern __shared__ uint64_t dyn[];
    const int nb = gridDim.x;
    uint64_t *tile_end = dyn;
    uint64_t *tile_pre = dyn + nb;
    uint64_t *own_q = dyn + 2 * nb;
    int32_t *s_slot = (int32_t *)(own_q + kTilePad);
    float *own_x = (float *)(s_slot + kTilePad);

    const int64_t N = a.N;
    const int64_t tile0 = (int64_t)blockIdx.x * kTile;                 // this block's first slot
    const int tlen = (int)min((int64_t)kTile, N - tile0);               // and its slot count
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * P;

    float st[P][M::NF];
    float lw[P], lwc[P];     // log-weight and its compensation term
    bool valid[P];
    unsigned epoch = 0;
    double logz = 0.0;
    int64_t nres = 0;
    int status = 0;
    float Mlast = 0.0f;
    bool alive = true;
    const double logN = log_f64((double)N);
    if (a.t0 > 0) {
        // resume: the run's scalars from the header, each particle from the checkpoint
        const SmcCkpt *h = (const SmcCkpt *)a.ckpt;
        const float *cs = (const float *)(a.ckpt + kCkptHeader);
        if (h->t != a.t0 || h->N != N || h->nf != M::NF) {
            status = PPL_E_ARG;
        } else {
            logz = h->logz;
            nres = h->nres;
            Mlast = h->mlast;
            status = h->status;
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            valid[p] = base + p < N;
#pragma unroll
            for (int f = 0; f < M::NF; ++f) st[p][f] = valid[p] ? cs[(size_t)f * N + base + p] : 0.0f;
            lw[p] = valid[p] ? cs[(size_t)M::NF * N + base + p] : -INFINITY;
            lwc[p] = valid[p] ? cs[(size_t)(M::NF + 1) * N + base + p] : 0.0f;
        }
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            valid[p] = base + p < N;
            M::init(a, (uint32_t)(base + p), st[p]);
            lw[p] = valid[p] ? 0.0f : -INFINITY;
            lwc[p] = 0.0f;
        }
    }

    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // Bookkeeping is the last wave's: it neither posts nor (up to 256 blocks) polls.
    // The normaliser of the last resampling is added to log Z-hat there while the
    // next factor's records are on their way.
    constexpr int kBook = kSmcThreads - 64;
    const bool book = threadIdx.x == kBook;
    double pend = 0.0;
    float pend_m = 0.0f;
    int64_t pend_s = -1;
    auto flush = [&]() {
        if (wv == kSmcWaves - 1 && pend_s >= 0) {
            const double inc = (double)pend_m + log_f64(pend) - logN;
            logz += inc;
            if (a.logz_tr && blockIdx.x == 0 && book) a.logz_tr[pend_s] = inc;
        }
        pend_s = -1;
    };
    if (threadIdx.x == 0) L.bad = 0;
    __syncthreads();
    // the factor pair's noise: two arrays, so that the choice between them is one of
    // values (an array's element at s mod 2 is an address and lives in scratch memory)
    float zn0[P], zn1[P];
    if constexpr (M::kNoise) {
#pragma unroll
        for (int p = 0; p < P; ++p) M::noise(a, a.t0 & ~(int64_t)1, (uint32_t)(base + p), zn0[p], zn1[p]);
    }
    for (int64_t s = a.t0; status == 0 && s < a.t1; ++s) {
        if (s == a.t0 || (s % kYChunk) == 0) {     // stage the chunk of observations holding factor s
            const int64_t c0 = s - s % kYChunk;
            __syncthreads();
            for (int i = threadIdx.x; i < kYChunk; i += kSmcThreads)
                ybuf[i] = (c0 + i < a.T) ? a.y[c0 + i] : 0.0f;
            __syncthreads();
        }
        const float ys = ybuf[s % kYChunk];
        // The slot index is re-materialised every factor: otherwise the compiler
        // hoists every per-slot address out of the factor loop and runs out of VGPRs.
        int jb = (int)base;
        asm volatile("" : "+v"(jb));
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float z = 0.0f;
            if constexpr (M::kNoise) z = (s & 1) ? zn1[p] : zn0[p];
            const float f = M::step(a, z, st[p], ys);
            if (valid[p]) kahan_add(lw[p], lwc[p], f);
        }
        // block partial for the ESS trigger
        float ml = -INFINITY;
#pragma unroll
        for (int p = 0; p < P; ++p) ml = fmaxf(ml, lw[p]);
        // Workgroup barriers of a factor: after the wave maxima, after the wave
        // sums, and the one of tagged_wait; every LDS word written between two of
        // them is next written after another two.
        ml = wave_max_dpp(ml);
        if (lane == 0) s_max[wv] = ml;
        __syncthreads();
        float mb = s_max[0];
#pragma unroll
        for (int w = 1; w < kSmcWaves; ++w) mb = fmaxf(mb, s_max[w]);
        float s1l = 0.0f, s2l = 0.0f;
        if (mb > -INFINITY) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const float e = expf(lw[p] - mb);
                s1l += e;
                s2l = fmaf(e, e, s2l);
            }
        }
        {
            const double u = wave_sum_dpp((double)s1l), v = wave_sum_dpp((double)s2l);
            if (lane == 0) {
                ldsd[wv] = u;
                ldsd[kSmcWaves + wv] = v;
            }
        }
        __syncthreads();
        ++epoch;
        if (threadIdx.x == 0) {
            double s1b = 0.0, s2b = 0.0;
#pragma unroll
            for (int w = 0; w < kSmcWaves; ++w) {
                s1b += ldsd[w];
                s2b += ldsd[kSmcWaves + w];
            }
            tagged_post<5>(a.rec, epoch, nb, {__float_as_uint(mb), hi32(s1b), lo32(s1b), hi32(s2b), lo32(s2b)});
        }
        flush();
        if constexpr (M::kNoise) {
            if ((s & 1) && s + 1 < a.t1) {
#pragma unroll
                for (int p = 0; p < P; ++p) M::noise(a, s + 1, (uint32_t)(jb + p), zn0[p], zn1[p]);
            }
        }
        if (!tagged_wait<5>(a.rec, a.bar, epoch, nb, L)) {
            alive = false;
            break;
        }
        float Mg;
        double S1, S2;
        merge_partials(L, nb, s_merge, Mg, S1, S2);
        Mlast = Mg;
        if (!(Mg > -INFINITY)) { status = PPL_E_ZERO_WEIGHT; break; }
        if (!(S1 > 0.0) || isnan(S1) || isnan(S2)) { status = PPL_E_NONFINITE; break; }
        const double ess = S1 * S1 / S2;
        const bool res = (s < a.T - 1) && (ess < (double)a.ess_frac * (double)N);
        if (blockIdx.x == 0 && book) {
            if (a.ess_trace) a.ess_trace[s] = ess;
            if (a.resampled) a.resampled[s] = res ? 1 : 0;
            if (a.logz_tr && !res) a.logz_tr[s] = 0.0;
        }
        if (!res) continue;
        if (a.elw_out && nres < a.max_events) {
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (valid[p]) a.elw_out[(size_t)nres * N + jb + p] = lw[p];
        }

        // ---- resampling: FP64 weights, normaliser, integer quantisation, tile scan
        uint64_t qx[P];          // exclusive prefixes within the thread
        uint64_t run = 0;
        double esl = 0.0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const double e = valid[p] ? exp_f64((double)lw[p] - (double)Mg) : 0.0;
            esl += e;
            qx[p] = run;
            run += (uint64_t)floor(ldexp(e, a.kbits));
        }
        const uint64_t incl = wave_scan_u64(run);
        {
            const double e = wave_sum_dpp(esl);
            if (lane == 63) {
                s_scan[wv] = incl;
                s_esum[wv] = e;
            }
        }
        __syncthreads();
        uint64_t off = incl - run;
#pragma unroll
        for (int w = 0; w < kSmcWaves; ++w)
            if (w < wv) off += s_scan[w];
        // The totals leave first; the tile itself is published while they are on
        // their way (a reader that is early finds an old tag and loads again).
        ++epoch;
        if (threadIdx.x == 0) {
            uint64_t btot = 0;
            double eb = 0.0;
#pragma unroll
            for (int w = 0; w < kSmcWaves; ++w) {
                btot += s_scan[w];
                eb += s_esum[w];
            }
            tagged_post<4>(a.rec, epoch, nb, {(uint32_t)(btot >> 32), (uint32_t)btot, hi32(eb), lo32(eb)});
        }
        const uint64_t qtag = qtag_of(nres);
        const uint32_t xtag = (uint32_t)(nres + 1);
        // The tile's prefix sums (and a one-field state) go to LDS, where this
        // block reads its own ancestors, and from there to memory with
        // coalesced stores (whole lines; the particle-major layout of the
        // registers would scatter each store over a wave's 64 particles).
#pragma unroll
        for (int p = 0; p < P; ++p) {
            own_q[padded(threadIdx.x * P + p)] = off + qx[p];
            if constexpr (kOwnX) own_x[padded(threadIdx.x * P + p)] = st[p][0];
        }
        if constexpr (!kOwnX) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (valid[p]) {
#pragma unroll
                    for (int f = 0; f < M::NF; ++f)
                        __hip_atomic_store(a.xtag + (size_t)f * N + jb + p,
                                           ((uint64_t)xtag << 32) | __float_as_uint(st[p][f]), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < tlen; i += kSmcThreads) {
            __hip_atomic_store(a.qtag + tile0 + i, qtag | own_q[padded(i)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if constexpr (kOwnX)
                __hip_atomic_store(a.xtag + tile0 + i, ((uint64_t)xtag << 32) | __float_as_uint(own_x[padded(i)]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        for (int i = threadIdx.x; i < kTilePad; i += kSmcThreads) s_slot[i] = 0;
        const uint4 rw = philox(0, 0, (uint32_t)s, (a.inst << 8) | kTagResample, a.key);
        if (!tagged_wait<4>(a.rec, a.bar, epoch, nb, L)) {
            alive = false;
            break;
        }
        unsigned *abort_flag = a.bar + 1;
        bool bad = false;

        // Tile prefixes and the normaliser sum, in the same order in every block:
        // every wave scans the records for itself (no workgroup barrier).
        int anc[P];
        {
            uint64_t tend[kRecGroups], S = 0;    // inclusive prefix of this lane's tiles
            double ev = 0.0;
#pragma unroll
            for (int g = 0; g < kRecGroups; ++g) {
                tend[g] = ~0ull;
                if (64 * g < nb) {
                    const int t = 64 * g + lane;
                    const uint64_t v = t < nb ? ((uint64_t)L.w[0][t] << 32) | L.w[1][t] : 0;
                    const uint64_t in = S + wave_scan_u64(v);
                    if (t < nb) {
                        tend[g] = in;
                        if (wv == 0) {
                            tile_pre[t] = in - v;
                            tile_end[t] = in;
                        }
                    }
                    S = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(in >> 32), 63) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)in, 63);
                    if (wv == kSmcWaves - 1) ev += wave_sum_dpp(t < nb ? from32(L.w[2][t], L.w[3][t]) : 0.0);
                }
            }
            pend = ev;
            pend_m = Mg;
            pend_s = s;
            const uint64_t U = __umul64hi(((uint64_t)rw.y << 32) | rw.x, S);
            ++nres;
            const uint64_t NN = (uint64_t)N;
            const SlotThreshold sn = divide_n(S, NN, a.inv_n);
            const uint64_t Sq = sn.quo, Sr = sn.rem;

            // Tiles of the ancestors of this block's first and last slot: the
            // first whose end exceeds the slot's threshold, counted over the lanes'
            // tiles.
            const int js0 = blockIdx.x * kTile;
            const int js1 = (int)min((int64_t)js0 + kTile, N) - 1;
            auto tile_of = [&](int j) {
                const uint64_t tau = (uint64_t)j * Sq + slot_threshold((uint32_t)j, Sr, U, NN, a.inv_n).quo;
                int t = 0;
#pragma unroll
                for (int g = 0; g < kRecGroups; ++g)
                    if (64 * g < nb) t += __popcll(__ballot(tend[g] <= tau));
                return min(t, nb - 1);
            };
            const int t0 = tile_of(js0), t1 = tile_of(js1);
            int32_t *anc_row = (a.anc_out && nres - 1 < a.max_events) ? a.anc_out + (size_t)(nres - 1) * N : nullptr;
            if (t1 - t0 < kScatterTiles) {
                // Slot j's ancestor is the last particle a whose exclusive prefix X_a
                // is <= tau_j, that is whose first slot f_a = min{j: X_a N <= j S + U}
                // = ceil((X_a N - U) / S) is <= j.  So every particle of those tiles
                // (this block's own from LDS, the others loaded once) marks slot f_a
                // with its index (the largest wins), and a running maximum over the
                // slots fills the rest: no staging of prefix sums and no search per
                // slot.  f_a is taken in FP64, whose error is below 2^-20 of a slot
                // for N < 2^31; where the value lies that near a whole number the 128-bit
                // products decide.
                const double dS = (double)S, rN = (double)N / dS, cU = (double)U / dS;
                int before = 0;                      // largest mark of a slot before this block's
                auto mark = [&](uint64_t X, int id) {
                    const double d = fma((double)X, rN, -cU), r = __builtin_rint(d);
                    int64_t f = (int64_t)__builtin_ceil(d);
                    if (fabs(d - r) < 0x1p-20) {
                        const int64_t j = (int64_t)r;
                        const unsigned __int128 lhs = (unsigned __int128)X * NN;
                        const unsigned __int128 rhs = (unsigned __int128)(uint64_t)max(j, (int64_t)0) * S + U;
                        f = j >= 0 && lhs <= rhs ? j : j + 1;
                    }
                    const int64_t q = f - js0;
                    if (q <= 0) before = max(before, id);
                    else if (q <= js1 - js0) atomicMax(&s_slot[padded((int)q)], id);
                };
                __syncthreads();                     // tile_pre
                const bool own_in = t0 <= (int)blockIdx.x && (int)blockIdx.x <= t1;
                bool own_done = !own_in;
                auto mark_own = [&]() {
                    const uint64_t pre = tile_pre[blockIdx.x];
                    const int id0 = ((int)blockIdx.x - t0) * kTile + 1;
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        const int i = threadIdx.x + k * kSmcThreads;
                        if (i < tlen) mark(pre + own_q[padded(i)], id0 + i);
                    }
                    own_done = true;
                };
                for (int t = t0; t <= t1; ++t) {
                    if (t == (int)blockIdx.x) continue;
                    const int64_t tb = (int64_t)t * kTile;
                    const int len = (int)min((int64_t)kTile, N - tb);
                    const uint64_t pre = tile_pre[t];
                    uint64_t v[P];
                    bool cur = false;
                    for (int tries = 0; !cur && tries < kBatchTries; ++tries) {
                        // all loads first (clamped in range), then the tags; a word that is
                        // not yet current makes the wave load the tile again
                        bool mine = !a.poll_all;
#pragma unroll
                        for (int k = 0; k < P; ++k)
                            v[k] = __hip_atomic_load(a.qtag + tb + min((int)threadIdx.x + k * kSmcThreads, len - 1),
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (!own_done) mark_own();   // while those loads run
#pragma unroll
                        for (int k = 0; k < P; ++k) mine = mine && (v[k] & ~kQMask) == qtag;
                        cur = __all(mine);
                        if (a.poll_all) break;
                    }
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        const int i = threadIdx.x + k * kSmcThreads;
                        if (i < len) {
                            const uint64_t x = cur ? v[k] & kQMask : read_q(a.qtag + tb + i, qtag, abort_flag, bad);
                            mark(pre + x, (t - t0) * kTile + 1 + i);
                        }
                    }
                }
                if (!own_done) mark_own();
                before = wave_max_u32((uint32_t)before);
                if (lane == 0 && before > 0) atomicMax(&s_slot[0], before);
                __syncthreads();
                uint32_t run_max = 0;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    run_max = max(run_max, (uint32_t)s_slot[padded(threadIdx.x * P + p)]);
                    anc[p] = (int)run_max;
                }
                const uint32_t upto = wave_scan_max_u32(run_max);
                uint32_t left = (uint32_t)__shfl_up((int)upto, 1, 64);
                if (lane == 0) left = 0;
                if (lane == 63) s_cnt[wv] = upto;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < kSmcWaves; ++w)
                    if (w < wv) left = max(left, s_cnt[w]);
                const int first = t0 * kTile - 1;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    anc[p] = first + max(max((int)left, anc[p]), 1);      // 1: only in a run given up
                    if (anc_row && jb + p < N) anc_row[jb + p] = anc[p];
                }
            } else {
                // Ancestors over many tiles (long runs of particles without weight):
                // each slot searches for itself.
                __syncthreads();                     // tile_pre, tile_end
                SlotThreshold th = slot_threshold((uint32_t)jb, Sr, U, NN, a.inv_n);
                int prev = t0 * kTile;
#pragma unroll 1
                for (int p = 0; p < P; ++p) {
                    const int j = jb + p;
                    if (j >= N) break;
                    if (p) slot_threshold_next(th, Sr, NN);
                    const uint64_t tau = (uint64_t)j * Sq + th.quo;
                    prev = find_ancestor_global(tau, N, nb, kTile, tile_end, tile_pre, a.qtag, qtag, prev, abort_flag,
                                                bad);
                    s_slot[padded(threadIdx.x * P + p)] = prev;
                    if (anc_row) anc_row[j] = prev;
                }
#pragma unroll
                for (int p = 0; p < P; ++p) anc[p] = s_slot[padded(threadIdx.x * P + p)];
            }
        }
        if constexpr (!MOVES) {
            // gather the ancestors' state: all loads first, then the tags; a word
            // that is not yet current sends the thread through the polling reads
            bool fresh = !a.poll_all;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (!valid[p]) continue;
                if (kOwnX && (uint64_t)(anc[p] - tile0) < (uint64_t)tlen) {
                    st[p][0] = own_x[padded((int)(anc[p] - tile0))];      // an ancestor of this block's own tile
                } else {
#pragma unroll
                    for (int f = 0; f < M::NF; ++f) {
                        const uint64_t v = __hip_atomic_load(a.xtag + (size_t)f * N + anc[p], __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                        fresh = fresh && (uint32_t)(v >> 32) == xtag;
                        st[p][f] = __uint_as_float((uint32_t)v);
                    }
                }
                lw[p] = 0.0f;
                lwc[p] = 0.0f;
            }
            if (!fresh) {
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    if (!valid[p]) continue;
                        if (kOwnX && (uint64_t)(anc[p] - tile0) < (uint64_t)tlen) continue;
#pragma unroll
                    for (int f = 0; f < M::NF; ++f)
                        st[p][f] = read_x(a.xtag + (size_t)f * N + anc[p], xtag, abort_flag, bad);
                }
            }
        } else {
            // resample-move: the gathered particles go through memory one at a
            // time, so only the moving particle's state occupies registers
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (!valid[p]) continue;
#pragma unroll
                for (int f = 0; f < M::NF; ++f)
                    a.xbuf2[(size_t)f * N + jb + p] = read_x(a.xtag + (size_t)f * N + anc[p], xtag, abort_flag, bad);
                lw[p] = 0.0f;
                lwc[p] = 0.0f;
            }
            double *arow = (a.alpha_out && nres - 1 < a.max_events)
                               ? a.alpha_out + (size_t)(nres - 1) * a.move_steps * N : nullptr;
#pragma unroll 1
            for (int p = 0; p < P; ++p) {
                const int j = jb + p;
                if (j >= N) break;
                MoveOf<M>::run(a, s, (uint32_t)j, a.xbuf2 + j, (size_t)N, arow, N);
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int f = 0; f < M::NF; ++f) st[p][f] = valid[p] ? a.xbuf2[(size_t)f * N + jb + p] : 0.0f;
            }
        }
        if (bad) L.bad = 1;      // a tagged read gave up: the next wait, or the check after the loop, sees it
    }
    __syncthreads();
    if (L.bad) alive = false;
    flush();

    // ---- stop: the run's state into the checkpoint
    const bool stopped = a.t1 < a.T;
    if (stopped && alive) {
        float *cs = (float *)(a.ckpt + kCkptHeader);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (!valid[p]) continue;
#pragma unroll
            for (int f = 0; f < M::NF; ++f) cs[(size_t)f * N + base + p] = st[p][f];
            cs[(size_t)M::NF * N + base + p] = lw[p];
            cs[(size_t)(M::NF + 1) * N + base + p] = lwc[p];
        }
        if (blockIdx.x == 0 && book) {
            SmcCkpt *h = (SmcCkpt *)a.ckpt;
            h->t = a.t1;
            h->N = N;
            h->nres = nres;
            h->nf = M::NF;
            h->status = status;
            h->logz = logz;
            h->mlast = Mlast;
        }
    }
    // ---- final normaliser (FP64) over the last epoch
    double ess_final = stopped ? 0.0 : (double)N;
    if (alive && status == 0 && a.T > 0 && !stopped) {
        double e1 = 0.0, e2 = 0.0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (valid[p]) {
                const double e = exp_f64((double)lw[p] - (double)Mlast);
                e1 += e;
                e2 += e * e;
            }
        }
        block_sum2_f64(e1, e2, ldsd);
        ++epoch;
        tagged_post<4>(a.rec, epoch, nb, {hi32(e1), lo32(e1), hi32(e2), lo32(e2)});
        if (!tagged_wait<4>(a.rec, a.bar, epoch, nb, L)) {
            alive = false;
        } else {
            const int t = threadIdx.x;
            double t1 = t < nb ? from32(L.w[0][t], L.w[1][t]) : 0.0;
            double t2 = t < nb ? from32(L.w[2][t], L.w[3][t]) : 0.0;
            block_sum2_f64(t1, t2, ldsd);
            const double inc = (double)Mlast + log_f64(t1) - logN;
            logz += inc;
            if (a.logz_tr && blockIdx.x == 0 && book) a.logz_tr[a.T - 1] = inc;
            ess_final = t1 * t1 / t2;
        }
    }
    if (!alive) status = PPL_E_HIP;

#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (!valid[p]) continue;
        const int64_t j = base + p;
        if (a.lw_out) a.lw_out[j] = lw[p];
        if (a.lat_out) {
#pragma unroll
            for (int f = 0; f < M::NF; ++f) a.lat_out[(size_t)f * N + j] = st[p][f];
        }
    }
    if (blockIdx.x == 0 && book) {
        a.scalars[0] = status ? (status == PPL_E_ZERO_WEIGHT ? -INFINITY : NAN) : logz;
        a.scalars[1] = status ? 0.0 : ess_final;
        a.scalars[2] = (double)nres;
        a.scalars[3] = (double)status;
        a.scalars[4] = (double)Mlast;
        a.scalars[5] = 0.0;
        a.scalars[6] = 0.0;
        a.scalars[7] = (double)N;
    }
}

// Clears the abort flag and the record lines' epochs (a fill kernel, so the
// launch sequence stays capturable).
__global__ void smc_reset_kernel(unsigned *bar, uint64_t *rec, int n_lines, uint64_t *tagged, int64_t n_tagged) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < kBarWords; i += stride) bar[i] = 0u;
    for (int64_t i = i0; i < (int64_t)n_lines * kRecWords; i += stride) rec[i] = 0u;
    for (int64_t i = i0; i < n_tagged; i += stride) tagged[i] = 0u;
}

// ------------------------------------------------------------------ host --
static int pick_p(int64_t N) {
    // particles per thread so that one block per CU covers N (up to 8)
    const int64_t per_cu = (N + 255) / 256;
    int P = 1;
    while (P < 8 && (int64_t)kSmcThreads * P < per_cu) P <<= 1;
    return P;
}

static int64_t smc_blocks(int64_t N, int P) { return (N + (int64_t)kSmcThreads * P - 1) / ((int64_t)kSmcThreads * P); }

struct SmcLayout {
    double *scal;
    unsigned *bar;
    uint64_t *rec, *qtag, *xtag;     // qtag and xtag adjacent: [N] then [NF][N]
    float *xbuf2;
    size_t bytes;
};

static SmcLayout smc_layout(void *ws, int NF, int64_t N, int64_t nb) {
    SmcLayout L;
    char *p = (char *)ws;
    size_t o = 0;
    auto take = [&](size_t n) { char *r = p + o; o += align_up(n, 256); return r; };
    L.scal = (double *)take(8 * sizeof(double));
    L.bar = (unsigned *)take(kBarWords * sizeof(unsigned));
    L.rec = (uint64_t *)take((size_t)2 * nb * kRecWords * sizeof(uint64_t));
    L.qtag = (uint64_t *)take((size_t)(NF + 1) * N * sizeof(uint64_t));
    L.xtag = L.qtag + N;
    L.xbuf2 = NF > 1 ? (float *)take((size_t)NF * N * sizeof(float)) : nullptr;   // mixture models only
    L.bytes = o;
    return L;
}

size_t smc_checkpoint_bytes(int model, int K, int64_t N) {
    const int NF = model == PPL_MODEL_LGSSM ? 1 : 2 * K;
    return kCkptHeader + align_up((size_t)(NF + 2) * N * sizeof(float), 256);
}

size_t smc_ws_bytes(int model, int K, int64_t N) {
    const int NF = model == PPL_MODEL_LGSSM ? 1 : 2 * K;
    const int P = pick_p(N);
    return smc_layout(nullptr, NF, N, smc_blocks(N, P)).bytes;
}

double *smc_scalars_ptr(const SmcArgs &a) { return a.out.d_scalars ? a.out.d_scalars : (double *)a.ws; }

template <class M, int P>
static int launch(SmcDev &d, int64_t nb, hipStream_t st) {
    auto kern = d.move_steps > 0 ? smc_persistent_kernel<M, P, true> : smc_persistent_kernel<M, P, false>;
    int dev = 0, ncu = 0, occ = 0;
    PPL_HIP(hipGetDevice(&dev));
    PPL_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    const int64_t tp = padded_size((int64_t)kSmcThreads * P);
    const size_t lds = (size_t)(2 * nb + tp) * sizeof(uint64_t) + (size_t)tp * sizeof(int32_t) +
                       (M::NF == 1 ? (size_t)tp * sizeof(float) : 0);
    PPL_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, kSmcThreads, lds));
    if ((int64_t)occ * ncu < nb)
        return fail(PPL_E_UNSUPPORTED, "SMC needs %lld co-resident blocks, device holds %d", (long long)nb, occ * ncu);
    // clears the barrier words, the record lines and the tagged resampling data
    // (so no word of an earlier call carries a tag this call looks for)
    const int64_t n_tagged = (int64_t)(d.xtag - d.qtag) + (int64_t)M::NF * d.N;
    const int reset_blocks = (int)std::min<int64_t>(1024, std::max<int64_t>(1, (n_tagged + 255) / 256));
    hipLaunchKernelGGL(smc_reset_kernel, dim3(reset_blocks), dim3(256), 0, st, d.bar, d.rec, (int)(2 * nb), d.qtag,
                       n_tagged);
    PPL_LAUNCH_CHECK("smc_reset_kernel");
    void *args[] = {&d};
    KernelTimer timer("smc_persistent_kernel", st);
    PPL_HIP(hipLaunchCooperativeKernel((const void *)kern, dim3((unsigned)nb), dim3(kSmcThreads), args, lds, st));
    timer.stop();
    return PPL_OK;
}

template <class M>
static int launch_p(SmcDev &d, int P, int64_t nb, hipStream_t st) {
    switch (P) {
        case 1: return launch<M, 1>(d, nb, st);
        case 2: return launch<M, 2>(d, nb, st);
        case 4: return launch<M, 4>(d, nb, st);
        case 8: return launch<M, 8>(d, nb, st);
    }
    return fail(PPL_E_UNSUPPORTED, "particles per thread %d", P);
}

int run_smc(const SmcArgs &a, hipStream_t st) {
    const int NF = a.model == PPL_MODEL_LGSSM ? 1 : 2 * a.K;
    const int P = pick_p(a.N);
    const int64_t nb = smc_blocks(a.N, P);
    // every block merges the per-block partials one per thread
    if (nb > kSmcMaxBlocks || nb > kSmcThreads)
        return fail(PPL_E_UNSUPPORTED, "SMC supports at most %lld particles",
                    (long long)std::min(kSmcMaxBlocks, kSmcThreads) * kSmcThreads * 8);
    if (a.T > 0x7fffffffLL) return fail(PPL_E_ARG, "too many factors");
    // a run passes at most 2 T + 1 barriers, each with its own epoch
    if (2 * a.T + 2 >= 0xffffffffLL) return fail(PPL_E_UNSUPPORTED, "barrier epoch would overflow");
    SmcLayout L = smc_layout(a.ws, NF, a.N, nb);
    SmcDev d{};
    d.y = a.y;
    d.T = a.T;
    d.N = a.N;
    d.K = a.K;
    d.key = make_key(a.seed);
    d.inst = a.inst;
    d.ess_frac = (float)a.ess_frac;
    for (int i = 0; i < 5; ++i) d.hyp[i] = (float)a.hyper[i];
    if (a.model == PPL_MODEL_LGSSM) d.lconst = -0.5 * log(2.0 * M_PI * a.hyper[2] * a.hyper[2]);
    else d.lconst = -0.5 * log(2.0 * M_PI) - log(a.hyper[1]);
    int c = 0;
    while (((int64_t)1 << c) < a.N) ++c;
    d.kbits = 62 - c;
    d.inv_n = ~0ull / (uint64_t)a.N;
    d.scalars = a.out.d_scalars ? a.out.d_scalars : L.scal;
    d.lw_out = (float *)a.out.d_log_weights;
    d.lat_out = (float *)a.out.d_latents;
    d.ess_trace = a.out.d_ess_trace;
    d.resampled = a.out.d_resampled;
    d.anc_out = a.out.d_ancestors;
    d.elw_out = a.out.d_event_lw;
    d.logz_tr = a.out.d_logz_trace;
    d.alpha_out = a.out.d_move_log_alpha;
    d.max_events = a.out.max_events;
    d.t0 = a.t_begin;
    d.t1 = a.t_end;
    d.ckpt = (char *)a.ckpt;
    d.move_steps = a.move_steps;
    // PPL_SMC_POLL_ALL=1 sends every tagged read through the polling path
    // (checking aid: the results must not change)
    {
        const char *e = getenv("PPL_SMC_POLL_ALL");
        d.poll_all = (e && e[0] == '1') ? 1 : 0;
    }
    d.move_lam = a.move_scale > 0.0 ? a.move_scale : 2.38 / sqrt(2.0 * a.K - 1.0);
    d.hyp64[0] = a.hyper[0];
    d.hyp64[1] = a.hyper[1];
    d.bar = L.bar;
    d.rec = L.rec;
    d.qtag = L.qtag;
    d.xtag = L.xtag;
    d.xbuf2 = L.xbuf2;
    if (a.model == PPL_MODEL_LGSSM) return launch_p<Lgssm>(d, P, nb, st);
    switch (a.K) {
        case 1: return launch_p<Gmm<1>>(d, P, nb, st);
        case 2: return launch_p<Gmm<2>>(d, P, nb, st);
        case 3: return launch_p<Gmm<3>>(d, P, nb, st);
        case 4: return launch_p<Gmm<4>>(d, P, nb, st);
        case 5: return launch_p<Gmm<5>>(d, P, nb, st);
        case 6: return launch_p<Gmm<6>>(d, P, nb, st);
        case 7: return launch_p<Gmm<7>>(d, P, nb, st);
        case 8: return launch_p<Gmm<8>>(d, P, nb, st);
    }
    return fail(PPL_E_ARG, "GMM K must be in 1..8");
}

}  // namespace ppl
