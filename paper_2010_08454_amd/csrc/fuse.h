// fuse.h -- pieces of the fused network kernels (the training pass and the
// inference network): weight fragments, one product, the LDS barrier.
#pragma once

#include <hip/hip_runtime.h>

#include "mlp.h"

namespace ppl {

typedef __bf16 fbf16x8_t __attribute__((ext_vector_type(8)));
typedef float ffloatx4_t __attribute__((ext_vector_type(4)));

// A product's weight fragments for this wave: fb[s][j] holds B rows
// 64 wave + 16 j + lane % 16, K entries 32 s + 8 (lane / 16) .. + 7, read from
// the fragment-order copy of the weights (frag_index: each load instruction
// reads 1 KB of consecutive bytes; from the [out][in] or [in][out] layout a
// wave's load touched 16 rows, 64 bytes of each).  They are loaded one product
// ahead (while the previous product's epilogue and the workgroup barrier run),
// so a product waits for global memory at most once.
typedef fbf16x8_t FuseFrags[8][4];

template <int KD, int S>
__device__ __forceinline__ void fuse_load_w(const uint16_t *Bw, fbf16x8_t (&fb)[S][4]) {
    static_assert(S >= KD / 32, "fragment buffer too short");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int fr = lane & 15, fk = (lane >> 4) * 8;
#pragma unroll
    for (int s = 0; s < KD / 32; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            fb[s][j] = *(const fbf16x8_t *)(Bw + frag_index(64 * wave + 16 * j + fr, 32 * s + fk, KD));
    __builtin_amdgcn_sched_barrier(0);       // keep the scheduler from sinking the loads into the MFMA loop
}

// acc[i][j][q] = C[16 i + 4 (lane / 16) + q][64 wave + 16 j + lane % 16] of
// C[32][256] = A[32][KD] B[256][KD]^T, B's fragments in fb.
template <int KD>
__device__ __forceinline__ void fuse_mma(const uint16_t *A, int lda, const FuseFrags &fb, ffloatx4_t (&acc)[2][4]) {
    const int lane = threadIdx.x & 63;
    const int fr = lane & 15, fk = (lane >> 4) * 8;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = ffloatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KD / 32; ++s) {
        fbf16x8_t fa[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[i] = *(const fbf16x8_t *)(A + (size_t)(16 * i + fr) * lda + 32 * s + fk);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[s][j], acc[i][j], 0, 0, 0);
    }
}

// Workgroup barrier for data exchanged through LDS only: waits for this
// wave's LDS operations (lgkmcnt 0) but leaves its global stores and the
// prefetched weight loads in flight (a full __syncthreads would wait for
// them at every layer).  Nothing the fused pass stores to global memory is
// read back by another wave of the workgroup.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);      // vmcnt and expcnt: no wait; lgkmcnt: 0
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// First mean of degree n in the network outputs of the polynomial model (8n
// means, then 8n log-scales, component-major).
__host__ __device__ constexpr int poly_head_off(int n) { return 12 + 8 * (n - 2) * (n + 1); }

}  // namespace ppl
