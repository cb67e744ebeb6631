// What the two files of bf16 attention kernels share.
#pragma once
#include "mfma.h"

namespace rev {

__device__ __forceinline__ bf16x8_t pack8(const float* p) {
    bf16x8_t r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)p[e];
    return r;
}

__device__ __forceinline__ void store4_bf16(bf16* p, float a, float b, float c, float d) {
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    bf16x4_t v;
    v[0] = (__bf16)a; v[1] = (__bf16)b; v[2] = (__bf16)c; v[3] = (__bf16)d;
    *reinterpret_cast<bf16x4_t*>(p) = v;
}

// attention_dma.hip: heads of 32, 64 or 80 features
bool attention_dma_takes(int dh);
int attention_forward_dma(hipStream_t s, const bf16* qkv, bf16* o, float* lse, int B, int T, int H, int dh, const int* key_len);
int attention_backward_dma(hipStream_t s, const bf16* qkv, const bf16* o, const bf16* dout, const float* lse, bf16* dqkv, float* delta,
                           int B, int T, int H, int dh, const int* key_len);

}  // namespace rev
