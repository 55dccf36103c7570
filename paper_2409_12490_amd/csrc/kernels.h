// Internal launch interface between the C ABI (api.hip) and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fast_div.h"

namespace cp {

constexpr int kHeadDim = 128;
constexpr int kMaxListBf16 = 6144;    // block-list entries the bf16 attention kernel keeps in LDS

// At the start of a kernel, every argument that its first loads need, in one go: the compiler loads an argument where it is used, one latency after
// another, three to five before the first load of a small kernel.  Layers of 1 x 2048 fp32 21.8 -> 21.3 us, 2 x 600 fp32 20.7 -> 20.0, 8/2 x 1000 22.9
// -> 22.1; estimate 4 x 700 12.2 -> 11.6, dense 2 x 512 6.64 -> 6.52.  (Not kept: in the selection 15.7 -> 15.9 us at 32/8 x 128K, with more scalar
// registers spilled.)
template <typename T>
__device__ __forceinline__ void ask_for_one(const T& x) { asm volatile("" ::"s"(x)); }
template <typename... T>
__device__ __forceinline__ void ask_for(const T&... x) { (ask_for_one(x), ...); }

struct Shape {
    int batch, hq, hkv, n, s, b, r, n1, n2;   // r = s / b
    int budget, local, list_len;
    int dtype;                                // 0 fp32, 1 bf16
    float attn_scale, score_scale, alpha;
    int softmax_domain;
    int64_t qs[3], kvs[3], os[3];             // element strides: batch, head, token
};

// Algorithm 1, max/min lines: representatives in the storage dtype.
// qrep [B,Hq,n1,2,128], krep [B,Hkv,n2,2,128]; index 0 = max, 1 = min.
hipError_t launch_pool(const Shape& sh, const void* q, const void* k, void* qrep, void* krep, hipStream_t st);

// Algorithm 1, score lines (four products, softmax, combine, mask, fusion).
// stats: score_stats_bytes() of scratch (bf16: per-chunk softmax statistics; fp32: unused, 0 bytes).
size_t score_stats_bytes(const Shape& sh);
hipError_t launch_score(const Shape& sh, const void* qrep, const void* krep, const float* prev, float* scores,
                        float* stats, hipStream_t st);

// Algorithm 2, top-k line.  shared: one list per (batch, KV head, segment) from the max of the scores of the
// KV head's query heads (idx [B,Hkv,n1,list_len], cnt [B,Hkv,n1]) instead of one per query head.
hipError_t launch_select(const Shape& sh, const float* scores, int32_t* idx, int32_t* cnt, bool shared, hipStream_t st);

// Algorithm 2 attention loop (idx != nullptr) or Eq. 2 dense causal attention (idx == nullptr).
// shared_lists: idx/cnt hold one list per KV head (see launch_select) instead of one per query head.
hipError_t launch_attn_bf16(const Shape& sh, const void* q, const void* k, const void* v, const int32_t* idx,
                            const int32_t* cnt, bool shared_lists, void* out, float* lse, hipStream_t st);
hipError_t launch_attn_fp32(const Shape& sh, const void* q, const void* k, const void* v, const int32_t* idx,
                            const int32_t* cnt, bool shared_lists, void* out, float* lse, hipStream_t st);

}  // namespace cp
