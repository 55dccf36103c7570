// What the two fp32 attention kernels share.
#pragma once
#include "kernels.h"

namespace cp {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef const __attribute__((address_space(4))) int32_t* scalar_list;   // read through scalar loads: wave-uniform addresses

struct Args32 {
    const float* q; const float* k; const float* v; const int32_t* idx; const int32_t* cnt;
    float* out; float* lse;
    int batch, hq, hkv, n, s, b, n1, list_len, qtiles;   // qtiles: per segment (sparse) or per sequence (dense)
    int shared_lists;                             // lists are per (batch, KV head, segment) instead of per query head
    float scale_log2e, scale;
    long long qs0, qs1, qs2, ks0, ks1, ks2, os0, os1, os2;
};

// Attention with fp32 factors split into fp16 pairs, and whether it is the better one here.
bool attn_fp32_split_better(const Shape& sh, bool sparse);
hipError_t launch_attn_fp32_split(const Shape& sh, Args32& a, hipStream_t st);

}  // namespace cp
