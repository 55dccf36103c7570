// What the two fp32 attention kernels share.
#pragma once
#include "kernels.h"
#include "work_order.h"

namespace cp {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef const __attribute__((address_space(4))) int32_t* scalar_list;   // read through scalar loads: wave-uniform addresses

namespace {

// Eight copies of 16 bytes per lane from memory (one base) to LDS at (lds_base + lane * 16) + 1 KiB * i: see the bf16 kernels.  A load needs one wait
// state after m0 and five after a vector instruction that writes its scalar address, which the compiler does not see in here.  One block of
// eight instead of a base, m0 and waits for each took 6 to 9 us off dense and block-sparse attention of 8 x 8192 tokens, 1 us off block-sparse 4 x 4096.
__device__ __forceinline__ void copy16x8(const void* sbase, const unsigned (&voff)[8], unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %9\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %9\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %9\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %9\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, %9\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %6, %9\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %7, %9\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %8, %9"
                 ::"s"(lds_base), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "v"(voff[4]), "v"(voff[5]), "v"(voff[6]), "v"(voff[7]), "s"(sbase)
                 : "memory", "scc");
}
// one, from an address per lane
__device__ __forceinline__ void copy16_far(const void* src, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(src) : "memory");
}

}  // namespace

struct Args32 {
    const float* q; const float* k; const float* v; const int32_t* idx; const int32_t* cnt;
    float* out; float* lse;
    int batch, hq, hkv, n, s, b, n1, list_len, qtiles;   // qtiles: per segment (sparse) or per sequence (dense)
    TileOrder order;                              // which row tile a workgroup takes; attn_fp32_kernel: in pairs alone
    int shared_lists;                             // lists are per (batch, KV head, segment) instead of per query head
    float scale_log2e, scale;
    long long qs0, qs1, qs2, ks0, ks1, ks2, os0, os1, os2;
};

// Row tiles of `rows`: those that exist, a segment's last one may be short; of the longest segment; workgroups launched for them; their order.
long long attn_fp32_row_tiles(const Shape& sh, bool sparse, int rows);
int attn_fp32_qtiles(const Shape& sh, bool sparse, int rows);
long long attn_fp32_grid(const Shape& sh, bool sparse, int rows);
TileOrder attn_fp32_order(const Shape& sh, bool sparse, int rows, int waves);

// Where 16 rows go to a workgroup: waves of a workgroup, and workgroups that share a row tile.
int attn_fp32_tile_waves(const Shape& sh, bool sparse);
int attn_fp32_tile_parts(const Shape& sh, bool sparse);

// Attention with fp32 factors split into three bf16 values, whether it is the better one here, and the waves of a workgroup.
bool attn_fp32_split_better(const Shape& sh, bool sparse);
int attn_fp32_split_waves(const Shape& sh, bool sparse);
hipError_t launch_attn_fp32_split(const Shape& sh, Args32& a, hipStream_t st);

}  // namespace cp
