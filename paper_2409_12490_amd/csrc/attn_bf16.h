// What the three bf16 attention kernels share: vector types, argument block, lane exchanges, the copy from memory to LDS.
#pragma once
#include "kernels.h"
#include "work_order.h"

namespace cp {

struct ArgsB {
    const uint16_t* q; const uint16_t* k; const uint16_t* v; const int32_t* idx; const int32_t* cnt;
    uint16_t* out; float* lse;
    int batch, hq, hkv, n, s, b, n1, list_len, qtiles;
    int group;                            // G = hq / hkv
    int shared_lists;                     // lists are per (batch, KV head, segment) instead of per query head
    float scale_log2e, scale;
    long long qs0, qs1, qs2, ks0, ks1, ks2, os0, os1, os2;
};

// Index arithmetic of the 256-row and the 128-row kernel, an argument of its own and their first: it is the first thing that they need, and the 32-row kernel
// reads fewer lines of arguments without it (behind the other arguments 0.4 us more for launches of one round, among them 0.15 us more for the smallest of the 32-row kernel).
struct ArgsIndex {
    WorkOrder order;
    FastDiv div_hkv, div_b;
};

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 v4bf16_lds;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;
#define LDS_PTR(T, off) ((__attribute__((address_space(3))) T*)(uintptr_t)(off))
typedef const __attribute__((address_space(4))) int32_t* scalar_list;   // read through scalar loads: wave-uniform addresses

constexpr float kLazyLog2 = 8.0f;        // how far a row's max may outgrow its reference point before O is rescaled

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
    union { uint4 u; bf16x8 b; } c; c.u = v; return c.b;
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) {
    union { u32x4 u; bf16x8 b; } c; c.u = v; return c.b;
}
// Keep a value computed at this point of the program (stops a load from staying pending into the loop).
__device__ __forceinline__ void pin(const bf16x8& v) { asm volatile("" ::"v"(v)); }

// 16 bytes per lane from global memory (uniform base + per-lane byte offset) straight into LDS at
// (lds_base + lane * 16); lds_base is wave-uniform.  Issued through inline asm so the compiler does not
// serialise later LDS reads of OTHER ring slots behind it; the matching s_waitcnt vmcnt is placed by hand
// before the tile barrier.  m0 is written here and not named as a clobber: it is a reserved register for the
// compiler, which keeps no value in it across statements and sets it anew before each use of its own (naming it
// only draws "clobber list contains reserved registers").  The compiler does not look into the asm for hazards: the load
// needs one wait state after m0 is written and five after a vector instruction (v_readfirstlane, or v_readlane where the
// compiler keeps a scalar in a vector register) has written sbase, so the asm waits for both itself.
__device__ __forceinline__ void dma16(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(voff), "s"(sbase)
                 : "memory");
}
// four of them, 1 KiB apart in LDS, from one base: three scalar instructions less for each but the first
__device__ __forceinline__ void dma16x4(const void* sbase, const unsigned (&voff)[4], unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %5\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %2, %5\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %5\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %5" ::"s"(lds_base), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(sbase)
                 : "memory", "scc");
}
__device__ __forceinline__ void dma16_far(const void* src, unsigned lds_base) {   // the same from an address per lane
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(src) : "memory");
}
__device__ __forceinline__ void dma4(const void* sbase, unsigned voff, unsigned lds_base) {   // the same with 4 bytes per lane
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_base), "v"(voff), "s"(sbase)
                 : "memory");
}

// The kernels here are compiled without IEEE mode, the device library with it, and a function is not inlined into one of the other
// mode: threadIdx, blockIdx and __umul24 would be calls, and all that follows from their results would count as divergent.  With the
// builtins: dense 32 heads x 32K tokens 7.03 -> 6.89 ms, x 2048 53.6 -> 51.4 us; block-sparse 32 x 32K in blocks of 16 689 -> 669, x 16K (16 blocks of 64)
// 368 -> 361, 2 x 32 x 64K (32 of 32) 2546 -> 2508.
__device__ __forceinline__ int thread_id() { return (int)__builtin_amdgcn_workitem_id_x(); }
__device__ __forceinline__ unsigned workgroup_id() { return __builtin_amdgcn_workgroup_id_x(); }
__device__ __forceinline__ unsigned mul24(unsigned x, unsigned y) { return (x & 0xffffffu) * (y & 0xffffffu); }   // one instruction

template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {   // into SGPRs; both halves unsigned, or the low one is sign-extended
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (const T*)(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ float half_max(float x) {      // max over lanes l and l^32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

}  // namespace

inline long long attn_bf16_kv_bytes(const Shape& sh) { return 4ll * sh.batch * sh.hkv * sh.n * kHeadDim; }

// Workgroups of `rows` query rows that a launch needs: a segment's last one may be short.
long long attn_bf16_row_tiles(const Shape& sh, bool sparse, int rows);

// Attention with 32-row workgroups whose waves split the keys, whether it is better here than the others, the waves, and the order of the workgroups.
bool attn_bf16_rows_better(const Shape& sh, bool sparse);
int attn_bf16_rows_waves(const Shape& sh, bool sparse);
TileOrder attn_bf16_rows_order(const Shape& sh, bool sparse, int waves);
hipError_t launch_attn_bf16_rows(const Shape& sh, ArgsB a, hipStream_t st);

// Attention over lists with 128-row workgroups, two to a compute unit, and whether it is better here than either.
bool attn_bf16_half_better(const Shape& sh);
hipError_t launch_attn_bf16_half(const Shape& sh, ArgsB a, hipStream_t st);

}  // namespace cp
