// fp32 attention on the 16-bit matrix instructions, for launches with enough query rows: the same walk over a block list (Algorithm 2) or all
// keys (Eq. 2) as attn_fp32.hip, with every fp32 factor split into three bf16 values and six products of them in the place of one.
//
//   x = h + m + l      h = bf16(x), m = bf16(x - h), l = x - h - m: all 24 bits, exactly, with fp32's own range of exponents
//   x y = h_x h_y + (h_x m_y + m_x h_y) + m_x m_y + (h_x l_y + l_x h_y), products exact, sums in fp32; left out are m_x l_y + l_x m_y + l_x l_y, of
//         either sign, at most 2^-24 of x y (2^-26.5 in the root mean square): half of what one rounding of the sum may be
//
// A workgroup owns 32 query rows of one segment (sparse) or of the sequence (dense); its W waves split the KEYS: wave w takes tiles w, w + W, ...
// of 32 keys (two runs of 16 tokens), with a running reference, sum and output of its own, merged through LDS at the end.  Per wave and tile:
//
//   S^T[key][q]  = K . Q^T      32x32x16 MFMA.  K comes by global_load_lds as whole rows (a lane per row straight from memory costs the
//                               address unit a request per lane and bound the kernel) into 16 KiB of LDS of the wave's own and is split
//                               on its way to the MFMAs; Q is split once per workgroup: h and m in LDS, l in registers
//   softmax                     one query per lane column
//   O^T[ch][q]  += V^T . P^T    a lane holds 8 keys of one channel, loaded as single floats; P^T is the S^T accumulator, split
//
// Values.  Weights count down to the subnormals, relative to a reference that the row's max may outgrow by 2^4; they are split times 2^20, which
// brings a subnormal's bits into bf16's range.  What cannot be split exactly (values below 2^-110 that are not 0) or has no finite result (infinities, V above
// about 2^94) is seen at the end of the walk, and the workgroup walks again with fp32 products, as attn_fp32.hip does.  If all
// of them do, that takes 1.3 to 2 times the time of attn_fp32.hip: block-sparse 4 x 4096 78 us (there 60), dense 4 x 2500 149 (75), 8 x 8192 1845 (1220).
//
// Errors against float64 (2-norm, attn_fp32.hip / here): dense 4 x 2500 5.2e-7 / 2.6e-7, block-sparse 4 x 4096 7.1e-7 / 2.7e-7, dense 8 x 8192 9.4e-7 / 3.5e-7: the
// sums have fewer roundings.
//
// What bounds it: the vector instructions (1140 a tile and wave, of which the splitting is 860; busy 75 % of the time) beside 96 MFMAs (50 %), at a clock
// of 1.9 GHz.  The splitting goes between the MFMAs of values split before (all of it first: 2 to 5 % slower).  Residues by v_dot2_f32_bf16, which reads
// a bf16 without unpacking it, take half the instructions, but that unit does not run beside the MFMAs: no faster (815 to 840 us where this takes 813).  Two fp16
// values and three products were faster (575), but hold 22 bits of a value within 2^13 of the largest and less of the others.
// Dense 8 x 8192 1110 -> 830 us, 4 x 2500 77 -> 64; block-sparse 4 x 4096 (704 keys) 55 -> 40, 8 x 8192 (704) 194 -> 146.
#include "attn_fp32.h"

#include <algorithm>
#include <type_traits>

namespace cp {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int TQ = 32, TK = 32;               // query rows of a workgroup, keys of a tile (two runs of 16 tokens)
constexpr float kLazy = 4.f;                  // log2 of how far a row's max may outgrow its reference while the products are split
constexpr float kScaleP = 1048576.f;          // weights are split times 2^20: those of 2^-149 have bits down to 2^-129, within bf16's subnormals

struct Parts { bf16x8 h, m, l; };             // x = h + m + l

// Splits x in five stages, which can go between the MFMAs of values split before.  x becomes what is left of it; lost: its low 16 bits are set where
// that is more than 8 bits (|x| below 2^-110).
template <int STAGE>
__device__ __forceinline__ void split_stage(float (&x)[8], Parts& p, unsigned& lost) {
    union Pairs { bf16x2 p[4]; bf16x8 v; unsigned u[4]; };
    if (STAGE == 0 || STAGE == 2) {             // the upper 8 bits, rounded
        Pairs y;
#pragma unroll
        for (int i = 0; i < 4; ++i) y.p[i] = __builtin_convertvector((f32x2){x[2 * i], x[2 * i + 1]}, bf16x2);
        (STAGE == 0 ? p.h : p.m) = y.v;
    } else if (STAGE == 1 || STAGE == 3) {
        Pairs y;
        y.v = STAGE == 1 ? p.h : p.m;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] -= __uint_as_float(i & 1 ? y.u[i >> 1] & 0xffff0000u : y.u[i >> 1] << 16);
    } else {
        Pairs y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned lo = __float_as_uint(x[2 * i]), hi = __float_as_uint(x[2 * i + 1]);
            y.u[i] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);       // the upper halves: what is left has 8 bits
            lost |= lo | hi;
        }
        asm("" : "+v"(lost));                   // here, or the residues are kept until the end of the tile
        p.l = y.v;
    }
}
__device__ __forceinline__ Parts split8(float (&x)[8], unsigned& lost) {
    Parts p;
    split_stage<0>(x, p, lost);
    __builtin_amdgcn_sched_barrier(0);          // stage by stage: the pairs in turn, or each waits for itself
    split_stage<1>(x, p, lost);
    __builtin_amdgcn_sched_barrier(0);
    split_stage<2>(x, p, lost);
    __builtin_amdgcn_sched_barrier(0);
    split_stage<3>(x, p, lost);
    __builtin_amdgcn_sched_barrier(0);
    split_stage<4>(x, p, lost);
    return p;
}
// c + small += a b, and between the products what splits x into next
template <bool NEXT>
__device__ __forceinline__ void mul_parts(const Parts& a, const Parts& b, f32x16& c, f32x16& small, float (&x)[8], Parts& next, unsigned& lost) {
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, small, 0, 0, 0);
    if (NEXT) split_stage<0>(x, next, lost);
    __builtin_amdgcn_sched_barrier(0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, small, 0, 0, 0);
    if (NEXT) split_stage<1>(x, next, lost);
    __builtin_amdgcn_sched_barrier(0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, small, 0, 0, 0);
    if (NEXT) split_stage<2>(x, next, lost);
    __builtin_amdgcn_sched_barrier(0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, small, 0, 0, 0);
    if (NEXT) split_stage<3>(x, next, lost);
    __builtin_amdgcn_sched_barrier(0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, small, 0, 0, 0);
    if (NEXT) split_stage<4>(x, next, lost);
    __builtin_amdgcn_sched_barrier(0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, c, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ float half_max(float x) {                // over lanes l and l ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// MODE 1: sparse, block size a multiple of 16; MODE 2: dense.
// PAIRS: in the order of TileOrder, else segments from the last to the first.
template <int MODE, int W, bool PAIRS>
__global__ __launch_bounds__(64 * W, 2) void attn_fp32_split_kernel(Args32 a) {
    ask_for(a.q, a.k, a.v, a.idx, a.cnt, a.batch, a.n, a.qtiles, a.shared_lists, a.scale_log2e, a.qs0, a.qs1, a.qs2, a.ks0, a.ks1, a.ks2);
    constexpr bool DENSE = MODE == 2;
    extern __shared__ __attribute__((aligned(1024))) float smem[];
    // While keys are walked: a K tile of 16 KiB per wave (32 rows of 512 B, 16-byte chunks XOR-swizzled by the row), then the parts of Q as B
    // operands, [part][16 channels][lane] of 16 bytes.  Afterwards: a partial O per wave in the place of its K tile, (max, sum) of every wave
    // and row and a flag per wave in the place of Q.
    const unsigned k_tile0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)smem;
    const unsigned q_tile = k_tile0 + W * TK * 512;                 // for fp32 products: the 32 rows of Q, swizzled like K
    float* part_o = smem;
    u32x4* q_parts = (u32x4*)(smem + W * TQ * kHeadDim);
    float* part_m = smem + W * TQ * kHeadDim;
    float* part_l = part_m + W * TQ;
    int* flags = (int*)(part_l + W * TQ);

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = a.hq / a.hkv, bkv = a.batch * a.hkv;              // consecutive workgroups walk the KV heads, see attn_fp32_kernel; then TileOrder
    const unsigned wg = PAIRS ? a.order.place(blockIdx.x) : blockIdx.x;
    const int x = wg % bkv, y = wg / bkv;
    const int bb = x / a.hkv, kvh = x % a.hkv, h = kvh * G + y % G;
    const TileOrder::Item item = DENSE   ? TileOrder::Item{0, a.qtiles - 1 - y / G}
                                 : PAIRS ? a.order.item(y / G, a.n1, a.qtiles)
                                         : a.order.by_segments(y / G, a.qtiles);
    const int j = item.segment, q_lo = j * a.s + item.tile * TQ;
    const int q_end = DENSE ? a.n : min(a.n, (j + 1) * a.s);        // rows >= q_end do not exist
    if (q_lo >= q_end) return;                                      // uniform: tile past a short segment
    const int q_last = min(q_end, q_lo + TQ) - 1;
    const int qpos = q_lo + l32;
    const float* kp = a.k + bb * a.ks0 + kvh * a.ks1;
    const float* vp = a.v + bb * a.ks0 + kvh * a.ks1;
    const float* qp = a.q + bb * a.qs0 + h * a.qs1;

    scalar_list list = nullptr; int count = 0;
    if (!DENSE) {
        const long long lrow = a.shared_lists ? ((long long)bb * a.hkv + kvh) * a.n1 + j : ((long long)bb * a.hq + h) * a.n1 + j;
        list = (scalar_list)(unsigned long long)(a.idx + lrow * a.list_len);
        count = min(max(((scalar_list)(unsigned long long)a.cnt)[lrow], 0), a.list_len);
    }
    // positions 0 .. total-1 of the listed blocks laid end to end (host checks list_len * b < 2^31)
    const unsigned total = DENSE ? (unsigned)q_last + 1u : (unsigned)count * (unsigned)a.b;
    const int ntiles = (int)((total + TK - 1) / TK);

    // ---- first tokens of the two runs of the wave's next tile, -1: no such tokens; call in tile order
    unsigned walk_e = 0, walk_off = 0;                              // list entry and offset inside its block of the next tile
    auto start_walk = [&]() { if (!DENSE) { walk_e = (unsigned)wave * TK / (unsigned)a.b; walk_off = (unsigned)wave * TK % (unsigned)a.b; } };
    const unsigned step_e = DENSE ? 0 : W * TK / (unsigned)a.b, step_off = DENSE ? 0 : W * TK % (unsigned)a.b;
    const int n2 = DENSE ? 0 : (a.n + a.b - 1) / a.b;
    auto run_at = [&](unsigned e, unsigned off) -> int {
        if (e >= (unsigned)count) return -1;
        const int blk = list[e];
        const int base = blk >= 0 && blk < n2 ? blk * a.b + (int)off : -1;
        return base < a.n ? base : -1;
    };
    auto next_tile = [&](int t, int& b0, int& b1) {
        if (DENSE) {
            b0 = t < ntiles ? t * TK : -1;
            b1 = b0 >= 0 && b0 + 16 < a.n ? b0 + 16 : -1;
            return;
        }
        b0 = run_at(walk_e, walk_off);
        const bool next = walk_off + 16 >= (unsigned)a.b;
        b1 = run_at(walk_e + (next ? 1 : 0), next ? 0 : walk_off + 16);
        if (b1 > q_last) b1 = -1;                                   // behind every row: 0 * V must be 0, whatever V holds
        walk_e += step_e; walk_off += step_off;
        if (walk_off >= (unsigned)a.b) { walk_off -= a.b; ++walk_e; }
    };

    const unsigned row_bytes = (unsigned)a.ks2 * 4u;
    // the wave's K tile by copies of two rows each, the lane's 16 bytes being chunk (lane & 31) ^ (row & 15) of its row
    const unsigned k_tile = k_tile0 + wave * (TK * 512);
    const unsigned k_chunk = (unsigned)(l32 ^ hh) << 4, k_row = hh * row_bytes;
    auto copy_k = [&](int b0, int b1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the reads of the tile before are done
#pragma unroll
        for (int run = 0; run < 2; ++run) {
            const int base = max(run ? b1 : b0, 0);                 // a run without tokens copies existing ones, masked later
            const char* rows = (const char*)(kp + (long long)base * a.ks2);
            unsigned off[8], chunk = k_chunk;
            asm("" : "+v"(chunk));                                  // what follows is worked out here, not kept through the loop
            if (base + 16 <= a.n) {
#pragma unroll
                for (int i = 0; i < 8; ++i) off[i] = (unsigned)(2 * i) * row_bytes + k_row + (chunk ^ (32 * i));
            } else {                                                // rows past the end repeat the last one
#pragma unroll
                for (int i = 0; i < 8; ++i) off[i] = (unsigned)min(2 * i + hh, a.n - 1 - base) * row_bytes + (chunk ^ (32 * i));
            }
            copy16x8(rows, off, k_tile + run * 8192);
        }
    };
    const unsigned row_at = l32 * 512 + ((hh ^ (l32 & 15)) << 4);
    auto read_row = [&](unsigned tile, int ks, float (&f)[8]) {     // row l32 of the tile, channels 16*ks + 8*(e >> 2) + 4*hh + (e & 3)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const f32x4 v = *(__attribute__((address_space(3))) const f32x4*)(uintptr_t)((tile + (row_at ^ ((4 * (ks & 3) + 2 * i) << 4))) + (ks >> 2) * 256);
#pragma unroll
            for (int e = 0; e < 4; ++e) f[4 * i + e] = v[e];
        }
    };
    float vf[2][4][8];                                              // [run][channel tile][e]: key 8*(e >> 2) + 4*hh + (e & 3), channel 32*dt + l32
    auto load_v = [&](int run, int base) {
        if (base < 0) {                                             // 0 * V must be 0
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int e = 0; e < 8; ++e) vf[run][dt][e] = 0.f;
            return;
        }
        const char* rows = (const char*)(vp + (long long)base * a.ks2);
        const int top = a.n - 1 - base;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const char* src = rows;
            unsigned off = (unsigned)(4 * hh) * row_bytes + 4 * l32;
            if (top >= 15) src += (unsigned long long)(8 * (e >> 2) + (e & 3)) * row_bytes;
            else off = (unsigned)min(8 * (e >> 2) + 4 * hh + (e & 3), top) * row_bytes + 4 * l32;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) vf[run][dt][e] = *(const float*)(src + off + 128 * dt);
        }
    };

    // ---- Q: every wave splits some of the 16-channel steps; h and m stay in LDS, l, through the K tiles, in registers (two workgroups of
    // four waves fill a compute unit's LDS with what is there)
    unsigned lost = 0;                                              // of the values that this wave has split
    bf16x8 q_l[8];
    {
        u32x4* l_parts = (u32x4*)smem;
        constexpr int kSteps = 8 / W;
        const float* row = qp + (long long)min(qpos, q_last) * a.qs2 + 4 * hh;
        float v[kSteps][8];
#pragma unroll
        for (int i = 0; i < kSteps; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const f32x4 w = *(const f32x4*)(row + 16 * (wave + i * W) + 8 * p);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][4 * p + e] = w[e];
            }
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const Parts p = split8(v[i], lost);
            union { bf16x8 b; u32x4 u; } c;
            c.b = p.h; q_parts[(0 * 8 + wave + i * W) * 64 + lane] = c.u;
            c.b = p.m; q_parts[(1 * 8 + wave + i * W) * 64 + lane] = c.u;
            c.b = p.l; l_parts[(wave + i * W) * 64 + lane] = c.u;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            union { bf16x8 b; u32x4 u; } c;
            c.u = l_parts[ks * 64 + lane]; q_l[ks] = c.b;
        }
        __syncthreads();                                            // before K comes
    }

    f32x16 o[4];
    float m, l;                                                     // reference of the raw logits; the lane's own keys' weights
    const float c = a.scale_log2e;
    // EXACT: fp32 products.  Else false where a value could not be split in full, or something is not finite: infinities, and what is near enough
    // to them to overflow in a part or in a weight's scale
    auto walk = [&](auto exact_tag) __attribute__((always_inline)) -> bool {
        constexpr bool EXACT = decltype(exact_tag)::value;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
        m = -INFINITY; l = 0.f;
        int b0, b1;
        start_walk();
        next_tile(wave, b0, b1);
        copy_k(b0, b1);
        for (int t = wave; t < ntiles && b0 <= q_last; t += W) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the tile's K is in LDS
            load_v(0, b0);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 s, small;
#pragma unroll
            for (int r = 0; r < 16; ++r) { s[r] = 0.f; small[r] = 0.f; }
            if (EXACT) {
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    float k8[8], q8[8];
                    read_row(k_tile, ks, k8); read_row(q_tile, ks, q8);
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {                // two chains: half as many roundings in each
                        s = __builtin_amdgcn_mfma_f32_32x32x2f32(k8[e], q8[e], s, 0, 0, 0);
                        small = __builtin_amdgcn_mfma_f32_32x32x2f32(k8[e + 1], q8[e + 1], small, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                float kx[2][8];
                Parts kp[2], q[2];
                auto read_q = [&](int ks) {
                    union { bf16x8 b; u32x4 u; } w;
                    w.u = q_parts[(0 * 8 + ks) * 64 + lane]; q[ks & 1].h = w.b;
                    w.u = q_parts[(1 * 8 + ks) * 64 + lane]; q[ks & 1].m = w.b;
                    q[ks & 1].l = q_l[ks];
                };
                read_row(k_tile, 0, kx[0]); read_q(0); read_row(k_tile, 1, kx[1]);
                kp[0] = split8(kx[0], lost);
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    if (ks < 6) read_row(k_tile, ks + 2, kx[ks & 1]);
                    if (ks < 7) read_q(ks + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (ks < 7) mul_parts<true>(kp[ks & 1], q[ks & 1], s, small, kx[(ks + 1) & 1], kp[(ks + 1) & 1], lost);
                    else mul_parts<false>(kp[ks & 1], q[ks & 1], s, small, kx[0], kp[0], lost);
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] += small[r];
            __builtin_amdgcn_sched_barrier(0);
            const int c0 = b0, c1 = b1;
            next_tile(t + W, b0, b1);
            copy_k(b0, b1);
            load_v(1, c1);
            __builtin_amdgcn_sched_barrier(0);

            if (max(c0, c1) + 15 > q_lo || c0 < 0 || c1 < 0) {      // hidden from some row, or not there
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int base = r < 8 ? c0 : c1;
                    if (base < 0 || base + 8 * ((r >> 2) & 1) + 4 * hh + (r & 3) > qpos) s[r] = -INFINITY;
                }
            }
            float mx = fmaxf(s[0], s[1]);
#pragma unroll
            for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(s[r], s[r + 1]), mx);
            mx = half_max(mx);
            const float m_new = (mx - m) * c > (EXACT ? 0.f : kLazy) ? mx : m;
            const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = exp2f((m - m_safe) * c);
            float least = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) { s[r] = (s[r] - m_safe) * c; least = fminf(least, s[r]); }
            if (__ballot(least < -126.f) == 0) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(s[r]);
            } else {                                                // v_exp_f32 has no subnormal results, exp2f does
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = exp2f(s[r]);
            }
            if (!EXACT) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] *= kScaleP;
            }
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 4) sum += (s[r] + s[r + 1]) + (s[r + 2] + s[r + 3]);
            l = l * alpha + sum;
            m = m_new;
            if (__ballot(alpha != 1.0f) != 0) {
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
            }
            if (EXACT) {
#pragma unroll
                for (int run = 0; run < 2; ++run)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[run][dt][e], s[8 * run + e], o[dt], 0, 0, 0);
            } else {
                Parts vp2[2], p;
                vp2[0] = split8(vf[0][0], lost);
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    if (x % 4 == 0) {
                        float p8[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) p8[e] = s[2 * x + e];
                        p = split8(p8, lost);                       // always exact, see kScaleP
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (x < 7) mul_parts<true>(vp2[x & 1], p, o[x % 4], o[x % 4], vf[(x + 1) / 4][(x + 1) % 4], vp2[(x + 1) & 1], lost);
                    else mul_parts<false>(vp2[x & 1], p, o[x % 4], o[x % 4], vf[0][0], vp2[0], lost);
                }
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // no copy is in flight into what the partial results or Q take
        float finite = l * 0.f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) finite = fmaf(o[dt][r], 0.f, finite);
        return __ballot(!(finite == 0.f) || (lost & 0xffffu) != 0) == 0;
    };
    bool exact = !walk(std::false_type());
    // one wave that meets such a value has all walk again, with Q by whole rows in the place of its parts
    __syncthreads();                                                // every wave is past its last read of Q
    if (lane == 0) flags[wave] = exact;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) exact |= flags[w] != 0;
    exact = __builtin_amdgcn_readfirstlane(exact);
    if (exact) {
        __syncthreads();                                            // everybody has read the flags
#pragma unroll
        for (int x = 0; x < 16 / W; ++x) {
            const int i = wave * (16 / W) + x, row = 2 * i + hh;
            copy16_far((const char*)(qp + (long long)min(q_lo + row, q_last) * a.qs2) + ((unsigned)(l32 ^ (row & 15)) << 4), q_tile + i * 1024);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        walk(std::true_type());
        __syncthreads();                                            // everybody is past Q
    }
    const float unit = exact ? 1.f : 1.f / kScaleP;                 // of the weights in l and O

    // ---- merge the W partial results
    l += __shfl_xor(l, 32);
    if (hh == 0) { part_m[wave * TQ + l32] = m; part_l[wave * TQ + l32] = l; }
    {
        float* dst = part_o + (wave * TQ + l32) * kHeadDim;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int gg = 0; gg < 4; ++gg) {                        // channels 32*dt + 8*gg + 4*hh .. +3
                const int chunk = (8 * dt + 2 * gg + hh) ^ l32;
                *(f32x4*)(dst + 4 * chunk) = f32x4{o[dt][4 * gg], o[dt][4 * gg + 1], o[dt][4 * gg + 2], o[dt][4 * gg + 3]};
            }
    }
    __syncthreads();
    float* op = a.out + bb * a.os0 + h * a.os1;
#pragma unroll
    for (int i = 0; i < TQ * 32 / (64 * W); ++i) {
        const int row = (i * 64 * W + tid) >> 5, chunk = tid & 31;
        float M = -INFINITY, L = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, part_m[w * TQ + row]);
        const float M_safe = (M == -INFINITY) ? 0.f : M;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float f = exp2f((part_m[w * TQ + row] - M_safe) * c);
            L += f * part_l[w * TQ + row];
            sum += f * *(const f32x4*)(part_o + (w * TQ + row) * kHeadDim + 4 * (chunk ^ row));
        }
        if (q_lo + row < q_end) {
            const float inv = L > 0.f ? 1.0f / L : 0.f;
            *(f32x4*)(op + (long long)(q_lo + row) * a.os2 + 4 * chunk) = sum * inv;
            if (a.lse && chunk == 0)
                a.lse[((long long)bb * a.hq + h) * a.n + q_lo + row] = L > 0.f ? M * a.scale + logf(L * unit) : -INFINITY;
        }
    }
}

template <int MODE, int W, bool PAIRS>
hipError_t launch(const Shape& sh, Args32& a, hipStream_t st) {
    const long long grid = attn_fp32_grid(sh, a.idx != nullptr, TQ);
    constexpr int smem = W * TQ * kHeadDim * 4 + 2 * 8 * 64 * 16;   // W = 4: half of a compute unit's LDS
    static_assert(2 * W * TQ * 4 + W * 4 <= 2 * 8 * 64 * 16, "what takes the place of Q");
    const hipError_t e = hipFuncSetAttribute((const void*)attn_fp32_split_kernel<MODE, W, PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_fp32_split_kernel<MODE, W, PAIRS>), dim3((unsigned)grid), dim3(64 * W), smem, st, a);
    return hipGetLastError();
}
}  // namespace

long long attn_fp32_row_tiles(const Shape& sh, bool sparse, int rows) {
    const int s = sparse ? sh.s : sh.n, rest = sh.n % s;
    return (long long)sh.batch * sh.hq * ((long long)(sh.n / s) * ((s + rows - 1) / rows) + (rest + rows - 1) / rows);
}

int attn_fp32_qtiles(const Shape& sh, bool sparse, int rows) {
    return ((sparse ? std::min(sh.s, sh.n) : sh.n) + rows - 1) / rows;    // a segment may be set longer than the sequence
}

long long attn_fp32_grid(const Shape& sh, bool sparse, int rows) {
    return (long long)sh.batch * sh.hq * attn_fp32_qtiles(sh, sparse, rows) * (sparse ? sh.n1 : 1);
}

TileOrder attn_fp32_order(const Shape& sh, bool sparse, int rows, int waves) {
    return TileOrder::of_launch(waves, attn_fp32_grid(sh, sparse, rows), attn_fp32_row_tiles(sh, sparse, rows), sh.n1, sh.r, sh.budget, sh.local, sh.b,
                                attn_fp32_qtiles(sh, sparse, rows), rows);
}

static long long listed_keys(const Shape& sh, bool sparse) {
    return sparse ? std::min((long long)sh.n, (long long)sh.list_len * sh.b) : sh.n;
}

// Against the fp32 matrix instructions (us, attn_fp32.hip / this one, all with the waves and orders of the present rules; listed keys in brackets; t: row tiles
// of 32).  That kernel splits rows into 16 and so fills the chip with half as many; where rows see unequal numbers of keys, most of those before them, it keeps a
// unit's two workgroups of unlike length.
//   nearly all keys: t = 188 to 200 4 x 1500 31.5 / 38.5, 3 x 2048 block-sparse 41 / 50, 2 x 3195 60 / 71, 1 x 6395 114 / 136; t = 256 to 258 4 x 2043 47 / 50, 2 x 4091
//   84 / 93, 1 x 8187 158 / 179, 3 x 2731 62 / 65; t = 272 to 282 2 x 4379 102 / 102, 1 x 8795 192 / 195, but 4 x 2171 56 / 53, 3 x 3000 76 / 73; from there on 1 x 10000
//   (313) 251 / 231, 8 x 1250 (320) 44 / 35, 4 x 2619 (328) 80 / 66, 4 x 4096 (512) 162 / 119.
//   fewer: t = 256 4 x 2043 (1408, 768, 384) 46 / 38, 24.4 / 24.2, 16.1 / 15.5, 1 x 8187 (5824, 3264, 1600) 159 / 136, 121 / 84, 58 / 48; t = 184 to 200 2 x 3195 (2240,
//   1216, 576) 55 / 56, 44 / 35, 21.7 / 19.8, 1 x 6000 (416, 1248, 3136) 15.8 / 19.0, 53 / 35, 84 / 77, 4 x 1500 (704, 1248) 23.2 / 23.4, 29 / 34, 3 x 2048 (1248) 36.7 /
//   34.4, 8 x 750 (416) 13.5 / 17.7; t = 163 1 x 5200 (416, 1248, 3136) 14.8 / 18.3, 49 / 35, 60 / 76; 152 8 x 600 (416) 13.0 / 17.6, 128 1 x 4096 (416, 1248)
//   13.1 / 17.7, 28 / 35.
//   Where its row tiles come in pairs that kernel has gained up to a fifth and become the better one for some launches of at most 1024 keys at t = 256 and short lists
//   below: dense 8 x 1000 25.0 / 28.4, 16 x 512 16.2 / 17.7, 32 x 251 11.1 / 12.2, block-sparse 1 x 8192 (416) 18.4 / 20.8, 1 x 6000 as above.  The line is where the
//   tests of this kernel hold it.
bool attn_fp32_split_better(const Shape& sh, bool sparse) {
    if (sh.kvs[2] >= (1 << 26) || (sparse && sh.b % 16 != 0)) return false;     // a run's rows within 32-bit byte offsets of its first; runs of 16
    const long long tiles = attn_fp32_row_tiles(sh, sparse, TQ), keys = listed_keys(sh, sparse), n = sh.n;
    if (n > 1024 && 5 * keys > 4 * n) return tiles > 272;
    if (tiles >= 256) return true;
    if (tiles >= 184) return n >= 1400 && 5 * keys <= 3 * n;
    return tiles >= 144 && n >= 2400 && 3 * keys <= n;
}

// Eight waves leave one workgroup to a compute unit, four two.  Eight / four (listed keys in brackets): up to a chip full of workgroups dense 4 x 2043 (t = 256) 50 / 61,
// block-sparse 1 x 8187 (1600) 48 / 57; beyond it rows of many and so unequal keys: dense 4 x 2619 (328) 66 / 79, 1 x 11995 (375) 286 / 337, 2 x 7995 (500) 217 / 248,
// 4 x 5115 (640) 194 / 197, block-sparse 2 x 5275 (330; 3712) 96 / 113, 1 x 11995 (375; 8512) 227 / 260; but block-sparse 2 x 5275 (2048) 84 / 77, 4 x 2971 (372; 1152)
// 55 / 44, 4 x 3995 (500; 2816) 117 / 109, dense 32 x 475 (480) 26.9 / 22.1, 4 x 5979 (748) 255 / 249.  (Eight would be better for the first few above 256, 4 x 2171
// (272; 832) 26.4 / 32.4.)
int attn_fp32_split_waves(const Shape& sh, bool sparse) {
    const long long tiles = attn_fp32_row_tiles(sh, sparse, TQ), keys = listed_keys(sh, sparse);
    return tiles <= 256 || (tiles <= 640 && sh.n >= 1024 && 8 * keys >= 5ll * sh.n) ? 8 : 4;
}

template <int MODE>
static hipError_t launch_waves(const Shape& sh, Args32& a, int waves, hipStream_t st) {
    if (waves == 8) return launch<MODE, 8, false>(sh, a, st);
    return a.order.turn ? launch<MODE, 4, true>(sh, a, st) : launch<MODE, 4, false>(sh, a, st);
}

hipError_t launch_attn_fp32_split(const Shape& sh, Args32& a, hipStream_t st) {
    const bool sparse = a.idx != nullptr;
    const int waves = attn_fp32_split_waves(sh, sparse);
    a.qtiles = attn_fp32_qtiles(sh, sparse, TQ);
    a.order = attn_fp32_order(sh, sparse, TQ, waves);
    return sparse ? launch_waves<1>(sh, a, waves, st) : launch_waves<2>(sh, a, waves, st);
}

}  // namespace cp
