// fp32 attention on the 16-bit matrix instructions, for launches with enough query rows: the same walk over a block list (Algorithm 2) or all
// keys (Eq. 2) as attn_fp32.hip, with every fp32 factor split into two fp16 values and three products of them in the place of one.
//
//   x * 2^e = h + l + r    h = fp16(x * 2^e), l = fp16(x * 2^e - h), |r| <= 2^-24 |x * 2^e| or 2^-25: what fp32 itself rounds away
//   x y 2^(e+f) = h_x h_y + h_x l_y + l_x h_y, products exact in fp32, sums in fp32; l_x l_y is left out (at most 2^-22, 2^-24 on average)
//
// A workgroup owns 32 query rows of one segment (sparse) or of the sequence (dense); its W waves split the KEYS: wave w takes tiles w, w + W, ...
// of 32 keys (two runs of 16 tokens), with a running reference, sum and output of its own, merged through LDS at the end.  Per wave and tile:
//
//   S^T[key][q]  = K . Q^T      32x32x16 MFMA.  K comes by global_load_lds as whole rows (a lane per row straight from memory costs the
//                               address unit a request per lane and bound the kernel) into 16 KiB of LDS of the wave's own and is split
//                               on its way to the MFMAs; Q is split once per workgroup and read from LDS
//   softmax                     one query per lane column
//   O^T[ch][q]  += V^T . P^T    a lane holds 8 keys of one channel, loaded as single floats; P^T is the S^T accumulator, split
//
// Scales and ranges.  Powers of two: one for Q, one each for the wave's K and V so far, set so that the largest value lies at 2^12..2^13 and
// set anew (O follows) where one reaches 2^15.  Every lane's largest Q, K and V must be at least 1/2 after scaling, or zero, so that l
// keeps its bits: the range of magnitudes in which all of a wave's rows and channels have to lie is 2^13 to 2^16.  Weights are relative to a reference that
// the row's max may outgrow by 2^4 and are split times 2^11: they are known to 2^-36 of the largest.  Where a value does not fit (infinities,
// rows that are 2^13 times smaller than others, Q or K above 2^72, V above 2^104) the workgroup walks again with fp32 products, weights relative to the
// true max and down to the subnormals, as attn_fp32.hip does.
//
// Errors against float64 (2-norm, attn_fp32.hip / here): dense 4 x 2500 5.2e-7 / 3.5e-7, block-sparse 4 x 4096 7.1e-7 / 3.6e-7, unit-scale logits 1.0e-7 /
// 0.9e-7, a channel of K 50 times the others 1.8e-6 / 8.2e-7.
//
// What bounds it: with 8 waves on a compute unit, one after another the vector instructions (750 a tile and wave, of which the splitting is 440), the MFMAs (48)
// and the caches: 32 rows read their keys anew, 32 KiB a tile, at 14 TB/s of L2 for 8 heads x 8192 tokens.  The matrix pipe is busy 31 % of the time, the
// vector unit 66 %, and the two hardly overlap.  Dense 8 x 8192 1090 -> 607 us, 4 x 2500 78 -> 54; block-sparse 4 x 4096 (704 keys) 57 -> 41.  On the way: K straight
// from memory as A operands 678 (dense 8 x 8192, with 4 products 723), products l_x l_y too 8 % slower and no more exact, scales left out 0 to 2 % faster, the
// largest values left out 3 %, residues by a conversion and an fma instead of v_fma_mix 5 % slower.
#include "attn_fp32.h"

#include <algorithm>
#include <type_traits>

namespace cp {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int TQ = 32, TK = 32;               // query rows of a workgroup, keys of a tile (two runs of 16 tokens)
constexpr float kTop = 32768.f, kBottom = 0.5f;    // scaled values: the largest of a lane is inside, or 0
constexpr int kFit = 12;                      // a scale is set to bring the largest value to 2^12 .. 2^13
constexpr int kMaxScale = 60;                 // log2 of the scales of Q and K: -60 .. 60, so that a product's is within fp32
constexpr int kLeastScaleV = -92, kMaxScaleV = 100;    // V up to 2^104: O, at most 2^kLazy * keys * |V|, stays within fp32
constexpr float kLazy = 4.f;                  // log2 of how far a row's max may outgrow its reference while the products are split
constexpr int kScaleP = 11;                   // weights, up to 2^kLazy, are split times 2^11

struct Parts { f16x8 h, l; };                 // x * scale = h + l, each rounded to nearest

__device__ __forceinline__ float pow2(int e) { return __uint_as_float((unsigned)(127 + e) << 23); }
__device__ __forceinline__ Parts split8(const float (&x)[8], float scale) {
    Parts p;
    f16x2 h[4]; float r[8], y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = x[i] * scale;
    __builtin_amdgcn_sched_barrier(0);          // stage by stage: the four pairs in turn, or each waits for itself
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = __builtin_convertvector((f32x2){y[2 * i], y[2 * i + 1]}, f16x2);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = fmaf(x[i], scale, -(float)h[i >> 1][i & 1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f16x2 l = __builtin_convertvector((f32x2){r[2 * i], r[2 * i + 1]}, f16x2);
        p.h[2 * i] = h[i][0]; p.h[2 * i + 1] = h[i][1]; p.l[2 * i] = l[0]; p.l[2 * i + 1] = l[1];
    }
    return p;
}
__device__ __forceinline__ void mul_parts(const Parts& a, const Parts& b, f32x16& c, f32x16& small) {
    small = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.l, b.h, small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h, b.l, small, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h, b.h, c, 0, 0, 0);
}
// A scale 2^e for values whose largest per lane is `most`: kept while all of them fit, else set anew from the wave's largest.  False: some
// lane's values, these or earlier ones (low: the least of their maxima), are too small beside the largest, or nothing fits them.
__device__ __forceinline__ bool fit(float most, int least, int max, int& e, float& low) {
    if (__ballot(!(most * pow2(e) < kTop)) != 0) {
        float top = most;
        for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
        e = __builtin_amdgcn_readfirstlane(127 + kFit - (int)(__float_as_uint(top) >> 23));
        if (e < least || e > max) { e = 0; return false; }
    }
    low = fminf(low, most > 0.f ? most : INFINITY);
    return __ballot(low * pow2(e) < kBottom) == 0;
}
__device__ __forceinline__ float half_max(float x) {                // over lanes l and l ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// MODE 1: sparse, block size a multiple of 16; MODE 2: dense.
template <int MODE, int W>
__global__ __launch_bounds__(64 * W, 2) void attn_fp32_split_kernel(Args32 a) {
    constexpr bool DENSE = MODE == 2;
    extern __shared__ __attribute__((aligned(1024))) float smem[];
    // While keys are walked: a K tile of 16 KiB per wave (32 rows of 512 B, 16-byte chunks XOR-swizzled by the row), then the parts of Q as B
    // operands, [part][16 channels][lane] of 16 bytes.  Afterwards: a partial O per wave in the place of its K tile, (max, sum) of every wave
    // and row and a flag per wave in the place of Q.
    const unsigned k_tile0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)smem;
    float* part_o = smem;
    u32x4* q_parts = (u32x4*)(smem + W * TQ * kHeadDim);
    float* part_m = smem + W * TQ * kHeadDim;
    float* part_l = part_m + W * TQ;
    int* flags = (int*)(part_l + W * TQ);

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = a.hq / a.hkv, bkv = a.batch * a.hkv;              // order of the workgroups: see attn_fp32_kernel
    const int x = blockIdx.x % bkv, y = blockIdx.x / bkv;
    const int bb = x / a.hkv, kvh = x % a.hkv, h = kvh * G + y % G;
    const int item = (DENSE ? a.qtiles : a.n1 * a.qtiles) - 1 - y / G;
    const int j = DENSE ? 0 : item / a.qtiles;
    const int q_lo = DENSE ? item * TQ : j * a.s + item % a.qtiles * TQ;
    const int q_end = DENSE ? a.n : min(a.n, (j + 1) * a.s);        // rows >= q_end do not exist
    if (q_lo >= q_end) return;                                      // uniform: tile past a short segment
    const int q_last = min(q_end, q_lo + TQ) - 1;
    const int qpos = q_lo + l32;
    const float* kp = a.k + bb * a.ks0 + kvh * a.ks1;
    const float* vp = a.v + bb * a.ks0 + kvh * a.ks1;
    const float* qrow = a.q + bb * a.qs0 + h * a.qs1 + (long long)min(qpos, q_last) * a.qs2 + 4 * hh;

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
        walk_e += step_e; walk_off += step_off;
        if (walk_off >= (unsigned)a.b) { walk_off -= a.b; ++walk_e; }
    };

    const unsigned row_bytes = (unsigned)a.ks2 * 4u;
    // the wave's K tile by copies of two rows each, the lane's 16 bytes being chunk (lane & 31) ^ (row & 15) of its row
    const unsigned k_tile = k_tile0 + wave * (TK * 512);
    const unsigned k_chunk = (unsigned)(l32 ^ hh) << 4, k_row = hh * row_bytes;
    unsigned run_off[8];                                            // byte offsets of the lane's pieces of a run
#pragma unroll
    for (int i = 0; i < 8; ++i) run_off[i] = (unsigned)(2 * i) * row_bytes + k_row + (k_chunk ^ (32 * i));
    auto copy_k = [&](int b0, int b1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the reads of the tile before are done
#pragma unroll
        for (int run = 0; run < 2; ++run) {
            const int base = run ? b1 : b0;
            if (base >= 0 && base + 16 <= a.n) {
                const char* rows = (const char*)(kp + (long long)base * a.ks2);
                copy16x8(rows, run_off, k_tile + run * 8192);
            } else {                                                // rows without a token copy an existing one, masked later
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int tok = min(max(base, 0) + 2 * i + hh, a.n - 1);
                    copy16_far((const char*)kp + (unsigned long long)(unsigned)tok * row_bytes + (k_chunk ^ (32 * i)), k_tile + run * 8192 + i * 1024);
                }
            }
        }
    };
    auto read_k = [&](int ks, float (&f)[8]) {                      // row l32 of the tile, channels 16*ks + 8*(e >> 2) + 4*hh + (e & 3)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const f32x4 v = *(__attribute__((address_space(3))) const f32x4*)(uintptr_t)(k_tile + l32 * 512 + (((4 * ks + 2 * i + hh) ^ (l32 & 15)) << 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) f[4 * i + e] = v[e];
        }
    };
    float kf[8][8];                                                 // row l32 of the tile, channels 16*ks + 8*(e >> 2) + 4*hh + (e & 3)
    auto load_k = [&](int b0, int b1) {                             // rows without a token read an existing one, masked later
        const int base = max(l32 < 16 ? b0 : b1, 0), tok = min(base + (l32 & 15), a.n - 1);
        const char* src = (const char*)kp + (unsigned long long)(unsigned)tok * row_bytes + 16 * hh;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const f32x4 v = *(const f32x4*)(src + 32 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e) kf[i >> 1][4 * (i & 1) + e] = v[e];
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

    // ---- Q: every wave splits some of the 16-channel steps, by one scale
    float* tops = part_m;                                           // largest and least row maximum of every wave's steps
    int eq = kMaxScale;
    bool exact;                                                     // workgroup-uniform: products of unsplit values
    {
        constexpr int kSteps = 8 / W > 0 ? 8 / W : 1;
        float v[kSteps][8], most = 0.f;
#pragma unroll
        for (int i = 0; i < kSteps; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const f32x4 w = *(const f32x4*)(qrow + 16 * (wave + i * W) + 8 * p);
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[i][4 * p + e] = w[e]; most = fmaxf(most, fabsf(w[e])); }
            }
        tops[tid] = most;                                           // [wave][lane]: rows l32, halves hh
        __syncthreads();
        float row = 0.f;                                            // of the lane's row and half over all steps
#pragma unroll
        for (int w = 0; w < W; ++w) row = fmaxf(row, tops[w * 64 + lane]);
        __syncthreads();                                            // Q's parts take their place
        float low = INFINITY;
        exact = !fit(row, -kMaxScale, kMaxScale, eq, low);
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const Parts p = split8(v[i], pow2(eq));
            union { f16x8 b; u32x4 u; } c;
            c.b = p.h; q_parts[(0 * 8 + wave + i * W) * 64 + lane] = c.u;
            c.b = p.l; q_parts[(1 * 8 + wave + i * W) * 64 + lane] = c.u;
        }
        __syncthreads();
    }

    f32x16 o[4];
    float m, l;                                                     // reference of the raw logits; the lane's own keys' weights
    const float c = a.scale_log2e;
    auto walk = [&](auto exact_tag) __attribute__((always_inline)) -> bool {
        constexpr bool EXACT = decltype(exact_tag)::value;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
        m = -INFINITY; l = 0.f;
        int ek = kMaxScale, ev = kMaxScaleV;                        // log2 of the scales of K and V
        float low_k = INFINITY, low_v = INFINITY;
        int b0, b1;
        start_walk();
        next_tile(wave, b0, b1);
        if (EXACT) load_k(b0, b1); else copy_k(b0, b1);
        for (int t = wave; t < ntiles && b0 <= q_last; t += W) {
            if (!EXACT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the tile's K is in LDS
            load_v(0, b0);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 s, small;
            if (EXACT) {
#pragma unroll
                for (int r = 0; r < 16; ++r) { s[r] = 0.f; small[r] = 0.f; }
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const f32x4 w = *(const f32x4*)(qrow + 16 * ks + 8 * i);
#pragma unroll
                        for (int e = 0; e < 4; e += 2) {            // two chains: half as many roundings in each
                            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[ks][4 * i + e], w[e], s, 0, 0, 0);
                            small = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[ks][4 * i + e + 1], w[e + 1], small, 0, 0, 0);
                        }
                    }
            } else {
                int tried;
                do {                                                // a second time where the tile asks for another scale
                    tried = ek;
                    const float scale = pow2(ek);
                    float most = 0.f, kn[8];
                    Parts qn;
                    auto read_q = [&](int ks) {
                        union { f16x8 b; u32x4 u; } w;
                        w.u = q_parts[(0 * 8 + ks) * 64 + lane]; qn.h = w.b;
                        w.u = q_parts[(1 * 8 + ks) * 64 + lane]; qn.l = w.b;
                    };
#pragma unroll
                    for (int r = 0; r < 16; ++r) { s[r] = 0.f; small[r] = 0.f; }
                    read_k(0, kn); read_q(0);
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        float kc[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) kc[e] = kn[e];
                        const Parts q = qn;
                        if (ks < 7) { read_k(ks + 1, kn); read_q(ks + 1); }
#pragma unroll
                        for (int e = 0; e < 8; e += 2) most = fmaxf(fmaxf(fabsf(kc[e]), fabsf(kc[e + 1])), most);
                        mul_parts(split8(kc, scale), q, s, small);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (!fit(most, -kMaxScale, kMaxScale, ek, low_k)) return false;
                } while (ek != tried);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] += small[r];
            __builtin_amdgcn_sched_barrier(0);
            const int c0 = b0, c1 = b1;
            next_tile(t + W, b0, b1);
            if (!EXACT) copy_k(b0, b1);
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
            const float unit = EXACT ? 1.f : pow2(-ek - eq);        // of the logits in s
            mx = half_max(mx) * unit;
            const float m_new = (mx - m) * c > (EXACT ? 0.f : kLazy) ? mx : m;
            const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
            float alpha = (m - m_safe) * c;
            if (EXACT) {                                            // weights count down to the smallest subnormal: v_exp_f32 has none
                alpha = exp2f(alpha);
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = exp2f((s[r] - m_safe) * c);
            } else {
                alpha = __builtin_amdgcn_exp2f(alpha);
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], unit, -m_safe) * c);
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
#pragma unroll
            for (int run = 0; run < 2; ++run) {
                if (EXACT) {
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[run][dt][e], s[8 * run + e], o[dt], 0, 0, 0);
                } else {
                    float p8[8], most = 0.f;
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                        for (int e = 0; e < 8; e += 2) most = fmaxf(fmaxf(fabsf(vf[run][dt][e]), fabsf(vf[run][dt][e + 1])), most);
                    const int before = ev;
                    if (!fit(most, kLeastScaleV, kMaxScaleV, ev, low_v)) return false;
                    if (ev != before) {
#pragma unroll
                        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                            for (int r = 0; r < 16; ++r) o[dt][r] *= pow2(max(ev - before, -126));      // less only where O is still 0
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) p8[e] = s[8 * run + e];
                    const Parts p = split8(p8, pow2(kScaleP));
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) {
                        mul_parts(split8(vf[run][dt], pow2(ev)), p, o[dt], o[dt]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (EXACT && run == 0) { load_k(b0, b1); __builtin_amdgcn_sched_barrier(0); }
            }
        }
        if (!EXACT) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= pow2(-ev - kScaleP);
        }
        return true;
    };
    if (!exact) exact = !walk(std::false_type());
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // no copy is in flight into what the partial results take
    // one wave that meets a value out of range has all walk again
    __syncthreads();                                                // every wave is past its last read of Q
    if (lane == 0) flags[wave] = exact;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) exact |= flags[w] != 0;
    exact = __builtin_amdgcn_readfirstlane(exact);
    if (exact) walk(std::true_type());

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
                a.lse[((long long)bb * a.hq + h) * a.n + q_lo + row] = L > 0.f ? M * a.scale + logf(L) : -INFINITY;
        }
    }
}

template <int MODE, int W>
hipError_t launch(const Shape& sh, Args32& a, hipStream_t st) {
    a.qtiles = ((a.idx ? min(sh.s, sh.n) : sh.n) + TQ - 1) / TQ;    // a segment may be set longer than the sequence
    const long long grid = (long long)sh.batch * sh.hq * a.qtiles * (a.idx ? sh.n1 : 1);
    constexpr int smem = W * TQ * kHeadDim * 4 + 2 * 8 * 64 * 16;   // W = 4: half of a compute unit's LDS
    static_assert(2 * W * TQ * 4 + W * 4 <= 2 * 8 * 64 * 16, "what takes the place of Q");
    const hipError_t e = hipFuncSetAttribute((const void*)attn_fp32_split_kernel<MODE, W>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_fp32_split_kernel<MODE, W>), dim3((unsigned)grid), dim3(64 * W), smem, st, a);
    return hipGetLastError();
}
}  // namespace

// Row tiles that exist: a segment's last tile may be short.
static long long row_tiles(const Shape& sh, bool sparse) {
    const int s = sparse ? sh.s : sh.n, rest = sh.n % s;
    return (long long)sh.batch * sh.hq * ((long long)(sh.n / s) * ((s + TQ - 1) / TQ) + (rest + TQ - 1) / TQ);
}

static long long listed_keys(const Shape& sh, bool sparse) {
    return sparse ? std::min((long long)sh.n, (long long)sh.list_len * sh.b) : sh.n;
}

// Against the fp32 matrix instructions (us, that kernel in its best form / this one; t: row tiles of 32).  That kernel splits rows into 16 and
// so fills the chip with half as many: t = 128 block-sparse 4 heads x 512 keys 13.5 / 18.8, 1 x 4096, 960 keys 26 / 30, dense 4 x 1000 23.4 / 26.4.  From t = 256 on
// it is always behind: block-sparse 8 x 1000, 400 keys 22.9 / 20.9, 2 x 4096 (256, 960 keys) 44 / 31, 4 x 4096 (512, 704) 57 / 41, 8 x
// 8192 (2048; 400, 1184, 4384) 147 / 109, 345 / 214, 898 / 504; dense 8 x 1000 35 / 29, 4 x 2500 (316) 78 / 54, 8 x 8192 1093 / 607.
// In between the two meet where rows are short or few: t = 192 3 x 2048, 1856 keys 44 / 45 and dense 46 / 47, 188 4 x 1500 dense 35 / 37, but 1 x 6000
// (188; 400, 960, 1856) 23 / 20.5, 43 / 31, 80 / 47; t = 163 1 x 5200 (400, 960, 3264) 22.9 / 20.0, 42 / 29, 72 / 74, 152 8 x 600, 400 keys 16 / 19.
bool attn_fp32_split_better(const Shape& sh, bool sparse) {
    if (sh.kvs[2] >= (1 << 26) || (sparse && sh.b % 16 != 0)) return false;     // a run's rows within 32-bit byte offsets of its first; runs of 16
    const long long tiles = row_tiles(sh, sparse), keys = listed_keys(sh, sparse);
    if (tiles >= 256) return true;
    if (tiles >= 184) return sh.n >= 2400 || (sparse && keys < 1536);
    return tiles >= 144 && sparse && sh.n >= 2400 && keys < 2400;
}

// Eight waves leave one workgroup to a compute unit, four two.  Eight / four: up to a chip full of workgroups block-sparse 1 x 8192 (t =
// 256; 400, 1184, 4384 keys) 22 / 26, 39 / 48, 98 / 136, dense 2 x 4096 81 / 111; beyond it rows of many or unequal keys: dense 4 x 2500
// (316) 54 / 71, 2 x 8192 (512) 176 / 220, 3 x 6000 (564) 162 / 169, block-sparse 2 x 6000 (376, 4384) 105 / 138, 3 x 3000 (282; 400, 960, 1856) 33 / 26,
// 37 / 40, 48 / 65; but 2 x 6000 (376, 960) 58 / 52, 4 x 4096 (512, 1856) 92 / 89; dense 3 x 8192 (768) 283 / 254.
hipError_t launch_attn_fp32_split(const Shape& sh, Args32& a, hipStream_t st) {
    const bool sparse = a.idx != nullptr;
    const long long tiles = row_tiles(sh, sparse), keys = listed_keys(sh, sparse);
    const bool eight = tiles <= 256 || (tiles <= 320 && keys >= 640) || (tiles < 600 && (!sparse || keys >= 3072));
    if (sparse) return eight ? launch<1, 8>(sh, a, st) : launch<1, 4>(sh, a, st);
    return eight ? launch<2, 8>(sh, a, st) : launch<2, 4>(sh, a, st);
}

}  // namespace cp
