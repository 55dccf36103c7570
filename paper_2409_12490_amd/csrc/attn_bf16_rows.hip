// bf16 MFMA flash attention for launches that cannot fill the chip with 256-row workgroups (attn_bf16.hip): few heads, short
// sequences, short segments.  The same arithmetic (bf16 operands, fp32 sums, P rounded to bf16 and the row sum taken over the
// rounded values) in another split: a workgroup owns 32 query rows and its W waves split the KEYS.  Wave w takes tiles w, w + W, ...
// of 32 keys, with a running max, sum and output of its own, and the W partial results are merged through LDS at the end.
//
//   S^T[key][q]   = K . Q^T     32x32x16 MFMA, A = K rows straight from memory to registers (a wave's keys are its own: nothing to
//                               share), B = Q fragments that stay in registers
//   softmax                     one query per lane column
//   O^T[ch][q]   += V^T . P^T   A = V through the transposing LDS read, from a tile of the wave's own that global_load_lds fills
//                               (two slots of 8 KiB); B = P^T, the S^T accumulators as they stand
//
// There is no barrier in the key loop.  V and then K of the next tile are asked for between QK and the softmax: loads
// return in order, so a wave whose K is there has its V too.
//
// What bounds it: up to a few hundred workgroups the latency of a tile (16 KB asked for one tile ahead; 1.5 us per tile and wave at 4
// heads x 3000 tokens), beyond that the caches: every 32 rows read their keys anew, eight times the bytes of the 256-row kernel
// (9 to 12 TB/s reached).  Dense 2 heads x 600 tokens 20.6 -> 9.6 us, 4 x 3000 72.7 -> 32.7, 2 x 8192 185 -> 88; block-sparse 2 x
// 5632 32.2 -> 25.7 (against the 256-row kernel, with 6 to 64 workgroups there); where that kernel fills the chip it is 2.4 times
// faster than this one.
#include "attn_bf16.h"

#include <algorithm>

namespace cp {
namespace {

constexpr int kRowsTQ = 32, kRowsTK = 32, kSlotBytes = kRowsTK * 256;
constexpr int kNoToken = 0x7fffffff;              // a key that does not exist: after every query

// MODE 0: sparse, any block size: every key of a tile has a token of its own.  MODE 1: sparse, block size a multiple of 32: a
// tile is 32 consecutive tokens, described by its first token on the scalar unit.  MODE 2: dense.
template <int MODE, int W>
__global__ __launch_bounds__(64 * W, 2) void attn_bf16_rows_kernel(ArgsB a) {
    constexpr bool DENSE = MODE == 2, RUN = MODE != 0;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    constexpr unsigned kStat = W * 2 * kSlotBytes;                  // behind the slots: (max, sum) [wave][row]

    const int tid = thread_id(), lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Consecutive workgroups walk the KV heads, so that a head's keys stay with few XCDs (workgroup id mod 8); inside one the row
    // tiles of a segment and head follow each other, and the segments with most keys, those at the end, come first.
    const int G = a.group, bkv = a.batch * a.hkv;
    const int wg = (int)workgroup_id(), x = wg % bkv, y = wg / bkv;
    const int bb = x / a.hkv, kvh = x % a.hkv;
    int h, j = 0, q_lo;
    if (DENSE) { h = kvh * G + y % G; q_lo = (a.qtiles - 1 - y / G) * kRowsTQ; }
    else {
        h = kvh * G + y / a.qtiles % G;
        j = a.n1 - 1 - y / a.qtiles / G;
        q_lo = j * a.s + y % a.qtiles * kRowsTQ;
    }
    const int q_end = DENSE ? a.n : min(a.n, (j + 1) * a.s);       // rows >= q_end do not exist
    if (q_lo >= q_end) return;                                     // uniform: tile past a short segment
    const int q_last = __builtin_amdgcn_readfirstlane(min(q_end, q_lo + kRowsTQ) - 1);
    const uint16_t* kp = uniform_ptr(a.k + bb * a.ks0 + kvh * a.ks1);
    const uint16_t* vp = uniform_ptr(a.v + bb * a.ks0 + kvh * a.ks1);

    scalar_list list = nullptr; int count = 0;
    if (!DENSE) {
        const long long lrow = a.shared_lists ? ((long long)bb * a.hkv + kvh) * a.n1 + j : ((long long)bb * a.hq + h) * a.n1 + j;
        list = (scalar_list)(unsigned long long)(a.idx + lrow * a.list_len);
        count = min(max(((scalar_list)(unsigned long long)a.cnt)[lrow], 0), a.list_len);
    }
    const int qpos = q_lo + l32;
    bf16x8 qf[8];
    {
        const uint16_t* src = a.q + bb * a.qs0 + h * a.qs1 + (long long)min(qpos, q_last) * a.qs2 + 8 * hh;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = as_bf16x8(*(const uint4*)(src + 16 * ks));
    }
    // positions 0 .. total-1 of the listed blocks laid end to end (host checks list_len * b < 2^31)
    const unsigned total = DENSE ? (unsigned)q_last + 1u : (unsigned)count * (unsigned)a.b;
    const int ntiles = (int)((total + kRowsTK - 1) / kRowsTK);

    // ---- MODE 1/2: first token of the wave's next tile, -1 past its last one; t: the dense tile --------------------
    unsigned walk_e = 0, walk_off = 0, step_e = 0, step_off = 0;    // list entry and offset inside its block of the next tile
    if (MODE == 1) {
        walk_e = (unsigned)wave * kRowsTK / (unsigned)a.b; walk_off = (unsigned)wave * kRowsTK % (unsigned)a.b;
        step_e = W * kRowsTK / (unsigned)a.b; step_off = W * kRowsTK % (unsigned)a.b;
    }
    const int n2 = MODE == 1 ? (a.n + a.b - 1) / a.b : 0;
    auto next_base = [&](int t) -> int {                            // call in tile order: t = wave, wave + W, ...
        if (DENSE) return t < ntiles ? t * kRowsTK : -1;
        int base = -1;
        while (base < 0 && walk_e < (unsigned)count) {              // entries outside the sequence have no tokens
            const int blk = list[walk_e];
            base = blk >= 0 && blk < n2 ? blk * a.b + (int)walk_off : -1;
            if (base >= a.n) base = -1;
            walk_e += step_e; walk_off += step_off;
            if (walk_off >= (unsigned)a.b) { walk_off -= a.b; ++walk_e; }
        }
        return base;
    };
    // ---- MODE 0: token of key l32 of tile t --------------------------------------------------------------------
    auto key_token = [&](int t) -> int {
        const unsigned p = (unsigned)t * kRowsTK + l32, e = p / (unsigned)a.b;
        const int blk = ((const int32_t*)(unsigned long long)list)[min(e, (unsigned)max(count - 1, 0))];
        const long long tk = (long long)blk * a.b + p % (unsigned)a.b;
        return t < ntiles && e < (unsigned)count && blk >= 0 && tk < a.n ? (int)tk : kNoToken;
    };

    // ---- loads: V rows 4*x + r4 into the slot (16-byte chunks swizzled by the row), K row l32 into registers ---------
    const unsigned tok_bytes = (unsigned)a.ks2 * 2u;                // host checks n * tok_bytes < 2^32, both < 2^24
    const int r4 = lane >> 4, vch = (lane & 15) ^ (4 * r4);
    const unsigned k_full = (unsigned)l32 * tok_bytes + hh * 16, v_full = (unsigned)r4 * tok_bytes + vch * 16;
    typedef const __attribute__((address_space(1))) char* global_bytes;
    bf16x8 kf[8];
    auto load_k = [&](const uint16_t* rows, unsigned off) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kf[ks] = as_bf16x8(*(const __attribute__((address_space(1))) u32x4*)((global_bytes)(unsigned long long)rows + off + 32 * ks));
    };
    auto load_tile = [&](int base, int tok, unsigned slot) {        // MODE 1/2: base; MODE 0: tok
        if (RUN) {
            const uint16_t* vrow = uniform_ptr(vp + (long long)base * a.ks2);
            unsigned koff = k_full;
            if (base + kRowsTK <= a.n) {
#pragma unroll
                for (int i = 0; i < 8; ++i) dma16(uniform_ptr(vrow + (long long)(4 * i) * a.ks2), v_full, slot + i * 1024);
            } else {                                                // rows past the end repeat the last token: after every query, masked
                const int top = a.n - 1 - base;
#pragma unroll
                for (int i = 0; i < 8; ++i) dma16(vrow, (unsigned)min(4 * i + r4, top) * tok_bytes + vch * 16, slot + i * 1024);
                koff = (unsigned)min(l32, top) * tok_bytes + hh * 16;
            }
            load_k(uniform_ptr(kp + (long long)base * a.ks2), koff);
        } else {                                                    // keys without a token read token 0 and are masked
            const unsigned row = (tok == kNoToken ? 0u : (unsigned)tok) * tok_bytes;
#pragma unroll
            for (int i = 0; i < 8; ++i) dma16(vp, (unsigned)__shfl((int)row, 4 * i + r4) + vch * 16, slot + i * 1024);
            load_k(kp, row + hh * 16);
        }
    };
    // V (transposed read, 16-lane groups): lane supplies row 4*hh + (i16 >> 2) (+16*t4, +8) and the 8-byte unit of channels
    // 32*dt + 16*gbit + 4*(i16 & 3); physical chunk = logical chunk ^ 4*(row & 3)
    const unsigned slot0 = lds0 + wave * 2 * kSlotBytes;
    const int i16 = lane & 15, gbit = (lane >> 4) & 1;
    unsigned va[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
        va[dt] = (4 * hh + (i16 >> 2)) * 256 + ((((unsigned)(dt ^ (i16 >> 2)) << 2) + 2 * gbit + ((i16 & 3) >> 1)) << 4) + (i16 & 1) * 8;
    auto read_v = [&](unsigned slot, int t4, int dt) -> bf16x8 {
        const unsigned ad = slot + va[dt] + t4 * 16 * 256;
        const v4bf16_lds lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(v4bf16_lds, ad));
        const v4bf16_lds hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(v4bf16_lds, ad + 8 * 256));
        bf16x8 f;
#pragma unroll
        for (int e = 0; e < 4; ++e) { f[e] = lo[e]; f[4 + e] = hi[e]; }
        return f;
    };

    f32x16 o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float c = a.scale_log2e, lazy_raw = kLazyLog2 / c;

    int base = -1, tok = kNoToken;
    // ascending lists: nothing is visible from the tile on whose first token is past the last row
    auto more = [&](int t) -> bool {
        if (RUN) return base >= 0 && base <= q_last;
        const int first = __builtin_amdgcn_readfirstlane(tok);
        return t < ntiles && (first <= q_last || first == kNoToken);
    };
    if (RUN) base = __builtin_amdgcn_readfirstlane(next_base(wave)); else tok = key_token(wave);
    if (more(wave)) load_tile(base, tok, slot0);
    unsigned slot = slot0;
    for (int t = wave; more(t); t += W) {
        const int this_base = base, this_tok = tok;
        if (RUN) base = __builtin_amdgcn_readfirstlane(next_base(t + W)); else tok = key_token(t + W);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // V and K of this tile
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned next_slot = slot ^ kSlotBytes;               // its last reads fed the PV of the tile before
        if (more(t + W)) load_tile(base, tok, next_slot);
        __builtin_amdgcn_sched_barrier(0);

        // ---- softmax: see the 256-row kernel
        if (RUN) {
            if (this_base + kRowsTK - 1 > q_lo) {
                const int lim = qpos - this_base - 4 * hh;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + (r & 3) > lim) s[r] = -INFINITY;
            }
        } else if (__builtin_amdgcn_ballot_w64(this_tok > q_lo) != 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (__shfl(this_tok, 8 * (r >> 2) + 4 * hh + (r & 3)) > qpos) s[r] = -INFINITY;
        }
        float mx = fmaxf(s[0], s[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(s[r], s[r + 1]), mx);
        mx = half_max(mx);
        const float m_new = (mx > m_run + lazy_raw) ? mx : m_run;
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_safe) * c);
        const float ms = m_safe * c;
        m_run = m_new;
        bf16x8 pf[2];
        bf16x2 one2; one2[0] = (__bf16)1.0f; one2[1] = (__bf16)1.0f;
        float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
        for (int t4 = 0; t4 < 2; ++t4) {
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[t4][e] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[8 * t4 + e], c, -ms));
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                bf16x2 pr; pr[0] = pf[t4][e]; pr[1] = pf[t4][e + 1];
                if (e & 2) rs1 = __builtin_amdgcn_fdot2_f32_bf16(pr, one2, rs1, false);
                else rs0 = __builtin_amdgcn_fdot2_f32_bf16(pr, one2, rs0, false);
            }
        }
        l_run = l_run * alpha + (rs0 + rs1);                        // per-half partial sums, merged at the end
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
#pragma unroll
        for (int t4 = 0; t4 < 2; ++t4)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_v(slot, t4, dt), pf[t4], o[dt], 0, 0, 0);
        slot = next_slot;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // no copy is in flight when the slots are written below

    // ---- merge the W partial results: out = sum_w 2^(c (m_w - M)) O_w / sum_w 2^(c (m_w - M)) l_w; a wave's O, 32 rows of 512 B with
    // the 16-byte chunks swizzled by the row, takes the place of its own two slots
    const float l_tot = half_sum(l_run);
    if (hh == 0) {
        *LDS_PTR(float, lds0 + kStat + (wave * 32 + l32) * 4) = m_run;
        *LDS_PTR(float, lds0 + kStat + (W * 32 + wave * 32 + l32) * 4) = l_tot;
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {                            // channels 32*dt + 8*gg + 4*hh .. +3
            const unsigned chunk = (unsigned)(8 * dt + 2 * gg + hh) ^ (unsigned)l32;
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(o[dt][4 * gg + e]);
            *LDS_PTR(u32x4, slot0 + l32 * 512 + chunk * 16) = w;
        }
    __syncthreads();
    uint16_t* ob = a.out + bb * a.os0 + h * a.os1;
#pragma unroll
    for (int i = 0; i < 8 / W; ++i) {                               // 16 threads to a row, 8 channels each
        const int row = i * 4 * W + (tid >> 4), pair = tid & 15;
        float M = -INFINITY, L = 0.f, sum[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[e] = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, *LDS_PTR(const float, lds0 + kStat + (w * 32 + row) * 4));
        const float M_safe = (M == -INFINITY) ? 0.f : M;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float f = __builtin_amdgcn_exp2f((*LDS_PTR(const float, lds0 + kStat + (w * 32 + row) * 4) - M_safe) * c);
            L += f * *LDS_PTR(const float, lds0 + kStat + (W * 32 + w * 32 + row) * 4);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const u32x4 v = *LDS_PTR(const u32x4, lds0 + w * 2 * kSlotBytes + row * 512 + (unsigned)((2 * pair + half) ^ row) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[4 * half + e] += f * __uint_as_float(v[e]);
            }
        }
        if (q_lo + row < q_end) {
            const float inv = L > 0.f ? 1.0f / L : 0.f;
            bf16x8 w;
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = (__bf16)(sum[e] * inv);
            union { bf16x8 b; u32x4 u; } cv; cv.b = w;
            *(u32x4*)(ob + (long long)(q_lo + row) * a.os2 + pair * 8) = cv.u;
            if (a.lse && pair == 0)
                a.lse[((long long)bb * a.hq + h) * a.n + q_lo + row] = L > 0.f ? M * a.scale + __logf(L) : -INFINITY;
        }
    }
}

template <int MODE, int W>
hipError_t launch(const ArgsB& a, unsigned grid, hipStream_t st) {
    constexpr int smem = W * 2 * kSlotBytes + 2 * W * 32 * 4;
    const hipError_t e = hipFuncSetAttribute((const void*)attn_bf16_rows_kernel<MODE, W>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_bf16_rows_kernel<MODE, W>), dim3(grid), dim3(64 * W), smem, st, a);
    return hipGetLastError();
}

}  // namespace

template <int W>
static hipError_t launch_waves(const Shape& sh, const ArgsB& a, unsigned grid, hipStream_t st) {
    if (!a.idx) return launch<2, W>(a, grid, st);
    return sh.b % 32 == 0 ? launch<1, W>(a, grid, st) : launch<0, W>(a, grid, st);
}

// Row tiles that exist: a segment's last tile may be short.
static long long row_tiles(const Shape& sh, bool sparse, int rows) {
    const int s = sparse ? sh.s : sh.n, rest = sh.n % s;
    return (long long)sh.batch * sh.hq * ((long long)(sh.n / s) * ((s + rows - 1) / rows) + (rest + rows - 1) / rows);
}

static long long listed_keys(const Shape& sh) { return std::min((long long)sh.n, (long long)sh.list_len * sh.b); }

// Few query rows: 256 of them to a workgroup leave compute units idle, 32 do not.  The lines lie where the two kernels meet (256-row against
// 32-row kernel).
//   block-sparse, blocks of 64 or 16: 16384 rows: 32 heads x 512 20.4 / 13.9 to 22.6 / 15.4 us, 8 x 2048 25.7 / 21.1 to 55 / 35, 1 x 16K
//   26.3 / 22.3 to 69 / 56; 24576 rows: 26.5 / 26.7 and 26.9 / 25.5, 26.1 / 30.2 to 69 / 59, 27.6 / 33.7 to 72 / 85.
//   dense, 32768 rows: 32 x 1024 30.9 / 30.5, 8 x 4096 98 / 86, 1 x 32K 722 / 590; 40960 rows: 37 / 40, 123 / 126, 903 / 938.
// Two 32-row workgroups fit a compute unit, and segments that are no multiple of 32 rows make more of them out of 16384 rows than the 512
// that fit the chip.  A second round costs as much as the first where all lists are as long, and more than the 256-row kernel takes
// where they are short: 16384 x 1 head, segments of 240 (552 workgroups), 6 blocks of 48 24.0 / 30.4, 10 of 40 27.4 / 33.7, 20 of
// 24 29.0 / 34.4, 40 of 48 67 / 62; 290 x 56 (616) 16.2 / 18.5; but 680 x 24 (552) 23.0 / 18.5, 2720 x 6 (546), 40 of 48 65 / 42; up
// to 540 workgroups (a short last tile per head) the 32-row kernel is never slower.  Segments of 48: more than 256 workgroups of
// 256 rows, 46 / 30.
bool attn_bf16_rows_better(const Shape& sh, bool sparse) {
    const long long rows = (long long)sh.batch * sh.hq * sh.n;
    if (!sparse) return rows <= 32768;
    if (rows > 16384) return false;
    const long long keys = listed_keys(sh);
    return row_tiles(sh, true, kRowsTQ) <= 540 || row_tiles(sh, true, 256) > 256 || keys >= 1536 || (keys >= 340 && sh.n <= 2 * keys);
}

// Eight waves where the workgroups are too few to give every compute unit two, and for dense rows of thousands of keys; four
// otherwise, two workgroups to a unit.  Eight against four waves: block-sparse, 8 heads x 1024 tokens 13.6 / 14.4 us (blocks of
// 32) and 15.3 / 17.1 (64), 2 x 8192 58 / 54 and 26 / 22; more than 256 workgroups out of 8192 rows: 8192 x 1, segments of 240, 60 blocks of 40
// 32 / 42, but 256 x 32 16.0 / 13.2; dense, one head x 16K 160 / 211, 2 x 8192 88 / 109, 2 x 16K 306 / 315, 8 x 2048 29 / 33, 8 x
// 4096 91 / 86, 32 x 512 15.3 / 13.1.
hipError_t launch_attn_bf16_rows(const Shape& sh, ArgsB a, hipStream_t st) {
    const int longest = a.idx ? std::min(sh.s, sh.n) : sh.n;          // a segment may be set longer than the sequence
    a.qtiles = (longest + kRowsTQ - 1) / kRowsTQ;
    const unsigned grid = (unsigned)((long long)sh.batch * sh.hq * a.qtiles * (a.idx ? sh.n1 : 1));
    const long long rows = (long long)sh.batch * sh.hq * sh.n;
    const bool eight = a.idx ? rows <= 8192 && (row_tiles(sh, true, kRowsTQ) <= 270 || listed_keys(sh) >= 340)
                             : rows <= 8192 || (sh.n >= 2048 && rows <= 16384) || sh.n >= 8192;
    return eight ? launch_waves<8>(sh, a, grid, st) : launch_waves<4>(sh, a, grid, st);
}

}  // namespace cp
