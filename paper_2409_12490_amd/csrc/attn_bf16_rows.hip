// bf16 MFMA flash attention for launches that cannot fill the chip with 256-row workgroups (attn_bf16.hip) or 128-row ones (attn_bf16_half.hip): few
// heads, short sequences, segments of up to 64 rows.  The same arithmetic (bf16 operands, fp32 sums, P rounded to bf16 and the row sum taken over the
// rounded values) in another split: a workgroup owns 32 query rows and its W waves split the KEYS.  Wave w takes tiles w, w + W, ...
// of 32 keys, with a running max, sum and output of its own, and the W partial results are merged through LDS at the end.
//
//   S^T[key][q]   = K . Q^T     32x32x16 MFMA, A = K rows from LDS, B = Q fragments that stay in registers
//   softmax                     one query per lane column
//   O^T[ch][q]   += V^T . P^T   A = V through the transposing LDS read; B = P^T, the S^T accumulators as they stand
//
// K and V tiles of the wave's own (8 KiB each) come by global_load_lds as whole rows.  There is no barrier in the key loop: K of the next tile is asked
// for when QK has read this one, V when PV has; each has half a tile's time to land, and loads return in order, so the other may be on its way.
//
// What bounds it: K as A operands straight from memory, a lane per row, asked the address unit of a compute unit for 512 pieces of 16 bytes a tile and Q for 512
// more per wave, one a cycle: that bound the kernel.  By whole rows it is 256 pieces of 64
// bytes: dense 2 heads x 600 tokens 9.9 -> 7.3 us, 4 x 3000 32.4 -> 20.5, 2 x 8192 88 -> 53; block-sparse 4 x 4000 (blocks of 16) 28.7 -> 18.6, 2 x 5632 24.7 ->
// 17.5, 8 x 1024 14.4 -> 10.6.  What is left is latency up to a few hundred workgroups, beyond that the caches (19 TB/s for dense 2 x 8192): every 32
// rows read their keys anew, eight times the bytes of the 256-row kernel.
#include "attn_bf16.h"

#include <algorithm>

namespace cp {
namespace {

constexpr int kRowsTQ = 32, kRowsTK = 32, kSlotBytes = kRowsTK * 256;
constexpr int kNoToken = 0x7fffffff;              // a key that does not exist: after every query

// MODE 0: sparse, any block size: every key of a tile has a token of its own.  MODE 1: sparse, block size a multiple of 16: a
// tile is two runs of 16 consecutive tokens, described by their first tokens on the scalar unit.  MODE 2: dense.
// PAIRS: in the order of TileOrder, else segments from the last to the first.
template <int MODE, int W, bool PAIRS>
__global__ __launch_bounds__(64 * W, 2) void attn_bf16_rows_kernel(ArgsB a, TileOrder order) {
    constexpr bool DENSE = MODE == 2, RUN = MODE != 0;
    ask_for(a.q, a.k, a.v, a.idx, a.cnt, a.batch, a.n, a.qtiles, a.group, a.scale_log2e, a.qs0, a.qs1, a.qs2, a.ks0, a.ks1, a.ks2);
    if (PAIRS) ask_for(order.turn);
    if (PAIRS && !DENSE) ask_for(order.full, order.past, order.by_full.mul, order.by_level.mul);
    if (!DENSE) ask_for(order.most, order.by_tiles.shift);
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    constexpr unsigned kQ = W * 2 * kSlotBytes;                     // behind the waves' K and V slots: Q
    constexpr unsigned kStat = kQ + kRowsTQ * 256;                  // (max, sum) [wave][row]

    const int tid = thread_id(), lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Consecutive workgroups walk the KV heads, so that a head's keys stay with few XCDs (workgroup id mod 8); then the query heads of a group, and inside a
    // head TileOrder.
    const int G = a.group, bkv = a.batch * a.hkv;
    const int wg = (int)(PAIRS ? order.place(workgroup_id()) : workgroup_id()), x = wg % bkv, y = wg / bkv;
    const int bb = x / a.hkv, kvh = x % a.hkv;
    int h, j = 0, q_lo;
    if (DENSE) { h = kvh * G + y % G; q_lo = (a.qtiles - 1 - y / G) * kRowsTQ; }
    else {
        h = kvh * G + y % G;
        const TileOrder::Item item = PAIRS ? order.item(y / G, a.n1, a.qtiles) : order.by_segments(y / G, a.qtiles);
        j = item.segment;
        q_lo = j * a.s + item.tile * kRowsTQ;
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
    // ---- Q, as whole rows to LDS by all waves, from there to the registers of each: a lane per row straight from memory, by every wave for
    // itself, asks the address unit for 512 * W pieces of 16 bytes
    const int r4 = lane >> 4, pch = lane & 15;                      // row inside a copy's four rows, chunk the lane's 16 bytes land in
    const uint16_t* qp = a.q + bb * a.qs0 + h * a.qs1;
#pragma unroll
    for (int i = 0; i < 8 / W; ++i) {
        const int row = 4 * (wave * (8 / W) + i) + r4;              // rows past the end repeat the last one; 16-byte chunks swizzled by the row
        dma16_far((const char*)(qp + (long long)min(q_lo + row, q_last) * a.qs2) + ((pch ^ (row & 15)) << 4), lds0 + kQ + (wave * (8 / W) + i) * 1024);
    }
    // positions 0 .. total-1 of the listed blocks laid end to end (host checks list_len * b < 2^31)
    const unsigned total = DENSE ? (unsigned)q_last + 1u : (unsigned)count * (unsigned)a.b;
    const int ntiles = (int)((total + kRowsTK - 1) / kRowsTK);

    // ---- MODE 1/2: first tokens of the two runs of the wave's next tile, -1: no such tokens; call in tile order
    unsigned walk_e = 0, walk_off = 0, step_e = 0, step_off = 0;    // list entry and offset inside its block of the next tile
    if (MODE == 1) {
        walk_e = (unsigned)wave * kRowsTK / (unsigned)a.b; walk_off = (unsigned)wave * kRowsTK % (unsigned)a.b;
        step_e = W * kRowsTK / (unsigned)a.b; step_off = W * kRowsTK % (unsigned)a.b;
    }
    const int n2 = MODE == 1 ? (a.n + a.b - 1) / a.b : 0;
    auto run_at = [&](unsigned e, unsigned off) -> int {
        if (e >= (unsigned)count) return -1;
        const int blk = list[e];
        const int at = blk >= 0 && blk < n2 ? blk * a.b + (int)off : -1;    // entries outside the sequence have no tokens
        return at < a.n ? at : -1;
    };
    int base0 = -1, base1 = -1;
    auto next_tile = [&](int t) {
        if (DENSE) {
            base0 = t < ntiles ? t * kRowsTK : -1;
            base1 = base0 >= 0 && base0 + 16 < a.n ? base0 + 16 : -1;
        } else {
            base0 = __builtin_amdgcn_readfirstlane(run_at(walk_e, walk_off));
            const bool over = walk_off + 16 >= (unsigned)a.b;
            base1 = __builtin_amdgcn_readfirstlane(run_at(walk_e + (over ? 1 : 0), over ? 0 : walk_off + 16));
            walk_e += step_e; walk_off += step_off;
            if (walk_off >= (unsigned)a.b) { walk_off -= a.b; ++walk_e; }
        }
    };
    // ---- MODE 0: token of key l32 of tile t --------------------------------------------------------------------
    auto key_token = [&](int t) -> int {
        const unsigned p = (unsigned)t * kRowsTK + l32, e = p / (unsigned)a.b;
        const int blk = ((const int32_t*)(unsigned long long)list)[min(e, (unsigned)max(count - 1, 0))];
        const long long tk = (long long)blk * a.b + p % (unsigned)a.b;
        return t < ntiles && e < (unsigned)count && blk >= 0 && tk < a.n ? (int)tk : kNoToken;
    };

    // ---- copies: rows 4*i + r4 of K and V into the wave's two slots, 16-byte chunks swizzled by the row (K: row & 15, V: 4 * (row & 3))
    const unsigned tok_bytes = (unsigned)a.ks2 * 2u;                // host checks n * tok_bytes < 2^32, both < 2^24
    const unsigned vch = (unsigned)(pch ^ (4 * r4)) << 4, kch = (unsigned)(pch ^ r4) << 4;   // K: of rows 16*x + r4, the others by the row's bits 2 and 3
    const unsigned k_slot = lds0 + wave * 2 * kSlotBytes, v_slot = k_slot + kSlotBytes;
    unsigned k_run[4], v_run[4];                                    // byte offsets of the lane's pieces of a run of 16 rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        k_run[i] = (unsigned)(4 * i + r4) * tok_bytes + (kch ^ (64 * i));
        v_run[i] = (unsigned)(4 * i + r4) * tok_bytes + vch;
    }
    int tok = kNoToken;                                             // MODE 0: of the lane's key of the next tile
    auto copy = [&](const uint16_t* from, bool is_k) {              // the next tile's; the reads of the tile before are done
        const unsigned slot = is_k ? k_slot : v_slot;
        auto chunk = [&](int i) { return is_k ? kch ^ (64 * (i & 3)) : vch; };
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (RUN) {
            const int first = max(base0, base1);                    // rows without a token repeat some of the tile's: masked
#pragma unroll
            for (int run = 0; run < 2; ++run) {
                const int at = run ? base1 : base0, from_tok = max(at >= 0 ? at : first, 0);
                const uint16_t* rows = uniform_ptr(from + (long long)from_tok * a.ks2);
                if (from_tok + 16 <= a.n) dma16x4(rows, is_k ? k_run : v_run, slot + run * 4096);
                else {                                            // past the end the last token: after every query, masked
                    const int top = a.n - 1 - from_tok;
#pragma unroll
                    for (int i = 0; i < 4; ++i) dma16(rows, (unsigned)min(4 * i + r4, top) * tok_bytes + chunk(i), slot + (4 * run + i) * 1024);
                }
            }
        } else {                                                    // keys without a token read token 0 and are masked
            const unsigned row = (tok == kNoToken ? 0u : (unsigned)tok) * tok_bytes;
#pragma unroll
            for (int i = 0; i < 8; ++i) dma16(from, (unsigned)__shfl((int)row, 4 * i + r4) + chunk(i), slot + i * 1024);
        }
    };
    const unsigned k_base = (k_slot + l32 * 256) | (unsigned)(((l32 & 15) ^ hh) << 4);   // K row l32, channels 16*ks + 8*hh: k_base ^ 32*ks
    // V (transposed read, 16-lane groups): lane supplies row 4*hh + (i16 >> 2) (+16*t4, +8) and the 8-byte unit of channels
    // 32*dt + 16*gbit + 4*(i16 & 3); physical chunk = logical chunk ^ 4*(row & 3)
    const int i16 = lane & 15, gbit = (lane >> 4) & 1;
    unsigned va[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
        va[dt] = (4 * hh + (i16 >> 2)) * 256 + ((((unsigned)(dt ^ (i16 >> 2)) << 2) + 2 * gbit + ((i16 & 3) >> 1)) << 4) + (i16 & 1) * 8;
    auto read_v = [&](int t4, int dt) -> bf16x8 {
        const unsigned ad = v_slot + va[dt] + t4 * 16 * 256;
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

    // ascending lists: nothing is visible from the tile on whose first token is past the last row
    auto more = [&](int t) -> bool {
        if (RUN) return t < ntiles && base0 <= q_last;
        const int first = __builtin_amdgcn_readfirstlane(tok);
        return t < ntiles && (first <= q_last || first == kNoToken);
    };
    if (RUN) next_tile(wave); else tok = key_token(wave);
    bool go = more(wave);
    if (go) {
        copy(kp, true); copy(vp, false);
        asm volatile("s_waitcnt vmcnt(16)" ::: "memory");           // the wave's share of Q has landed
    } else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    bf16x8 qf[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = as_bf16x8(*LDS_PTR(const u32x4, lds0 + kQ + l32 * 256 + (((2 * ks + hh) ^ (l32 & 15)) << 4)));
    for (int t = wave; go; t += W) {
        const int this0 = base0, this1 = base1, this_tok = tok;
        if (RUN) next_tile(t + W); else tok = key_token(t + W);
        const bool next = more(t + W);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");            // K of this tile; its V may be on the way
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        bf16x8 kf[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kf[ks] = as_bf16x8(*LDS_PTR(const u32x4, k_base ^ (unsigned)(32 * ks)));
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (next) copy(kp, true);
        __builtin_amdgcn_sched_barrier(0);

        // ---- softmax: see the 256-row kernel
        if (RUN) {
            if (max(this0, this1) + 15 > q_lo || this0 < 0 || this1 < 0) {   // hidden from some row, or not there
#pragma unroll
                for (int run = 0; run < 2; ++run) {
                    const int at = run ? this1 : this0;
                    int lim = at < 0 ? -1 : qpos - at - 4 * hh;
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        if (8 * (r >> 2) + (r & 3) > lim) s[8 * run + r] = -INFINITY;
                        asm("" : "+v"(lim));                        // see the 256-row kernel
                    }
                }
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
        if (next) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // V of this tile; K of the next may be on the way
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int t4 = 0; t4 < 2; ++t4)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_v(t4, dt), pf[t4], o[dt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (next) copy(vp, false);
        go = next;
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
            *LDS_PTR(u32x4, k_slot + l32 * 512 + chunk * 16) = w;
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

template <int MODE, int W, bool PAIRS>
hipError_t launch(const ArgsB& a, TileOrder order, unsigned grid, hipStream_t st) {
    constexpr int smem = W * 2 * kSlotBytes + kRowsTQ * 256 + 2 * W * 32 * 4;
    const hipError_t e = hipFuncSetAttribute((const void*)attn_bf16_rows_kernel<MODE, W, PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_bf16_rows_kernel<MODE, W, PAIRS>), dim3(grid), dim3(64 * W), smem, st, a, order);
    return hipGetLastError();
}

}  // namespace

template <int MODE>
static hipError_t launch_waves(const Shape& sh, const ArgsB& a, int waves, unsigned grid, hipStream_t st) {
    const TileOrder order = attn_bf16_rows_order(sh, MODE != 2, waves);
    if (waves == 8) return launch<MODE, 8, false>(a, order, grid, st);
    return order.turn ? launch<MODE, 4, true>(a, order, grid, st) : launch<MODE, 4, false>(a, order, grid, st);
}

// Row tiles that exist: a segment's last tile may be short.
long long attn_bf16_row_tiles(const Shape& sh, bool sparse, int rows) {
    const int s = sparse ? sh.s : sh.n, rest = sh.n % s;
    return (long long)sh.batch * sh.hq * ((long long)(sh.n / s) * ((s + rows - 1) / rows) + (rest + rows - 1) / rows);
}

static int rows_qtiles(const Shape& sh, bool sparse) {
    return ((sparse ? std::min(sh.s, sh.n) : sh.n) + kRowsTQ - 1) / kRowsTQ;      // a segment may be set longer than the sequence
}

static long long rows_grid(const Shape& sh, bool sparse) { return (long long)sh.batch * sh.hq * rows_qtiles(sh, sparse) * (sparse ? sh.n1 : 1); }

TileOrder attn_bf16_rows_order(const Shape& sh, bool sparse, int waves) {
    return TileOrder::of_launch(waves, rows_grid(sh, sparse), attn_bf16_row_tiles(sh, sparse, kRowsTQ), sh.n1, sh.r, sh.budget, sh.local, sh.b,
                                rows_qtiles(sh, sparse), kRowsTQ);
}

static long long listed_keys(const Shape& sh) { return std::min((long long)sh.n, (long long)sh.list_len * sh.b); }

// Few query rows: 256 of them to a workgroup leave compute units idle, 32 do not; where 256 fill the chip that kernel reads the keys once for eight
// row tiles and takes two thirds of the time.  The lines lie where this kernel meets the other two (us, the better one of those / this one, all in the orders of
// work_order.h; segments of 512, blocks of 64; keys listed in brackets; t: row tiles of 32).
//   block-sparse, up to t = 540 always: 32 heads x 500 15.9 / 9.8, 1 x 16384 (960, 2624, 4672) 25.3 / 19.0, 61 / 37, 104 / 58.
//   t = 576 to 657, keys few beside the sequence lose: 1 x 19000 (832, 1344) 23.3 / 25.4, 34.3 / 34.2, 2 x 9500 (960, 1344) 26.0 / 26.2, 34.1 / 29.6, but 4 x 4700
//   (960) 25.3 / 19.8, 8 x 2300 25.4 / 16.4.
//   t = 700 to 880: 8 x 3500 (960) 25.6 / 25.3, 1 x 24000 (1344) 34.8 / 35.1, 2 x 14000 (1344) 34.5 / 37.1, 4 x 7000 (1344) 33.9 / 34.6, but 8 x 3500 (2624) 61 / 43,
//   2 x 14000 (2624) 62 / 57, 32 x 850 (832) 20.3 / 17.5.
//   t = 900 to 1024: 8 x 4096 (960, 1344, 2624) 25.7 / 27.2, 33.9 / 33.6, 61 / 49, 4 x 8192 (2624) 62 / 58, 2 x 16384 (2624, 4672) 62 / 64, 105 / 101, 32 x 1000 (832)
//   23.2 / 20.5, 16 x 2000 (1600) 39.5 / 31.0; of 178 launches at most twice as long as their keys (eight numbers of heads) this kernel takes 0.64 to 0.90 of
//   the time on average, 0.53 to 1.04 in each; t = 1500: 32 x 1500 (1344) 35.1 / 36.1, 8 x 6000 (4672) 105.4 / 104.9.
//   segments of 128 rows and less leave half of a 256-row workgroup empty, at any length (most of those of 65 to 128 rows are the 128-row kernel's, which is asked
//   first, attn_bf16_half_better): against 256 rows 32 heads x 8192, segments of 128 (416, 1184, 4256) 127 / 122, 269 / 235, 676 / 589, of 64 (592) 312 / 156; segments
//   of 192 (480) 103 / 128.
//   dense, 49152 rows: 32 x 1500 40 / 36, 8 x 6000 147 / 109, 4 x 12000 280 / 208; 65536 rows: 32 x 2000 53 / 57, 8 x 8192 205 / 192, 2 x 32768 745 /
//   720; 32 x 1750 48.9 / 49.5; 96000 rows: 8 x 12000 323 / 389.
bool attn_bf16_rows_better(const Shape& sh, bool sparse) {
    const long long rows = (long long)sh.batch * sh.hq * sh.n;
    if (!sparse) return rows <= 49152 || (rows <= 65536 && sh.n >= 4096);
    const long long keys = listed_keys(sh), tiles = attn_bf16_row_tiles(sh, true, kRowsTQ), wide = attn_bf16_row_tiles(sh, true, 256);
    if (tiles <= 540) return true;
    if (8 * wide >= 4 * tiles) return true;
    if (8 * wide >= 2 * tiles) return tiles <= 1200 || keys >= 512;
    if (tiles <= 660) return keys >= 1300 || sh.n <= 5 * keys;
    return tiles <= 1024 && (sh.n <= 2 * keys || (tiles <= 900 ? keys >= 1300 && sh.n <= 8 * keys : keys >= 2400 && 2ll * sh.n <= 7 * keys));
}

// Eight waves where the workgroups are too few to give every compute unit two, and for long rows of unequal length; four otherwise, two workgroups to
// a unit.  Four against eight waves: block-sparse, t = 256 8 x 1000 13.3 / 10.7 us, 1 x 8192 (1312, 4672 keys) 18.6 / 13.9, 48 / 32; t = 375
// 1 x 12000 (1312, 4672) 22.5 / 24.9, 52 / 56, 8 x 1500 (960, 1312) 15.2 / 17.5, 17.9 / 17.3, 4 x 3000 (2624) 30 / 25, 2 x 6000 (4672) 49 / 35; t = 500 8 x 2000
// 18.5 / 22.1; dense, 32 x 256 6.4 / 6.8, 8 x 1000 12.0 / 10.2, 1 x 16K 140 / 99, 8 x 2000 21.5 / 19.9, 32 x 500 9.2 / 11.5, 8 x 3000 32 / 38.
int attn_bf16_rows_waves(const Shape& sh, bool sparse) {
    const long long tiles = attn_bf16_row_tiles(sh, sparse, kRowsTQ), keys = listed_keys(sh);
    const bool eight = sparse ? tiles <= 270 || (tiles <= 400 && 10ll * sh.n <= 13 * keys)
                              : (tiles <= 270 && sh.n >= 512) || (tiles <= 520 && sh.n >= 1024);
    return eight ? 8 : 4;
}

hipError_t launch_attn_bf16_rows(const Shape& sh, ArgsB a, hipStream_t st) {
    const bool sparse = a.idx != nullptr;
    a.qtiles = rows_qtiles(sh, sparse);
    const unsigned grid = (unsigned)rows_grid(sh, sparse);
    const int waves = attn_bf16_rows_waves(sh, sparse);
    if (!sparse) return launch_waves<2>(sh, a, waves, grid, st);
    return sh.b % 16 == 0 ? launch_waves<1>(sh, a, waves, grid, st) : launch_waves<0>(sh, a, waves, grid, st);
}

}  // namespace cp
