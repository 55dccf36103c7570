// bf16 MFMA flash attention over a block list with 128-row workgroups of four waves, two to a compute unit: for segments that leave part of a
// 256-row workgroup (attn_bf16.hip) empty, and for launches of short lists.  Block sizes are multiples of 16.
//
// The arithmetic and the split inside a workgroup are those of the 256-row kernel, and so are the results, bit for bit: a wave owns 32 query rows, K
// and V tiles of 64 keys go to LDS by global_load_lds, S^T = K . Q^T, softmax with one query per lane column, O^T += V^T . P^T with V through the
// transposing LDS read.  A wave alternates between a matrix phase, PV(t-1) interleaved with QK(t), and the softmax of tile t.  Its partner on the
// SIMD is a wave of the unit's other workgroup, at a phase of its own; the two share nothing, so the prologue and the epilogue of one run under the
// key loop of the other.
//
// LDS: two slots each for K and V (64 KiB) and the tiles' descriptions, so that two workgroups fit.  Step t asks for V(t) and K(t+1), whose slots were
// read for the last time in step t-1, behind its matrix phase and waits for them at its end: one barrier per step.  Asked for before the matrix phase
// they delay it: 32 heads x 8192 tokens (segments of 128, 416 keys) 83.0 against 75.5 us, 2 x 8 x 93184 (672 keys) 614 against 603; only for long
// lists it is the better place (4256 keys 427 against 442).
//
// What bounds it: neither the matrix pipe (37 % busy) nor the vector unit (35 %) nor the caches (6.8 TB/s) alone, at a power-bound clock of 2.0 GHz: two waves to a SIMD take
// turns at phases that depend on each other, and short items start and end often.  It reads the keys twice as often as the 256-row kernel and is 7 to 15 %
// slower where that has no empty waves.  2 x 8 x 93184 tokens: 466 GFLOP in 581 us, 0.80 PFLOP/s; the 32-row kernel, which reads the keys four
// times as often, took 988.
#include "attn_bf16.h"

#include <algorithm>

namespace cp {
namespace {

constexpr int TQ = 128, WQ = 32, TK = 64;         // query rows of a workgroup and of a wave; keys of a tile
constexpr int kWaves = TQ / WQ;
constexpr int kTileBytes = TK * 256;
constexpr int kKOff = 0, kVOff = 2 * kTileBytes;  // two slots each
constexpr int kTabOff = 4 * kTileBytes;           // sparse: first tokens of the four runs of every tile
constexpr int kTabMax = 12 * 1024;                // of 80 KiB: lists of up to 49152 keys.  Longer ones are for the other two kernels, with segments of 65 to 128
                                                  // rows for the 32-row one, which takes 1.3 times the time (4256 keys)
constexpr int kOutPitch = 272;                    // epilogue staging: one output row + 16 B, in bytes
constexpr unsigned kRound = 512;                  // workgroups that the chip holds
constexpr int kLook = 3;                          // LDS fragments read ahead of their MFMAs
static_assert(kWaves * WQ * kOutPitch <= 4 * kTileBytes, "epilogue staging reuses the slots");

// A tile is four runs of 16 consecutive tokens, described by their first tokens (-1: no such tokens): four copies of 16 bytes per lane, from a base each, 4 KiB apart in LDS (see dma16)
__device__ __forceinline__ void dma16_runs(const void* b0, const void* b1, const void* b2, const void* b3, unsigned voff, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, %3\n\ts_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\t"
                 "s_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5" ::"s"(lds_base), "v"(voff), "s"(b0), "s"(b1), "s"(b2), "s"(b3)
                 : "memory", "scc");
}

__global__ __launch_bounds__(64 * kWaves, 2) void attn_bf16_half_kernel(ArgsIndex ix, ArgsB a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int tid = thread_id(), lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // every argument in one go, as in the 256-row kernel
    ask_for(ix.order.full, ix.order.by_kv.shift, ix.div_hkv.mul, ix.div_b.mul, a.q, a.k, a.v, a.idx, a.cnt, a.n, a.s, a.qs0, a.qs1, a.qs2, a.ks0, a.ks1, a.ks2, a.list_len,
            a.scale_log2e);
    const WorkOrder::Item item = ix.order.item(workgroup_id(), kRound, (unsigned)a.group, (unsigned)a.n1, (unsigned)a.qtiles);
    const int bb = (int)ix.div_hkv.div((unsigned)item.bkv), g = item.bkv - bb * a.hkv, h = g * a.group + item.gq, j = item.segment, qt = item.tile;
    const int q_lo = j * a.s + qt * TQ;
    const int q_end = min(a.n, (j + 1) * a.s);
    if (q_lo >= q_end) return;                                   // uniform: tile past a short segment
    const int q_last = min(q_end, q_lo + TQ) - 1;
    int wq_lo = q_lo + WQ * wave;
    asm("" : "+v"(wq_lo));                                       // what a wave sees of a tile stays in vector registers, as in the 256-row kernel
    const int wq_last = min(q_end, wq_lo + WQ) - 1;              // < wq_lo when the wave has no rows
    const int qpos = wq_lo + l32;

    const uint16_t* qp = a.q + bb * a.qs0 + h * a.qs1;
    const uint16_t* kp = uniform_ptr(a.k + bb * a.ks0 + g * a.ks1);
    const uint16_t* vp = uniform_ptr(a.v + bb * a.ks0 + g * a.ks1);
    const int r4 = lane >> 4, pch = lane & 15;                   // row inside a copy's four rows, chunk the lane's 16 bytes land in

    // ---- Q: the wave's 32 rows as whole rows to LDS (where V comes later), swizzled like K
    const unsigned q_lds = lds0 + kVOff + wave * (WQ * 256);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 4 * i + r4;                              // rows past the end repeat the last one
        dma16_far((const char*)(qp + (long long)min(q_lo + WQ * wave + row, q_last) * a.qs2) + ((pch ^ (row & 15)) << 4), q_lds + i * 1024);
    }
    // ---- the runs of all tiles, worked out once by all threads -----------------------------------------------
    const long long lrow = a.shared_lists ? ((long long)bb * a.hkv + g) * a.n1 + j : ((long long)bb * a.hq + h) * a.n1 + j;
    const int32_t* list = uniform_ptr(a.idx + lrow * a.list_len);
    const int cnt = *(scalar_list)(unsigned long long)uniform_ptr(a.cnt + lrow);
    const int count = min(max(cnt, 0), a.list_len);
    int ntiles = (int)(((unsigned)count * (unsigned)a.b + TK - 1) / TK);
    const int blocks = (int)ix.div_b.div((unsigned)(a.n + a.b - 1));
    for (int x = tid; x < 4 * ntiles; x += 64 * kWaves) {
        const unsigned p = 16u * (unsigned)x, e = ix.div_b.div(p);
        const int blk = list[min(e, (unsigned)a.list_len - 1u)];
        const int tok = blk * a.b + (int)(p - e * (unsigned)a.b);
        // entries outside the sequence have no tokens
        *LDS_PTR(int, lds0 + kTabOff + 4 * x) = e < (unsigned)count && blk >= 0 && blk < blocks && tok < a.n ? tok : -1;
    }
    __syncthreads();
    while (ntiles > 0) {                                     // trailing tiles that no row sees: lane l looks at the l-th last one
        const i32x4 d = *LDS_PTR(const i32x4, lds0 + kTabOff + 16 * max(ntiles - 1 - lane, 0));
        bool sees = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) sees |= d[i] >= 0 && d[i] <= q_last;
        const unsigned long long seen = __builtin_amdgcn_ballot_w64(sees && lane < ntiles);
        ntiles -= seen ? (int)__builtin_ctzll(seen) : min(ntiles, 64);
        if (seen) break;
    }
    ntiles = __builtin_amdgcn_readfirstlane(ntiles);
    struct Runs { int at[4]; };
    auto runs_of = [&](int t) -> Runs {
        Runs r;
        const i32x4 d = *LDS_PTR(const i32x4, lds0 + kTabOff + 16 * t);
#pragma unroll
        for (int i = 0; i < 4; ++i) r.at[i] = __builtin_amdgcn_readfirstlane(d[i]);
        return r;
    };
    // ---- tile loader: the wave fills rows 16*i + 4*wave .. + 3 ----------------------------------------------
    const unsigned tok_bytes = (unsigned)a.ks2 * 2u;             // host checks n * tok_bytes < 2^32, both < 2^24
    const unsigned kch = (unsigned)(pch ^ (4 * wave + r4)) << 4, vch = (unsigned)(pch ^ (4 * r4)) << 4;   // swizzles: row & 15, 4 * (row & 3)
    const unsigned lane_row = (unsigned)(4 * wave + r4) * tok_bytes;
    auto issue = [&](const uint16_t* base, unsigned chunk, const Runs& r, unsigned to) {
        const int most = max(max(r.at[0], r.at[1]), max(r.at[2], r.at[3])), least = min(min(r.at[0], r.at[1]), min(r.at[2], r.at[3]));
        if (least >= 0 && most <= a.n - 16) {                    // uniform: all runs exist in full
            const char* at = (const char*)base;
            dma16_runs(at + (unsigned)r.at[0] * tok_bytes, at + (unsigned)r.at[1] * tok_bytes, at + (unsigned)r.at[2] * tok_bytes,
                       at + (unsigned)r.at[3] * tok_bytes, lane_row + chunk, to + 4 * wave * 256);
            return;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = r.at[i];                              // rows without a token read token 0 or the last one, masked later
            dma16(base, mul24(at < 0 ? 0u : (unsigned)min(at + 4 * wave + r4, a.n - 1), tok_bytes) + chunk, to + (16 * i + 4 * wave) * 256);
        }
    };

    // ---- per-lane LDS read addresses, in the slot that is read next ------------------------------------------
    unsigned ka[8], va[4];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) ka[ks] = ((lds0 + kKOff + l32 * 256) | (unsigned)(((l32 & 15) ^ hh) << 4)) ^ (ks << 5);
    const int i16 = lane & 15, gbit = (lane >> 4) & 1;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
        va[dt] = lds0 + kVOff + (4 * hh + (i16 >> 2)) * 256 + ((((unsigned)(dt ^ (i16 >> 2)) << 2) + 2 * gbit + ((i16 & 3) >> 1)) << 4) + (i16 & 1) * 8;
    f32x16 o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float c = a.scale_log2e, lazy_raw = kLazyLog2 / c;
    bf16x8 qf[8];

    // ---- the phases: fragment j of kind 0: QK alone (16), 1: PV alone (16), 2: PV interleaved with QK in groups of four (32)
    bf16x8 ring[kLook + 1];
    auto frag_read = [&](int kind, int j, bf16x8& f) __attribute__((always_inline)) {
        const bool is_v = kind == 1 || (kind == 2 && (j & 7) < 4);
        if (is_v) {
            const unsigned ad = va[j & 3] + (kind == 1 ? j >> 2 : j >> 3) * 16 * 256;
            const v4bf16_lds lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(v4bf16_lds, ad));
            const v4bf16_lds hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(v4bf16_lds, ad + 8 * 256));
#pragma unroll
            for (int e = 0; e < 4; ++e) { f[e] = lo[e]; f[4 + e] = hi[e]; }
        } else {
            const int ks = kind == 0 ? j >> 1 : 2 * (j >> 3) + (((j & 7) - 4) >> 1);
            f = as_bf16x8(*LDS_PTR(const u32x4, ka[ks] + (j & 1) * 32 * 256));
        }
    };
    auto run_frags = [&](int kind, f32x16 (&s)[2], const bf16x8 (&pf)[4]) __attribute__((always_inline)) {
        const int n = kind == 2 ? 32 : 16;
        if (kind != 1) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
        }
#pragma unroll
        for (int j = 0; j < kLook; ++j) frag_read(kind, j, ring[j]);
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            if (j < n) {
                if (j + kLook < n) frag_read(kind, j + kLook, ring[(j + kLook) % (kLook + 1)]);
                const bf16x8& f = ring[j % (kLook + 1)];
                if (kind == 1 || (kind == 2 && (j & 7) < 4))
                    o[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pf[kind == 1 ? j >> 2 : j >> 3], o[j & 3], 0, 0, 0);
                else
                    s[j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[kind == 0 ? j >> 1 : 2 * (j >> 3) + (((j & 7) - 4) >> 1)], s[j & 1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // key row 16*run + kr of the tile is token at[run] + kr, visible up to min(qpos, n - 1); a missing run is masked whole
    auto mask = [&](f32x16 (&s)[2], const Runs& r) {
        const int top = min(qpos, a.n - 1) - 4 * hh;
#pragma unroll
        for (int run = 0; run < 4; ++run) {
            int lim = r.at[run] < 0 ? -1 : top - r.at[run];
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (8 * g2 + i > lim) s[run >> 1][8 * (run & 1) + 4 * g2 + i] = -INFINITY;
                    asm("" : "+v"(lim));                         // or each comparison is built on the others
                }
        }
    };
    // S^T tile -> P^T fragments; running max / sum; O rescaled where a row's max has outgrown its reference point by more than 2^kLazyLog2
    auto softmax = [&](f32x16 (&s)[2], bf16x8 (&pf)[4]) {
        float mx = fmaxf(s[0][0], s[0][1]), my = fmaxf(s[1][0], s[1][1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) {
            mx = fmaxf(fmaxf(s[0][r], s[0][r + 1]), mx);
            my = fmaxf(fmaxf(s[1][r], s[1][r + 1]), my);
        }
        mx = half_max(fmaxf(mx, my));
        const float m_new = (mx > m_run + lazy_raw) ? mx : m_run;
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_safe) * c);
        const float ms = m_safe * c;
        m_run = m_new;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kt][r] = __builtin_amdgcn_exp2f(fmaf(s[kt][r], c, -ms));
        bf16x2 one2; one2[0] = (__bf16)1.0f; one2[1] = (__bf16)1.0f;
        float rs0 = 0.f, rs1 = 0.f;                              // the row sum adds up the rounded values that PV uses
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[t4][e] = (__bf16)s[t4 >> 1][8 * (t4 & 1) + e];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                bf16x2 pr; pr[0] = pf[t4][e]; pr[1] = pf[t4][e + 1];
                if (e & 2) rs1 = __builtin_amdgcn_fdot2_f32_bf16(pr, one2, rs1, false);
                else rs0 = __builtin_amdgcn_fdot2_f32_bf16(pr, one2, rs0, false);
            }
        }
        l_run = l_run * alpha + (rs0 + rs1);                     // per-half partial sums, merged at the end
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
    };

    // ---- K of tile 0, Q to registers -------------------------------------------------------------------------
    Runs cur = runs_of(0), next = runs_of(ntiles > 1 ? 1 : 0);
    if (ntiles > 0) issue(kp, kch, cur, lds0 + kKOff);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = as_bf16x8(*LDS_PTR(const u32x4, q_lds + l32 * 256 + (((2 * ks + hh) ^ (l32 & 15)) << 4)));
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) pin(qf[ks]);
    __syncthreads();                                             // everybody's K, and nobody reads Q in LDS any more

    f32x16 s[2]; bf16x8 pf[4];
    bool have_p = false;                                         // P^T of tile t-1 waits for its PV
    int k_step = kTileBytes, v_step = -kTileBytes;               // to the other slot; step t reads K(t) and V(t-1)
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) va[dt] += kTileBytes;
    for (int t = 0; t < ntiles; ++t) {
        bool act = false, full = true;                           // a row of the wave sees a key; all of its rows see all of them
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            act |= cur.at[i] >= 0 && cur.at[i] <= wq_last;
            full &= cur.at[i] >= 0 && cur.at[i] + 15 <= wq_lo && cur.at[i] + 16 <= a.n;
        }
        __builtin_amdgcn_s_setprio(3);
        if (have_p && act) run_frags(2, s, pf);
        else if (act) run_frags(0, s, pf);
        else if (have_p) run_frags(1, s, pf);
        __builtin_amdgcn_s_setprio(0);
        issue(vp, vch, cur, lds0 + kVOff + (t & 1) * kTileBytes);
        if (t + 1 < ntiles) issue(kp, kch, next, lds0 + kKOff + ((t + 1) & 1) * kTileBytes);
        const i32x4 ahead = *LDS_PTR(const i32x4, lds0 + kTabOff + 16 * min(t + 2, ntiles - 1));
        if (act) {
            if (!full) mask(s, cur);
            softmax(s, pf);
        }
        have_p = act;
        cur = next;
#pragma unroll
        for (int i = 0; i < 4; ++i) next.at[i] = __builtin_amdgcn_readfirstlane(ahead[i]);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) ka[ks] += k_step;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) va[dt] += v_step;
        k_step = -k_step; v_step = -v_step;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    if (have_p) run_frags(1, s, pf);

    // ---- epilogue: O^T[ch][q] / l -> out[q][ch], transposed through LDS so that global stores are whole rows -----
    const float l_tot = half_sum(l_run);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    __syncthreads();                                             // every wave is past its last tile reads
    const unsigned stage = lds0 + wave * (WQ * kOutPitch);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
            bf16x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = (__bf16)(o[dt][4 * gg + i] * inv);
            *LDS_PTR(bf16x4, stage + l32 * kOutPitch + (32 * dt + 8 * gg + 4 * hh) * 2) = w;
        }
    uint16_t* ob = a.out + bb * a.os0 + h * a.os1;
#pragma unroll
    for (int x = 0; x < 8; ++x) {                                // the wave reads back only what it wrote itself
        const int row = 4 * x + r4;
        const u32x4 val = *LDS_PTR(const u32x4, stage + row * kOutPitch + pch * 16);
        if (wq_lo + row < q_end) *(u32x4*)(ob + (long long)(wq_lo + row) * a.os2 + pch * 8) = val;
    }
    if (a.lse && hh == 0 && qpos < q_end)
        a.lse[((long long)bb * a.hq + h) * a.n + qpos] = l_tot > 0.f ? m_run * a.scale + __logf(l_tot) : -INFINITY;
}

// LDS for the runs of every tile
long long table_bytes(const Shape& sh) { return ((long long)sh.list_len * sh.b + TK - 1) / TK * 16; }

}  // namespace

// The line lies where this kernel meets the other two (us, the better one of those / this one, all in the orders of work_order.h; t: row tiles of 32, w: 256-row
// workgroups).
//   Segments of 65 to 128 rows: 2 x 8 heads x 93184 tokens (672 keys) 978 / 580; 32 x 8192 (416, 1184, 4256) 122 / 71, 235 / 151, 589 / 393; blocks of 16,
//   32 x 20000 (672) 413 / 249, 32 x 60000 (3296) 4679 / 2942; segments of 96 157 / 122; t = 1400 to 1500: 16 x 2800 (1184) 40 / 34, 32 x 1500 29 / 22.  Below, lists
//   that are short beside the sequence: t = 750 to 1024: 8 x 3000 (672, 1184) 21.4 / 20.3, 27.2 / 31.1, 4 x 6000 (416, 1440) 16.9 / 14.9, 34.8 / 36.6, 8 x 4096
//   (416, 2208) 17.7 / 15.3, 47 / 53; t = 560 to 660: 2 x 9000 (672) 21.8 / 20.2, 4 x 4500 (416, 672) 16.0 / 14.7, 18.3 / 20.1, 2 x 10500 (2208) 50 / 53.
//   Up to 64 rows half of this kernel is empty too: 32 x 8192, segments of 64 156 / 167.
//   Segments that fill a quarter less of its workgroups: of 384 32 x 4096, 8192, 32768 (1440) 109 / 82, 205 / 168, 879 / 717, of 320 114 / 94, 239 / 196, 1010 / 816, of
//   288 118 / 108, 249 / 208, 1055 / 897; as much of either: of 192 32 x 8192 (480, 1248) 103 / 97, 193 / 198, 32 x 32768 (736) 527 / 545.
//   Else it reads the keys twice as often and loses (32 x 16384, segments of 512, 1600 keys 345 / 368, 32 x 50000 1069 / 1157), but not where 256-row
//   workgroups leave half of the chip idle (w = 128: 8 x 4000 (832, 1600) 24.0 / 23.0, 37.3 / 39.4, the better one of 256 rows 39.8; w = 188 to 256: 8 x 6000 25.7 / 26.3,
//   41.6 / 44.8, 32 x 1500 24.5 / 25.1, 8 x 8000 27.5 / 27.8, 45.3 / 47.8, 32 x 2000 26.2 / 26.8, 41.8 / 45.2, 16 x 4000 27.2 / 27.7, 44.0 / 47.1) and for short
//   lists of blocks of an odd multiple of 16, whose keys that kernel takes one by one: w = 512 (528, 784 keys) 46.0 / 41.2, 58.3 / 54.0, w = 2048 188 / 164, 240 / 221,
//   w = 6272 (336, 528) 419 / 360, 539 / 487; 1232 to 1296 keys, w = 512 to 1504 83 / 79, 171 / 160, 238 / 227, but w = 6272 1043 / 1054 and heads of
//   their own KV head 16/16 x 30000 (w = 2400; 400, 80; 1280) 377 / 388, x 131072 (w = 8752; 480, 48; 912) 1009 / 1020.
bool attn_bf16_half_better(const Shape& sh) {
    if (sh.b % 16 != 0 || table_bytes(sh) > kTabMax) return false;
    const long long tiles = attn_bf16_row_tiles(sh, true, WQ), wide = attn_bf16_row_tiles(sh, true, 256), halves = attn_bf16_row_tiles(sh, true, TQ);
    const long long keys = std::min((long long)sh.n, (long long)sh.list_len * sh.b);
    if (8 * wide >= 2 * tiles)                                   // half of the 256-row workgroups is empty
        return 8 * wide < 4 * tiles && (tiles >= 1400 || (tiles > 700 && 5ll * sh.n >= 22 * keys) || (tiles > 540 && sh.n >= 10 * keys));
    if (attn_bf16_rows_better(sh, true)) return false;
    if (wide <= 256) return halves <= 256;
    return 8 * wide >= 5 * halves || (sh.b % 32 != 0 && (keys <= 768 || (keys <= 1100 && wide <= 4200) || (keys <= 1300 && wide <= 1600)));
}

hipError_t launch_attn_bf16_half(const Shape& sh, ArgsB a, hipStream_t st) {
    ArgsIndex ix;
    ix.div_hkv = FastDiv(sh.hkv); ix.div_b = FastDiv(sh.b);
    a.qtiles = (std::min(sh.s, sh.n) + TQ - 1) / TQ;              // a segment may be set longer than the sequence
    ix.order = WorkOrder(sh.batch * sh.hkv, a.group, sh.n1, a.qtiles, kRound, attn_bf16_kv_bytes(sh));
    const int smem = kTabOff + (int)((table_bytes(sh) + 1023) & ~1023ll);
    const hipError_t e = hipFuncSetAttribute((const void*)attn_bf16_half_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_bf16_half_kernel, dim3((unsigned)((long long)sh.batch * sh.hq * sh.n1 * a.qtiles)), dim3(64 * kWaves), smem, st, ix, a);
    return hipGetLastError();
}

}  // namespace cp
