// fp32 attention: Algorithm 2's per-segment loop over a block list, or Eq. 2 dense causal attention when no list is
// given.  fp32 operands, products and sums throughout (v_mfma_f32_16x16x4_f32 is an fp32 fused multiply-add).
//
// A workgroup owns 16 * RT query rows of one segment (sparse) or of the sequence (dense); its W waves split the KEYS:
// wave w takes tiles w, w + W, ... of 16 keys, with a running max, sum and output of its own, and the W partial
// results are merged through LDS at the end.  Per wave and tile:
//
//   S^T[key][q]  = K . Q^T      A = K rows, B = Q rows; both sides take the channels in the order 16*kk + 4*g + e
//                               (g = lane group), so that one 16-byte load per lane feeds four MFMAs
//   softmax                     one query per lane column, keys 4*g + r: in-lane, then over the four lane groups
//   O^T[ch][q]  += V^T . P^T    B = P^T is the S^T accumulator as it stands (MFMA r contracts keys 4*g + r); A = V, whose
//                               rows come in as 16-byte pieces: channel tile (half, e) holds channels 64*half + 4*i + e
//
// K and V go from memory straight to registers: the waves of a workgroup read different keys, so there is nothing to
// share through LDS, and the fp32 matrix rate is a sixteenth of the bf16 one: 16 KB per 2048 * RT matrix cycles and wave
// are 16 (RT = 2, MODE 0) to 32 (RT = 1) bytes per clock and compute unit, within what L2 delivers.  V of a tile is asked for
// before its QK, K of the next tile before its softmax and PV.
//
// Values: a wave takes its weights relative to the true max of the row among its keys, so they are at most 1, and weights down to
// the smallest subnormal count; O overflows for |V| above 3.4e38 / (number of keys) at the earliest.  (A max that may outgrow its
// reference by 2^8, as in the bf16 kernel, saves most rescalings of O, 4 % of the time, and overflows 256 times earlier.)
//
// This kernel takes the launches that are too small for attn_fp32_split.hip, and the block sizes and strides that are not for it.
//
// What bounds it: latency, where few workgroups fill the chip (one head x 2048 tokens, 384 keys: 9.8 us, against 85 of a vector-FMA loop over
// 32 x 32 tiles in LDS), and the fp32 matrix instructions, which share their units with the vector instructions (measured: a wave's softmax and address
// arithmetic add their time to the MFMAs of all waves of the SIMD).  So the key loop keeps them few: tiles of 16 consecutive tokens with their
// addresses on the scalar unit (MODE 1/2), O rescaled only in tiles where some row's max moves.
#include "attn_fp32.h"

namespace cp {
namespace {

__device__ __forceinline__ float group_max(float x) {               // over the four lane groups: lanes l, l^16, l^32, l^48
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// C workgroups (blockIdx.y) share a row tile, each with its part of the channels of V and O: see attn_fp32_tile_parts.
// MODE 0: any block size and any stride (dense if there is no list): every key of a tile has a token of its own.  MODE 1: sparse, block size a multiple of
// 16: a tile is 16 consecutive tokens, described by its first token on the scalar unit.  MODE 2: dense.
// PAIRS: two workgroups to a compute unit in the order of TileOrder, whose arithmetic the other launches do without (0.1 to 0.35 us of 10 to 30).
template <int MODE, int RT, int W, int C, bool PAIRS>
__global__ __launch_bounds__(64 * W, MODE == 0 ? 1 : 4 - RT) void attn_fp32_kernel(Args32 a) {
    ask_for(a.q, a.k, a.v, a.idx, a.cnt, a.batch, a.n, a.qtiles, a.shared_lists, a.scale_log2e, a.qs0, a.qs1, a.qs2, a.ks0, a.ks1, a.ks2);
    constexpr bool RUN = MODE != 0;
    constexpr int TQ = 16 * RT, TK = 16;
    constexpr int kNoToken = 0x7fffffff;                            // a key that does not exist: after every query
    const bool dense = MODE == 2 || (MODE == 0 && !a.idx);
    constexpr int CH = kHeadDim / C, CHUNKS = CH / 4;               // channels of the output
    const int part = C > 1 ? blockIdx.y : 0;
    constexpr int PIECES = CH / 64;                                 // a lane's floats of a row of V: PIECES of four, 64 apart
    __shared__ __attribute__((aligned(1024))) float part_o[W * TQ * CH];     // 16-byte chunks XOR-swizzled by the row
    __shared__ float part_m[W * TQ], part_l[W * TQ];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, g = lane >> 4;

    // Consecutive workgroups walk the KV heads, so that a head's keys stay with few XCDs (workgroup id mod 8); the tiles
    // with most keys, those at the end of the sequence, come first.
    const int G = a.hq / a.hkv, bkv = a.batch * a.hkv;
    const unsigned wg = PAIRS ? a.order.place(blockIdx.x) : blockIdx.x;
    const int x = wg % bkv, y = wg / bkv;
    const int bb = x / a.hkv, kvh = x % a.hkv, h = kvh * G + y % G;
    int j, q_lo;
    if (PAIRS && !dense) {
        const TileOrder::Item item = a.order.item(y / G, a.n1, a.qtiles);
        j = item.segment; q_lo = j * a.s + item.tile * TQ;
    } else {
        const int item = (dense ? a.qtiles : a.n1 * a.qtiles) - 1 - y / G;
        j = dense ? 0 : item / a.qtiles;
        q_lo = dense ? item * TQ : j * a.s + item % a.qtiles * TQ;
    }
    const int q_end = dense ? a.n : min(a.n, (j + 1) * a.s);       // rows >= q_end do not exist
    if (q_lo >= q_end) return;                                     // uniform: tile past a short segment
    const int q_last = min(q_end, q_lo + TQ) - 1;
    const float* kp = a.k + bb * a.ks0 + kvh * a.ks1;
    const float* vp = a.v + bb * a.ks0 + kvh * a.ks1 + part * CH;

    scalar_list list = nullptr; int count = 0;
    if (!dense) {
        const long long lrow = a.shared_lists ? ((long long)bb * a.hkv + kvh) * a.n1 + j : ((long long)bb * a.hq + h) * a.n1 + j;
        list = (scalar_list)(unsigned long long)(a.idx + lrow * a.list_len);
        count = min(max(((scalar_list)(unsigned long long)a.cnt)[lrow], 0), a.list_len);
    }
    f32x4 qf[RT][8];
    // MODE 1/2: Q comes by whole rows to LDS, once per workgroup, 16-byte chunks XOR-swizzled by the row, and into registers from there: a lane per row
    // straight from memory, by every wave for itself, asks the address unit for 512 * W pieces of 16 bytes, one a cycle.  One head x 2048
    // tokens, block-sparse (384 keys) 12.1 -> 11.6 us, dense 42.2 -> 40.6, x 512 dense 14.1 -> 13.1.  (K and V the same way, with a tile of
    // each in LDS, 14.8: with one wave to a SIMD the way through LDS costs more than the address unit did.)
    const unsigned lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)part_o;
    if (RUN) {
        static_assert(!RUN || (RT == 1 && W * CH >= kHeadDim), "16 rows of Q take the place of partial Os");
        const int l32 = lane & 31, hh = lane >> 5;
#pragma unroll
        for (int x = 0; x < 8 / W; ++x) {
            const int i = wave * (8 / W) + x;
            copy16_far((const char*)(a.q + bb * a.qs0 + h * a.qs1 + (long long)min(q_lo + 2 * i + hh, q_last) * a.qs2) + (((unsigned)(l32 ^ hh) << 4) ^ (32 * i)), lds + i * 1024);
        }
    } else {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int row = q_lo + 16 * rt + c16;
            const float* src = a.q + bb * a.qs0 + h * a.qs1 + (long long)min(row, q_last) * a.qs2 + 4 * g;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) qf[rt][kk] = *(const f32x4*)(src + 16 * kk);
        }
    }
    // positions 0 .. total-1 of the listed blocks laid end to end (host checks list_len * b < 2^31)
    const unsigned total = dense ? (unsigned)q_last + 1u : (unsigned)count * (unsigned)a.b;
    const int ntiles = (int)((total + TK - 1) / TK);

    // ---- MODE 1/2: first token of the wave's next tile, -1 past its last one; t: the dense tile --------------------
    unsigned walk_e = 0, walk_off = 0;                              // list entry and offset inside its block of the next tile
    if (MODE == 1) { walk_e = (unsigned)wave * TK / (unsigned)a.b; walk_off = (unsigned)wave * TK % (unsigned)a.b; }
    const unsigned step_e = MODE == 1 ? W * TK / (unsigned)a.b : 0, step_off = MODE == 1 ? W * TK % (unsigned)a.b : 0;
    const int n2 = MODE == 1 ? (a.n + a.b - 1) / a.b : 0;
    auto next_base = [&](int t) -> int {                            // call in tile order: t = wave, wave + W, ...
        if (MODE == 2) return t < ntiles ? t * TK : -1;
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
    // ---- MODE 0: token of the lane's key c16 of tile t ---------------------------------------------------------
    auto key_token = [&](int t) -> int {
        const unsigned p = (unsigned)t * TK + c16;
        if (dense) return p < total ? (int)p : kNoToken;
        const unsigned e = p / (unsigned)a.b;
        const int blk = ((const int32_t*)(unsigned long long)list)[min(e, (unsigned)max(count - 1, 0))];
        const long long tk = (long long)blk * a.b + p % (unsigned)a.b;
        return t < ntiles && e < (unsigned)count && blk >= 0 && tk < a.n ? (int)tk : kNoToken;
    };

    f32x4 kf[8], vf[4][PIECES];
    auto load_k = [&](const float* rows, unsigned off) {            // 32-bit byte offset from a wave-uniform address (MODE 1/2)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) kf[kk] = *(const f32x4*)((const char*)rows + off + 64 * kk);
    };
    auto load_v = [&](int r, const float* rows, unsigned off) {
#pragma unroll
        for (int hf = 0; hf < PIECES; ++hf) vf[r][hf] = *(const f32x4*)((const char*)rows + off + 256 * hf);
    };
    // MODE 1/2: the lane's offsets inside a tile of 16 existing tokens.  In the last, ragged tile of the sequence the rows
    // past its end repeat the last token; they lie after every query and are masked.
    const unsigned row_bytes = (unsigned)a.ks2 * 4u;
    const unsigned k_full = c16 * row_bytes + 16 * g;
    unsigned v_full[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v_full[r] = (4 * g + r) * row_bytes + 16 * c16;
    auto load_k_run = [&](int base) {
        const int b0 = max(base, 0);
        unsigned off = k_full;
        if (b0 + TK > a.n) off = min(c16, a.n - 1 - b0) * row_bytes + 16 * g;
        load_k(kp + (long long)b0 * a.ks2, off);
    };
    auto load_v_run = [&](int base) {
        unsigned off[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) off[r] = v_full[r];
        if (base + TK > a.n) {
#pragma unroll
            for (int r = 0; r < 4; ++r) off[r] = min(4 * g + r, a.n - 1 - base) * row_bytes + 16 * c16;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) load_v(r, vp + (long long)base * a.ks2, off[r]);
    };
    auto load_k_token = [&](int tok) { load_k(kp + (long long)(tok == kNoToken ? 0 : tok) * a.ks2 + 4 * g, 0u); };

    f32x4 o[RT][PIECES][4];
    float m[RT], l[RT];                                             // m: running max of the raw logits
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m[rt] = -INFINITY; l[rt] = 0.f;
#pragma unroll
        for (int hf = 0; hf < PIECES; ++hf)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[rt][hf][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    int base = -1, tok = kNoToken;
    if (RUN) {
        base = next_base(wave); load_k_run(base);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");            // the wave's share of Q has landed; K is younger
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[0][kk] = *(__attribute__((address_space(3))) const f32x4*)(uintptr_t)(lds + c16 * 512 + (((4 * kk + g) ^ c16) << 4));
    }
    else { tok = key_token(wave); load_k_token(tok); }
    // ascending lists: nothing is visible from the tile on whose first token is past the last row
    auto more = [&](int t) -> bool {
        if (RUN) return base >= 0 && base <= q_last;
        const int first = __builtin_amdgcn_readfirstlane(tok);
        return t < ntiles && (first <= q_last || first == kNoToken);
    };
    for (int t = wave; more(t); t += W) {
        const int nbase = RUN ? next_base(t + W) : 0;
        int ktok[4];                                                // MODE 0: the tokens of the accumulator rows 4*g + r
        if (RUN) load_v_run(base);
        else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                ktok[r] = __shfl(tok, 4 * g + r);
                load_v(r, vp + (long long)(ktok[r] == kNoToken ? 0 : ktok[r]) * a.ks2 + 4 * c16, 0u);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 s[RT][2 / RT];                                        // two accumulator chains in flight
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 2 / RT; ++i) s[rt][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    s[rt][e % (2 / RT)] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kk][e], qf[rt][kk][e], s[rt][e % (2 / RT)], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const bool hidden = RUN ? base + TK - 1 > q_lo : __ballot(tok > q_lo) != 0;      // by some row
        const bool missing = !RUN && __ballot(tok == kNoToken) != 0;
        if (RUN) load_k_run(nbase);
        else { tok = key_token(t + W); load_k_token(tok); }
        __builtin_amdgcn_sched_barrier(0);

#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if (RT == 1) s[rt][0] += s[rt][2 / RT - 1];
            f32x4& z = s[rt][0];
            if (hidden) {
                const int qpos = q_lo + 16 * rt + c16;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if ((RUN ? base + 4 * g + r : ktok[r]) > qpos) z[r] = -INFINITY;
            }
            float mx = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
            // weights are taken from the row's true max, so that no P is above 1 and O grows no faster than the sum of |V|
            const float m_new = fmaxf(m[rt], group_max(mx));
            const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
            float alpha = (m[rt] - m_safe) * a.scale_log2e;
#pragma unroll
            for (int r = 0; r < 4; ++r) z[r] = (z[r] - m_safe) * a.scale_log2e;
            if (__ballot(fminf(fminf(fminf(z[0], z[1]), fminf(z[2], z[3])), alpha) < -126.f) == 0) {
                alpha = __builtin_amdgcn_exp2f(alpha);
#pragma unroll
                for (int r = 0; r < 4; ++r) z[r] = __builtin_amdgcn_exp2f(z[r]);
            } else {                                                // v_exp_f32 has no subnormal results, exp2f does
                alpha = exp2f(alpha);
#pragma unroll
                for (int r = 0; r < 4; ++r) z[r] = exp2f(z[r]);
            }
            l[rt] = l[rt] * alpha + ((z[0] + z[1]) + (z[2] + z[3]));   // the lane's own keys; the lane groups are added at the end
            m[rt] = m_new;
            if (__ballot(alpha != 1.0f) != 0) {
#pragma unroll
                for (int hf = 0; hf < PIECES; ++hf)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[rt][hf][e] *= alpha;
            }
        }
        if (missing) {                                              // 0 * V must be 0, whatever token 0 holds
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (ktok[r] == kNoToken) {
#pragma unroll
                    for (int hf = 0; hf < PIECES; ++hf) vf[r][hf] = 0.f;
                }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int hf = 0; hf < PIECES; ++hf)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        o[rt][hf][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][hf][e], s[rt][0][r], o[rt][hf][e], 0, 0, 0);
        base = nbase;
    }

    if (RUN) __syncthreads();                                       // everybody has read Q
    // ---- merge the W partial results: out = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w ----------------------
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        l[rt] += __shfl_xor(l[rt], 16); l[rt] += __shfl_xor(l[rt], 32);
        const int row = 16 * rt + c16;
        if (g == 0) { part_m[wave * TQ + row] = m[rt]; part_l[wave * TQ + row] = l[rt]; }
        float* dst = part_o + (wave * TQ + row) * CH;
#pragma unroll
        for (int hf = 0; hf < PIECES; ++hf)
#pragma unroll
            for (int r = 0; r < 4; ++r) {                           // channels 64*hf + 16*g + 4*r .. +3
                const int chunk = (16 * hf + 4 * g + r) ^ (c16 & (CHUNKS - 1));
                *(f32x4*)(dst + 4 * chunk) = f32x4{o[rt][hf][0][r], o[rt][hf][1][r], o[rt][hf][2][r], o[rt][hf][3][r]};
            }
    }
    __syncthreads();
    float* op = a.out + bb * a.os0 + h * a.os1 + part * CH;
#pragma unroll
    for (int c = 0; c < (TQ * CHUNKS + 64 * W - 1) / (64 * W); ++c) {
        const int row = (c * 64 * W + tid) / CHUNKS, chunk = tid % CHUNKS;
        if (row >= TQ) break;                                       // eight waves, half of the channels
        float M = -INFINITY, L = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, part_m[w * TQ + row]);
        const float M_safe = (M == -INFINITY) ? 0.f : M;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float f = exp2f((part_m[w * TQ + row] - M_safe) * a.scale_log2e);
            L += f * part_l[w * TQ + row];
            sum += f * *(const f32x4*)(part_o + (w * TQ + row) * CH + 4 * (chunk ^ (row & 15 & (CHUNKS - 1))));
        }
        const int qpos = q_lo + row;
        if (qpos < q_end) {
            const float inv = L > 0.f ? 1.0f / L : 0.f;
            *(f32x4*)(op + (long long)qpos * a.os2 + 4 * chunk) = sum * inv;
            if (a.lse && chunk == 0 && part == 0)
                a.lse[((long long)bb * a.hq + h) * a.n + qpos] = L > 0.f ? M * a.scale + logf(L) : -INFINITY;
        }
    }
}

template <int MODE, int RT, int W, int C>
hipError_t launch(const Shape& sh, Args32& a, hipStream_t st) {
    const bool sparse = a.idx != nullptr;
    const dim3 grid((unsigned)attn_fp32_grid(sh, sparse, 16 * RT), C);
    a.qtiles = attn_fp32_qtiles(sh, sparse, 16 * RT);
    if constexpr (MODE != 0 && W == 4 && C == 1) {
        a.order = attn_fp32_order(sh, sparse, 16 * RT, W);
        if (a.order.turn) {
            hipLaunchKernelGGL((attn_fp32_kernel<MODE, RT, W, C, true>), grid, dim3(64 * W), 0, st, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((attn_fp32_kernel<MODE, RT, W, C, false>), grid, dim3(64 * W), 0, st, a);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_tiled(const Shape& sh, Args32& a, hipStream_t st) {
    const bool sparse = a.idx != nullptr, eight = attn_fp32_tile_waves(sh, sparse) == 8;
    if (attn_fp32_tile_parts(sh, sparse) == 2) return eight ? launch<MODE, 1, 8, 2>(sh, a, st) : launch<MODE, 1, 4, 2>(sh, a, st);
    return eight ? launch<MODE, 1, 8, 1>(sh, a, st) : launch<MODE, 1, 4, 1>(sh, a, st);
}

}  // namespace

// 16 rows to a workgroup: what is left to this kernel are launches that 32 rows would not fill the chip with, or not evenly (attn_fp32_split_better).
// Eight waves split a long row further, four are better where rows are short.  Attention alone, us, four / eight waves (row tiles in brackets): dense 8
// heads x 512 tokens (256) 13.5 / 14.6, 1 x 3000 (188) 57.5 / 56.2; block-sparse 1 x 2100 (132; 384 keys) 12.0 / 12.4, 1 x 3000 (188; 1056) 25.4 / 24.0,
// 1 x 4000 (250; 1216) 28.3 / 27.2, 2 x 1500 (188; all keys) 34.1 / 31.8.  Rows of more than 1024 keys have eight at any number of tiles, because their
// sums are longer with four: 1 head x 1025 to 2048 tokens is 3.49e-7 from float64 with four, 3.15e-7 with eight (four in the two workgroups of
// attn_fp32_tile_parts would take up to 6 % less: dense 1 x 1025 19.3 / 20.4, 1 x 2048 34.3 / 35.9; block-sparse 1 x 1500 (94; 1280) 27.6 / 28.1, 1 x
// 2048 (128; all keys) 36.4 / 36.2).
int attn_fp32_tile_waves(const Shape& sh, bool sparse) {
    return (sparse ? min((long long)sh.n, (long long)sh.list_len * sh.b) : sh.n) > 1024 ? 8 : 4;
}

// Up to 128 row tiles two workgroups take a tile, each with half of its channels of V and O: the products of Q and K are made twice, 48 matrix
// instructions a tile of keys instead of 64, on compute units that would be idle.  One / two workgroups (row tiles), the same bits: block-sparse 1 x
// 2048 (128; 384 keys) 11.6 / 10.2, 1 x 915 (58, all keys) 22.4 / 18.8, 2 x 1000 (126; 640) 16.5 / 13.9, 1 x 1500 (94; 768) 18.9 / 16.1; dense 1 x 512
// (32) 13.0 / 11.0, 3 x 600 (114) 15.4 / 13.1, 1 x 2048 (128) 40.1 / 35.9. Above, some units get two: 3 x 1300 (246) 23.8 / 36.2, 2 x 1500 (188) 31.4 /
// 44.4.  Four workgroups gain no more on 64 tiles and less (1 x 915 18.6, dense 1 x 1000 19.4 against 19.0).
int attn_fp32_tile_parts(const Shape& sh, bool sparse) { return attn_fp32_row_tiles(sh, sparse, 16) <= 128 ? 2 : 1; }

hipError_t launch_attn_fp32(const Shape& sh, const void* q, const void* k, const void* v, const int32_t* idx,
                            const int32_t* cnt, bool shared_lists, void* out, float* lse, hipStream_t st) {
    Args32 a;
    a.q = (const float*)q; a.k = (const float*)k; a.v = (const float*)v; a.idx = idx; a.cnt = cnt;
    a.out = (float*)out; a.lse = lse;
    a.batch = sh.batch; a.hq = sh.hq; a.hkv = sh.hkv; a.n = sh.n; a.s = sh.s; a.b = sh.b; a.n1 = sh.n1; a.list_len = sh.list_len;
    a.shared_lists = shared_lists ? 1 : 0;
    a.scale = sh.attn_scale; a.scale_log2e = sh.attn_scale * 1.4426950408889634f;
    a.qs0 = sh.qs[0]; a.qs1 = sh.qs[1]; a.qs2 = sh.qs[2];
    a.ks0 = sh.kvs[0]; a.ks1 = sh.kvs[1]; a.ks2 = sh.kvs[2];
    a.os0 = sh.os[0]; a.os1 = sh.os[1]; a.os2 = sh.os[2];
    const bool near = sh.kvs[2] < (1 << 26);                        // a tile's rows are within 32-bit byte offsets of its first
    if (attn_fp32_split_better(sh, idx != nullptr)) return launch_attn_fp32_split(sh, a, st);
    if (!idx && near) return launch_tiled<2>(sh, a, st);
    if (idx && near && sh.b % 16 == 0) return launch_tiled<1>(sh, a, st);
    return launch<0, 2, 4, 1>(sh, a, st);
}

}  // namespace cp
