// Algorithm 2 "Pruned Attention", the line  I = argtop_k(S[j], B / block size),
// plus the local and diagonal blocks that are always kept.
//
// One wavefront per (batch, head, segment) row.  The row lives in registers (lane l owns blocks
// l, l+64, ...).  Scores are mapped to order-preserving unsigned keys; the k-th largest key is found
// by an MSB-first radix search (one wave-wide count per bit: a compare per key, the lane masks counted on the
// scalar unit) that stops at the first bit whose count is exactly k; everything above it is taken, ties at
// the threshold go to the smallest indices, and the result is compacted in index order, so the
// list comes out ascending.  Long rows are first thinned to the few keys that can be among the k largest; the longest are
// not held in registers but read twice.
#include "kernels.h"

namespace cp {
namespace {

struct SelectArgs {
    const float* scores; int32_t* idx; int32_t* cnt;
    long long rows;            // B*H*n1 lists (H = query heads, or KV heads when the lists are shared)
    int n1, n2, r, budget, local, list_len;
    int group;                 // shared lists: query heads per KV head, whose scores are merged by max
};


__device__ __forceinline__ uint32_t ordered_key(float x) {
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0;                       // -0 ranks with +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// key of block i for list row `row`: the row's own score, or (SHARED) the largest score of the block among the
// query heads of the row's KV head (scores [B, Hq, n1, n2], query head = KV head * group + member)
template <bool SHARED>
__device__ __forceinline__ uint32_t row_key(const SelectArgs& a, long long row, int j, int i) {
    if (!SHARED) return ordered_key(a.scores[row * a.n2 + i]);
    const long long bh = row / a.n1;
    uint32_t kx = 0;
    for (int g2 = 0; g2 < a.group; ++g2)
        kx = max(kx, ordered_key(a.scores[((bh * a.group + g2) * a.n1 + j) * a.n2 + i]));
    return kx;
}

__device__ __forceinline__ int wave_sum(int v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// The k-th largest of the wave's 64 * N keys (padding keys are 0 and never counted): MSB-first radix search, one
// wave-wide count per bit (a compare per key, the lane masks counted on the scalar unit).  It stops at the first
// bit whose count is exactly k: the keys at or above that trial value are then the k largest (the k-th and the
// (k+1)-th differ), and the value returned separates them just as well as the k-th key itself.
// Always: count(key >= result) >= k, provided k keys are non-zero.
template <int N>
__device__ __forceinline__ uint32_t kth_largest(const uint32_t (&key)[N], int k) {
    uint32_t thr = 0;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t trial = thr | (1u << bit);
        int c = 0;
#pragma unroll
        for (int m = 0; m < N; ++m) c += (int)__popcll(__ballot(key[m] >= trial));
        if (c >= k) thr = trial;
        if (c == k) break;
    }
    return thr;
}

// Writes, in slot order (slot m, then lane), the index of every key above thr and of the first keys equal to thr
// until k are taken; returns how many were written.  index(m) = the block index of the lane's key m.
template <int N, typename Index>
__device__ __forceinline__ int take_largest(const uint32_t (&key)[N], uint32_t thr, int k, int n_slots, int lane,
                                            int32_t* out, Index index) {
    int above = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) above += (int)__popcll(__ballot(key[m] > thr));
    int ties_left = k - above;                         // the keys equal to thr that still fit (0 if none is)
    int written = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        if (m >= n_slots) break;                        // wave-uniform
        const bool valid = key[m] != 0u;                // padding keys are 0, the key of a score never is
        const bool tie = valid && key[m] == thr;
        const unsigned long long tie_mask = __ballot(tie);
        const int tie_rank = __popcll(tie_mask & ((1ull << lane) - 1ull));
        const bool take = valid && (key[m] > thr || (tie && tie_rank < ties_left));
        const unsigned long long take_mask = __ballot(take);
        if (take) out[written + __popcll(take_mask & ((1ull << lane) - 1ull))] = index(m);
        written += __popcll(take_mask);
        ties_left -= min(ties_left, (int)__popcll(tie_mask));
        __builtin_amdgcn_sched_barrier(0);              // keeps the ballot masks of one step from piling up in SGPRs
    }
    return written;
}

constexpr int kCandPerLane = 4;                         // the prefilter keeps at most 64 * 4 candidates per row
constexpr int kPrefilterMaxK = 128;                     // and is used for k up to half that many buckets

// The search over one row with PER_LANE keys per lane (64 * PER_LANE >= the row's candidates).
// Long rows are thinned first: the lane's keys fall into four buckets (slot mod 4), so the wave has 256 bucket
// maxima; the k-th largest of them, T, has at least k keys at or above it, so the k largest keys of the row are
// among the keys >= T (about k..1.4 k of them when large scores are spread over the lanes).  Those are compacted
// in index order into the wave's LDS region (at most 4 per lane) and the exact search runs on them: the same list,
// ties included, with a fraction of the compares.  A row with more than 256 keys >= T (many equal scores) is
// searched in full.
// THIN: not for rows of more than 2048 blocks, which come here with k above 256 only (without it, 32 heads x 128K tokens in blocks of 32, k = 300 177 -> 89 us).
// merged: the row's keys in LDS (SHARED), else they come from the scores.
template <int PER_LANE, bool SHARED, bool THIN>
__device__ __forceinline__ int select_row(const SelectArgs& a, long long row, int n_cand, int kj, int lane,
                                          int32_t* out, uint2* cand, const uint32_t* merged) {
    uint32_t key[PER_LANE];
#pragma unroll
    for (int m = 0; m < PER_LANE; ++m) {
        const int i = m * 64 + lane;
        const uint32_t kx = SHARED ? merged[min(i, n_cand - 1)] : row_key<false>(a, row, 0, min(i, a.n2 - 1));   // unconditional load: no per-element exec masks to keep
        key[m] = (i < n_cand) ? kx : 0u;                   // 0 is below every trial threshold: never counted
    }
    if (THIN && PER_LANE > kCandPerLane && kj <= kPrefilterMaxK) {
        uint32_t top[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int m = 0; m < PER_LANE; ++m) top[m & 3] = max(top[m & 3], key[m]);
        const uint32_t T = kth_largest<4>(top, kj);        // > 0: the row has kj <= 128 valid keys in distinct buckets
        int total = 0;
#pragma unroll
        for (int m = 0; m < PER_LANE; ++m) total += (int)__popcll(__ballot(key[m] >= T));
        if (T != 0u && total <= 64 * kCandPerLane) {        // wave-uniform
            int base = 0;
#pragma unroll
            for (int m = 0; m < PER_LANE; ++m) {
                const bool in = key[m] >= T;
                const unsigned long long mask = __ballot(in);
                if (in) cand[base + __popcll(mask & ((1ull << lane) - 1ull))] = make_uint2(key[m], (unsigned)(m * 64 + lane));
                base += (int)__popcll(mask);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the wave reads back what its own lanes wrote: LDS operations of a wave complete in order
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            uint32_t ck[kCandPerLane]; int ci[kCandPerLane];
#pragma unroll
            for (int c = 0; c < kCandPerLane; ++c) {
                const int pos = c * 64 + lane;
                const uint2 e = cand[min(pos, 64 * kCandPerLane - 1)];
                ck[c] = pos < total ? e.x : 0u; ci[c] = (int)e.y;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // before the region is written for the wave's next row
            const uint32_t thr = kth_largest<kCandPerLane>(ck, kj);
            return take_largest<kCandPerLane>(ck, thr, kj, (total + 63) / 64, lane, out, [&](int c) { return ci[c]; });
        }
    }
    const uint32_t thr = kth_largest<PER_LANE>(key, kj);
    return take_largest<PER_LANE>(key, thr, kj, (n_cand + 63) / 64, lane, out, [&](int m) { return m * 64 + lane; });
}

// The group's scores of a list's first n blocks, merged by max, to LDS, by the whole workgroup: several loads of a head's row in flight
__device__ __forceinline__ void merge_group(const SelectArgs& a, long long row, int j, int n, uint32_t* merged) {
    const float* src = a.scores + ((row / a.n1 * a.group) * a.n1 + j) * a.n2;
    const long long step = (long long)a.n1 * a.n2;             // to the next head's row
    for (int i = threadIdx.x; i < n; i += 256) {
        uint32_t kx = 0;
        int g2 = 0;
        for (; g2 + 4 <= a.group; g2 += 4) {
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = src[(g2 + u) * step + i];
#pragma unroll
            for (int u = 0; u < 4; ++u) kx = max(kx, ordered_key(x[u]));
        }
        for (; g2 < a.group; ++g2) kx = max(kx, ordered_key(src[g2 * step + i]));
        merged[i] = kx;
    }
}

// behind the `written` chosen blocks: the local blocks, then the segment's own, then -1
__device__ __forceinline__ void finish_row(const SelectArgs& a, long long row, int n_cand, int diag_hi, int written, int lane, int32_t* out) {
    const int fixed = diag_hi - n_cand;
    for (int x = lane; x < fixed; x += 64) out[written + x] = n_cand + x;
    const int total = written + fixed;
    for (int x = total + lane; x < a.list_len; x += 64) out[x] = -1;
    if (lane == 0) a.cnt[row] = total;
}

// SHARED: a workgroup per list: its four waves merge the scores of the group's query heads into LDS,
// several loads of a head's row in flight, then one of them searches.  With one wave per list, its loads head after head,
// 32 query heads x 128K tokens in blocks of 64 took 44 us for 8 KV heads and 71 us for 4; now 15 and 14 (67 MB of scores).
// MAX_PER_LANE: 64 * MAX_PER_LANE >= n2, a multiple of 8.  A row early in the sequence has few candidates: the
// search is compiled for eight row lengths (eighths of the maximum) and a wave takes the shortest that holds its row.
template <int MAX_PER_LANE, bool SHARED>
__global__ __launch_bounds__(256) void select_kernel(SelectArgs a) {
    const int lane = threadIdx.x & 63;
    const long long row = SHARED ? (long long)blockIdx.x : (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.rows) return;
    const int j = (int)(row % a.n1);
    const int diag_lo = j * a.r;
    const int diag_hi = min(a.n2, diag_lo + a.r);
    const int n_local = min(a.local, diag_lo);
    const int n_cand = diag_lo - n_local;
    const int kj = min(a.budget, n_cand);
    int32_t* out = a.idx + row * a.list_len;
    constexpr bool THIN = MAX_PER_LANE <= 32;
    __shared__ uint2 cand_all[SHARED ? 1 : 4][THIN ? 64 * kCandPerLane : 1];
    uint2* cand = cand_all[SHARED ? 0 : threadIdx.x >> 6];
    __shared__ uint32_t merged[SHARED ? 64 * MAX_PER_LANE : 1];
    if (SHARED) {                                              // the whole workgroup merges the group's scores, one wave searches
        merge_group(a, row, j, kj > 0 ? n_cand : 0, merged);
        __syncthreads();
        if (threadIdx.x >= 64) return;
    }

    int written = 0;
    if (kj > 0) {
        constexpr int E = MAX_PER_LANE / 8;
        const int eighths = (n_cand + 64 * E - 1) / (64 * E);          // wave-uniform, 1 .. 8
        switch (eighths) {
            case 1: written = select_row<1 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            case 2: written = select_row<2 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            case 3: written = select_row<3 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            case 4: written = select_row<4 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            case 5: written = select_row<5 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            case 6: written = select_row<6 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            case 7: written = select_row<7 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
            default: written = select_row<8 * E, SHARED, THIN>(a, row, n_cand, kj, lane, out, cand, merged); break;
        }
    }
    finish_row(a, row, n_cand, diag_hi, written, lane, out);
}


// Rows longer than 4096 blocks, k > kStreamMaxK: one 256-thread workgroup per row, thread t owns blocks t, t+256, ...; the same
// radix search with the wave counts added up through LDS, and a compaction whose prefix runs over the four waves.
constexpr int kWideThreads = 256, kWidePerThread = 32;       // 8192 blocks
template <bool SHARED>
__global__ __launch_bounds__(kWideThreads) void select_wide_kernel(SelectArgs a) {
    __shared__ int part[2][4];                             // double-buffered per-wave partial counts
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long row = blockIdx.x;
    const int j = (int)(row % a.n1);
    const int diag_lo = j * a.r;
    const int diag_hi = min(a.n2, diag_lo + a.r);
    const int n_local = min(a.local, diag_lo);
    const int n_cand = diag_lo - n_local;
    const int kj = min(a.budget, n_cand);
    int32_t* out = a.idx + row * a.list_len;

    uint32_t key[kWidePerThread];
#pragma unroll
    for (int m = 0; m < kWidePerThread; ++m) {
        const int i = m * kWideThreads + tid;
        const uint32_t kx = row_key<SHARED>(a, row, j, min(i, a.n2 - 1));
        key[m] = (i < n_cand) ? kx : 0u;                   // 0 is below every trial threshold: never counted
    }
    int step = 0;
    auto block_sum = [&](int v) {                          // same value in every thread; one barrier per call
        v = wave_sum(v);
        if (lane == 0) part[step & 1][wave] = v;
        __syncthreads();
        const int t = part[step & 1][0] + part[step & 1][1] + part[step & 1][2] + part[step & 1][3];
        ++step;
        return t;
    };
    int written = 0;
    if (kj > 0) {                                          // uniform over the workgroup
        uint32_t thr = 0;
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t trial = thr | (1u << bit);
            int c = 0;
#pragma unroll
            for (int m = 0; m < kWidePerThread; ++m) c += (key[m] >= trial) ? 1 : 0;
            const int t = block_sum(c);
            if (t >= kj) thr = trial;
            if (t == kj) break;                            // uniform: exactly the list, see select_row
        }
        int above = 0;
#pragma unroll
        for (int m = 0; m < kWidePerThread; ++m) above += (key[m] > thr) ? 1 : 0;
        int ties_left = kj - block_sum(above);             // >= 1 by construction of thr
#pragma unroll
        for (int m = 0; m < kWidePerThread; ++m) {
            if (m * kWideThreads >= n_cand) break;          // uniform
            const int i = m * kWideThreads + tid;
            const bool valid = key[m] != 0u;
            const bool tie = valid && key[m] == thr;
            // ties before this thread in index order: earlier waves of this step, then earlier lanes
            const unsigned long long tie_mask = __ballot(tie);
            const int tie_w = (int)__popcll(tie_mask);
            if (lane == 0) part[step & 1][wave] = tie_w;
            __syncthreads();
            int tie_before = 0, tie_all = 0;
            for (int w = 0; w < 4; ++w) { const int x = part[step & 1][w]; tie_all += x; if (w < wave) tie_before += x; }
            ++step;
            const int tie_rank = tie_before + (int)__popcll(tie_mask & ((1ull << lane) - 1ull));
            const bool take = valid && (key[m] > thr || (tie && tie_rank < ties_left));
            const unsigned long long take_mask = __ballot(take);
            if (lane == 0) part[step & 1][wave] = (int)__popcll(take_mask);
            __syncthreads();
            int take_before = 0, take_all = 0;
            for (int w = 0; w < 4; ++w) { const int x = part[step & 1][w]; take_all += x; if (w < wave) take_before += x; }
            ++step;
            if (take) out[written + take_before + (int)__popcll(take_mask & ((1ull << lane) - 1ull))] = i;
            written += take_all;
            ties_left -= min(ties_left, tie_all);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const int fixed = diag_hi - n_cand;
    for (int x = tid; x < fixed; x += kWideThreads) out[written + x] = n_cand + x;
    const int total = written + fixed;
    for (int x = total + tid; x < a.list_len; x += kWideThreads) out[x] = -1;
    if (tid == 0) a.cnt[row] = total;
}

// ---------------------------------------------------------------------------------------------
// Long rows: the same search, the row streamed instead of held in registers.
//
// A wave reads its row twice, 16 bytes to a lane and load.  First pass: the maxima of 64 * NB buckets (lane, load mod NB/4, key of the
// load); their k-th largest, T, has at least k keys at or above it.  Second pass: the keys >= T, in index order, to the wave's LDS
// region, where the exact search runs on at most 2 * NB of them per lane.  With k at most half of the buckets they fit unless many
// scores are equal or the large ones share few buckets.  Then those above T are tried (many scores of 0: fewer than k are left, and T is
// the k-th largest), and at last the row is searched where it lies, pass after pass from the L2 cache.
//
// Bound by the vector unit (about 25 instructions per four keys in both passes) and, for few rows, by the latency of the loads.  In
// registers a row of 4096 blocks holds 64 keys per lane: few waves to a SIMD, and a count or a compaction step for every one of them.
// Per-head lists of 32 heads, in registers / streamed: 128K tokens in blocks of 32, k = 64, 78 / 45 us (with many zeros 186 / 52), k = 128 79 / 46;
// in blocks of 16 (a workgroup per row, a barrier per bit), k = 128, 136 / 62, k = 256 136 / 69; 94505 tokens, segments of 128, 78 / 55.
// Shared lists of 4 KV heads 36 / 25 (blocks of 32), 8 KV heads 134 / 50 (16).
// Eight loads in flight: 65 instead of 62 and 61 instead of 55 us.
// ---------------------------------------------------------------------------------------------
constexpr int kStreamAhead = 4;                         // loads in flight
constexpr int kStreamMaxK = 256;                        // the largest k that is streamed
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_row;    // four scores of a row, which starts anywhere

// f(u, i, key) for every four keys of the lane, in index order, until it returns false (the same for the whole wave): key[e] belongs
// to block i + e, and is 0 past the candidates; u numbers the loads in flight
template <bool SHARED, typename F>
__device__ __forceinline__ void for_keys(const float* src, const uint32_t* merged, int n2, int n_cand, int lane, F f) {
    for (int c0 = 0; c0 < n_cand; c0 += 256 * kStreamAhead) {
        uint32_t key[kStreamAhead][4];
        int at[kStreamAhead];
#pragma unroll
        for (int u = 0; u < kStreamAhead; ++u) {
            at[u] = min(c0 + 256 * u + 4 * lane, SHARED ? (n2 + 3) / 4 * 4 - 4 : n2 - 4);   // the last four of the row, if it ends before
            if (SHARED) {
#pragma unroll
                for (int e = 0; e < 4; ++e) key[u][e] = merged[at[u] + e];
            } else {
                const f32x4_row x = *(const f32x4_row*)(src + at[u]);
#pragma unroll
                for (int e = 0; e < 4; ++e) key[u][e] = __float_as_uint(x[e]);
            }
        }
#pragma unroll
        for (int u = 0; u < kStreamAhead; ++u) {
            const int i = c0 + 256 * u + 4 * lane;
            if (c0 + 256 * u >= n_cand) break;          // wave-uniform
            if (!SHARED) {
#pragma unroll
                for (int e = 0; e < 4; ++e) key[u][e] = ordered_key(__uint_as_float(key[u][e]));
            }
            if (c0 + 256 * u + 256 > n_cand) {          // keys below i are another lane's
#pragma unroll
                for (int e = 0; e < 4; ++e) key[u][e] = at[u] + e >= i && at[u] + e < n_cand ? key[u][e] : 0u;
            }
            if (!f(u, at[u], key[u])) return;
        }
    }
}

// Appends, in index order, what `in` says of the wave's 256 keys; put(position, e) stores one.  Returns how many.
template <typename Put>
__device__ __forceinline__ int append(const bool (&in)[4], Put put) {
    int before = 0, all = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const unsigned long long mask = __ballot(in[e]);
        before = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, before));
        all += (int)__popcll(mask);
    }
    if (all == 0) return 0;                             // wave-uniform
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (in[e]) put(before++, e);
    return all;
}

// The kj largest of the `total` <= 64 * N keys in the wave's LDS region, which hold them
template <int N>
__device__ __forceinline__ int search_candidates(const uint2* cand, int total, int kj, int lane, int32_t* out) {
    uint32_t key[N]; int at[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
        const uint2 e = cand[c * 64 + lane];
        key[c] = c * 64 + lane < total ? e.x : 0u; at[c] = (int)e.y;
    }
    const uint32_t thr = kth_largest<N>(key, kj);
    return take_largest<N>(key, thr, kj, (total + 63) / 64, lane, out, [&](int c) { return at[c]; });
}

template <int NB, bool SHARED>
__device__ __forceinline__ int select_streamed(const float* src, const uint32_t* merged, int n2, int n_cand, int kj, int lane,
                                               int32_t* out, uint2* cand) {
    constexpr int kRoom = 2 * 64 * NB;
    uint32_t top[NB];
#pragma unroll
    for (int x = 0; x < NB; ++x) top[x] = 0u;
    for_keys<SHARED>(src, merged, n2, n_cand, lane, [&](int u, int, const uint32_t (&key)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) top[u % (NB / 4) * 4 + e] = max(top[u % (NB / 4) * 4 + e], key[e]);
        return true;
    });
    const uint32_t T = kth_largest<NB>(top, kj);
    uint32_t largest = 0u;
#pragma unroll
    for (int x = 0; x < NB; ++x) largest = max(largest, top[x]);
    for (int o = 32; o > 0; o >>= 1) largest = max(largest, (uint32_t)__shfl_xor((int)largest, o));
    auto count = [&](uint32_t a, uint32_t b, uint32_t c, int (&n)[3]) {      // keys >= a, b, c; none of them 0
        n[0] = n[1] = n[2] = 0;
        for_keys<SHARED>(src, merged, n2, n_cand, lane, [&](int, int, const uint32_t (&key)[4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                n[0] += (int)__popcll(__ballot(key[e] >= a));
                n[1] += (int)__popcll(__ballot(key[e] >= b));
                n[2] += (int)__popcll(__ballot(key[e] >= c));
            }
            return true;
        });
    };
    int n[3] = {0, 0, 0};
    uint32_t least = max(T, 1u), thr = T;
    for (int tries = 0; tries < 2; ++tries) {
        int total = 0;
        for_keys<SHARED>(src, merged, n2, n_cand, lane, [&](int, int i, const uint32_t (&key)[4]) {
            bool in[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) in[e] = key[e] >= least;
            const int base = total;
            total += append(in, [&](int pos, int e) { if (base + pos < kRoom) cand[base + pos] = make_uint2(key[e], (unsigned)(i + e)); });
            return total <= kRoom;
        });
        if (total <= kRoom) {                           // wave-uniform
            // the wave reads back what its own lanes wrote: LDS operations of a wave complete in order
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            return total <= 64 * NB ? search_candidates<NB>(cand, total, kj, lane, out) : search_candidates<2 * NB>(cand, total, kj, lane, out);
        }
        // Too many.  Without those equal to T they may fit; if fewer than k are left then, the k-th largest is T itself
        if (T != largest && tries == 0) count(T + 1, T + 1, T + 1, n);
        if (n[0] < kj || n[0] > kRoom) break;
        least = T + 1;
    }
    if (n[0] >= kj) {                                   // two bits of the k-th largest per pass, from the highest that T, below it, and the largest differ in
        int bit = (31 - __clz(T ^ largest)) | 1;        // of the pair
        thr = (largest >> bit >> 1) << bit << 1;
        for (; bit > 0; bit -= 2) {
            const uint32_t one = 1u << (bit - 1);
            count(thr + one, thr + 2 * one, thr + 3 * one, n);
            const int digit = n[2] >= kj ? 3 : n[1] >= kj ? 2 : n[0] >= kj ? 1 : 0;
            thr += digit * one;
            if (digit > 0 && n[digit - 1] == kj) break; // exactly the list
        }
        n[0] = 0;
        if (thr != largest) count(thr + 1, thr + 1, thr + 1, n);
    }
    int ties_left = kj - n[0], written = 0;             // n[0]: keys above thr
    for_keys<SHARED>(src, merged, n2, n_cand, lane, [&](int, int i, const uint32_t (&key)[4]) {
        bool in[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) in[e] = key[e] > thr;
        if (ties_left > 0) {                            // wave-uniform
            bool tie[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) tie[e] = key[e] == thr && key[e] != 0u;
            const int ties = append(tie, [&](int pos, int e) { in[e] = pos < ties_left; });
            ties_left -= min(ties_left, ties);
        }
        const int base = written;
        written += append(in, [&](int pos, int e) { out[base + pos] = i + e; });
        return written < kj;
    });
    return written;
}

// PER_LANE: 64 * PER_LANE >= n2 (SHARED: the merged scores in LDS)
template <int NB, bool SHARED, int PER_LANE>
__global__ __launch_bounds__(256) void select_stream_kernel(SelectArgs a) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long row = SHARED ? (long long)blockIdx.x : (long long)blockIdx.x * 4 + wave;
    if (row >= a.rows) return;
    const int j = (int)(row % a.n1);
    const int diag_lo = j * a.r, diag_hi = min(a.n2, diag_lo + a.r);
    const int n_cand = diag_lo - min(a.local, diag_lo), kj = min(a.budget, n_cand);
    int32_t* out = a.idx + row * a.list_len;
    __shared__ uint2 cand_all[SHARED ? 1 : 4][2 * 64 * NB];
    __shared__ uint32_t merged[SHARED ? 64 * PER_LANE : 1];
    if (SHARED) {
        merge_group(a, row, j, kj > 0 ? n_cand : 0, merged);
        __syncthreads();
        if (threadIdx.x >= 64) return;
    }
    int written = 0;
    if (kj > 0) written = select_streamed<NB, SHARED>(a.scores + row * a.n2, merged, a.n2, n_cand, kj, lane, out, cand_all[SHARED ? 0 : wave]);
    finish_row(a, row, n_cand, diag_hi, written, lane, out);
}

}  // namespace

template <bool SHARED, int PER_LANE>
static hipError_t launch_stream(const SelectArgs& a, unsigned grid, hipStream_t st) {
    if (a.budget <= 128) hipLaunchKernelGGL((select_stream_kernel<4, SHARED, PER_LANE>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((select_stream_kernel<8, SHARED, PER_LANE>), dim3(grid), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <bool SHARED>
hipError_t launch_select_impl(const Shape& sh, const float* scores, int32_t* idx, int32_t* cnt, hipStream_t st) {
    SelectArgs a;
    a.scores = scores; a.idx = idx; a.cnt = cnt;
    a.rows = (long long)sh.batch * (SHARED ? sh.hkv : sh.hq) * sh.n1;
    a.group = sh.hq / sh.hkv;
    a.n1 = sh.n1; a.n2 = sh.n2; a.r = sh.r; a.budget = sh.budget; a.local = sh.local; a.list_len = sh.list_len;
    const unsigned grid = (unsigned)(SHARED ? a.rows : (a.rows + 3) / 4);
    // Streamed: rows of more than 2048 blocks.  Up to there a wave holds its row without losing the company of others (per-head lists in
    // registers / streamed, 32 heads x 128K tokens in blocks of 64: 18.8 / 24.2 us; shared ones 17.4 / 16.1, but 20000 tokens in blocks of 16
    // 9.6 / 10.3).  k above 256 would need 1024 buckets (32 heads, k = 300 of 2063 blocks: 22 / 34 us, with many zeros 30 / 67).
    if (sh.n2 <= 64 * 8) hipLaunchKernelGGL((select_kernel<8, SHARED>), dim3(grid), dim3(256), 0, st, a);
    else if (sh.n2 <= 64 * 32) hipLaunchKernelGGL((select_kernel<32, SHARED>), dim3(grid), dim3(256), 0, st, a);
    else if (sh.budget <= kStreamMaxK) {
        return sh.n2 <= 64 * 64 ? launch_stream<SHARED, 64>(a, grid, st) : launch_stream<SHARED, 128>(a, grid, st);
    } else if (sh.n2 <= 64 * 64) hipLaunchKernelGGL((select_kernel<64, SHARED>), dim3(grid), dim3(256), 0, st, a);
    else {
        if (a.rows > 0x7fffffffLL || sh.n2 > kWideThreads * kWidePerThread) return hipErrorInvalidValue;
        hipLaunchKernelGGL(select_wide_kernel<SHARED>, dim3((unsigned)a.rows), dim3(kWideThreads), 0, st, a);
    }
    return hipGetLastError();
}

// A KV head with one query head has that head's list: the per-head kernel, four rows to a workgroup.  (A workgroup per list, where rows are held in registers, 128K
// tokens in blocks of 32, k = 300, a wave / a workgroup: 256 lists 35 / 35 us, 512 35 / 38, 8192 88 / 123.)
hipError_t launch_select(const Shape& sh, const float* scores, int32_t* idx, int32_t* cnt, bool shared, hipStream_t st) {
    return shared && sh.hq != sh.hkv ? launch_select_impl<true>(sh, scores, idx, cnt, st) : launch_select_impl<false>(sh, scores, idx, cnt, st);
}

}  // namespace cp
