// Algorithm 1 "Estimation of Query Criticality in One Layer" on gfx950.
//
//   pool_kernel   element-wise max/min representatives of every query segment and key block
//                 (the reshape + max/min lines).  Streams Q and K once: HBM-bound.
//   score_kernel  four representative products, row softmax over blocks, (S1+S3)/2 vs (S2+S4)/2,
//                 element-wise max, block causal mask, layer fusion.
#include "kernels.h"

namespace cp {
namespace {

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
// both inputs hold exact bf16 values, so taking the upper halves loses nothing
__device__ __forceinline__ uint32_t pack_bf16_exact(float lo, float hi) {
    return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u);
}

// 16 bytes that are read once: streamed past the caches (measured: 6.2 instead of 5.4 TB/s for the pooling pass)
typedef __attribute__((ext_vector_type(4))) unsigned pool_u32x4;
__device__ __forceinline__ uint4 load_once(const void* p) {
    const pool_u32x4 x = __builtin_nontemporal_load((const pool_u32x4*)p);
    return make_uint4(x[0], x[1], x[2], x[3]);
}

struct PoolArgs {
    const void* q; const void* k; void* qrep; void* krep;
    int n, s, b, n1, n2, hq, hkv;
    long long q_groups, k_groups;          // B*Hq*n1, B*Hkv*n2
    long long q_wgs;                       // workgroups that pool Q; the rest pool K
    int q_split, k_split;                  // waves that share one group: 1, 2, 4 or 8
    long long qs0, qs1, qs2, ks0, ks1, ks2;
};

constexpr int kPoolWaves = 8;

// 16 bytes of one token row, as floats
template <typename T> struct PoolVec;
template <> struct PoolVec<uint16_t> {
    static constexpr int kElems = 8;
    static __device__ __forceinline__ void widen(const uint4& v, float (&x)[8]) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[2 * e] = bf16_lo(w[e]); x[2 * e + 1] = bf16_hi(w[e]); }
    }
    static __device__ __forceinline__ uint4 narrow(const float (&x)[8]) {
        return make_uint4(pack_bf16_exact(x[0], x[1]), pack_bf16_exact(x[2], x[3]), pack_bf16_exact(x[4], x[5]), pack_bf16_exact(x[6], x[7]));
    }
};
template <> struct PoolVec<float> {
    static constexpr int kElems = 4;
    static __device__ __forceinline__ void widen(const uint4& v, float (&x)[4]) {
        x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y); x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
    }
    static __device__ __forceinline__ uint4 narrow(const float (&x)[4]) {
        return make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
    }
};

// A group is a segment of Q or a block of K; `split` waves of a workgroup share one and merge through LDS.  A lane owns 16 bytes
// of a token row, kLanes lanes cover the row, a wave kRows rows per load with eight loads in flight (a batch).
//
// Bound by HBM for long sequences (1.34 GB at 32 + 8 heads x 128K tokens: 5.7 to 6.4 TB/s; a plain copy moves 5.2 here) and by
// the latency of a wave's batches, one after another, for short ones: with a wave to a group, 2000 tokens took 11.7 us.
template <typename T>
__global__ __launch_bounds__(64 * kPoolWaves) void pool_kernel(PoolArgs a) {
    constexpr int E = PoolVec<T>::kElems, kLanes = kHeadDim / E, kRows = 64 / kLanes, kLoads = 8, kBatch = kLoads * kRows;
    __shared__ __attribute__((aligned(16))) float part[kPoolWaves][2][kHeadDim];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool is_q = (long long)blockIdx.x < a.q_wgs;
    const int split = is_q ? a.q_split : a.k_split;
    const int slot = wave / split, share = wave % split;
    const long long gid = (is_q ? (long long)blockIdx.x : (long long)blockIdx.x - a.q_wgs) * (kPoolWaves / split) + slot;
    const bool there = gid < (is_q ? a.q_groups : a.k_groups);
    const int chunk = lane % kLanes, rsub = lane / kLanes;
    float hi[E], lo[E];
#pragma unroll
    for (int e = 0; e < E; ++e) { hi[e] = -INFINITY; lo[e] = INFINITY; }
    auto merge = [&](const uint4& v) {
        float x[E];
        PoolVec<T>::widen(v, x);
#pragma unroll
        for (int e = 0; e < E; ++e) { hi[e] = fmaxf(hi[e], x[e]); lo[e] = fminf(lo[e], x[e]); }
    };
    if (there) {
        const int groups = is_q ? a.n1 : a.n2, heads = is_q ? a.hq : a.hkv, size = is_q ? a.s : a.b;
        const int i = (int)(gid % groups); const long long bh = gid / groups;
        const int h = (int)(bh % heads), bb = (int)(bh / heads);
        const long long stride = is_q ? a.qs2 : a.ks2;
        const T* src = (is_q ? (const T*)a.q + bb * a.qs0 + h * a.qs1 : (const T*)a.k + bb * a.ks0 + h * a.ks1) + chunk * E;
        const int t0 = i * size, t1 = (int)min((long long)a.n, (long long)t0 + size);
        int t = t0 + share * kBatch;
        for (; t + kBatch <= t1; t += split * kBatch) {
            const T* p = src + (long long)(t + rsub) * stride;
            uint4 v[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) v[u] = load_once(p + (long long)(kRows * u) * stride);
#pragma unroll
            for (int u = 0; u < kLoads; ++u) merge(v[u]);
        }
        if (t < t1) {                          // the group's last, short batch: rows past the end repeat its last row
            uint4 v[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) v[u] = load_once(src + (long long)min(t + kRows * u + rsub, t1 - 1) * stride);
#pragma unroll
            for (int u = 0; u < kLoads; ++u) merge(v[u]);
        }
    }
#pragma unroll
    for (int o = kLanes; o < 64; o *= 2)
#pragma unroll
        for (int e = 0; e < E; ++e) { hi[e] = fmaxf(hi[e], __shfl_xor(hi[e], o)); lo[e] = fminf(lo[e], __shfl_xor(lo[e], o)); }
    if (split > 1) {                           // uniform over the workgroup
        if (rsub == 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) { part[wave][0][chunk * E + e] = hi[e]; part[wave][1][chunk * E + e] = lo[e]; }
        }
        __syncthreads();
        if (share != 0) return;
        for (int w = 1; w < split; ++w)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                hi[e] = fmaxf(hi[e], part[wave + w][0][chunk * E + e]);
                lo[e] = fminf(lo[e], part[wave + w][1][chunk * E + e]);
            }
    }
    if (there && rsub == 0) {
        T* dst = (T*)(is_q ? a.qrep : a.krep) + gid * 2 * kHeadDim;
        *(uint4*)(dst + chunk * E) = PoolVec<T>::narrow(hi);
        *(uint4*)(dst + kHeadDim + chunk * E) = PoolVec<T>::narrow(lo);
    }
}

// ---------------------------------------------------------------------------------------------
// score, fp32: fp32 MFMAs, whole rows of logits in LDS.
// ---------------------------------------------------------------------------------------------
struct ScoreArgs {
    const void* qrep; const void* krep; const float* prev; float* scores;
    float* stats;                          // bf16 path: per-chunk softmax statistics (see score_kernel)
    int hq, hkv, n1, n2, r, domain;
    int nchunk, n1_pad;
    int parts;                             // bf16 path: waves that share a group and split the tiles of a chunk (1, 2, 4, 8)
    int wg_groups;                         // groups of 16 * GPW segments (bf16) or segments (fp32) per workgroup
    int wg_heads;                          // bf16 path: query heads of one KV head whose groups are numbered through
    float scale, alpha;
};
constexpr int kScoreWaves = 8;             // waves per workgroup of the bf16 score kernel
constexpr int kTileBlocks = 32;            // blocks per MFMA tile
constexpr int kTileBytes = kTileBlocks * 2 * kHeadDim * 2;   // max row + min row per block, bf16
constexpr int kChunkTiles = 8;             // tiles per workgroup, all of them in LDS (128 KiB)
constexpr int kScoreChunk = kChunkTiles * kTileBlocks;
constexpr int kScoreWgs = 256;             // workgroups that fill the chip, one to a compute unit

// A workgroup takes up to eight segments of a (batch, head), i.e. 16 columns (segment, max/min representative) of Z^T = K_rep .
// Q_rep^T, and all blocks: 16x16x4 fp32 MFMAs over tiles of eight blocks (A = 16 representative rows of K straight from memory, B =
// the columns), logits to LDS as [column][K representative][block], then row softmax, (S1+S3)/2 vs (S2+S4)/2, mask, fusion.
// Bound by latency: one chain of loads, products, two passes over the row, stores.  Estimate step against one segment per
// workgroup with vector FMAs, each thread reading the 1 KiB of a block's representatives by itself: one head x 2048 tokens 12.0 ->
// 9.1 us, 8 x 8192 in blocks of 16 45 -> 30, 2 x 64K in blocks of 32 167 -> 85 (pooling included); error against float64 half as large (two accumulator chains).
constexpr int kScore32Waves = 8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
__host__ __device__ inline int score32_pitch(int n2) { return 2 * n2 + 1; }   // floats per column; odd: columns fall on different banks
__global__ __launch_bounds__(64 * kScore32Waves) void score_fp32_kernel(ScoreArgs a) {
    extern __shared__ float smem[];
    constexpr float kLog2e = 1.4426950408889634f;
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int segs = a.wg_groups, pitch = score32_pitch(a.n2);
    float* z = smem;                                        // [2 * segs][pitch]
    float* inv = smem + 2 * segs * pitch;                   // [2 * segs][2]
    const int j0 = blockIdx.x * segs, h = blockIdx.y, bb = blockIdx.z;
    const long long qrow0 = ((long long)bb * a.hq + h) * a.n1;
    const float* krep = (const float*)a.krep + ((long long)bb * a.hkv + h / (a.hq / a.hkv)) * a.n2 * 2 * kHeadDim;
    const int n_seg = min(segs, a.n1 - j0);                 // of this workgroup
    f32x4 qf[8];                                            // column c16: both sides take the channels in the order 16*kk + 4*g + e
    {
        const float* src = (const float*)a.qrep + (qrow0 + j0) * 2 * kHeadDim + min(c16, 2 * n_seg - 1) * kHeadDim + 4 * g;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[kk] = *(const f32x4*)(src + 16 * kk);
    }
    const int col = c16, seg = j0 + (c16 >> 1);
    const int dom = a.domain == 0 ? a.n2 : min(a.n2, (seg + 1) * a.r);
    for (int t = wave; 8 * t < a.n2; t += kScore32Waves) {
        const float* src = krep + (long long)min(16 * t + c16, 2 * a.n2 - 1) * kHeadDim + 4 * g;
        f32x4 kf[8];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) kf[kk] = *(const f32x4*)(src + 16 * kk);
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kk][e], qf[kk][e], acc[e & 1], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {                       // K row 4*g + r of the tile: block 2*g + r/2, representative r & 1
            const int i = 8 * t + 2 * g + (r >> 1);
            if (col < 2 * n_seg && i < a.n2) z[col * pitch + (r & 1) * a.n2 + i] = i < dom ? (acc[0][r] + acc[1][r]) * a.scale : -INFINITY;
        }
    }
    __syncthreads();
    for (int x = wave; x < 4 * n_seg; x += kScore32Waves) { // one wave to a row of logits
        float* row = z + (x >> 1) * pitch + (x & 1) * a.n2;
        float m = -INFINITY;
        for (int i = lane; i < a.n2; i += 64) m = fmaxf(m, row[i]);
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        float sum = 0.f;
        for (int i = lane; i < a.n2; i += 64) {
            const float e = exp2f((row[i] - m) * kLog2e);
            row[i] = e;
            sum += e;
        }
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) inv[x] = 1.0f / sum;
    }
    __syncthreads();
    for (int s = 0; s < n_seg; ++s) {
        const int vis = min(a.n2, (j0 + s + 1) * a.r);      // first block wholly after the segment
        const float* zmax = z + 2 * s * pitch;              // of Q_max: K_max, K_min; then of Q_min
        const float* zmin = zmax + pitch;
        const long long row = (qrow0 + j0 + s) * a.n2;
        for (int i = tid; i < a.n2; i += 64 * kScore32Waves) {
            float sc = 0.f;
            if (i < vis) {
                const float s1 = zmax[i] * inv[4 * s], s2 = zmax[a.n2 + i] * inv[4 * s + 1];
                const float s3 = zmin[i] * inv[4 * s + 2], s4 = zmin[a.n2 + i] * inv[4 * s + 3];
                sc = fmaxf((s1 + s3) * 0.5f, (s2 + s4) * 0.5f);
            }
            if (a.prev) sc = a.alpha * sc + (1.0f - a.alpha) * a.prev[row + i];
            if (fabsf(sc) < 1.17549435e-38f) sc = 0.f;
            a.scores[row + i] = sc;
        }
    }
}


// ---------------------------------------------------------------------------------------------
// score, bf16: the four representative products as bf16 MFMA GEMMs (representatives are exact bf16
// values, so every product is exact and only the fp32 accumulation rounds).
//
// The blocks of a (batch, head) are cut into tiles of 32 and the tiles into chunks of eight; a workgroup keeps the K
// representatives of one chunk in LDS (128 KiB, copied once by global_load_lds, 16-byte pieces XOR-swizzled by the block) and
// its 8 waves walk groups of 16 * GPW segments over them, with no further barrier.  Z^T = K_rep . Q_rep^T: the A operand is
// a tile of 32 blocks of K_max (then K_min), the B operand, column = (segment, max/min representative), stays in registers.
// A lane then holds, for its column, 16 blocks of the tile in registers: the softmax statistics over blocks are in-lane
// reductions plus one exchange between the wave halves, and the two query representatives of a segment sit in neighbouring lanes
// (one DPP exchange per score).  A short sequence has fewer groups than waves: `parts` waves then share a group and split
// its tiles.
//
//   PASS 0   per chunk and column: max and sum of 2^(c z - max) of the two products  -> stats
//   PASS 1   merges the chunk statistics, recomputes the products of its chunk, normalises, combines (S1+S3)/2 vs
//            (S2+S4)/2, masks, fuses, stores.  Tiles that lie wholly after a group are written without any product.
//   PASS 2   both in one launch, for rows of a single chunk (n2 <= 256): the statistics stay in LDS.
//
// A chunk is four tiles from the front of the row and the four that mirror them from its end, so that every workgroup has the
// same share of the causal half.
//
// What bounds it: PASS 0 the vector unit (171 vector instructions, 34 of them exponentials, per 16 segments and tile: 53K of
// the 106K busy cycles of a compute unit at 2 x 32 heads x 64K tokens, the MFMAs beside them) and the 5 to 7 us until a chunk has
// landed; PASS 1 the latency of S' and of the stores (2.7 TB/s there).  Against eight waves that streamed their chunk
// through two 32 KiB buffers, with a barrier per 64 blocks and 128 segments of one chunk to a workgroup, the estimate step takes,
// same pooling: 32 heads x 2000 tokens 19.2 -> 13.7 us (one launch less), x 4096 20.3 -> 16.1, x 16K 48.4 -> 37.6, 2 x 2 heads x 84K
// 57 -> 37, 32 x 128K 268 -> 263, 2 x 32 x 64K with fusion 373 -> 356, 8 x 128K in blocks of 16 with fusion 351 -> 320.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
#define SCORE_LDS(T, off) ((__attribute__((address_space(3))) T*)(uintptr_t)(off))

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
    union { uint4 u; bf16x8 b; } c; c.u = v; return c.b;
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) {
    union { u32x4 u; bf16x8 b; } c; c.u = v; return c.b;
}
__device__ __forceinline__ float halves_max(float x) {     // max over lanes l and l ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float neighbour(float x) {      // the value of lane l ^ 1
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));
}

// z[gg][b2][r] = K_rep(b2)[block 8*(r>>2) + 4*hh + (r&3) of the tile] . Q_rep[column of group gg]; tile: its LDS address.
// The two products alternate; every fragment feeds GPW MFMAs and is read kAhead of them ahead.
template <int GPW>
__device__ __forceinline__ void score_tile(unsigned tile, int l32, int hh, const bf16x8 (&qf)[GPW][8], f32x16 (&z)[GPW][2]) {
    constexpr int kAhead = 4;
    const unsigned base = tile + l32 * 512;
    const int sw = l32 & 15;
    auto read = [&](int j) { return as_bf16x8(*SCORE_LDS(const u32x4, base + (j & 1) * 256 + (((2 * (j >> 1) + hh) ^ sw) << 4))); };
    bf16x8 kf[kAhead];
#pragma unroll
    for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
            for (int r = 0; r < 16; ++r) z[gg][b2][r] = 0.f;
#pragma unroll
    for (int j = 0; j < kAhead; ++j) kf[j] = read(j);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
#pragma unroll
        for (int gg = 0; gg < GPW; ++gg)
            z[gg][j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j % kAhead], qf[gg][j >> 1], z[gg][j & 1], 0, 0, 0);
        if (j + kAhead < 16) kf[j % kAhead] = read(j + kAhead);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int PASS, int GPW>
__global__ __launch_bounds__(64 * kScoreWaves, 2) void score_kernel(ScoreArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char score_lds[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)score_lds;
    constexpr unsigned kRed = kChunkTiles * kTileBytes;     // behind the tiles: (max, sum) [wave][product][column], PASS 2
    constexpr float kLog2e = 1.4426950408889634f;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x, bh0 = blockIdx.z * a.wg_heads, h0 = bh0 % a.hq, bb = bh0 / a.hq;
    const int col_waves = kScoreWaves / a.parts, part = wave / col_waves;
    const int g_first = blockIdx.y * a.wg_groups + wave % col_waves;
    const int head_groups = (a.n1 + 16 * GPW - 1) / (16 * GPW);
    const int g_end = min(head_groups * a.wg_heads, (int)(blockIdx.y + 1) * a.wg_groups);
    // first block of tile lt of the chunk
    auto tile_begin = [&](int lt) { return kTileBlocks * (lt < kChunkTiles / 2 ? chunk * (kChunkTiles / 2) + lt
                                                          : a.nchunk * kChunkTiles - 1 - (chunk * (kChunkTiles / 2) + lt - kChunkTiles / 2)); };
    // first block wholly after segment j (of those that exist)
    auto seen_end = [&](int j) { return min(a.n2, (min(j, a.n1 - 1) + 1) * a.r); };
    // ---- K representatives -> LDS: wave w copies tile w, row = 2 * block + representative, 256 B; blocks past the last one repeat
    // it; a tile that nobody needs is left out
    {
        static_assert(kScoreWaves == kChunkTiles, "a wave copies a tile");
        const int b0 = tile_begin(wave);
        const int last = a.wg_heads > 1 ? a.n1 - 1 : g_end * 16 * GPW - 1;      // (several heads: the last segment is among them)
        if (b0 < (PASS == 1 || a.domain == 1 ? seen_end(last) : a.n2)) {
            const uint16_t* ksrc = (const uint16_t*)a.krep + ((long long)bb * a.hkv + h0 / (a.hq / a.hkv)) * a.n2 * 2 * kHeadDim;
            const unsigned long long pv = (unsigned long long)ksrc;
            const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)pv);
            const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(pv >> 32));
            const void* sbase = (const void*)(((unsigned long long)hi << 32) | lo);
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int row = 4 * x + (lane >> 4);
                const int blk = min(b0 + (row >> 1), a.n2 - 1);
                const int lc = (lane & 15) ^ ((row >> 1) & 15);
                const unsigned voff = (unsigned)(((blk * 2 + (row & 1)) * kHeadDim + lc * 8) * 2);
                const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + wave * kTileBytes + 1024u * x);
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(sbase)
                             : "memory");   // m0: reserved for the compiler, which sets it anew before each use of its own
            }
        }
    }
    const float cs = a.scale * kLog2e;                      // logits in log2 units
    const bool vec = (a.n2 & 3) == 0;                       // rows of scores are 16-byte aligned
    const int rep = l32 & 1;
    bool landed = false;
    // Every wave takes the body at least once and meets the barriers in it: with parts > 1 or PASS 2 it has at most one group (the
    // host sees to that), else there is only the first one, behind which all copies have landed
    const bool joint = PASS == 2 || a.parts > 1;
    for (int g = g_first; g < g_end || !landed; g += col_waves) {
        const bool active = g < g_end;                      // wave-uniform
        const int head = min(g, g_end - 1) / head_groups;   // of this workgroup
        const int j0 = (g - head * head_groups) * 16 * GPW;
        const long long qrow0 = (long long)(bh0 + head) * a.n1;  // row of segment 0 of this (batch, head) in scores
        const int vis_hi = seen_end(j0 + 16 * GPW - 1);     // first block after the last segment of the group
        int seg[GPW], vis[GPW];
        bf16x8 qf[GPW][8];
#pragma unroll
        for (int gg = 0; gg < GPW; ++gg) {
            seg[gg] = j0 + 16 * gg + (l32 >> 1);
            vis[gg] = seen_end(seg[gg]);
            const uint16_t* src = (const uint16_t*)a.qrep + ((qrow0 + min(seg[gg], a.n1 - 1)) * 2 + rep) * kHeadDim + 8 * hh;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) qf[gg][ks] = as_bf16x8(*(const uint4*)(src + 16 * ks));
        }
        // statistics of product b2, column col: stats[((bh * nchunk + chunk) * 2 + b2) * 2 + (0: max, 1: sum)][col]
        const long long cols = 2LL * a.n1_pad, chunk_step = 4 * cols;
        float* stats = a.stats + (long long)(bh0 + head) * a.nchunk * chunk_step;
        float mx[GPW][2], inv[GPW][2];
        if (PASS == 1) {                                    // merge: the lane does product b2 = hh, its column's other lane the other one
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg) {
                float M = -INFINITY, L = 0.f;
                const float* from = stats + 2 * hh * cols + 2 * min(seg[gg], a.n1_pad - 1) + rep;
                constexpr int kAhead = 8;
                for (int c0 = 0; c0 < a.nchunk; c0 += kAhead) {
                    float mc[kAhead], lc[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const float* at = from + min(c0 + u, a.nchunk - 1) * chunk_step;
                        mc[u] = at[0]; lc[u] = at[cols];
                    }
                    float mn = M;
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (c0 + u >= a.nchunk) { mc[u] = -INFINITY; lc[u] = 0.f; }
                        mn = fmaxf(mn, mc[u]);
                    }
                    const float ms = (mn == -INFINITY) ? 0.f : mn;
                    L *= exp2f(M - ms);
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) L += lc[u] * exp2f(mc[u] - ms);
                    M = mn;
                }
                const float own_m = (M == -INFINITY) ? 0.f : M;
                const float own_i = L > 0.f ? 1.0f / L : 0.f;
                const auto rm = __builtin_amdgcn_permlane32_swap(__float_as_uint(own_m), __float_as_uint(own_m), false, false);
                const auto ri = __builtin_amdgcn_permlane32_swap(__float_as_uint(own_i), __float_as_uint(own_i), false, false);
                const float oth_m = __uint_as_float(hh ? rm[0] : rm[1]);   // the value of lane l ^ 32
                const float oth_i = __uint_as_float(hh ? ri[0] : ri[1]);
                mx[gg][0] = hh ? oth_m : own_m; mx[gg][1] = hh ? own_m : oth_m;
                inv[gg][0] = hh ? oth_i : own_i; inv[gg][1] = hh ? own_i : oth_i;
            }
        }
        // S' of the lane's eight scores of a tile and group, asked for one tile ahead
        float4 pv[GPW][2];
        const bool fused4 = PASS != 0 && a.prev && vec && active;
        auto fetch_prev = [&](int lt) {
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
                for (int g2 = 0; g2 < 2; ++g2) {
                    const int i = lt < kChunkTiles ? tile_begin(lt) + 4 * hh + 8 * (2 * g2 + rep) : a.n2;
                    if (fused4 && i < a.n2 && seg[gg] < a.n1) pv[gg][g2] = *(const float4*)(a.prev + (qrow0 + seg[gg]) * a.n2 + i);
                }
        };
        if (PASS != 0) fetch_prev(part);
        if (!landed) {                                      // every wave's copies are in LDS
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            landed = true;
        }
        if (PASS != 1) {
            float m[GPW][2], l[GPW][2];
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) { m[gg][b2] = -INFINITY; l[gg][b2] = 0.f; }
            for (int lt = part; lt < kChunkTiles; lt += a.parts) {
                const int b0 = tile_begin(lt);
                if (!active || b0 >= (a.domain == 0 ? a.n2 : vis_hi)) continue;
                f32x16 z[GPW][2];
                score_tile<GPW>(lds0 + lt * kTileBytes, l32, hh, qf, z);
#pragma unroll
                for (int gg = 0; gg < GPW; ++gg) {
                    const int dom = a.domain == 0 ? a.n2 : vis[gg];
                    const int dom_lo = a.domain == 0 ? a.n2 : seen_end(j0 + 16 * gg);
                    if (cs > 0.f && b0 + kTileBlocks <= dom_lo) {
                        // every block of the tile counts for every column: no masks, the scale folded into one fma
#pragma unroll
                        for (int b2 = 0; b2 < 2; ++b2) {
                            const f32x16& x = z[gg][b2];
                            float mt = fmaxf(x[0], x[1]);
#pragma unroll
                            for (int r = 2; r < 16; r += 2) mt = fmaxf(fmaxf(x[r], x[r + 1]), mt);
                            mt = halves_max(mt) * cs;
                            const float mn = fmaxf(m[gg][b2], mt);
                            float sum = 0.f;
#pragma unroll
                            for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(x[r], cs, -mn));
                            l[gg][b2] = l[gg][b2] * __builtin_amdgcn_exp2f(m[gg][b2] - mn) + sum;
                            m[gg][b2] = mn;
                        }
                        continue;
                    }
#pragma unroll
                    for (int b2 = 0; b2 < 2; ++b2) {
                        float v[16];
                        float mt = -INFINITY;
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            v[r] = (b0 + 4 * hh + 8 * (r >> 2) + (r & 3) < dom) ? z[gg][b2][r] * cs : -INFINITY;
                            mt = fmaxf(mt, v[r]);
                        }
                        mt = halves_max(mt);
                        const float mn = fmaxf(m[gg][b2], mt);
                        const float ms = (mn == -INFINITY) ? 0.f : mn;
                        float sum = 0.f;
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum += exp2f(v[r] - ms);
                        l[gg][b2] = l[gg][b2] * exp2f(m[gg][b2] - ms) + sum;        // per-half partial sums under a common max
                        m[gg][b2] = mn;
                    }
                }
            }
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) l[gg][b2] = halves_sum(l[gg][b2]);
            if (joint) {                                    // merge the parts of the group (the host keeps GPW at 1 here)
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2)
                    if (hh == 0) *SCORE_LDS(f32x2, lds0 + kRed + ((wave * 2 + b2) * 32 + l32) * 8) = f32x2{m[0][b2], l[0][b2]};
                __syncthreads();
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) {
                    float M = -INFINITY, L = 0.f;
                    for (int x = 0; x < a.parts; ++x)
                        M = fmaxf(M, (*SCORE_LDS(const f32x2, lds0 + kRed + (((x * col_waves + wave % col_waves) * 2 + b2) * 32 + l32) * 8))[0]);
                    const float ms = (M == -INFINITY) ? 0.f : M;
                    for (int x = 0; x < a.parts; ++x) {
                        const f32x2 e = *SCORE_LDS(const f32x2, lds0 + kRed + (((x * col_waves + wave % col_waves) * 2 + b2) * 32 + l32) * 8);
                        L += e[1] * exp2f(e[0] - ms);
                    }
                    m[0][b2] = M; l[0][b2] = L;
                }
            }
            if (PASS == 0) {
                if (hh == 0 && part == 0 && active) {
#pragma unroll
                    for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
                        for (int b2 = 0; b2 < 2; ++b2) {
                            float* at = stats + chunk * chunk_step + 2 * b2 * cols + 2 * seg[gg] + rep;
                            at[0] = m[gg][b2]; at[cols] = l[gg][b2];
                        }
                }
                continue;
            }
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) {
                    mx[gg][b2] = (m[gg][b2] == -INFINITY) ? 0.f : m[gg][b2];
                    inv[gg][b2] = l[gg][b2] > 0.f ? 1.0f / l[gg][b2] : 0.f;
                }
        }
        if (!active) continue;
        // 2^(c z + fold) = 2^(c z - max) / sum / 2; usable when every column of the wave has a positive sum
        float fold[GPW][2];
        bool folds[GPW];
#pragma unroll
        for (int gg = 0; gg < GPW; ++gg) {
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) fold[gg][b2] = -mx[gg][b2] + __log2f(inv[gg][b2]) - 1.0f;
            folds[gg] = cs > 0.f && __builtin_amdgcn_ballot_w64(inv[gg][0] > 0.f && inv[gg][1] > 0.f) == ~0ull;
        }
        for (int lt = part; lt < kChunkTiles; lt += a.parts) {
            const int b0 = tile_begin(lt);
            float4 now[GPW][2];
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
                for (int g2 = 0; g2 < 2; ++g2) now[gg][g2] = pv[gg][g2];
            fetch_prev(lt + a.parts);
            if (b0 >= a.n2) continue;
            const int i0 = b0 + 4 * hh;
            f32x16 z[GPW][2];
            if (b0 < vis_hi) score_tile<GPW>(lds0 + lt * kTileBytes, l32, hh, qf, z);
#pragma unroll
            for (int gg = 0; gg < GPW; ++gg) {
                // S1 = (max,max), S2 = (max,min), S3 = (min,max), S4 = (min,min): the lane has the products of its
                // query representative with K_max (b2 = 0) and K_min (b2 = 1), its neighbour those of the other one
                float sc[16];
                const bool full = b0 + kTileBlocks <= seen_end(j0 + 16 * gg);       // visible to every segment of the sixteen
                if (b0 >= seen_end(j0 + 16 * gg + 15)) {                            // to none
#pragma unroll
                    for (int r = 0; r < 16; ++r) sc[r] = 0.f;
                } else if (folds[gg] && full) {                                     // 1/sum and the 1/2 of the average are in the exponent
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float p0 = __builtin_amdgcn_exp2f(fmaf(z[gg][0][r], cs, fold[gg][0]));
                        const float p1 = __builtin_amdgcn_exp2f(fmaf(z[gg][1][r], cs, fold[gg][1]));
                        sc[r] = fmaxf(p0 + neighbour(p0), p1 + neighbour(p1));
                    }
                } else {
                    const int dom = a.domain == 0 ? a.n2 : vis[gg];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int i = i0 + 8 * (r >> 2) + (r & 3);
                        const bool in_dom = i < dom;
                        const float p0 = in_dom ? exp2f(z[gg][0][r] * cs - mx[gg][0]) * inv[gg][0] : 0.f;
                        const float p1 = in_dom ? exp2f(z[gg][1][r] * cs - mx[gg][1]) * inv[gg][1] : 0.f;
                        const float t0 = p0 + neighbour(p0), t1 = p1 + neighbour(p1);
                        sc[r] = (i < vis[gg]) ? fmaxf(t0, t1) * 0.5f : 0.f;
                    }
                }
                // both lanes of a pair hold the segment's 16 scores: representative 0 stores blocks 0-7 and 16-23 of
                // the lane half's 16, representative 1 the rest, four consecutive blocks at a time
                if (seg[gg] < a.n1) {
                    const long long row = (qrow0 + seg[gg]) * a.n2;
#pragma unroll
                    for (int g2 = 0; g2 < 2; ++g2) {
                        const int i = i0 + 8 * (2 * g2 + rep);  // wave-varying but only two values: both compiled
                        float w[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] = rep ? sc[4 * (2 * g2 + 1) + e] : sc[4 * (2 * g2) + e];
                        const float old[4] = {now[gg][g2].x, now[gg][g2].y, now[gg][g2].z, now[gg][g2].w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (a.prev) w[e] = a.alpha * w[e] + (1.0f - a.alpha) * (vec ? old[e] : i + e < a.n2 ? a.prev[row + i + e] : 0.f);
                            if (fabsf(w[e]) < 1.17549435e-38f) w[e] = 0.f;
                        }
                        if (vec) {
                            if (i < a.n2) *(float4*)(a.scores + row + i) = make_float4(w[0], w[1], w[2], w[3]);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (i + e < a.n2) a.scores[row + i + e] = w[e];
                        }
                    }
                }
            }
        }
    }
}

}  // namespace

// Every wave of a group gets at least one batch, and two where there are enough groups to fill the chip.  The whole estimate step
// with 1 / 2 / 4 / 8 waves per segment: 32 heads x 2000 tokens 26.8 / 22.2 / 19.6 / 19.2 us, x 4096 35.7 / 26.4 / 21.3 / 20.3, x 128K
// (512 tokens a segment) 280 / 269 / 271 / 267 and, with Q token-major, 315 / 273 / 275 / 274; two batches of 256-token segments
// (batch 2, 64K) 364 at four waves, 375 at eight with one batch each.  fp32, 8 heads x 8192: 47 / 31 / 23 / 19.
static int pool_split(const Shape& sh, int size, long long groups) {
    const int batch = sh.dtype == 1 ? 32 : 16;
    int split = 1;
    while (split < kPoolWaves && 2 * split * batch <= size && (groups * split < 4096 || 4 * split * batch <= size)) split *= 2;
    return split;
}

hipError_t launch_pool(const Shape& sh, const void* q, const void* k, void* qrep, void* krep, hipStream_t st) {
    PoolArgs a;
    a.q = q; a.k = k; a.qrep = qrep; a.krep = krep;
    a.n = sh.n; a.s = sh.s; a.b = sh.b; a.n1 = sh.n1; a.n2 = sh.n2; a.hq = sh.hq; a.hkv = sh.hkv;
    a.q_groups = (long long)sh.batch * sh.hq * sh.n1;
    a.k_groups = (long long)sh.batch * sh.hkv * sh.n2;
    a.qs0 = sh.qs[0]; a.qs1 = sh.qs[1]; a.qs2 = sh.qs[2];
    a.ks0 = sh.kvs[0]; a.ks1 = sh.kvs[1]; a.ks2 = sh.kvs[2];
    a.q_split = pool_split(sh, sh.s, a.q_groups); a.k_split = pool_split(sh, sh.b, a.k_groups);
    a.q_wgs = (a.q_groups * a.q_split + kPoolWaves - 1) / kPoolWaves;
    const unsigned grid = (unsigned)(a.q_wgs + (a.k_groups * a.k_split + kPoolWaves - 1) / kPoolWaves);
    if (sh.dtype == 1) hipLaunchKernelGGL(pool_kernel<uint16_t>, dim3(grid), dim3(64 * kPoolWaves), 0, st, a);
    else hipLaunchKernelGGL(pool_kernel<float>, dim3(grid), dim3(64 * kPoolWaves), 0, st, a);
    return hipGetLastError();
}

// Scratch for the statistics of every chunk, padded to 128 segments.  A single chunk keeps them in LDS; the factor for short
// sequences leaves room for up to eight partial statistics per chunk, which the kernel merges in LDS now: callers may hold
// buffers of this size, so it stays.
size_t score_stats_bytes(const Shape& sh) {
    if (sh.dtype != 1) return 0;
    const size_t room = sh.n1 <= 16 ? 8 : sh.n1 <= 32 ? 4 : sh.n1 <= 64 ? 2 : 1;
    const size_t nchunk = (size_t)((sh.n2 + kScoreChunk - 1) / kScoreChunk) * room;
    const size_t n1_pad = (size_t)((sh.n1 + 127) / 128) * 128;
    return (size_t)sh.batch * sh.hq * nchunk * 2 * 2 * (2 * n1_pad) * sizeof(float);
}

template <int PASS, int GPW>
static hipError_t launch_score_pass(const ScoreArgs& a, dim3 grid, hipStream_t st) {
    constexpr int smem = kChunkTiles * kTileBytes + (PASS == 1 ? 0 : kScoreWaves * 2 * 32 * 8);
    const hipError_t e = hipFuncSetAttribute((const void*)score_kernel<PASS, GPW>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((score_kernel<PASS, GPW>), grid, dim3(64 * kScoreWaves), smem, st, a);
    return hipGetLastError();
}

hipError_t launch_score(const Shape& sh, const void* qrep, const void* krep, const float* prev, float* scores,
                        float* stats, hipStream_t st) {
    ScoreArgs a;
    a.qrep = qrep; a.krep = krep; a.prev = prev; a.scores = scores; a.stats = stats;
    a.hq = sh.hq; a.hkv = sh.hkv; a.n1 = sh.n1; a.n2 = sh.n2; a.r = sh.r; a.domain = sh.softmax_domain;
    a.scale = sh.score_scale; a.alpha = sh.alpha;
    a.nchunk = (sh.n2 + kScoreChunk - 1) / kScoreChunk;
    a.n1_pad = (sh.n1 + 127) / 128 * 128;
    a.parts = 1; a.wg_groups = kScoreWaves; a.wg_heads = 1;
    if (sh.dtype == 1) {
        const long long heads = (long long)sh.batch * sh.hq;
        if (heads > 65535) return hipErrorInvalidValue;
        // Few segments: as many workgroups as the chip holds, the waves without a group of their own sharing one.  Many: pairs
        // of groups per wave, which halve the LDS reads per MFMA (estimate at 32 heads x 128K 263 against 271 us, 8 x 128K in
        // blocks of 16 320 / 349), and, with more than four workgroups to a compute unit, more groups to a workgroup,
        // so that a chunk is copied less often.
        const int sixteens = (sh.n1 + 15) / 16;
        auto wgs = [&](int groups) { return heads * a.nchunk * ((groups + a.wg_groups - 1) / a.wg_groups); };
        const bool pairs = a.nchunk > 1 && sixteens > kScoreWaves && heads * a.nchunk * ((sixteens + 2 * kScoreWaves - 1) / (2 * kScoreWaves)) >= kScoreWgs;
        const int groups = pairs ? (sixteens + 1) / 2 : sixteens;
        if (!pairs)
            while (a.parts < kChunkTiles && (a.wg_groups / 2 >= groups || wgs(groups) < kScoreWgs)) { a.parts *= 2; a.wg_groups /= 2; }
        while (a.parts == 1 && a.nchunk > 1 && a.wg_groups < groups && wgs(groups) >= 4 * kScoreWgs) a.wg_groups *= 2;
        // One workgroup holds all groups of a head and there are still two for every compute unit: the heads of a KV head share a
        // copied chunk (estimate, 2 x 32 heads x 64K 330 -> 319 us without S', 359 with it either way; 32 x 128K in blocks of 32 407 -> 402).
        while (pairs && a.wg_groups >= groups * a.wg_heads && (a.hq / a.hkv) % (2 * a.wg_heads) == 0 && heads / a.wg_heads * a.nchunk >= 2 * kScoreWgs) {
            a.wg_heads *= 2; a.wg_groups *= 2;
        }
        const dim3 grid(a.nchunk, (groups * a.wg_heads + a.wg_groups - 1) / a.wg_groups, (unsigned)(heads / a.wg_heads));
        if (a.nchunk == 1) return launch_score_pass<2, 1>(a, grid, st);
        const hipError_t e = pairs ? launch_score_pass<0, 2>(a, grid, st) : launch_score_pass<0, 1>(a, grid, st);
        if (e != hipSuccess) return e;
        return pairs ? launch_score_pass<1, 2>(a, grid, st) : launch_score_pass<1, 1>(a, grid, st);
    }
    // as many segments to a workgroup as leave one for every compute unit and fit their rows of logits in LDS
    const long long heads = (long long)sh.batch * sh.hq;
    auto bytes = [&](int segs) { return (2 * (size_t)segs * score32_pitch(sh.n2) + 4 * segs) * sizeof(float); };
    int segs = 8;
    while (segs > 1 && (bytes(segs) > 128 * 1024 || heads * ((sh.n1 + segs - 1) / segs) < kScoreWgs)) segs /= 2;
    a.wg_groups = segs;
    const hipError_t e = hipFuncSetAttribute((const void*)score_fp32_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes(segs));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(score_fp32_kernel, dim3((sh.n1 + segs - 1) / segs, sh.hq, sh.batch), dim3(64 * kScore32Waves), bytes(segs), st, a);
    return hipGetLastError();
}

}  // namespace cp
