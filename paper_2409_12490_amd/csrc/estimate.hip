// Algorithm 1 "Estimation of Query Criticality in One Layer" on gfx950.
//
//   pool_kernel   element-wise max/min representatives of every query segment and key block
//                 (the reshape + max/min lines).  Streams Q and K once: HBM-bound.
//   score_kernel  four representative products, row softmax over blocks, (S1+S3)/2 vs (S2+S4)/2,
//                 element-wise max, block causal mask, layer fusion.
#include "kernels.h"

#include <type_traits>

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
    unsigned q_groups, k_groups;           // B*Hq*n1, B*Hkv*n2
    unsigned q_wgs;                        // workgroups that pool Q; the rest pool K
    int q_split, k_split;                  // log2 of the waves that share one group
    int q_across, k_across;                // consecutive groups: 0 along a head, 1 across the heads (see launch_pool)
    FastDiv div_n1, div_n2, div_hq, div_hkv;
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
// Bound by HBM for long sequences (1.34 GB at 32 + 8 heads x 128K tokens: 194 to 215 us, 6.2 to 6.9 TB/s; a plain copy moves 5.2
// here) and by the latency of a wave's batches, one after another, for short ones: with a wave to a group, 2000 tokens took 11.7 us.
template <typename T>
__global__ __launch_bounds__(64 * kPoolWaves) void pool_kernel(PoolArgs a) {
    constexpr int E = PoolVec<T>::kElems, kLanes = kHeadDim / E, kRows = 64 / kLanes, kLoads = 8, kBatch = kLoads * kRows;
    __shared__ __attribute__((aligned(16))) float part[kPoolWaves][2][kHeadDim];
    ask_for(a.q, a.k, a.qrep, a.krep, a.q_wgs, a.q_split, a.k_split, a.q_across, a.k_across, a.div_n1.mul, a.div_hkv.shift, a.qs0, a.qs1, a.qs2, a.ks0, a.ks1, a.ks2);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool is_q = blockIdx.x < a.q_wgs;
    const int log_split = is_q ? a.q_split : a.k_split, split = 1 << log_split;
    const int slot = wave >> log_split, share = wave & (split - 1);
    const unsigned gid = (is_q ? blockIdx.x : blockIdx.x - a.q_wgs) * (kPoolWaves >> log_split) + slot;
    const bool there = gid < (is_q ? a.q_groups : a.k_groups);
    const int groups = is_q ? a.n1 : a.n2, heads = is_q ? a.hq : a.hkv;
    int i = 0, h = 0, bb = 0;
    if (there) {
        const FastDiv by_group = is_q ? a.div_n1 : a.div_n2, by_head = is_q ? a.div_hq : a.div_hkv;
        if (is_q ? a.q_across : a.k_across) {
            const unsigned x = by_head.div(gid);
            h = (int)(gid - x * heads); bb = (int)by_group.div(x); i = (int)(x - (unsigned)bb * groups);
        } else {
            const unsigned x = by_group.div(gid);
            i = (int)(gid - x * groups); bb = (int)by_head.div(x); h = (int)(x - (unsigned)bb * heads);
        }
    }
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
        const int size = is_q ? a.s : a.b;
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
        // the group's last, short batch: rows past the end repeat its last row.  Half a batch has a form of its own, or the smallest groups
        // would ask for everything twice (32 heads x 9000 tokens in groups of 16: 20.3 against 17.6 us)
        auto last = [&](auto loads) {
            constexpr int N = decltype(loads)::value;
            uint4 v[N];
#pragma unroll
            for (int u = 0; u < N; ++u) v[u] = load_once(src + (long long)min(t + kRows * u + rsub, t1 - 1) * stride);
#pragma unroll
            for (int u = 0; u < N; ++u) merge(v[u]);
        };
        if (t + kBatch / 2 < t1) last(std::integral_constant<int, kLoads>());
        else if (t < t1) last(std::integral_constant<int, kLoads / 2>());
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
        T* dst = (T*)(is_q ? a.qrep : a.krep) + (((long long)bb * heads + h) * groups + i) * 2 * kHeadDim;
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
    // bf16 path: the sixteens of segments of a KV head's query heads are dealt to gridDim.y workgroups: share_least each, the first
    // share_more one more
    int group, share_least, share_more;
    FastDiv div_chunks, div_groups;        // nchunk; sixteens of a head
    int segs;                              // fp32 path: segments per workgroup
    float scale, alpha;
};
constexpr int kScoreWaves = 8;             // waves per workgroup of the bf16 score kernel
constexpr int kTileBlocks = 32;            // blocks per MFMA tile
constexpr int kTileBytes = kTileBlocks * 2 * kHeadDim * 2;   // max row + min row per block, bf16
constexpr int kChunkTiles = 8;             // tiles per workgroup, all of them in LDS (128 KiB)
constexpr int kScoreChunk = kChunkTiles * kTileBlocks;
constexpr int kScoreWgs = 256;             // workgroups that fill the chip, one to a compute unit
constexpr unsigned kMaxGridYZ = 65535;     // the largest second and third extent of a grid

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
    ask_for(a.qrep, a.krep, a.prev, a.scores, a.hq, a.n1, a.n2, a.segs, a.scale, a.alpha);
    const int segs = a.segs, pitch = score32_pitch(a.n2);
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
// The blocks of a (batch, KV head) are cut into tiles of 32 and the tiles into chunks of eight; a workgroup keeps the K
// representatives of one chunk in LDS (128 KiB, copied once by global_load_lds, 16-byte pieces XOR-swizzled by the block) and
// its 8 waves take groups of 16 segments, of any of the KV head's query heads, one each per round.  Z^T = K_rep . Q_rep^T: the A operand
// is a tile of 32 blocks of K_max (then K_min), the B operand, column = (segment, max/min representative), stays in registers.
// A lane then holds, for its column, 16 blocks of the tile in registers: the softmax statistics over blocks are in-lane
// reductions plus one exchange between the wave halves, and the two query representatives of a segment sit in neighbouring lanes
// (one DPP exchange per score).  In a last round of at most four groups `parts` waves share a group and split its tiles.
//
//   PASS 0   per chunk and column: max and sum of 2^(c z - max) of the two products  -> stats
//   PASS 1   merges the chunk statistics, recomputes the products of its chunk, normalises, combines (S1+S3)/2 vs
//            (S2+S4)/2, masks, fuses, stores.  Tiles that lie wholly after a group are written without any product.
//   PASS 2   both in one launch, for rows of a single chunk (n2 <= 256): the statistics stay in LDS.
//
// A chunk is four tiles from the front of the row and the four that mirror them from its end, so that every workgroup has the
// same share of the causal half.  Rows of scores start at any multiple of 4 bytes; 16 bytes of one go in one access all the same.
//
// What bounds it: PASS 0 the vector unit (171 vector instructions, 34 of them exponentials, per 16 segments and tile) and the 5 to 7
// us until a chunk has landed; PASS 1 the latency of S' and of the stores.  With one workgroup to a compute unit, what the groups leave
// over after whole rounds of whole workgroups decides (score_shares).  The two passes, in us, against (a) eight waves that streamed
// their chunk through two 32 KiB buffers, 128 segments of one head and chunk to a workgroup, and (b) this kernel with groups of one head in
// fixed eights: 32 / 8 heads x 66000 tokens, segments of 256, blocks of 32: (a) 104, (b) 139, now 72; segments of 128, blocks of 16,
// with S': 551, 822, 342; x 131072 (512, 64): 60, 60, 53, with S' 61, 66, 58; 2 x 32 x 65536 (256, 32) with S' 154, 146, 121;
// 8 x 131072 (128, 16) 195, 209, 183; x 16384 (512, 64) 20, 9.8, 9.6.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_row;   // four scores of a row, which starts anywhere
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

// z[b2][r] = K_rep(b2)[block 8*(r>>2) + 4*hh + (r&3) of the tile] . Q_rep[column]; tile: its LDS address.
// The two products alternate; every fragment is read kAhead MFMAs ahead.
__device__ __forceinline__ void score_tile(unsigned tile, int l32, int hh, const bf16x8 (&qf)[8], f32x16 (&z)[2]) {
    constexpr int kAhead = 4;
    const unsigned base = tile + l32 * 512;
    const int sw = l32 & 15;
    auto read = [&](int j) { return as_bf16x8(*SCORE_LDS(const u32x4, base + (j & 1) * 256 + (((2 * (j >> 1) + hh) ^ sw) << 4))); };
    bf16x8 kf[kAhead];
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
        for (int r = 0; r < 16; ++r) z[b2][r] = 0.f;
#pragma unroll
    for (int j = 0; j < kAhead; ++j) kf[j] = read(j);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        z[j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j % kAhead], qf[j >> 1], z[j & 1], 0, 0, 0);
        if (j + kAhead < 16) kf[j % kAhead] = read(j + kAhead);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int PASS>
__global__ __launch_bounds__(64 * kScoreWaves, 2) void score_kernel(ScoreArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char score_lds[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)score_lds;
    constexpr unsigned kRed = kChunkTiles * kTileBytes;     // behind the tiles: (max, sum) [wave][product][column], PASS 0 and 2
    constexpr float kLog2e = 1.4426950408889634f;
    ask_for(a.qrep, a.krep, a.prev, a.scores, a.stats, a.hq, a.n1, a.n2, a.nchunk, a.group, a.share_least, a.share_more, a.div_chunks.mul, a.div_groups.mul, a.scale);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid (x, shares, z): unit x + X z is a chunk of a (batch, KV head)
    const unsigned unit = blockIdx.z * gridDim.x + blockIdx.x;
    const int share = blockIdx.y, shares = gridDim.y;
    const int kv = (int)a.div_chunks.div(unit), chunk = (int)unit - kv * a.nchunk;
    // the sixteens of segments of the KV head's query heads, numbered through: dealt in eights to and fro, so that rows lie together and
    // nobody has all the late segments, which see most blocks (one by one, every shares-th, PASS 1 takes 125 instead of 94 us at
    // 32 / 4 heads x 128K, 256 a segment, blocks of 32, and 36 instead of 28 at 32 / 8 (512, 64)), the rest one by one
    const int head_groups = (a.n1 + 15) / 16;
    const int mine = a.share_least + (share < a.share_more ? 1 : 0), whole = a.share_least / kScoreWaves * kScoreWaves;
    // first block of tile lt of the chunk; four tiles (f) come from the front of the row, four (b) from its end, in the order f b f b b f b f,
    // of which 1, 2 or 4 waves that take every first, second or fourth tile get equal shares
    auto tile_begin = [&](int lt) {
        const int x = chunk * (kChunkTiles / 2) + (lt >> 1);
        return kTileBlocks * (((lt ^ (lt >> 2)) & 1) ? a.nchunk * kChunkTiles - 1 - x : x);
    };
    // first block wholly after segment j (of those that exist)
    auto seen_end = [&](int j) { return min(a.n2, (min(j, a.n1 - 1) + 1) * a.r); };
    // ---- K representatives -> LDS: wave w copies tile w, row = 2 * block + representative, 256 B; blocks past the last one repeat
    // it; a tile without a block is left out
    {
        static_assert(kScoreWaves == kChunkTiles, "a wave copies a tile");
        const int b0 = tile_begin(wave);
        if (b0 < a.n2) {
            const unsigned long long pv = (unsigned long long)((const uint16_t*)a.krep + (long long)kv * a.n2 * 2 * kHeadDim);
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
                // m0: reserved for the compiler, which sets it anew before each use of its own.  The wait: one state after m0, five after
                // the v_readfirstlane behind sbase, which the compiler does not see in here
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(sbase)
                             : "memory");
            }
        }
    }
    const float cs = a.scale * kLog2e;                      // logits in log2 units
    const int rep = l32 & 1;
    for (int first = 0; first < mine; first += kScoreWaves) {       // every wave takes every round and meets the barriers in it
        const int left = mine - first;                      // parts: waves that share a group of the last round and split its tiles
        const int parts = left > 4 ? 1 : left > 2 ? 2 : left > 1 ? 4 : 8;
        const int col_waves = kScoreWaves / parts, part = wave / col_waves, slot = wave % col_waves;
        const bool active = slot < left;                    // wave-uniform
        const int g = first < whole ? first * shares + (first & kScoreWaves ? shares - 1 - share : share) * kScoreWaves + slot
                                    : whole * shares + share + min(slot, left - 1) * shares;
        const int gh = (int)a.div_groups.div(g);
        const int bh = kv * a.group + gh, j0 = (g - gh * head_groups) * 16;
        const long long qrow0 = (long long)bh * a.n1;       // row of segment 0 of this (batch, head) in scores
        const int vis_lo = seen_end(j0), vis_hi = seen_end(j0 + 15);    // first block after the first / last segment of the group
        const int seg = j0 + (l32 >> 1), vis = seen_end(seg);
        const long long row = (qrow0 + seg) * a.n2;
        bf16x8 qf[8];
        {
            const uint16_t* src = (const uint16_t*)a.qrep + ((qrow0 + min(seg, a.n1 - 1)) * 2 + rep) * kHeadDim + 8 * hh;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) qf[ks] = as_bf16x8(*(const uint4*)(src + 16 * ks));
        }
        // statistics of product b2, column col: stats[((bh * nchunk + chunk) * 2 + b2) * 2 + (0: max, 1: sum)][col]
        const long long cols = 2LL * a.n1_pad, chunk_step = 4 * cols;
        float* stats = a.stats + (long long)bh * a.nchunk * chunk_step;
        float mx[2], inv[2];
        if (PASS == 1) {                                    // merge: the lane does product b2 = hh, its column's other lane the other one
            float M = -INFINITY, L = 0.f;
            const float* from = stats + 2 * hh * cols + 2 * seg + rep;
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
            mx[0] = hh ? oth_m : own_m; mx[1] = hh ? own_m : oth_m;
            inv[0] = hh ? oth_i : own_i; inv[1] = hh ? own_i : oth_i;
        }
        // S' of the lane's eight scores of tile lt, asked for two tiles ahead
        struct Prev { f32x4_row v[2]; } prev[2];
        auto fetch_prev = [&](int lt, Prev& to) {
            if (!a.prev || !active || seg >= a.n1 || lt >= kChunkTiles) return;
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2) {
                const int i = tile_begin(lt) + 4 * hh + 8 * (2 * g2 + rep);
                const float* at = a.prev + row + i;
                if (i + 4 <= a.n2) to.v[g2] = *(const f32x4_row*)at;
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (i + e < a.n2) to.v[g2][e] = at[e];
                }
            }
        };
        if (PASS != 0) { fetch_prev(part, prev[0]); fetch_prev(part + parts, prev[1]); }
        if (first == 0) {                                   // every wave's copies are in LDS
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        if (PASS != 1) {
            float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};
            const int dom = a.domain == 0 ? a.n2 : vis, dom_lo = a.domain == 0 ? a.n2 : vis_lo, dom_hi = a.domain == 0 ? a.n2 : vis_hi;
            for (int lt = part; lt < kChunkTiles; lt += parts) {
                const int b0 = tile_begin(lt);
                if (!active || b0 >= dom_hi) continue;
                f32x16 z[2];
                score_tile(lds0 + lt * kTileBytes, l32, hh, qf, z);
                if (cs > 0.f && b0 + kTileBlocks <= dom_lo) {
                    // every block of the tile counts for every column: no masks, the scale folded into one fma
#pragma unroll
                    for (int b2 = 0; b2 < 2; ++b2) {
                        const f32x16& x = z[b2];
                        float mt = fmaxf(x[0], x[1]);
#pragma unroll
                        for (int r = 2; r < 16; r += 2) mt = fmaxf(fmaxf(x[r], x[r + 1]), mt);
                        mt = halves_max(mt) * cs;
                        const float mn = fmaxf(m[b2], mt);
                        float sum = 0.f;
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(x[r], cs, -mn));
                        l[b2] = l[b2] * __builtin_amdgcn_exp2f(m[b2] - mn) + sum;
                        m[b2] = mn;
                    }
                    continue;
                }
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) {
                    float v[16];
                    float mt = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        v[r] = (b0 + 4 * hh + 8 * (r >> 2) + (r & 3) < dom) ? z[b2][r] * cs : -INFINITY;
                        mt = fmaxf(mt, v[r]);
                    }
                    mt = halves_max(mt);
                    const float mn = fmaxf(m[b2], mt);
                    const float ms = (mn == -INFINITY) ? 0.f : mn;
                    float sum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum += exp2f(v[r] - ms);
                    l[b2] = l[b2] * exp2f(m[b2] - ms) + sum;            // per-half partial sums under a common max
                    m[b2] = mn;
                }
            }
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) l[b2] = halves_sum(l[b2]);
            if (parts > 1) {                                // merge the parts of the group
                auto red = [&](int w, int b2) { return SCORE_LDS(f32x2, lds0 + kRed + ((w * 2 + b2) * 32 + l32) * 8); };
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2)
                    if (hh == 0) *red(wave, b2) = f32x2{m[b2], l[b2]};
                __syncthreads();
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) {
                    float M = -INFINITY, L = 0.f;
                    for (int x = 0; x < parts; ++x) M = fmaxf(M, (*red(x * col_waves + slot, b2))[0]);
                    const float ms = (M == -INFINITY) ? 0.f : M;
                    for (int x = 0; x < parts; ++x) {
                        const f32x2 e = *red(x * col_waves + slot, b2);
                        L += e[1] * exp2f(e[0] - ms);
                    }
                    m[b2] = M; l[b2] = L;
                }
            }
            if (PASS == 0) {
                if (hh == 0 && part == 0 && active) {
#pragma unroll
                    for (int b2 = 0; b2 < 2; ++b2) {
                        float* at = stats + chunk * chunk_step + 2 * b2 * cols + 2 * seg + rep;
                        at[0] = m[b2]; at[cols] = l[b2];
                    }
                }
                continue;
            }
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) {
                mx[b2] = (m[b2] == -INFINITY) ? 0.f : m[b2];
                inv[b2] = l[b2] > 0.f ? 1.0f / l[b2] : 0.f;
            }
        }
        if (!active) continue;
        // 2^(c z + fold) = 2^(c z - max) / sum / 2; usable when every column of the wave has a positive sum
        float fold[2];
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) fold[b2] = -mx[b2] + __log2f(inv[b2]) - 1.0f;
        const bool folds = cs > 0.f && __builtin_amdgcn_ballot_w64(inv[0] > 0.f && inv[1] > 0.f) == ~0ull;
        auto write_tile = [&](int lt, const Prev& old) {
            const int b0 = tile_begin(lt), i0 = b0 + 4 * hh;
            if (b0 >= a.n2) return;
            // S1 = (max,max), S2 = (max,min), S3 = (min,max), S4 = (min,min): the lane has the products of its
            // query representative with K_max (b2 = 0) and K_min (b2 = 1), its neighbour those of the other one
            float sc[16];
            if (b0 >= vis_hi) {                             // visible to no segment of the sixteen
#pragma unroll
                for (int r = 0; r < 16; ++r) sc[r] = 0.f;
            } else {
                f32x16 z[2];
                score_tile(lds0 + lt * kTileBytes, l32, hh, qf, z);
                if (folds && b0 + kTileBlocks <= vis_lo) {  // to every one: 1/sum and the 1/2 of the average are in the exponent
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float p0 = __builtin_amdgcn_exp2f(fmaf(z[0][r], cs, fold[0]));
                        const float p1 = __builtin_amdgcn_exp2f(fmaf(z[1][r], cs, fold[1]));
                        sc[r] = fmaxf(p0 + neighbour(p0), p1 + neighbour(p1));
                    }
                } else {
                    const int dom = a.domain == 0 ? a.n2 : vis;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int i = i0 + 8 * (r >> 2) + (r & 3);
                        const bool in_dom = i < dom;
                        const float p0 = in_dom ? exp2f(z[0][r] * cs - mx[0]) * inv[0] : 0.f;
                        const float p1 = in_dom ? exp2f(z[1][r] * cs - mx[1]) * inv[1] : 0.f;
                        const float t0 = p0 + neighbour(p0), t1 = p1 + neighbour(p1);
                        sc[r] = (i < vis) ? fmaxf(t0, t1) * 0.5f : 0.f;
                    }
                }
            }
            // both lanes of a pair hold the segment's 16 scores: representative 0 stores blocks 0-7 and 16-23 of
            // the lane half's 16, representative 1 the rest, four consecutive blocks at a time
            if (seg < a.n1) {
#pragma unroll
                for (int g2 = 0; g2 < 2; ++g2) {
                    const int i = i0 + 8 * (2 * g2 + rep);  // wave-varying but only two values: both compiled
                    f32x4_row w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        w[e] = rep ? sc[4 * (2 * g2 + 1) + e] : sc[4 * (2 * g2) + e];
                        if (a.prev) w[e] = a.alpha * w[e] + (1.0f - a.alpha) * old.v[g2][e];
                        if (fabsf(w[e]) < 1.17549435e-38f) w[e] = 0.f;
                    }
                    float* to = a.scores + row + i;
                    if (i + 4 <= a.n2) *(f32x4_row*)to = w;
                    else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (i + e < a.n2) to[e] = w[e];
                    }
                }
            }
        };
        for (int lt = part; lt < kChunkTiles; lt += 2 * parts) {
            write_tile(lt, prev[0]);
            fetch_prev(lt + 2 * parts, prev[0]);
            if (lt + parts < kChunkTiles) {
                write_tile(lt + parts, prev[1]);
                fetch_prev(lt + 3 * parts, prev[1]);
            }
        }
    }
}

}  // namespace

// Every wave of a group gets at least one batch, and two where there are enough groups to fill the chip.  The whole estimate step
// with 1 / 2 / 4 / 8 waves per segment, at the time the split came in: 32 heads x 2000 tokens 26.8 / 22.2 / 19.6 / 19.2 us, x 4096 35.7 /
// 26.4 / 21.3 / 20.3, x 128K (512 tokens a segment) 280 / 269 / 271 / 267; two batches of 256-token segments (batch 2, 64K) 364
// at four waves, 375 at eight with one batch each.  fp32, 8 heads x 8192: 47 / 31 / 23 / 19.
static int pool_split(const Shape& sh, int size, long long groups) {    // log2 of the waves
    const int batch = sh.dtype == 1 ? 32 : 16;
    int x = 0;
    while ((1 << x) < kPoolWaves && (2 << x) * batch <= size && (groups << x < 4096 || (4 << x) * batch <= size)) ++x;
    return x;
}

hipError_t launch_pool(const Shape& sh, const void* q, const void* k, void* qrep, void* krep, hipStream_t st) {
    PoolArgs a;
    a.q = q; a.k = k; a.qrep = qrep; a.krep = krep;
    a.n = sh.n; a.s = sh.s; a.b = sh.b; a.n1 = sh.n1; a.n2 = sh.n2; a.hq = sh.hq; a.hkv = sh.hkv;
    a.q_groups = (unsigned)sh.batch * sh.hq * sh.n1;                // below 2^31: make_shape, and n2 <= 8192 here
    a.k_groups = (unsigned)sh.batch * sh.hkv * sh.n2;
    a.qs0 = sh.qs[0]; a.qs1 = sh.qs[1]; a.qs2 = sh.qs[2];
    a.ks0 = sh.kvs[0]; a.ks1 = sh.kvs[1]; a.ks2 = sh.kvs[2];
    a.q_split = pool_split(sh, sh.s, a.q_groups); a.k_split = pool_split(sh, sh.b, a.k_groups);
    // Token-major tensors (the heads of a token lie together) are walked across the heads: along a head the waves in flight, a few heads
    // of many, all read at strides of a whole token.  Pooling along / across them, 32 / 8 heads x 66000 tokens, 512 a segment, 132 / 108
    // us, x 33000 60 / 55, x 128K 211 / 213; 2 x 32 / 4 x 66000 227 / 190.
    a.q_across = sh.qs[1] < sh.qs[2]; a.k_across = sh.kvs[1] < sh.kvs[2];
    a.div_n1 = FastDiv(sh.n1); a.div_n2 = FastDiv(sh.n2); a.div_hq = FastDiv(sh.hq); a.div_hkv = FastDiv(sh.hkv);
    const unsigned q_slots = kPoolWaves >> a.q_split, k_slots = kPoolWaves >> a.k_split;
    a.q_wgs = (a.q_groups + q_slots - 1) / q_slots;
    const unsigned grid = a.q_wgs + (a.k_groups + k_slots - 1) / k_slots;
    if (sh.dtype == 1) hipLaunchKernelGGL(pool_kernel<uint16_t>, dim3(grid), dim3(64 * kPoolWaves), 0, st, a);
    else hipLaunchKernelGGL(pool_kernel<float>, dim3(grid), dim3(64 * kPoolWaves), 0, st, a);
    return hipGetLastError();
}

// Scratch for the statistics of every chunk, padded to 128 segments.  The kernel needs none for a single chunk and `room` times less
// for a short sequence (the partial statistics of its waves are merged in LDS).  The size is part of the interface: it decides which calls
// critiprefill_estimate_static refuses, and those stay the same.
size_t score_stats_bytes(const Shape& sh) {
    if (sh.dtype != 1) return 0;
    const size_t room = sh.n1 <= 16 ? 8 : sh.n1 <= 32 ? 4 : sh.n1 <= 64 ? 2 : 1;
    const size_t nchunk = (size_t)((sh.n2 + kScoreChunk - 1) / kScoreChunk) * room;
    const size_t n1_pad = (size_t)((sh.n1 + 127) / 128) * 128;
    return (size_t)sh.batch * sh.hq * nchunk * 2 * 2 * (2 * n1_pad) * sizeof(float);
}

// Workgroups that the groups of a KV head's query heads are dealt to.  A workgroup copies its chunk (about 0.6 of a round: 6 us, rounds of
// 8 in PASS 0 and 15 in PASS 1), takes its rounds of eight groups and shares out the rest, 1, 1/2, 1/4 or 1/8 of a round; the chip runs
// kScoreWgs of them at a time.  Taken: the number with the least time by this account, among those that give a workgroup up to
// six whole rounds and a rest of 1, 2, 4 or 8.
static int score_shares(int groups, long long chunks) {        // chunks: of all (batch, KV head)
    int best = 1;
    double least = 1e30;
    for (int rounds = 0; rounds <= 6; ++rounds)
        for (int rest = 1; rest <= kScoreWaves; rest *= 2) {
            const int share = min(groups, rounds * kScoreWaves + rest), n = (groups + share - 1) / share;
            const int mine = (groups + n - 1) / n, left = mine % kScoreWaves;
            const double time = 0.6 + mine / kScoreWaves + (left == 0 ? 0.0 : left > 4 ? 1.0 : left > 2 ? 0.5 : left > 1 ? 0.25 : 0.125);
            const double all = time * (double)((chunks * n + kScoreWgs - 1) / kScoreWgs);
            if (all < least && n <= (int)kMaxGridYZ) { least = all; best = n; }
        }
    return best;
}

template <int PASS>
static hipError_t launch_score_pass(const ScoreArgs& a, dim3 grid, hipStream_t st) {
    constexpr int smem = kChunkTiles * kTileBytes + (PASS == 1 ? 0 : kScoreWaves * 2 * 32 * 8);
    const hipError_t e = hipFuncSetAttribute((const void*)score_kernel<PASS>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(score_kernel<PASS>, grid, dim3(64 * kScoreWaves), smem, st, a);
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
    if (sh.dtype == 1) {
        if ((long long)sh.batch * sh.hq > 65535) return hipErrorInvalidValue;
        const unsigned units = (unsigned)sh.batch * sh.hkv * a.nchunk;
        const int head_groups = (sh.n1 + 15) / 16, groups = sh.hq / sh.hkv * head_groups;
        const int shares = score_shares(groups, units);
        a.group = sh.hq / sh.hkv; a.share_least = groups / shares; a.share_more = groups % shares;
        a.div_chunks = FastDiv(a.nchunk); a.div_groups = FastDiv(head_groups);
        // workgroups that copy the same chunk on one XCD (workgroup id mod 8) where that leaves no XCD short
        const unsigned across = units % 8 == 0 && units / 8 <= kMaxGridYZ ? 8 : units;
        const dim3 grid(across, shares, units / across);
        if (a.nchunk == 1) return launch_score_pass<2>(a, grid, st);
        const hipError_t e = launch_score_pass<0>(a, grid, st);
        return e != hipSuccess ? e : launch_score_pass<1>(a, grid, st);
    }
    const long long heads = (long long)sh.batch * sh.hq;
    // as many segments to a workgroup as leave one for every compute unit and fit their rows of logits in LDS
    auto bytes = [&](int segs) { return (2 * (size_t)segs * score32_pitch(sh.n2) + 4 * segs) * sizeof(float); };
    int segs = 8;
    while (segs > 1 && (bytes(segs) > 128 * 1024 || heads * ((sh.n1 + segs - 1) / segs) < kScoreWgs)) segs /= 2;
    a.segs = segs;
    const hipError_t e = hipFuncSetAttribute((const void*)score_fp32_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes(segs));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(score_fp32_kernel, dim3((sh.n1 + segs - 1) / segs, sh.hq, sh.batch), dim3(64 * kScore32Waves), bytes(segs), st, a);
    return hipGetLastError();
}

}  // namespace cp
