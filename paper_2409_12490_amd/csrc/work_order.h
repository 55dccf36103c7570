// Which (batch, query head, segment, row tile) a workgroup of block-sparse attention takes.  The orders decide the time alone.
//
// WorkOrder: the kernels with 256 and 128 rows to a workgroup (attn_bf16.hip, attn_bf16_half.hip).
//
// A compute unit takes the next workgroup in order when it is free, and each of the 8 XCDs every eighth workgroup, so the order decides how evenly
// the units finish and what the caches hold.  The heaviest come first: segments from the last to the first, all heads of one, and (head, segment)
// pairs in rounds that fill the chip once, a round at its last row tile, which sees most keys, then the same pairs at the one before.  With the tiles
// of a segment in one round the units that get first tiles get them again in the next, and with segments in ascending order the long ones of the last
// heads are left over.  One KV head after another, ascending segments -> this order (us; (segment, block; blocks listed)): 32/8 heads x 3000 tokens
// (512, 64; 32) 113 -> 74, 4000 (16) 86 -> 81, 4096 (64) 188 -> 128, 7000 (256, 32; 32) 149 -> 142, 8000 (512, 64; 32) 267 -> 253, 16384 (16) 363 -> 349,
// 32/4 x 24000 (32) 828 -> 808, 2 x 32/8 x 12340 (512, 32; 67) 879 -> 832; 128-row workgroups 32/8 x 8192 (128, 32; 128) 440 -> 389, (32) 158 -> 153.  A
// model of units that take the next workgroup when they are free (5.5 us and 1.65 per tile of 64 keys) gives the same gains; what it leaves at
// 32/8 x 16384 is 3 % above an even split.
//
// Launches of less than two rounds and one workgroup more to each of the 256 units take all pairs at their last row tile before any at the one before: by
// rounds the units that take a third workgroup have two long ones.  By rounds / all pairs: 8/2 x 18523 (512, 32; 16) 88.8 / 84.2, 20443 (512, 64; 16)
// 124.9 / 120.1, 16/16 x 8283 (512, 32; 16) 83.3 / 72.2, 128-row workgroups 4/2 x 37083 (256, 16; 4) 41.5 / 39.7.  With more, the tiles of a segment come too
// far apart: 16/16 x 47963 (1024, 64; 32) 942 / 969, 128-row 32/8 x 6123 (256, 16; 4) 44.4 / 46.7, 8/2 x 20443 (256, 16; 30) 71.8 / 73.5.
//
// Consecutive workgroups walk the KV heads of a set.  Up to 64 MiB of keys and values all KV heads are one set, which leaves fewer rounds that are
// not full (36/12 x 10000 in sets of 4 376 instead of 366).  More of them are walked 8, 4, 2 or 1 at a time, the largest of these that divides
// their number, so that every eighth workgroup, an XCD's, reads the keys of one KV head: all together / in sets, 2 x 32/8 x 34000 (256, 32; 32)
// 1371 / 1336 (sets of 4 1333), 65536 2668 / 2581 (2583); 36/12 x 14000 (512, 64; 32) 535 / 529, 49152 1976 / 1912; 40/10 x 65536 2906 / 2810.  An
// odd number goes one at a time, and an XCD gets neighbouring segments of a round, whose lists are alike (every eighth of them / neighbours: 25/5 x
// 65536 1806 / 1746, 9/3 x 100000 1003 / 975, 15/15 x 40000 704 / 680; not for one KV head alone, 8/1 x 9000 (256, 32; 32) 63.5 -> 67.6).
#pragma once
#include "fast_div.h"

namespace cp {

struct WorkOrder {
    struct Item { int bkv, gq, segment, tile; };    // (batch, KV head), query head in its group
    unsigned full, rest, set_kv, neighbours;   // pairs in whole rounds and behind them; KV heads of a set; whether an XCD gets neighbouring pairs
    FastDiv by_round, by_rest, by_set, by_heads, by_kv;

    WorkOrder() = default;
    // bkv = batch * hkv, group = query heads of a KV head, n1 segments of qtiles row tiles, workgroups that fill the chip, bytes of K and V
    WorkOrder(unsigned bkv, unsigned group, unsigned n1, unsigned qtiles, unsigned round, long long kv_bytes) {
        const unsigned least = bkv & (0u - bkv);        // the largest power of two that divides it
        set_kv = kv_bytes <= (64ll << 20) ? bkv : least < 8 ? least : 8;
        neighbours = set_kv < bkv && set_kv == 1;
        const unsigned set_heads = set_kv * group;
        const unsigned pairs = bkv * group * n1;
        rest = pairs * qtiles < 2 * round + 256 ? pairs : pairs % round;
        full = pairs - rest;
        by_round = FastDiv(round * qtiles); by_rest = FastDiv(rest ? rest : 1);
        by_set = FastDiv(set_heads * n1); by_heads = FastDiv(set_heads); by_kv = FastDiv(set_kv);
    }
    __host__ __device__ __forceinline__ Item item(unsigned wg, unsigned round, unsigned group, unsigned n1, unsigned qtiles) const {    // round as a constant of the kernel
        Item t; unsigned u;
        const unsigned set_heads = set_kv * group;
        if (wg < full * qtiles) {
            const unsigned rd = by_round.div(wg), y = wg - rd * round * qtiles;
            t.tile = (int)(qtiles - 1 - y / round);
            const unsigned p = y % round;
            u = rd * round + (neighbours ? p % 8 * (round / 8) + p / 8 : p);
        } else {
            const unsigned y = wg - full * qtiles, z = by_rest.div(y);
            t.tile = (int)(qtiles - 1 - z);
            u = full + y - z * rest;
        }
        const unsigned set = by_set.div(u), v = u - set * set_heads * n1, level = by_heads.div(v), x = v - level * set_heads, gq = by_kv.div(x);
        t.segment = (int)(n1 - 1 - level);
        t.gq = (int)gq;
        t.bkv = (int)(set * set_kv + x - gq * set_kv);
        return t;
    }
};

// The order of the kernels with 32 and 16 rows to a workgroup (attn_bf16_rows.hip, attn_fp32_split.hip, attn_fp32.hip) inside a head.
//
// Every launch but those of in_pairs: segments from the last to the first, and the row tiles of a segment, which read the same keys, after one
// another.
//
// In pairs: workgroups of four waves, two to a compute unit, where the chip holds all of them.  Row tiles come by the keys that they see, most
// first, and the workgroup that comes 256 after another joins it on its unit, so the first 256 come with the longest last (turn = 256) and long and
// short ones share a unit.  A segment whose list is full sees `past` tiles' worth of keys before it and those up to the tile; the others, at the
// start of the sequence, see all keys up to the tile.  The lists on the GPU may say otherwise: the order decides the time alone.
//
// Attention alone, us (segment, block; blocks listed).  Segments from the last to the first / by keys without the turn / in pairs: bf16 4 heads x
// 4000 tokens (512, 16; 64) 21.1 / 19.5 / 19.3, 2 x 8000 (512, 64; 40) 37.9 / 34.4 / 34.1; fp32 4 x 4096 (256, 64; 6) 44.9 / 42.6 / 41.1, (512, 64; 20)
// 98 / 89 / 85, 4 x 3000 (256, 64; 4) 35.2 / 28.8 / 28.6, 2 x 6000 (512, 64; 4) 46 / 38 / 35; 16-row tiles 8 x 700 (256, 32; 4) 15.6 / 16.7 / 13.5, 8 x 900
// (512, 64; 4) 25.5 / 25.0 / 22.7, dense 8 x 800 25.5 / 25.5 / 19.5, 16 x 400 15.7 / 15.7 / 12.3, 12 x 600 21.5 / 21.5 / 16.7.
// More workgroups than the chip holds, by keys / segments from the last to the first.  The tiles of a segment come half a launch apart by keys, and
// its keys from memory again: bf16 batch 4 x 8/8 x 30000 (128, 8; 100) 1083 / 999, 12/12 x 60000 800 / 759, 32/8 x 32768 (64, 16; 10) 418 / 408; just
// above the chip long ones share a unit: 16/4 x 1100 (512, 64; 4) 18.4 / 13.5, 4/2 x 4700 (14) 28.5 / 23.4, 32/8 x 900 (4) 18.3 / 17.7; fp32 8/2 x 3000
// 101 / 94.  By keys is better for few KV heads of short lists, 8/2 x 60000 (64, 16; 20) 242 / 253, 2/1 x 12000 (256, 64; 30) 46.4 / 48.8; over 215
// launches it is 0.8 % behind.
struct TileOrder {
    // Not where many workgroups find no rows, past the end of a short last segment, and leave their places to others: fp32 8 x 600 (512, 64; 4; 208 of
    // 512) would take 20.0 instead of 14.7, but 8 x 900 (56 of 512) gains as above.
    static bool in_pairs(long long wgs, long long with_rows) { return wgs > 256 && wgs <= 512 && 8 * (wgs - with_rows) <= wgs; }

    struct Item { int segment, tile; };
    unsigned turn;                        // workgroups at the front that come in the opposite order, see in_pairs
    unsigned full, past, most;            // segments with full lists; a tile's rows of keys each; what the last tile of the others sees
    FastDiv by_full, by_level, by_tiles;  // full, full + 1, qtiles

    TileOrder() : turn(0), full(0), past(0), most(0) {}
    // by_keys: else the segments from the last to the first, tile by tile
    TileOrder(int n1, int r, int budget, int local, int b, int qtiles, int rows, bool by_keys) : turn(0) {
        const long long blocks = (long long)budget + local, keys = blocks * b / rows;
        const unsigned early = !by_keys || blocks > (long long)n1 * r ? n1 : (unsigned)((blocks + r - 1) / r);
        full = n1 - early; most = early * qtiles;
        past = full == 0 || keys > most ? most : (unsigned)(keys + qtiles < most ? most - qtiles : keys);    // for segments of no multiple of a tile's rows
        by_full = FastDiv(full ? full : 1); by_level = FastDiv(full + 1); by_tiles = FastDiv(qtiles);
    }
    // The order of a launch of `wgs` workgroups, of which `with_rows` have rows.
    static TileOrder of_launch(int waves, long long wgs, long long with_rows, int n1, int r, int budget, int local, int b, int qtiles, int rows) {
        const bool pairs = waves == 4 && in_pairs(wgs, with_rows);
        TileOrder o(n1, r, budget, local, b, qtiles, rows, pairs);
        if (pairs) o.turn = 256;
        return o;
    }
    __host__ __device__ __forceinline__ unsigned place(unsigned id) const { return id < turn ? turn - 1 - id : id; }
    // segments from the last to the first
    __host__ __device__ __forceinline__ Item by_segments(unsigned rank, unsigned qtiles) const {
        const unsigned at = most - 1 - rank, segment = by_tiles.div(at);
        return {(int)segment, (int)(at - segment * qtiles)};
    }
    // by the keys that they see
    __host__ __device__ __forceinline__ Item item(unsigned rank, unsigned n1, unsigned qtiles) const {
        const unsigned above = (past + qtiles - most) * full;    // of full segments, with more keys than all others
        unsigned seen, x;                 // tiles' worth of keys; which of those that see as many
        if (rank < above) {
            const unsigned level = by_full.div(rank);
            x = rank - level * full; seen = past + qtiles - level;
        } else if (rank -= above; rank < (most - past) * (full + 1)) {
            const unsigned level = by_level.div(rank);
            x = rank - level * (full + 1); seen = most - level;
        } else {
            x = full; seen = past - (rank - (most - past) * (full + 1));
        }
        if (x < full) return {(int)(n1 - 1 - x), (int)(seen - past - 1)};
        const unsigned segment = by_tiles.div(seen - 1);
        return {(int)segment, (int)(seen - 1 - segment * qtiles)};
    }
};

}  // namespace cp
