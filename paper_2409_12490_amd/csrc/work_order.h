// Which (batch, query head, segment, row tile) a workgroup of block-sparse attention takes (256-row and 128-row bf16 kernels).
//
// A compute unit takes the next workgroup in order when it is free, and each of the 8 XCDs every eighth workgroup, so the order decides how evenly the units finish and
// what the caches hold.  The heaviest come first: segments from the last to the first, all heads of one, and (head, segment) pairs in rounds that fill the chip once, a
// round at its last row tile, which sees most keys, then the same pairs at the one before.  With the tiles of a segment in one round the units that get first tiles get
// them again in the next, and with segments in ascending order the long ones of the last heads are left over.  Heads of one KV head after another, ascending segments -> this order (us):
// 32/8 heads x 3000 tokens (512, 64; 32 blocks) 112 -> 73, 4000 (16) 86 -> 81, 4096 (64) 188 -> 123, 7000 (256, 32; 32) 150 -> 143, 8000 (32) 265 -> 255, 16384 (16) 360 -> 351, 32/4 x
// 24000 (32) 825 -> 805, 2 x 32/8 x 12340 (512, 32; 67) 880 -> 838; 128-row workgroups 32/8 x 8192 (128, 32; 128) 443 -> 394.  A model of units that take the next workgroup
// when they are free (5.5 us and 1.65 per tile of 64 keys) gives the same gains; what it leaves at 32/8 x 16384 is 3 % above an even split.
//
// Consecutive workgroups walk the KV heads, so that one's keys stay with one XCD or two.  More than 64 MiB of keys and values are walked eight KV heads at a time, one to
// an XCD (16 / 8 at a time: 2 x 32/8 x 12340 815 / 809, 34000 (256, 32; 32) 1319 / 1303, 65536 2480 / 2435).  Smaller ones are walked all together: fewer
// rounds that are not full.
#pragma once
#include "fast_div.h"

namespace cp {

struct WorkOrder {
    struct Item { int bkv, gq, segment, tile; };    // (batch, KV head), query head in its group
    unsigned full, rest, set_kv, set_heads;    // pairs in whole rounds and behind them; KV heads and heads of a set
    FastDiv by_round, by_rest, by_set, by_heads, by_kv;

    WorkOrder() = default;
    // bkv = batch * hkv, group = query heads of a KV head, n1 segments of qtiles row tiles, workgroups that fill the chip, bytes of K and V
    WorkOrder(unsigned bkv, unsigned group, unsigned n1, unsigned qtiles, unsigned round, long long kv_bytes) {
        set_kv = bkv % 8 == 0 && kv_bytes > (64ll << 20) ? 8 : bkv;
        set_heads = set_kv * group;
        const unsigned pairs = bkv * group * n1;
        rest = pairs % round; full = pairs - rest;
        by_round = FastDiv(round * qtiles); by_rest = FastDiv(rest ? rest : 1);
        by_set = FastDiv(set_heads * n1); by_heads = FastDiv(set_heads); by_kv = FastDiv(set_kv);
    }
    __host__ __device__ __forceinline__ Item item(unsigned wg, unsigned round, unsigned n1, unsigned qtiles) const {    // round as a constant of the kernel
        Item t; unsigned u;
        if (wg < full * qtiles) {
            const unsigned rd = by_round.div(wg), y = wg - rd * round * qtiles;
            t.tile = (int)(qtiles - 1 - y / round);
            u = rd * round + y % round;
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

}  // namespace cp
