"""The order of workgroups of block-sparse attention (WorkOrder, TileOrder), compiled for the CPU from the header the kernels include: every (KV head, query head,
segment, row tile) exactly once, whatever the numbers of heads and segments leave over after whole rounds, and the heaviest first."""
import ctypes
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_12490_amd", "csrc")
PROGRAM = """
#define __host__
#define __device__
#define __forceinline__ inline
#include "work_order.h"
extern "C" void order(unsigned bkv, unsigned group, unsigned n1, unsigned qtiles, unsigned round, long long kv_bytes, int* out) {
    const cp::WorkOrder o(bkv, group, n1, qtiles, round, kv_bytes);
    for (unsigned wg = 0; wg < bkv * group * n1 * qtiles; ++wg) {
        const auto t = o.item(wg, round, group, n1, qtiles);
        out[4 * wg] = t.bkv; out[4 * wg + 1] = t.gq; out[4 * wg + 2] = t.segment; out[4 * wg + 3] = t.tile;
    }
}
extern "C" void tiles(int n1, int r, int budget, int local, int b, int qtiles, int rows, long long wgs, int by_keys, int pairs, int* out) {
    cp::TileOrder o(n1, r, budget, local, b, qtiles, rows, by_keys);
    if (pairs) o.turn = 256;
    for (long long wg = 0; wg < wgs; ++wg) {
        const unsigned heads = (unsigned)(wgs / (n1 * qtiles)), place = o.place((unsigned)wg);
        const auto t = o.item(place / heads, n1, qtiles);
        out[3 * wg] = place % heads; out[3 * wg + 1] = t.segment; out[3 * wg + 2] = t.tile;
    }
}
extern "C" int launched(int waves, long long wgs, long long with_rows, int n1, int r, int budget, int local, int b, int qtiles, int rows, int* out) {
    const cp::TileOrder o = cp::TileOrder::of_launch(waves, wgs, with_rows, n1, r, budget, local, b, qtiles, rows);
    for (int rank = 0; rank < n1 * qtiles; ++rank) {
        const auto t = o.turn ? o.item(rank, n1, qtiles) : o.by_segments(rank, qtiles), u = o.item(rank, n1, qtiles);
        if (t.segment != u.segment || t.tile != u.tile) return -1;
        out[2 * rank] = t.segment; out[2 * rank + 1] = t.tile;
    }
    return o.turn;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    compiler = shutil.which("g++") or shutil.which("clang++") or shutil.which("c++")
    if compiler is None:
        pytest.skip("no C++ compiler")
    where = tmp_path_factory.mktemp("work_order")
    (where / "f.cpp").write_text(PROGRAM)
    subprocess.run([compiler, "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(where / "f.cpp"), "-o", str(where / "f.so")], check=True)
    lib = ctypes.CDLL(str(where / "f.so"))
    lib.order.argtypes = [ctypes.c_uint] * 5 + [ctypes.c_longlong, np.ctypeslib.ndpointer(np.int32)]
    lib.tiles.argtypes = [ctypes.c_int] * 7 + [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, np.ctypeslib.ndpointer(np.int32)]
    lib.order.restype = lib.tiles.restype = None
    lib.launched.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong] + [ctypes.c_int] * 7 + [np.ctypeslib.ndpointer(np.int32)]
    return lib


@pytest.fixture(scope="module")
def order(lib):
    return lib.order


@pytest.mark.parametrize("round_", [256, 512])
@pytest.mark.parametrize("kv_bytes", [1 << 26, (1 << 26) + 1])
def test_each_item_once(order, round_, kv_bytes):
    for bkv, group, n1, qtiles in [(1, 1, 1, 1), (1, 1, 1, 3), (8, 4, 8, 1), (8, 4, 8, 2), (8, 4, 33, 2), (16, 4, 129, 1), (24, 1, 11, 5), (17, 1, 31, 2), (5, 5, 40, 2), (6, 3, 57, 4), (12, 3, 40, 2), (5, 1, 9, 2), (16, 8, 4, 2), (2, 1, 257, 1)]:
        out = np.full((bkv * group * n1 * qtiles, 4), -1, np.int32)
        order(bkv, group, n1, qtiles, round_, kv_bytes, out)
        what = (bkv, group, n1, qtiles)
        assert (out >= 0).all() and (out < np.array([bkv, group, n1, qtiles])).all(), what
        assert len(np.unique(out, axis=0)) == len(out), what
        at_a_time = math.gcd(bkv, 8) if kv_bytes > 1 << 26 else bkv
        last_tile = out[out[:, 3] == qtiles - 1]
        if at_a_time == 1 < bkv:                              # an XCD, every eighth workgroup, has neighbouring pairs of a round
            whole = 0 if bkv * group * n1 * qtiles < 2 * round_ + 256 else len(last_tile) // round_ * round_
            last_tile[:whole] = last_tile[:whole].reshape(-1, round_ // 8, 8, 4).transpose(0, 2, 1, 3).reshape(-1, 4)
        for first in range(0, bkv, at_a_time):                # the segments of a set of KV heads, from the last to the first
            segments = last_tile[last_tile[:, 0] // at_a_time == first // at_a_time, 2]
            assert (np.diff(segments) <= 0).all(), what
        assert (np.diff(last_tile[:, 0] // at_a_time) >= 0).all(), what       # set after set; in each an XCD, every eighth workgroup, has one KV head to read
        assert (last_tile[:, 0] % at_a_time == np.arange(len(last_tile)) % at_a_time).all(), what


@pytest.mark.parametrize("bkv,group,n1,qtiles,round_", [(2, 4, 37, 2, 256), (8, 4, 10, 2, 256), (16, 1, 23, 2, 256), (8, 4, 11, 2, 256), (3, 1, 85, 3, 256), (2, 4, 79, 2, 512), (16, 1, 39, 2, 512), (2, 4, 53, 3, 512)])
def test_few_rounds_come_by_row_tiles(order, bkv, group, n1, qtiles, round_):
    """Launches of less than two rounds and a workgroup to each of the 256 units: every pair at its last row tile, the longest, before any at the one before."""
    assert round_ < bkv * group * n1 * qtiles < 2 * round_ + 256
    out = np.full((bkv * group * n1 * qtiles, 4), -1, np.int32)
    order(bkv, group, n1, qtiles, round_, 1 << 20, out)
    assert (np.diff(out[:, 3]) <= 0).all() and len(np.unique(out, axis=0)) == len(out)


@pytest.mark.parametrize("heads", [1, 3, 8])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("s,b", [(16, 16), (96, 32), (128, 128), (255, 51), (256, 32), (512, 64)])
def test_each_row_tile_once(lib, heads, rows, s, b):
    r, qtiles = s // b, (s + rows - 1) // rows
    for n1 in (1, 2, 5, 16, 33):
        wgs = heads * n1 * qtiles
        for budget, local in [(0, 0), (1, 0), (3, 2), (6, 1), (17, 0), (40, 1), (2000, 2), (2**30, 2**30)]:
            for by_keys, pairs in [(0, 0), (1, 0), (1, 1)]:
                if pairs and not 256 < wgs <= 512:
                    continue
                out = np.full((wgs, 3), -1, np.int32)
                lib.tiles(n1, r, budget, local, b, qtiles, rows, wgs, by_keys, pairs, out)
                what = (n1, budget, local, by_keys, pairs)
                assert (out >= 0).all() and (out < np.array([heads, n1, qtiles])).all(), what
                assert len(np.unique(out, axis=0)) == len(out), what
                if pairs:                                     # the longest 256 with the longest last
                    out[:256] = out[:256][::-1].copy()
                if not by_keys:
                    assert (np.diff(out[:, 1] * qtiles + out[:, 2]) <= 0).all(), what
                elif s % rows == 0 and (budget + local) * b % rows == 0:
                    keys = np.minimum((budget + local) * b, out[:, 1].astype(np.int64) * s) + rows * (out[:, 2] + 1)
                    assert (np.diff(keys) <= 0).all(), what


@pytest.mark.parametrize("waves,wgs,with_rows,pairs", [(4, 256, 256, 0), (4, 257, 257, 1), (4, 512, 512, 1), (4, 513, 513, 0), (4, 4096, 4096, 0), (4, 1 << 20, 1 << 20, 0), (8, 257, 257, 0),
                                                       (8, 512, 512, 0), (8, 4096, 4096, 0), (4, 512, 448, 1), (4, 512, 447, 0), (4, 384, 336, 1), (4, 384, 335, 0)])
def test_order_of_a_launch(lib, waves, wgs, with_rows, pairs):
    """Long and short row tiles in pairs where the chip holds all workgroups of four waves, two to a compute unit, and one in eight at most is past the end.  In every other launch the row tiles of
    a segment stay together: they read the same keys."""
    for n1, s, b, rows, budget in [(64, 64, 16, 32, 20), (200, 48, 16, 32, 60), (33, 128, 8, 32, 100), (16, 512, 64, 32, 6), (9, 256, 32, 16, 4)]:
        qtiles = -(-s // rows)
        out = np.full((n1 * qtiles, 2), -1, np.int32)
        assert lib.launched(waves, wgs, with_rows, n1, s // b, budget, 1, b, qtiles, rows, out) == (256 if pairs else 0)
        together = (out.reshape(n1, qtiles, 2)[:, :, 0] == np.arange(n1)[::-1, None]).all()
        assert together == (not pairs), (n1, s, b)
