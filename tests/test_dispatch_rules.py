"""The library's dispatch rules on the CPU, on both sides of their lines: which attention kernel, and how the fp32 kernel divides a launch."""
import pytest

from tests import helpers as H


def workload(dtype, heads, kv_heads, n, s, b, k, L=1):
    return H.small_workload("rules", 1, heads, kv_heads, n, s, b, k, L, dtype=dtype)


@pytest.mark.parametrize("n,s,b,k,kernel", [
    (50000, 256, 16, 31, "128"), (131072, 256, 16, 31, "128"), (50000, 256, 16, 32, "256"),           # 768 and 784 keys, 6272 and 16384 workgroups of 256 rows
    (33000, 256, 16, 51, "128"), (34000, 256, 16, 51, "256"), (33000, 256, 16, 52, "256"),            # 1088 and 1104 keys, 4128 and 4256 workgroups
    (12800, 256, 16, 64, "128"), (12801, 256, 16, 64, "256"), (12800, 256, 16, 65, "256"),            # 1296 and 1312 keys, 1600 and 1632 workgroups
    (11000, 480, 48, 16, "128"), (50000, 480, 48, 16, "256"),
    (50000, 512, 32, 8, "256"),                                                                       # blocks of 32
])
def test_blocks_of_odd_multiples_of_16(n, s, b, k, kernel):
    assert H.attention_kernel(workload("bf16", 32, 8, n, s, b, k)) == kernel


@pytest.mark.parametrize("heads,n,s,b,k,kernel", [
    ((32, 8), 1000, 512, 64, 4, "32"), ((32, 8), 1024, 512, 64, 4, "32"), ((32, 8), 1025, 512, 64, 4, "256"),    # 1024 row tiles, 832 keys; 1056
    ((16, 4), 1664, 512, 64, 4, "32"), ((16, 4), 1665, 512, 64, 4, "128"),                                       # at most twice the keys
    ((16, 4), 2000, 512, 64, 16, "32"), ((8, 2), 4000, 512, 64, 32, "32"), ((8, 2), 4000, 512, 64, 16, "128"), ((8, 2), 4096, 512, 64, 32, "32"),
    ((1, 1), 32768, 512, 64, 247, "32"), ((1, 1), 32768, 512, 64, 160, "32"), ((1, 1), 32768, 512, 64, 100, "128"), ((1, 1), 32769, 512, 64, 247, "256"),
])
def test_rows_of_32_up_to_1024_row_tiles(heads, n, s, b, k, kernel):
    assert H.attention_kernel(workload("bf16", *heads, n, s, b, k)) == kernel


@pytest.mark.parametrize("heads,n,route", [(1, 2048, "fp32 2x8"), (1, 2049, "fp32 1x8"), (2, 1024, "fp32 2x4"), (2, 1025, "fp32 1x8"), (8, 256, "fp32 2x4"), (8, 257, "fp32 1x4"), (1, 1025, "fp32 2x8"), (1, 1024, "fp32 2x4")])
def test_shared_row_tiles_up_to_128(heads, n, route):
    """Dense: 128 and 129 or more row tiles of 16; more than 1024 keys have eight waves."""
    assert H.attention_route(workload("fp32", heads, heads, n, 512, 64, 4), False) == route


@pytest.mark.parametrize("dtype,heads,n,route", [
    ("fp32", 16, 256, "fp32 1x4"), ("fp32", 16, 257, "fp32 1x4 pairs"), ("fp32", 16, 480, "fp32 1x4 pairs"), ("fp32", 12, 650, "fp32 1x4 pairs"),     # 256, 272, 480 and 492 workgroups
    ("fp32", 32, 512, "split 4 pairs"), ("fp32", 32, 513, "split 4"), ("fp32", 32, 256, "split 8"), ("fp32", 32, 257, "split 4 pairs"),
    ("bf16", 32, 256, "32 4"), ("bf16", 32, 257, "32 4 pairs"), ("bf16", 32, 512, "32 4 pairs"), ("bf16", 32, 513, "32 4"), ("bf16", 8, 2048, "32 8"),
])
def test_pairs_where_the_chip_holds_all(dtype, heads, n, route):
    """Dense: more than 256 and at most 512 workgroups of four waves."""
    assert H.attention_route(workload(dtype, heads, heads, n, 512, 64, 4), False) == route


@pytest.mark.parametrize("dtype,heads,n,route", [
    ("bf16", 16, 896, "32 4 pairs"), ("bf16", 16, 960, "32 4 pairs"), ("bf16", 16, 864, "32 4"),       # 512 workgroups, of which 64, 32 and 80 past the end
    ("fp32", 8, 896, "fp32 1x4 pairs"), ("fp32", 8, 864, "fp32 1x4"),
])
def test_no_pairs_where_many_are_past_the_end(dtype, heads, n, route):
    """Block-sparse, segments of 512: one workgroup in eight may be past the end of the last one."""
    assert H.attention_route(workload(dtype, heads, heads, n, 512, 64, 4)) == route
