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
