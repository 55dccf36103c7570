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
