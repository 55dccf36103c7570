"""The division by multiplication that the bf16 attention kernel's index arithmetic uses, restated here and compared with integer
division at the edges of its range (0 <= n < 2^31, 1 <= d < 2^31): multiples of d and their neighbours, powers of two, the largest n."""
import random


def fast_div(d):
    shift = 0
    while (1 << shift) < d:
        shift += 1
    mul = ((((1 << shift) - d) << 32) // d + 1) & 0xffffffff

    def div(n):
        t = ((mul * n) >> 32) + n
        assert t < 1 << 32                                   # the sum stays in 32 bits
        return t >> shift
    return div


def test_exact_over_the_range():
    g = random.Random(1)
    top = (1 << 31) - 1
    divisors = [1, 2, 3, 5, 7, 255, 256, 257, 65535, 65537, top, top - 1, 1 << 30, (1 << 30) + 1]
    divisors += [g.randrange(1, 1 << g.randrange(1, 31)) for _ in range(400)]
    for d in divisors:
        div = fast_div(d)
        ns = {0, 1, d - 1, d, min(top, d + 1), top, top // d * d, max(0, top // d * d - 1)}
        for _ in range(50):
            x = d * g.randrange(0, top // d + 1)
            ns |= {x, max(0, x - 1), min(top, x + 1), g.randrange(0, top + 1)}
        assert all(div(n) == n // d for n in ns), d
