"""The 256-row bf16 attention kernel asks for its first tiles by entries that it reads ahead of the list's copy in LDS: short lists (fewer
blocks, or halves of a tile, than it reads ahead), rows whose unused tail holds plausible block numbers instead of -1, lists of more than 512
entries.  Against the checker, with the bar of the other bf16 attention tests."""
import numpy as np
import pytest

from tests.test_gpu_bf16_wide import check, dev, lists, make
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s,kernel", [(64, 256, "256"), (128, 256, "256"), (192, 768, "256"), (32, 256, "256"), (96, 768, "256"), (192, 384, "128"), (96, 288, "128")],
                         ids=["b64", "b128", "b192", "b32", "b96", "b192_128_rows", "b96_128_rows"])
def test_blocks_behind_the_count(b, s, kernel):
    w, q, k, v = make(1, 40, 4, 1201, s, b, 5, 1)
    assert H.attention_kernel(w) == kernel
    idx, cnt = lists(w, w.n_q_heads)
    ref, ref_cnt = idx.copy(), cnt.copy()
    for h in range(w.n_q_heads):
        for j in range(w.n_segments):
            keep = min(int(cnt[0, h, j]), 1 + (h + j) % 5)
            ref[0, h, j, keep:] = -1
            ref_cnt[0, h, j] = keep
            idx[0, h, j, keep:] = (h + np.arange(idx.shape[3] - keep)) % max(1, j * w.blocks_per_segment)    # blocks that the rows would see
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, ref_cnt))
    todo = [(0, h, j) for h in (0, 1, 2, 3, 4, 39) for j in range(w.n_segments)]
    check(w, out, lse, q, k, v, ref, ref_cnt, todo)


@pytest.mark.parametrize("b", [32, 64])
def test_lists_of_more_than_512_entries(b):
    w, q, k, v = make(1, 2 if b == 32 else 1, 1, 520 * b + 64, 512, b, 515, 1)
    assert H.attention_kernel(w) == "256"
    idx, cnt = lists(w, w.n_q_heads)
    assert cnt.max() > 512
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, idx, cnt, [(0, 0, j) for j in (0, 1, w.n_segments - 2, w.n_segments - 1)])
