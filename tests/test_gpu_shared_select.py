"""select_shared with every row length of its kernels and group sizes around the four scores it loads at a time: bit-exact against the
checker's rule on the same scores, ties, zeros and negative (fused) scores among them."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n_blocks", [7, 512, 513, 2048, 4095, 4100])
@pytest.mark.parametrize("group,budget", [(1, 32), (4, 129), (5, 17), (8, 64)])
def test_lists_bit_exact(n_blocks, group, budget):
    b = 16
    w = H.small_workload("shsel", 1, 2 * group, 2, n_blocks * b, 512, b, budget, 1)
    g = np.random.default_rng(n_blocks + group)
    S = (g.standard_normal((1, 2 * group, w.n_segments, w.n_blocks)) * 1e-3).astype(np.float32)
    S[..., ::3] = np.float32(2e-3)                                     # ties
    S[:, :, -1, ::2] = 0.0
    Sg = O.shared_group_scores(S, 2)
    idx_o, cnt_o = O.select(Sg, 512, b, budget, 1)
    q = torch.empty((1, 2 * group, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    k = torch.empty((1, 2, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    idx_g, cnt_g = H.gpu_select_shared(w, q, k, torch.from_numpy(S).to(DEV))
    H.check_selection(Sg, idx_o, cnt_o, idx_g, cnt_g, w, exact=True)


@pytest.mark.parametrize("n_blocks,heads", [(300, 3), (2049, 1), (4096, 5), (4099, 2)])
def test_one_query_head_per_kv_head(n_blocks, heads):
    """With as many KV heads as query heads the shared lists are the per-head lists, whichever kernel makes them."""
    b = 16
    w = H.small_workload("single", 2, heads, heads, n_blocks * b, 512, b, 33, 1)
    S = torch.rand((2, heads, w.n_segments, w.n_blocks), generator=torch.Generator().manual_seed(n_blocks)).to(DEV)
    S[..., ::5] = 0.5                                                  # ties
    q = torch.empty((2, heads, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    for mine, theirs in zip(H.gpu_select_shared(w, q, q, S), H.gpu_select(w, q, q, S)):
        assert torch.equal(mine, theirs)
