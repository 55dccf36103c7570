"""Lists from rows of more than 2048 blocks, per head and shared: streamed for budgets up to 256, held in registers (up to 4096 blocks) or
searched by a workgroup each above.  With row ends that no load divides, at the edges of both bucket counts, bit-exact against the checker's rule on the same scores.  The score layouts reach every way out
of the search: few candidates, more than one search's worth, too many equal to the threshold (found again above it, or ties to be
counted out), and large scores that share their buckets (searched in the row itself)."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def scores(kind, shape, g):
    S = g.random(shape, dtype=np.float32) * 1e-3
    if kind == "zeros":
        S[g.random(shape) < 0.99] = 0.0
    elif kind == "few_values":
        S = np.round(g.standard_normal(shape) * 2).astype(np.float32)
    elif kind == "one_bucket":
        S[..., 5::256] += 1.0
        S[..., 7::64] += 0.5
    elif kind == "buckets_in_front":
        S[..., : shape[-1] // 3] += 1.0
        S[..., ::512] += 1.0
    elif kind == "constant":
        S[...] = 0.25
    return S


@pytest.mark.parametrize("kind", ["spread", "zeros", "few_values", "one_bucket", "buckets_in_front", "constant"])
@pytest.mark.parametrize("n_blocks,budget", [(2049, 1), (2051, 128), (3000, 129), (4096, 64), (4099, 256), (8190, 128), (8192, 200)])
def test_rows(n_blocks, budget, kind):
    b = 16
    w = H.small_workload("stream", 1, 2, 1, n_blocks * b, 1024, b, budget, 1)
    print(n_blocks, budget, kind, flush=True)
    S = scores(kind, (1, 2, w.n_segments, w.n_blocks), np.random.default_rng(n_blocks + budget))
    q = torch.empty((1, 2, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    k = torch.empty((1, 1, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    idx_o, cnt_o = O.select(S, 1024, b, budget, 1)
    H.check_selection(S, idx_o, cnt_o, *H.gpu_select(w, q, k, torch.from_numpy(S).to(DEV)), w, exact=True)
    Sg = O.shared_group_scores(S, 1)
    idx_o, cnt_o = O.select(Sg, 1024, b, budget, 1)
    H.check_selection(Sg, idx_o, cnt_o, *H.gpu_select_shared(w, q, k, torch.from_numpy(S).to(DEV)), w, exact=True)


@pytest.mark.parametrize("kind", ["spread", "zeros", "one_bucket", "constant"])
@pytest.mark.parametrize("n_blocks,budget", [(2051, 129), (3000, 256), (4097, 31)])
def test_rows_of_a_group(n_blocks, budget, kind):
    b = 16
    w = H.small_workload("streamsh", 1, 6, 2, n_blocks * b, 256, b, budget, 2)
    S = scores(kind, (1, 6, w.n_segments, w.n_blocks), np.random.default_rng(n_blocks + budget))
    Sg = O.shared_group_scores(S, 2)
    idx_o, cnt_o = O.select(Sg, 256, b, budget, 2)
    q = torch.empty((1, 6, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    k = torch.empty((1, 2, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
    H.check_selection(Sg, idx_o, cnt_o, *H.gpu_select_shared(w, q, k, torch.from_numpy(S).to(DEV)), w, exact=True)


@pytest.mark.parametrize("kind", ["spread", "zeros", "few_values", "constant"])
@pytest.mark.parametrize("n_blocks,budget", [(2049, 257), (3001, 300), (4096, 257), (4096, 1000), (4099, 257), (8192, 300), (8192, 2000)])
def test_budgets_above_the_stream(n_blocks, budget, kind):
    """Per head; shared between two query heads; and shared with one query head to a KV head, few lists and many."""
    b, s = 16, 1024
    for heads, kv, seg in [(2, 1, s), (2, 2, s), (2, 2, 128)] if n_blocks == 4096 else [(2, 1, s), (2, 2, s)]:
        w = H.small_workload("above", 1, heads, kv, n_blocks * b, seg, b, budget, 1)
        print(n_blocks, budget, kind, heads, kv, w.n_segments, flush=True)
        S = scores(kind, (1, heads, w.n_segments, w.n_blocks), np.random.default_rng(n_blocks + budget))
        q = torch.empty((1, heads, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
        k = torch.empty((1, kv, w.seq_len, 128), dtype=torch.bfloat16, device=DEV)
        if kv == 1:
            idx_o, cnt_o = O.select(S, seg, b, budget, 1)
            H.check_selection(S, idx_o, cnt_o, *H.gpu_select(w, q, k, torch.from_numpy(S).to(DEV)), w, exact=True)
        Sg = O.shared_group_scores(S, kv)
        idx_o, cnt_o = O.select(Sg, seg, b, budget, 1)
        H.check_selection(Sg, idx_o, cnt_o, *H.gpu_select_shared(w, q, k, torch.from_numpy(S).to(DEV)), w, exact=True)
