"""A whole layer captured into a graph and replayed several times on new inputs, eager work in between: every replay equals the eager
result bit for bit.  Every attention kernel, one and several score chunks, rows that are streamed by the selection, shared lists."""
import pytest
import torch

from paper_2409_12490_amd import binding as B
from paper_2409_12490_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [
    # Hq Hkv    n    s    b   k  dtype, kernel of the block-sparse attention
    (4, 2, 2100, 256, 64, 5, "bf16", "32"),      # one score chunk
    (8, 2, 4500, 256, 16, 9, "bf16", "256"),     # several chunks
    (16, 4, 2950, 128, 32, 10, "bf16", "128"),
    (2, 1, 33100, 512, 16, 9, "bf16", "128"),    # 2069 blocks
    (4, 1, 1200, 128, 32, 4, "fp32", "fp32"),
    (8, 2, 1003, 256, 64, 3, "fp32", "split"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_replays_equal_eager(case):
    Hq, Hkv, n, s, b, k, dtype, kernel = case
    w = H.small_workload("capture", 1, Hq, Hkv, n, s, b, k, 1, dtype=dtype, unit_variance=True)
    assert H.attention_kernel(w) == kernel
    sets = [[t.to(DEV) for t in synth.make_qkv(w.replace(seed=w.seed + i), threads=4)] for i in range(3)]
    q, k_, v = (t.clone() for t in sets[0])
    out = torch.empty_like(q)
    p = H.params_for(w, q, k_, out=out)
    S, ws = B.alloc_scores(p), B.alloc_workspace(p)
    (idx, cnt), (sidx, scnt) = B.alloc_lists(p), B.alloc_shared_lists(p)
    shared, dense = torch.empty_like(q), torch.empty_like(q)

    def layer():
        B.critiprefill_estimate(p, q, k_, None, S, ws)
        B.critiprefill_select(p, S, idx, cnt)
        B.critiprefill_sparse_attn(p, q, k_, v, idx, cnt, out, None)
        B.critiprefill_select_shared(p, S, sidx, scnt)
        B.critiprefill_sparse_attn_shared(p, q, k_, v, sidx, scnt, shared, None)
        B.critiprefill_dense_causal_attn(p, q, k_, v, dense, None)

    results = (S, idx, cnt, out, sidx, scnt, shared, dense)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        layer()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer()
    for fresh in sets + sets[:1]:
        for mine, new in zip((q, k_, v), fresh):
            mine.copy_(new)
        layer()
        torch.cuda.synchronize()
        eager = [t.clone() for t in results]
        for t in results:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, e) for a, e in zip(results, eager))
