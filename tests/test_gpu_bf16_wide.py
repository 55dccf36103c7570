"""The 256-row bf16 attention kernel: shared lists, logits far from the unit scale, repeated runs; and the 32-row kernel at some 17000 to 34000
rows: segments far longer than a workgroup, negative counts, several dense batches with head counts that are no powers of two (the same of the 256-row
kernel is in test_gpu_bf16_lines.py); in every tile mode (blocks of 64, of 32, of other sizes, dense).  Against the
checker on sampled segments and rows, with the bars of the other bf16 attention tests."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from paper_2409_12490_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def make(Bt, Hq, Hkv, n, s, b, k, L, gain=1.0):
    w = H.small_workload("wide", Bt, Hq, Hkv, n, s, b, k, L, unit_variance=True)
    assert Bt * Hq * n > 16384
    q, k_, v = synth.make_qkv(w, threads=8)
    return w, (q.float() * gain).to(q.dtype), (k_.float() * gain).to(k_.dtype), v


def lists(w, heads, seed=3):
    S = np.random.default_rng(seed).random((w.batch, heads, w.n_segments, w.n_blocks), dtype=np.float32)
    return O.select(S, w.segment_size, w.block_size, w.budget_blocks, w.local_blocks)


def sample(w):
    """(batch, head, segment) triples: the corners and the middle of each axis."""
    heads = sorted({0, 1, w.n_q_heads // 2, w.n_q_heads - 1})
    segs = sorted({0, 1, w.n_segments // 2, w.n_segments - 1} & set(range(w.n_segments)))
    return [(i, h, j) for i in range(w.batch) for h in heads for j in segs]


def check(w, out, lse, q, k, v, idx, cnt, todo, tol=2e-2):
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), idx, cnt, w.segment_size, w.block_size, segments=todo)
    out, lse = out.float().cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(out).all()
    for (i, h, j) in todo:
        rows = slice(j * w.segment_size, min(w.seq_len, (j + 1) * w.segment_size))
        assert H.max_abs(out[i, h, rows], o_ref[i, h, rows]) <= tol, (i, h, j)
        assert H.max_abs(lse[i, h, rows], lse_ref[i, h, rows]) <= 2e-2, (i, h, j)


def dev(*arrays):
    return [(torch.from_numpy(a) if isinstance(a, np.ndarray) else a).to(DEV) for a in arrays]


@pytest.mark.parametrize("b,s", [(64, 512), (32, 256), (24, 240)], ids=["b64", "b32", "b24"])
def test_shared_lists(b, s):
    w, q, k, v = make(2, 12, 3, 1403, s, b, 5, 1)
    assert H.attention_kernel(w) == "256"
    idx, cnt = lists(w, w.n_kv_heads)
    out, lse = H.gpu_sparse_shared(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, *O.expand_shared_lists(idx, cnt, w.n_q_heads), sample(w))


@pytest.mark.parametrize("gain", [6.0, 0.05], ids=["peaked", "flat"])
@pytest.mark.parametrize("b", [64, 32, 16])
def test_peaked_and_flat_logits(b, gain):
    """Logits 36 and 0.0025 times as large: the reference point of a row moves again and again, or never after the first tile."""
    w, q, k, v = make(1, 20, 5, 1701, 256, b, 6, 1, gain)
    assert H.attention_kernel(w) == "256"
    idx, cnt = lists(w, w.n_q_heads)
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, idx, cnt, sample(w))


@pytest.mark.parametrize("gain", [6.0, 1.0, 0.05])
def test_dense_batches(gain):
    w, q, k, v = make(2, 12, 3, 1403, 512, 64, 5, 1, gain)
    assert H.attention_kernel(w, False) == "32"
    assert w.batch * w.n_q_heads * w.seq_len > 32768
    out, lse = (t.float().cpu().numpy() for t in H.gpu_dense(w, *dev(q, k, v)))
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    rows = np.unique(np.concatenate([np.arange(40), np.arange(w.seq_len - 40, w.seq_len), np.random.default_rng(1).integers(0, w.seq_len, 60)]))
    o_ref, lse_ref = O.dense_causal_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), rows=rows)
    assert H.max_abs(out[:, :, rows], o_ref) <= 2e-2
    assert H.max_abs(lse[:, :, rows], lse_ref) <= 2e-2


@pytest.mark.parametrize("b", [64, 32, 16])
def test_long_segments_drop_many_trailing_tiles(b):
    """Segments of 8192 tokens: the first query tile of one sees 4 of its own 128 tiles of 64 keys."""
    w, q, k, v = make(1, 3, 1, 9001, 8192, b, 4, 0)
    assert H.attention_kernel(w) == "32"
    idx, cnt = lists(w, w.n_q_heads)
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, idx, cnt, [(0, 2, 0), (0, 0, 1), (0, 2, 1)])


@pytest.mark.parametrize("b", [64, 32, 16])
def test_negative_and_zero_counts(b):
    w, q, k, v = make(1, 20, 1, 1000, 256, b, 3, 1)
    assert H.attention_kernel(w) == "32"
    idx, cnt = lists(w, w.n_q_heads)
    bad, ref = cnt.copy(), cnt.copy()
    bad[0, 0, 1], bad[0, 19, 2], bad[0, 10, 3] = -3, -(1 << 31), 0
    ref[0, 0, 1] = ref[0, 19, 2] = ref[0, 10, 3] = 0
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, bad))
    todo = [(0, h, j) for h in (0, 10, 19) for j in range(w.n_segments)]
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), idx, ref, 256, b, segments=todo)
    for h in (0, 10, 19):
        assert H.max_abs(out[0, h].float().cpu().numpy(), o_ref[0, h]) <= 2e-2
        assert np.array_equal(np.isneginf(lse[0, h].cpu().numpy()), np.isneginf(lse_ref[0, h]))


@pytest.mark.parametrize("b", [64, 32, 16])
def test_run_twice_bit_identical(b):
    w, q, k, v = make(1, 20, 5, 1701, 256, b, 6, 1)
    assert H.attention_kernel(w) == "256"
    args = dev(q, k, v, *lists(w, w.n_q_heads))
    first, second = H.gpu_sparse(w, *args), H.gpu_sparse(w, *args)
    assert all(torch.equal(x, y) for x, y in zip(first, second))
    first, second = H.gpu_dense(w, *args[:3]), H.gpu_dense(w, *args[:3])
    assert all(torch.equal(x, y) for x, y in zip(first, second))
