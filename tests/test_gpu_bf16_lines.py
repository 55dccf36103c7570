"""The bf16 attention kernels on both sides of the lines between them: 32-row workgroups for rows that leave 256-row ones idle and for segments of up
to 64, blocks that are odd multiples of 16 as pairs of runs (also an odd number of runs, and runs that end inside a tile), four and eight waves; 128-row
ones for segments of up to 128 and a few short lists; and the 256-row kernel's special cases at row counts that are its own.
Against the checker on sampled segments and rows, with the bars of the other bf16 attention tests."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from paper_2409_12490_amd import synth
from tests import helpers as H
from tests.test_gpu_bf16_wide import check, dev, lists, sample

pytestmark = pytest.mark.gpu


def make(Bt, Hq, Hkv, n, s, b, k, L, gain=1.0):
    w = H.small_workload("lines", Bt, Hq, Hkv, n, s, b, k, L, unit_variance=True)
    q, k_, v = synth.make_qkv(w, threads=8)
    return w, (q.float() * gain).to(q.dtype), (k_.float() * gain).to(k_.dtype), v


SPARSE = [
    # Bt Hq Hkv  n     s    b    k   L, rows of a workgroup
    (1, 2, 1, 1003, 112, 16, 9, 1, "32"),          # runs of 16, odd numbers of them; segments of 112: a last row tile of 16
    (1, 3, 3, 777, 240, 48, 6, 1, "32"), (2, 5, 5, 901, 160, 80, 4, 1, "32"), (1, 4, 2, 2050, 96, 32, 20, 0, "32"),
    (1, 8, 2, 1500, 512, 64, 20, 1, "32"),         # 376 row tiles, nearly all keys: eight waves; and four:
    (1, 8, 2, 1500, 512, 64, 2, 1, "32"),
    (1, 16, 4, 4100, 128, 32, 40, 1, "128"),       # segments of 128, 2064 row tiles
    (1, 16, 4, 4100, 128, 32, 8, 0, "128"),
    (1, 4, 2, 3001, 128, 32, 40, 1, "32"),         # 376 row tiles
    (1, 32, 8, 1300, 64, 16, 30, 2, "32"),         # segments of 64
    (1, 9, 3, 2051, 256, 32, 40, 1, "32"),         # 585 row tiles, 1.4 times the keys
    (1, 2, 1, 9501, 512, 64, 3, 1, "128"),         # 594 row tiles of few keys
    (1, 7, 7, 3301, 256, 32, 60, 1, "32"),         # 728 row tiles, keys enough
    (1, 16, 4, 2001, 512, 64, 30, 1, "32"),        # 1008 row tiles, all keys
    (1, 17, 17, 2001, 512, 64, 30, 1, "256"),      # 1071
    (1, 17, 17, 2001, 512, 64, 3, 1, "256"),       # of few keys
]


@pytest.mark.parametrize("shape", SPARSE, ids=lambda t: "x".join(map(str, t[:8])))
def test_sparse(shape):
    w, q, k, v = make(*shape[:8])
    assert H.attention_kernel(w) == shape[8]
    idx, cnt = lists(w, w.n_q_heads)
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, idx, cnt, sample(w))


@pytest.mark.parametrize("b", [16, 48, 64])
@pytest.mark.parametrize("token_major", [False, True])
def test_bad_lists_in_32_row_workgroups(b, token_major):
    """Entries outside the sequence have no tokens, entries behind the count are not read, counts outside the list are clamped."""
    s = 192
    w, q, k, v = make(1, 6, 2, 1100, s, b, 5, 1)
    idx, cnt = lists(w, w.n_q_heads)
    bad, bad_cnt, ref, ref_cnt = idx.copy(), cnt.copy(), idx.copy(), cnt.copy()
    for h in range(w.n_q_heads):
        for j in range(w.n_segments):
            c = int(cnt[0, h, j])
            bad[0, h, j, c:] = 0
            keep = list(idx[0, h, j, :c])
            if c > 3:
                bad[0, h, j, 1], bad[0, h, j, 2] = -1 - h, -(1 << 31)
                del keep[1:3]
            if (h + j) % 5 == 4:
                bad_cnt[0, h, j], keep = -h, []
            ref[0, h, j] = -1
            ref[0, h, j, :len(keep)] = keep
            ref_cnt[0, h, j] = len(keep)
    if token_major:
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
    dq, dk, dv = (x.to("cuda") for x in (q, k, v))
    out, lse = H.gpu_sparse(w, dq, dk, dv, *dev(bad, bad_cnt))
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), ref, ref_cnt, s, b)
    assert H.max_abs(out.float().cpu().numpy(), o_ref) <= 2e-2
    assert np.array_equal(np.isneginf(lse.cpu().numpy()), np.isneginf(lse_ref))


@pytest.mark.parametrize("shape", [(1, 32, 8, 256), (1, 8, 2, 1000), (1, 16, 4, 1000), (1, 33, 11, 1003), (2, 6, 2, 4100), (1, 32, 8, 1536), (1, 32, 8, 1537),
                                   (1, 16, 4, 4096), (1, 16, 4, 4097), (2, 20, 4, 1403)], ids=lambda t: "x".join(map(str, t)))
@pytest.mark.parametrize("gain", [1.0, 6.0])
def test_dense(shape, gain):
    w, q, k, v = make(*shape, 512, 64, 5, 1, gain)
    out, lse = (t.float().cpu().numpy() for t in H.gpu_dense(w, *dev(q, k, v)))
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    rows = np.unique(np.concatenate([np.arange(33), np.arange(w.seq_len - 33, w.seq_len), np.random.default_rng(1).integers(0, w.seq_len, 30)]))
    heads = sorted({0, w.n_q_heads - 1})
    G = w.n_q_heads // w.n_kv_heads
    o_ref, lse_ref = O.dense_causal_attention(synth.to_f64(q)[:, heads], synth.to_f64(k)[:, [h // G for h in heads]], synth.to_f64(v)[:, [h // G for h in heads]], rows=rows)
    assert H.max_abs(out[:, heads][:, :, rows], o_ref) <= 2e-2
    assert H.max_abs(lse[:, heads][:, :, rows], lse_ref) <= 2e-2


@pytest.mark.parametrize("b", [64, 32, 16])
def test_256_rows_many_trailing_tiles(b):
    w, q, k, v = make(1, 5, 1, 9001, 8192, b, 4, 0)
    assert H.attention_kernel(w) == "256"
    idx, cnt = lists(w, w.n_q_heads)
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, idx, cnt, [(0, 2, 0), (0, 0, 1), (0, 4, 1)])


@pytest.mark.parametrize("b", [64, 32, 16])
def test_256_rows_negative_and_zero_counts(b):
    w, q, k, v = make(1, 40, 2, 1000, 256, b, 3, 1)
    assert H.attention_kernel(w) == "256"
    idx, cnt = lists(w, w.n_q_heads)
    bad, ref = cnt.copy(), cnt.copy()
    bad[0, 0, 1], bad[0, 39, 2], bad[0, 10, 3] = -3, -(1 << 31), 0
    ref[0, 0, 1] = ref[0, 39, 2] = ref[0, 10, 3] = 0
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, bad))
    todo = [(0, h, j) for h in (0, 10, 39) for j in range(w.n_segments)]
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), idx, ref, 256, b, segments=todo)
    for h in (0, 10, 39):
        assert H.max_abs(out[0, h].float().cpu().numpy(), o_ref[0, h]) <= 2e-2
        assert np.array_equal(np.isneginf(lse[0, h].cpu().numpy()), np.isneginf(lse_ref[0, h]))
