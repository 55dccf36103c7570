"""The bf16 attention kernels with 32-row workgroups whose waves split the keys (4 or 8 waves; blocks of multiples of 16 and of other sizes; dense) and
with 256-row workgroups (blocks of 64, of 32, of other sizes; dense).  Ragged lengths, last tiles of one token, segments shorter than a row
tile, lists that hold bad entries.  Bars of the other bf16 attention tests."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from paper_2409_12490_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"

SHAPES = [
    # Hq Hkv    n    s    b   k  L, rows of a workgroup: block-sparse, dense
    (1, 1, 1, 16, 16, 1, 0, "32", "32"),             # one query, one key
    (2, 1, 33, 32, 32, 2, 0, "32", "32"),            # a last tile of one token
    (4, 2, 2047, 256, 64, 5, 1, "32", "32"),         # 256 row tiles: eight waves
    (4, 2, 2049, 96, 96, 4, 0, "32", "32"),          # 260: blocks of 96
    (2, 2, 1003, 24, 8, 9, 1, "32", "32"),           # a token per key; segments of 24
    (3, 1, 1500, 144, 48, 6, 1, "32", "32"),         # blocks of 48
    (16, 4, 1024, 512, 128, 2, 1, "32", "32"),
    (16, 4, 1025, 512, 128, 2, 1, "32", "32"),       # 528 row tiles
    (40, 8, 1025, 512, 128, 2, 1, "256", "32"),      # blocks of 64s
    (24, 8, 777, 256, 32, 6, 0, "32", "32"),         # four waves
    (48, 8, 777, 256, 32, 6, 0, "256", "32"),        # blocks of 32
    (24, 8, 1399, 64, 16, 5, 2, "32", "32"),
    (40, 8, 1399, 240, 24, 5, 2, "256", "256"),      # a token per key
    (32, 8, 2100, 192, 96, 3, 1, "256", "256"),      # blocks of 96
    (2, 1, 8200, 512, 64, 4, 1, "32", "32"),         # dense with eight waves
    (1, 1, 16001, 240, 48, 5, 1, "32", "32"),        # 534 row tiles
    (1, 1, 16321, 240, 48, 5, 1, "128", "32"),       # 545 row tiles, short lists
    (1, 1, 16321, 240, 48, 40, 0, "32", "32"),       # long ones
    (32, 8, 250, 240, 48, 6, 0, "32", "32"),         # 8000 rows in 288 tiles, 250 keys: four waves
    (3, 1, 77, 4096, 64, 2, 1, "32", "32"),          # a segment longer than the sequence
    (24, 8, 800, 4096, 16, 2, 1, "32", "32"),
    (48, 16, 800, 4096, 16, 2, 1, "256", "32"),
]


def lists(w, seed):
    S = np.random.default_rng(seed).random((1, w.n_q_heads, w.n_segments, w.n_blocks), dtype=np.float32)
    return O.select(S, w.segment_size, w.block_size, w.budget_blocks, w.local_blocks)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda c: "x".join(map(str, c[:7])))
def test_both_kernels_against_checker(shape):
    Hq, Hkv, n, s, b, k, L, sparse, dense = shape
    w = H.small_workload("rows", 1, Hq, Hkv, n, s, b, k, L, unit_variance=n > 1)
    assert (H.attention_kernel(w), H.attention_kernel(w, False)) == (sparse, dense)
    q, k_, v = synth.make_qkv(w, threads=8)
    qf, kf, vf = (synth.to_f64(t) for t in (q, k_, v))
    # token-major storage, as a model's projections leave it
    qd, kd, vd = (t.to(DEV).transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k_, v))
    idx, cnt = lists(w, n)
    heads, segs = sorted({0, Hq // 2, Hq - 1}), sorted({0, 1, w.n_segments // 2, w.n_segments - 1} & set(range(w.n_segments)))
    todo = [(0, h, j) for h in heads for j in segs]
    o_ref, lse_ref = O.sparse_attention(qf, kf, vf, idx, cnt, s, b, segments=todo)
    out, lse = (t.float().cpu().numpy() for t in H.gpu_sparse(w, qd, kd, vd, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV)))
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    for (_, h, j) in todo:
        rows = slice(j * s, min(n, (j + 1) * s))
        assert H.max_abs(out[0, h, rows], o_ref[0, h, rows]) <= H.TOL_OUT["bf16"], (h, j)
        assert H.max_abs(lse[0, h, rows], lse_ref[0, h, rows]) <= 2e-2, (h, j)
    rows = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n), np.random.default_rng(1).integers(0, n, 40)]))
    G = Hq // Hkv
    out, lse = (t.float().cpu().numpy() for t in H.gpu_dense(w, qd, kd, vd))
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    for h in heads:
        d_ref, dl_ref = O.dense_causal_attention(qf[:, h:h + 1], kf[:, h // G:h // G + 1], vf[:, h // G:h // G + 1], rows=rows)
        assert H.max_abs(out[:, h:h + 1, rows], d_ref) <= H.TOL_OUT["bf16"], h
        assert H.max_abs(lse[:, h:h + 1, rows], dl_ref) <= 2e-2, h


@pytest.mark.parametrize("b", [64, 32, 16])
@pytest.mark.parametrize("heads", [2, 20, 40], ids=["32_rows", "32_rows_more", "256_rows"])
def test_bad_and_empty_lists(heads, b):
    """Empty lists, a count past the row, negative and too large entries: masked, as in the tests of the 256-row kernel."""
    w = H.small_workload("badrows", 1, heads, 1, 1000, 256, b, 3, 1)
    assert H.attention_kernel(w) == ("256" if heads == 40 else "32")
    q, k, v = synth.make_qkv(w, threads=4)
    idx, cnt = lists(w, b)
    bad, bad_cnt, ref, ref_cnt = idx.copy(), cnt.copy(), idx.copy(), cnt.copy()
    bad_cnt[0, 0, 1] = 1_000_000
    bad_cnt[0, 0, 2] = ref_cnt[0, 0, 2] = 0
    bad[0, 1, 2, :2] = [w.n_blocks + 5, 1 << 30]; bad_cnt[0, 1, 2] = 2; ref_cnt[0, 1, 2] = 0
    bad[0, 1, 3, 0] = -4; bad_cnt[0, 1, 3] = 1; ref_cnt[0, 1, 3] = 0
    todo = [(0, h, j) for h in (0, 1) for j in range(w.n_segments)]
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), ref, ref_cnt, 256, b, segments=todo)
    out, lse = H.gpu_sparse(w, q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(bad).to(DEV), torch.from_numpy(bad_cnt).to(DEV))
    assert H.max_abs(out[0, :2].float().cpu().numpy(), o_ref[0, :2]) <= H.TOL_OUT["bf16"]
    assert np.array_equal(np.isneginf(lse[0, :2].cpu().numpy()), np.isneginf(lse_ref[0, :2]))
