"""The fp32 attention kernels at the borders of their variants: fp32 products or split ones, keys divided between 4 or 8 waves,
tiles of consecutive tokens or one token per key.  Against the fp64 checker with the fp32 bars of the other tests
(unit-variance inputs, so logits of a few units: 128 products and the weighted sum round to about 1e-6)."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from paper_2409_12490_amd import binding as B
from paper_2409_12490_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"

SHAPES = [
    # Hq Hkv   n     s    b    k  L, routes: block-sparse, dense (attention_route)
    (1, 1, 1, 16, 16, 1, 0, "fp32 2x4", "fp32 2x4"),              # one query, one key
    (2, 1, 271, 128, 16, 3, 1, "fp32 2x4", "fp32 2x4"),           # 16 rows, 4 waves, most of them without a tile; a last tile of 15 tokens
    (2, 2, 1553, 288, 48, 40, 0, "fp32 1x8", "fp32 1x8"),         # 16 rows, 8 waves; 48 does not divide 8 x 16 keys
    (8, 4, 1601, 128, 32, 60, 1, "split 8", "split 8"),         # split products, 8 waves; a last row tile of one row
    (8, 2, 2064, 256, 64, 4, 1, "split 4", "split 8"),          # split: 4 waves for the short lists, 8 for dense
    (16, 4, 3120, 512, 128, 16, 0, "split 4", "split 4"),       # split, 4 waves: many workgroups
    (1, 1, 2048, 128, 32, 8, 0, "fp32 2x4", "fp32 2x8"),          # 128 row tiles: two workgroups to a tile, each with half of the channels
    (2, 1, 1009, 255, 51, 9, 1, "fp32 tokens", "fp32 2x4"),          # the same dense; block-sparse a token per key
    (2, 2, 1001, 256, 16, 70, 1, "fp32 2x4", "fp32 2x4"),         # 126 row tiles, long lists; a last tile of nine rows
    (3, 1, 688, 344, 43, 9, 1, "fp32 tokens", "fp32 1x4"),           # dense 129 row tiles: one workgroup to a tile
    (8, 2, 700, 256, 32, 4, 1, "fp32 1x4 pairs", "fp32 1x4 pairs"),           # 352 row tiles of 16, two workgroups to a compute unit: long and short in pairs
    (8, 2, 600, 512, 64, 4, 0, "fp32 1x4", "fp32 1x4 pairs"),           # block-sparse: too many of 512 past the end of the last segment for that
    (4, 2, 3000, 256, 64, 4, 1, "split 4 pairs", "split 8"),          # 376 split tiles of 32 rows in pairs
    (3, 1, 500, 72, 24, 4, 1, "fp32 tokens", "fp32 2x4"),            # blocks of 24: one token per key; segments no multiple of a row tile
    (1, 1, 2048, 256, 64, 20, 0, "fp32 2x8", "fp32 2x8"),          # the same with eight waves: rows of more than 1024 keys
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda c: "x".join(map(str, c[:7])))
def test_variants_against_checker(shape):
    Hq, Hkv, n, s, b, k, L, sparse, dense = shape
    w = H.small_workload("fp32tiles", 1, Hq, Hkv, n, s, b, k, L, dtype="fp32", unit_variance=n > 1)
    assert (H.attention_route(w), H.attention_route(w, False)) == (sparse, dense)
    q, k_, v = synth.make_qkv(w, threads=8)
    qf, kf, vf = (synth.to_f64(t) for t in (q, k_, v))
    q, k_, v = q.to(DEV), k_.to(DEV), v.to(DEV)
    g = np.random.default_rng(n)
    Sd = g.random((1, Hq, w.n_segments, w.n_blocks), dtype=np.float32)
    idx, cnt = O.select(Sd, s, b, k, L)
    heads, segs = sorted({0, Hq - 1}), sorted({0, w.n_segments // 2, w.n_segments - 1})
    todo = [(0, h, j) for h in heads for j in segs]
    o_ref, lse_ref = O.sparse_attention(qf, kf, vf, idx, cnt, s, b, segments=todo)
    out, lse = (t.cpu().numpy() for t in H.gpu_sparse(w, q, k_, v, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV)))
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    for (_, h, j) in todo:
        rows = slice(j * s, min(n, (j + 1) * s))
        assert H.max_abs(out[0, h, rows], o_ref[0, h, rows]) <= H.TOL_OUT["fp32"], (h, j)
        assert H.max_abs(lse[0, h, rows], lse_ref[0, h, rows]) <= 1e-4, (h, j)
    rows = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n), g.integers(0, n, 40)]))
    d_ref, dl_ref = O.dense_causal_attention(qf, kf, vf, rows=rows)
    out, lse = (t.cpu().numpy() for t in H.gpu_dense(w, q, k_, v))
    assert np.isfinite(out).all()
    assert H.max_abs(out[:, :, rows], d_ref) <= H.TOL_OUT["fp32"]
    assert H.max_abs(lse[:, :, rows], dl_ref) <= 1e-4


def test_token_stride_beyond_32_bit_offsets():
    """A token stride of 2^26 elements (256 MB): byte offsets inside a tile of 16 tokens no longer fit 32 bits."""
    n, stride = 19, 1 << 26
    w = H.small_workload("wide", 1, 1, 1, n, 16, 16, 1, 0, dtype="fp32", unit_variance=True)
    q, k, v = synth.make_qkv(w)
    rows = torch.empty((n - 1) * stride + 256, dtype=torch.float32, device=DEV)
    kd = rows.as_strided((1, 1, n, 128), (0, 0, stride, 1), 0)
    vd = rows.as_strided((1, 1, n, 128), (0, 0, stride, 1), 128)
    kd.copy_(k); vd.copy_(v)
    qd = q.to(DEV)
    d_ref, _ = O.dense_causal_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v))
    out, _ = H.gpu_dense(w, qd, kd, vd)
    assert H.max_abs(out.cpu().numpy(), d_ref) <= H.TOL_OUT["fp32"]
    idx, cnt = O.select(np.ones((1, 1, w.n_segments, w.n_blocks), np.float32), 16, 16, 1, 0)      # every block: dense again
    out, _ = H.gpu_sparse(w, qd, kd, vd, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))
    assert H.max_abs(out.cpu().numpy(), d_ref) <= H.TOL_OUT["fp32"]


def _logits(row):
    """K of one head whose logits with an all-ones first channel of Q are ``row`` (the scale 1/sqrt(128) taken out)."""
    k = torch.zeros((1, 1, len(row), 128), dtype=torch.float32)
    k[0, 0, :, 0] = torch.tensor(row, dtype=torch.float32) * 128 ** 0.5
    return k


@pytest.mark.parametrize("b", [16, 24, 0], ids=["runs", "tokens", "dense"])
@pytest.mark.parametrize("case", ["large_values", "subnormal_weights"])
def test_value_range(case, b):
    """Weights stay at most 1 and count down to the subnormals.  large_values: keys with V = 3e37 in the tiles of one wave, the later ones
    with a logit 5 above the first (a factor of 148); a weight above 11 would overflow.  subnormal_weights: keys whose weight is exp(-90) = 8e-40 beside one
    of weight 1 and V = 0, with V = 2^118. The logits are exact up to one rounding, 90 * 2^-24 = 5e-6 relative in a weight; a
    subnormal of 8e-40 is known to 2^-19 = 2e-6."""
    n = 300
    row = [-20.0 if case == "large_values" else -90.0] * n
    v = torch.full((1, 1, n, 128), 1.0 if case == "large_values" else 2.0 ** 118, dtype=torch.float32)
    row[0] = 0.0
    if case == "large_values":
        row[64] = row[128] = 5.0                                  # later tiles of the same wave, with four waves and with eight
        v[0, 0, [0, 64, 128]] = 3e37
    else:
        v[0, 0, 0] = 0.0
    k, q = _logits(row), torch.zeros((1, 1, n, 128), dtype=torch.float32)
    q[..., 0] = 1.0
    w = H.small_workload("range", 1, 1, 1, n, b * 25 or 16, b or 16, 25, 0, dtype="fp32")
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    if b:
        idx, cnt = O.select(np.ones((1, 1, w.n_segments, w.n_blocks), np.float32), b * 25, b, 25, 0)    # every block
        out, lse = H.gpu_sparse(w, qd, kd, vd, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))
    else:
        out, lse = H.gpu_dense(w, qd, kd, vd)
    ref, lse_ref = O.dense_causal_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v))
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=2e-5)
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=0, atol=2e-5)


@pytest.mark.parametrize("b,s", [(32, 128), (24, 72)], ids=["runs", "tokens"])
def test_batches(b, s):
    """Batch and head offsets of block-sparse (a run of tokens per tile, a token per key), shared and dense attention: three batches, groups of
    two heads, token-major storage, every row of every head."""
    w = H.small_workload("fp32batch", 3, 6, 3, 307, s, b, 3, 1, dtype="fp32", unit_variance=True)
    q, k, v = synth.make_qkv(w, threads=4)
    qf, kf, vf = (synth.to_f64(t) for t in (q, k, v))
    qd, kd, vd = (t.to(DEV).transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    Sd = np.random.default_rng(b).random((3, 6, w.n_segments, w.n_blocks), dtype=np.float32)
    idx, cnt = O.select(Sd, s, b, 3, 1)
    runs = [(O.sparse_attention(qf, kf, vf, idx, cnt, s, b), H.gpu_sparse(w, qd, kd, vd, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))),
            (O.dense_causal_attention(qf, kf, vf), H.gpu_dense(w, qd, kd, vd))]
    idx, cnt = O.select(O.shared_group_scores(Sd, 3), s, b, 3, 1)
    runs.append((O.sparse_attention(qf, kf, vf, *O.expand_shared_lists(idx, cnt, 6), s, b),
                 H.gpu_sparse_shared(w, qd, kd, vd, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))))
    for (o_ref, lse_ref), (out, lse) in runs:
        assert H.max_abs(out.cpu().numpy(), o_ref) <= H.TOL_OUT["fp32"]
        assert H.max_abs(lse.cpu().numpy(), lse_ref) <= 1e-4


def test_segment_far_longer_than_the_sequence():
    """A segment set longer than the sequence launches no workgroups past its end: with 2^28 tokens to a segment they would be 2^24, more
    than a launch takes."""
    n = 100
    w = H.small_workload("longseg", 1, 1, 1, n, 1 << 28, 1 << 14, 1, 0, dtype="fp32", unit_variance=True)
    q, k, v = synth.make_qkv(w)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    idx = torch.full((1, 1, 1, (1 << 14) + 1), -1, dtype=torch.int32, device=DEV)
    idx[..., 0] = 0
    out, _ = H.gpu_sparse(w, qd, kd, vd, idx, torch.ones((1, 1, 1), dtype=torch.int32, device=DEV))
    d_ref, _ = O.dense_causal_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v))
    assert H.max_abs(out.cpu().numpy(), d_ref) <= H.TOL_OUT["fp32"]


@pytest.mark.parametrize("n,others", [(600, 8), (1024, 3), (1025, 2), (1333, 2), (2048, 2)])
@pytest.mark.parametrize("b", [16, 0], ids=["runs", "dense"])
def test_a_shared_row_tile_has_the_same_bits(n, others, b):
    """Two workgroups share the row tiles of small launches, each with half of the channels.  That changes no sum: the head's result is, bit for bit, that of the same
    head among others, where a tile has one workgroup and its keys are split between as many waves (four, or eight for more than 1024 keys)."""
    one = H.small_workload("alone", 1, 1, 1, n, 512, b or 64, 130 if b else 40, 1, dtype="fp32", unit_variance=True)
    many = H.small_workload("among", 1, others, others, n, 512, b or 64, 130 if b else 40, 1, dtype="fp32", unit_variance=True)
    assert H.attention_kernel(one, bool(b)) == H.attention_kernel(many, bool(b)) == "fp32"
    waves = 8 if n > 1024 else 4
    assert H.attention_route(one, bool(b)) == f"fp32 2x{waves}" and H.attention_route(many, bool(b)).startswith(f"fp32 1x{waves}")
    q, k, v = (t.to(DEV) for t in synth.make_qkv(many, threads=8))
    Sd = np.random.default_rng(n).random((1, others, many.n_segments, many.n_blocks), dtype=np.float32)
    idx, cnt = (torch.from_numpy(x).to(DEV) for x in O.select(Sd, 512, b or 64, many.budget_blocks, 1))
    for h in (0, others - 1):
        q1, k1, v1 = (t[:, h:h + 1].clone() for t in (q, k, v))
        if b:
            lists = [t[:, h:h + 1].clone() for t in (idx, cnt)]
            pair = H.gpu_sparse(many, q, k, v, idx, cnt), H.gpu_sparse(one, q1, k1, v1, *lists)
        else:
            pair = H.gpu_dense(many, q, k, v), H.gpu_dense(one, q1, k1, v1)
        for all_heads, alone in zip(*pair):
            assert torch.equal(all_heads[:, h:h + 1], alone)
