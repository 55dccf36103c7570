"""fp32 attention on fp16 pairs (launches with enough row tiles): edges of tiles and runs, both wave counts, block sizes, layouts, shared lists and
bad lists, values that change their scale on the way and values that no scale fits.

Tolerances: as the other fp32 attention tests where inputs are of unit scale.  Relative errors (2-norm): a factor is known to 2^-24, products are
exact, sums of n terms in fp32 to about sqrt(n) 2^-24 of their size; 1e-6 = 16 * 2^-24 covers 32 channels-steps, a few hundred keys and the exponential."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from paper_2409_12490_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def make(Bt, Hq, Hkv, n, s, b, k, L, seed=7):
    w = H.small_workload("split", Bt, Hq, Hkv, n, s, b, k, L, dtype="fp32", seed=seed, unit_variance=True)
    q, k_, v = synth.make_qkv(w, threads=8)
    return w, q.to(DEV), k_.to(DEV), v.to(DEV)


def lists(w, heads, seed=3):
    S = np.random.default_rng(seed).random((w.batch, heads, w.n_segments, w.n_blocks), dtype=np.float32)
    return O.select(S, w.segment_size, w.block_size, w.budget_blocks, w.local_blocks)


def tiles(w, sparse):
    s = w.segment_size if sparse else w.seq_len
    rest = w.seq_len % s
    return w.batch * w.n_q_heads * (w.seq_len // s * -(-s // 32) + -(-rest // 32))


def exact(q, k, v, visible):
    """softmax(q k^T / sqrt(d)) v in float64; visible [.., rows, keys]."""
    z = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()) / q.shape[-1] ** 0.5
    z = z.masked_fill(~visible, float("-inf"))
    lse = torch.logsumexp(z, -1)
    return torch.matmul((z - lse.unsqueeze(-1)).exp(), v.double()), lse


def dense_exact(w, q, k, v):
    G = w.n_q_heads // w.n_kv_heads
    i = torch.arange(w.seq_len, device=DEV)
    return exact(q, k.repeat_interleave(G, 1), v.repeat_interleave(G, 1), i[None] <= i[:, None])


def rel(x, y):
    return float((x.double() - y).norm() / y.norm())


def sampled(w):
    heads = sorted({0, 1, w.n_q_heads - 1})
    segs = sorted({0, 1, w.n_segments // 2, w.n_segments - 1} & set(range(w.n_segments)))
    return [(i, h, j) for i in range(w.batch) for h in heads for j in segs]


def check(w, out, lse, q, k, v, idx, cnt):
    todo = sampled(w)
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q.cpu()), synth.to_f64(k.cpu()), synth.to_f64(v.cpu()), idx, cnt, w.segment_size, w.block_size, segments=todo)
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(out).all()
    for (i, h, j) in todo:
        rows = slice(j * w.segment_size, min(w.seq_len, (j + 1) * w.segment_size))
        assert H.max_abs(out[i, h, rows], o_ref[i, h, rows]) <= H.TOL_OUT["fp32"], (i, h, j)
        assert H.max_abs(lse[i, h, rows], lse_ref[i, h, rows]) <= H.TOL_OUT["fp32"], (i, h, j)


SPARSE = [
    # Bt, Hq, Hkv, n, s, b, k, L: runs of 16 that pair up across blocks, odd numbers of them, ragged ends inside a run
    (1, 8, 2, 1003, 128, 16, 5, 1), (1, 8, 2, 1400, 144, 16, 20, 0), (1, 8, 4, 1601, 112, 16, 9, 1), (2, 5, 5, 900, 256, 32, 7, 1), (1, 12, 3, 1111, 240, 48, 6, 2),
    (1, 16, 1, 1000, 320, 80, 4, 1), (1, 10, 2, 1025, 512, 64, 3, 1), (1, 3, 1, 2900, 256, 128, 6, 0), (2, 4, 2, 2100, 512, 64, 24, 1), (1, 2, 1, 4100, 4096, 64, 8, 0),
]


@pytest.mark.parametrize("shape", SPARSE, ids=lambda t: "x".join(map(str, t)))
@pytest.mark.parametrize("token_major", [False, True])
def test_sparse(shape, token_major):
    w, q, k, v = make(*shape)
    assert tiles(w, True) >= 256
    idx, cnt = lists(w, w.n_q_heads)
    if token_major:
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
    out, lse = H.gpu_sparse(w, q, k, v, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))
    check(w, out, lse, q, k, v, idx, cnt)


@pytest.mark.parametrize("shape", [(1, 8, 2, 1000), (1, 8, 2, 1003), (2, 5, 5, 833), (1, 4, 2, 2065), (1, 20, 4, 1031), (1, 32, 8, 257), (1, 300, 300, 17), (1, 260, 1, 33)],
                         ids=lambda t: "x".join(map(str, t)))
def test_dense(shape):
    w, q, k, v = make(*shape, 256, 64, 4, 1)
    assert tiles(w, False) >= 256
    out, lse = H.gpu_dense(w, q, k, v)
    o_ref, lse_ref = dense_exact(w, q, k, v)
    assert rel(out, o_ref) <= 1e-6 and rel(lse, lse_ref) <= 1e-6
    assert float((out - o_ref).abs().max()) <= H.TOL_OUT["fp32"]


def test_shared_lists():
    w, q, k, v = make(2, 8, 2, 700, 128, 32, 5, 1)
    idx, cnt = lists(w, w.n_kv_heads)
    out, lse = H.gpu_sparse_shared(w, q, k, v, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))
    check(w, out, lse, q, k, v, *O.expand_shared_lists(idx, cnt, w.n_q_heads))


@pytest.mark.parametrize("b", [16, 64])
def test_bad_lists_and_counts(b):
    """Entries outside the sequence have no tokens, entries behind the count are not read, counts outside the list are clamped."""
    w, q, k, v = make(1, 10, 2, 1000, 256, b, 5, 1)
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
    out, lse = H.gpu_sparse(w, q, k, v, torch.from_numpy(bad).to(DEV), torch.from_numpy(bad_cnt).to(DEV))
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q.cpu()), synth.to_f64(k.cpu()), synth.to_f64(v.cpu()), ref, ref_cnt, 256, b)
    assert H.max_abs(out.cpu().numpy(), o_ref) <= H.TOL_OUT["fp32"]
    assert np.array_equal(np.isneginf(lse.cpu().numpy()), np.isneginf(lse_ref))


def test_run_twice_and_powers_of_two():
    """The scales follow the values: powers of two in V come out exactly, powers of two between Q and K do not show at all."""
    w, q, k, v = make(1, 8, 2, 1003, 256, 32, 6, 1)
    idx, cnt = (torch.from_numpy(x).to(DEV) for x in lists(w, 8))
    out, lse = H.gpu_sparse(w, q, k, v, idx, cnt)
    for e in (-70, 0, 40, 90):
        again, lse2 = H.gpu_sparse(w, q, k, v * 2.0 ** e, idx, cnt)
        assert torch.equal(again, out * 2.0 ** e) and torch.equal(lse2, lse)
    for e in (-30, 30):
        again, lse2 = H.gpu_sparse(w, q * 2.0 ** e, k * 2.0 ** -e, v, idx, cnt)
        assert torch.equal(again, out) and torch.equal(lse2, lse)


GROW = {"k_grows": ("k", 200.0), "v_grows": ("v", 3000.0), "v_shrinks": ("v", 1 / 500.0), "v_apart": ("v", 1e-9), "v_far_apart": ("v", 1e25), "q_rows_apart": ("q", 1e-7)}


@pytest.mark.parametrize("case", GROW)
@pytest.mark.parametrize("shape", [(1, 8, 2, 1003), (1, 24, 2, 1003)], ids=["eight", "four"])
def test_scales_on_the_way(case, shape):
    """Values that outgrow the scale of a wave's first tiles (set anew), or lie too far apart for one scale (walked again with fp32 products)."""
    w, q, k, v = make(*shape, 256, 64, 4, 1)
    which, factor = GROW[case]
    x = {"q": q, "k": k, "v": v}[which]
    x[:, :, 300:] *= factor
    if which == "k":
        q = q / 50                                             # logits within fp32's exponent and a few hundred
    out, lse = H.gpu_dense(w, q, k, v)
    o_ref, lse_ref = dense_exact(w, q, k, v)
    # per row, relative to it: rows before 300 see only the small or large part.  k_grows: logits of a few hundred, known to 2^-24 of themselves
    err = (out.double() - o_ref).norm(dim=3) / o_ref.norm(dim=3)
    assert float(err.max()) <= (2e-4 if which == "k" else 4e-6)
    assert rel(lse, lse_ref) <= 1e-6


@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 3e38])
@pytest.mark.parametrize("which", ["v", "k"])
def test_values_that_fit_no_scale(which, bad):
    """One bad value at token 700: what is after it takes it, what is in earlier segments' rows does not."""
    w, q, k, v = make(1, 8, 2, 1003, 256, 64, 4, 1)
    o_ref, _ = dense_exact(w, q, k, v)
    x = {"k": k, "v": v}[which]
    x[0, 1, 700, 5] = bad
    out, _ = H.gpu_dense(w, q, k, v)
    assert rel(out[:, :4], o_ref[:, :4]) <= 1e-6                # the other KV head
    assert rel(out[:, 4:, :640], o_ref[:, 4:, :640]) <= 1e-6
    if which == "v":
        after = out[0, 4:, 700:, 5]
        if bad == 3e38:
            ref, _ = dense_exact(w, q, k, v)
            assert rel(after, ref[0, 4:, 700:, 5]) <= 1e-5
        else:
            assert not torch.isfinite(after).any()
        rest = [c for c in range(128) if c != 5]
        assert rel(out[0, 4:, 700:, rest], o_ref[0, 4:, 700:, rest]) <= 1e-6


def test_segment_longer_than_the_sequence():
    """A segment set longer than the sequence launches no workgroups past its end."""
    w, q, k, v = make(1, 10, 2, 900, 65536, 64, 4, 1)
    idx, cnt = lists(w, w.n_q_heads)
    out, lse = H.gpu_sparse(w, q, k, v, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))
    check(w, out, lse, q, k, v, idx, cnt)
