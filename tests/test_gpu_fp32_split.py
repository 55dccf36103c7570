"""fp32 attention on triples of bf16 (launches with enough row tiles): edges of tiles and runs, both wave counts, block sizes, layouts, shared lists and
bad lists, values, weights and channels of any size beside each other, values that cannot be split.

Tolerances: as the other fp32 attention tests where inputs are of unit scale.  Relative errors (2-norm): factors are exact, products known to
2^-24, sums of n terms in fp32 to about sqrt(n) 2^-24 of their size; 1e-6 = 16 * 2^-24 covers the channels, a few hundred keys and the exponential."""
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
    (1, 16, 1, 1000, 320, 80, 4, 1), (1, 10, 2, 1025, 512, 64, 3, 1), (1, 3, 1, 2900, 256, 128, 6, 0), (2, 4, 2, 2100, 512, 64, 24, 1), (1, 3, 1, 4100, 4096, 64, 8, 0),
]


@pytest.mark.parametrize("shape", SPARSE, ids=lambda t: "x".join(map(str, t)))
@pytest.mark.parametrize("token_major", [False, True])
def test_sparse(shape, token_major):
    w, q, k, v = make(*shape)
    assert H.attention_kernel(w) == "split"
    idx, cnt = lists(w, w.n_q_heads)
    if token_major:
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
    out, lse = H.gpu_sparse(w, q, k, v, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV))
    check(w, out, lse, q, k, v, idx, cnt)


@pytest.mark.parametrize("shape", [(1, 8, 2, 1000), (1, 8, 2, 1003), (2, 5, 5, 833), (1, 6, 2, 2065), (1, 20, 4, 1031), (1, 32, 8, 257), (1, 300, 300, 17), (1, 260, 1, 33)],
                         ids=lambda t: "x".join(map(str, t)))
def test_dense(shape):
    w, q, k, v = make(*shape, 256, 64, 4, 1)
    assert H.attention_kernel(w, False) == "split"
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
    """Powers of two in V come out exactly, powers of two between Q and K do not show at all."""
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
    """Values that grow or shrink on the way through the sequence."""
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


def every_block(w, b):
    """Lists that hold every block: dense attention again."""
    return [torch.from_numpy(x).to(DEV) for x in O.select(np.ones((w.batch, w.n_q_heads, w.n_segments, w.n_blocks), np.float32), w.segment_size, b, 25, 0)]


LIGHT = {
    # logit of the light keys, their V, V of token 0 (logit 0)
    "v1": (-17.0, 1.0, 0.0), "v1_lighter": (-25.0, 1.0, 0.0), "v_large": (-25.0, 2.0 ** 70, 0.0), "v_2_100": (-25.0, 2.0 ** 100, 0.0),
    "v_beside_1": (-28.0, 2.0 ** 30, 1.0), "subnormal": (-90.0, 2.0 ** 60, 0.0), "subnormal_2_118": (-90.0, 2.0 ** 118, 0.0),
}


@pytest.mark.parametrize("b", [16, 0], ids=["runs", "dense"])
@pytest.mark.parametrize("case", LIGHT)
def test_light_keys(case, b):
    """Keys of small weight count where the heavy one has a small V: down to the subnormal weights, at any size of V.  Logits are exact up to one
    rounding, 90 * 2^-24 = 5e-6 relative in a weight; a subnormal weight of 8e-40 is known to 2^-19 = 2e-6."""
    n, H_ = 300, 32
    logit, light, heavy = LIGHT[case]
    w = H.small_workload("light", 1, H_, H_, n, b * 25 or 16, b or 16, 25, 0, dtype="fp32")
    q = torch.zeros((1, H_, n, 128), dtype=torch.float32, device=DEV)
    k, v = torch.zeros_like(q), torch.full_like(q, light)
    q[..., 0] = 1.0
    k[:, :, 1:, 0] = logit * 128 ** 0.5
    v[:, :, 0] = heavy
    assert H.attention_kernel(w, bool(b)) == "split"
    out, lse = H.gpu_sparse(w, q, k, v, *every_block(w, b)) if b else H.gpu_dense(w, q, k, v)
    ref, lse_ref = O.dense_causal_attention(synth.to_f64(q[:, :1].cpu()), synth.to_f64(k[:, :1].cpu()), synth.to_f64(v[:, :1].cpu()))
    for h in (0, 7, 31):
        np.testing.assert_allclose(out[:, h].cpu().numpy(), ref[:, 0], rtol=2e-5)
        np.testing.assert_allclose(lse[:, h].cpu().numpy(), lse_ref[:, 0], rtol=0, atol=2e-5)


def test_a_single_key_returns_its_value():
    """A row that sees one key has that key's V, bit for bit: no operand is held in fewer bits than it came in."""
    w, q, k, v = make(2, 32, 8, 333, 256, 64, 4, 1)
    out, _ = H.gpu_dense(w, q, k, v)
    assert torch.equal(out[:, :, 0], v.repeat_interleave(4, 1)[:, :, 0])


@pytest.mark.parametrize("e", [10, 24, 36, 60])
@pytest.mark.parametrize("which", ["v", "qk", "kq"])
def test_channels_apart(which, e):
    """A power of two in some channels of V comes out of the same channels, exactly; between channels of Q and K it does not show."""
    w, q, k, v = make(1, 8, 2, 1003, 256, 32, 6, 1)
    idx, cnt = (torch.from_numpy(x).to(DEV) for x in lists(w, 8))
    out, lse = H.gpu_sparse(w, q, k, v, idx, cnt)
    d = torch.ones(128, device=DEV)
    d[32:64] = d[100] = 2.0 ** -e
    if which == "v":
        again, lse2 = H.gpu_sparse(w, q, k, v * d, idx, cnt)
        assert torch.equal(again, out * d) and torch.equal(lse2, lse)
    else:
        again, lse2 = H.gpu_sparse(w, *((q * d, k / d) if which == "qk" else (q / d, k * d)), v, idx, cnt)
        assert torch.equal(again, out) and torch.equal(lse2, lse)


@pytest.mark.parametrize("factor", [1e4, 1e10, 1e25])
@pytest.mark.parametrize("first", [2, 34])
def test_later_values_larger(first, factor):
    """What a row may not see does not show in it, whatever its size."""
    w, q, k, v = make(1, 8, 2, 1003, 256, 64, 4, 1)
    out, lse = H.gpu_dense(w, q, k, v)
    v[:, :, first:] *= factor
    again, lse2 = H.gpu_dense(w, q, k, v)
    o_ref, lse_ref = dense_exact(w, q, k, v)
    err = (again.double() - o_ref).norm(dim=3) / o_ref.norm(dim=3)
    assert float(err.max()) <= 4e-6
    assert torch.equal(again[:, :, :first], out[:, :, :first]) and torch.equal(lse, lse2)


@pytest.mark.parametrize("which", ["v", "k", "q"])
def test_values_below_the_split(which):
    """Values too small for three bf16 parts (below 2^-110): a power of two between Q and K, or in V, still does not show but for the rounding of other
    sums (fp32 products take over)."""
    w, q, k, v = make(1, 8, 2, 1003, 256, 32, 6, 1)
    idx, cnt = (torch.from_numpy(x).to(DEV) for x in lists(w, 8))
    out, lse = H.gpu_sparse(w, q, k, v, idx, cnt)
    e = 2.0 ** -112                                           # unit-scale values keep their 24 bits above 2^-149 (but for those below 2^-14)
    args = {"v": (q, k, v * e), "k": (q / e, k * e, v), "q": (q * e, k / e, v)}[which]
    again, lse2 = H.gpu_sparse(w, *args, idx, cnt)
    assert rel(again, out.double() * (e if which == "v" else 1.0)) <= 2e-6
    assert rel(lse2, lse.double()) <= 1e-6


def test_infinities():
    """An infinite value goes to what sees it, as an infinity; a key at minus infinity is as good as not there."""
    w, q, k, v = make(1, 8, 2, 1003, 256, 64, 4, 1)
    o_ref, _ = dense_exact(w, q, k, v)
    x = v.clone()
    x[0, 1, 700, 5] = float("inf")
    out, _ = H.gpu_dense(w, q, k, x)
    assert torch.isposinf(out[0, 4:, 704:, 5]).all()          # rows of later workgroups, which see all keys of its tile
    rest = [c for c in range(128) if c != 5]
    assert rel(out[0, 4:, :, rest], o_ref[0, 4:, :, rest]) <= 1e-6
    q, y = q.clone(), k.clone()
    q[..., 3] = q[..., 3].abs() + 0.1
    y[0, :, 700, 3] = -float("inf")
    out, lse = H.gpu_dense(w, q, y, v)
    visible = torch.ones(1003, 1003, dtype=torch.bool, device=DEV).tril()
    visible[:, 700] = False
    y[0, :, 700, 3] = 0.0
    o_ref, lse_ref = exact(q, y.repeat_interleave(4, 1), v.repeat_interleave(4, 1), visible)
    assert rel(out, o_ref) <= 1e-6 and rel(lse, lse_ref) <= 1e-6


def test_runs_behind_the_last_row():
    """A tile's second run that lies behind the workgroup's last row is not touched: segments of three runs behind an odd number of blocks, so that the
    second and third of a segment share a tile, of which the rows of its first 32 see one."""
    w, q, k, v = make(1, 8, 2, 1203, 48, 16, 5, 0)
    assert H.attention_kernel(w) == "split"
    idx, cnt = (torch.from_numpy(x).to(DEV) for x in lists(w, 8))
    out, lse = H.gpu_sparse(w, q, k, v, idx, cnt)
    first = 10 * 48 + 32
    k[:, :, first:first + 16, 7] = float("inf")
    v[:, :, first:first + 16] = float("inf")
    again, lse2 = H.gpu_sparse(w, q, k, v, idx, cnt)
    assert torch.equal(again[:, :, :first], out[:, :, :first]) and torch.equal(lse2[:, :, :first], lse[:, :, :first])
