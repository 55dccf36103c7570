"""Block-sparse bf16 attention where the 128-row kernel takes it: segments of 65 to 128 rows, of 320 and 384, blocks of odd multiples of 16 in
short lists, 256-row workgroups for half of the chip; last segments and row tiles of every length, runs that end with the sequence or inside a tile, lists whose blocks end
inside a tile.  Against the checker on sampled segments, with the bars of the other bf16 attention tests."""
import numpy as np
import pytest
import torch

from oracle import critiprefill_oracle as O
from paper_2409_12490_amd import synth
from tests import helpers as H
from tests.test_gpu_bf16_wide import check, dev, lists, sample

pytestmark = pytest.mark.gpu


def make(Bt, Hq, Hkv, n, s, b, k, L, gain=1.0):
    w = H.small_workload("half", Bt, Hq, Hkv, n, s, b, k, L, unit_variance=True)
    q, k_, v = synth.make_qkv(w, threads=8)
    return w, (q.float() * gain).to(q.dtype), (k_.float() * gain).to(k_.dtype), v


SHAPES = [
    # Bt Hq Hkv  n     s    b    k   L
    (1, 16, 4, 2950, 128, 32, 10, 1), (1, 16, 4, 4013, 96, 16, 12, 1), (1, 17, 17, 3501, 112, 112, 5, 0), (2, 4, 2, 9001, 128, 32, 4, 1),
    (1, 16, 4, 2945, 128, 128, 3, 2),        # a last segment of one row
    (1, 32, 8, 1900, 192, 48, 6, 1), (1, 16, 4, 3100, 384, 64, 5, 1),
    (1, 32, 8, 3300, 256, 16, 20, 1),        # two 128-row tiles, runs of 16
    (1, 16, 4, 4100, 320, 64, 3, 1), (1, 8, 2, 4000, 512, 64, 4, 1),
    (2, 8, 2, 3999, 208, 16, 7, 0),          # 13 blocks of 16 to a segment: lists that end inside a tile
    (1, 8, 1, 8300, 128, 32, 3, 1),          # 520 (query head, segment) pairs of a KV head: a round of 512 and a part of one
    (1, 16, 1, 8400, 256, 16, 4, 0),         # 528, of two row tiles each
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda t: "x".join(map(str, t)))
@pytest.mark.parametrize("gain", [1.0, 6.0])
def test_sparse(shape, gain):
    w, q, k, v = make(*shape, gain)
    assert H.attention_kernel(w) == "128"
    idx, cnt = lists(w, w.n_q_heads)
    out, lse = H.gpu_sparse(w, *dev(q, k, v, idx, cnt))
    check(w, out, lse, q, k, v, idx, cnt, sample(w))


@pytest.mark.parametrize("k,kernel", [(382, "128"), (383, "32")])
def test_longest_lists(k, kernel):
    """Lists of 49152 keys, the most that the kernel's table of tiles holds; one block more is for the 32-row kernel."""
    w, q, k_, v = make(1, 1, 1, 49200, 128, 128, k, 1)
    assert H.attention_kernel(w) == kernel
    idx, cnt = lists(w, 1)
    assert cnt.max() == min(k + 2, w.n_blocks)
    out, lse = H.gpu_sparse(w, *dev(q, k_, v, idx, cnt))
    check(w, out, lse, q, k_, v, idx, cnt, [(0, 0, j) for j in (0, 100, w.n_segments - 2, w.n_segments - 1)])


@pytest.mark.parametrize("shape", [(8, 2, 4000, 512, 64, 4, 1), (8, 2, 4000, 512, 32, 30, 1), (8, 2, 4000, 512, 16, 80, 1), (7, 1, 4100, 480, 48, 30, 1)],
                         ids=["b64", "b32", "b16", "b48"])
@pytest.mark.parametrize("gain", [1.0, 6.0])
def test_same_bits_as_256_rows(shape, gain):
    """The same sequences once in a launch of this kernel and once, twice over, in one that the 256-row kernel takes."""
    one, q, k, v = make(1, *shape, gain)
    two = make(2, *shape)[0]
    assert (H.attention_kernel(one), H.attention_kernel(two)) == ("128", "256")
    idx, cnt = lists(one, one.n_q_heads)
    args = dev(q, k, v, idx, cnt)
    out, lse = H.gpu_sparse(one, *args)
    out2, lse2 = H.gpu_sparse(two, *(x.repeat(2, *[1] * (x.dim() - 1)) for x in args))
    for i in (0, 1):
        assert torch.equal(out2[i], out[0]) and torch.equal(lse2[i], lse[0])


@pytest.mark.parametrize("shape", [(1, 16, 4, 2950, 128, 32, 10, 1), (1, 32, 8, 3300, 256, 16, 20, 1)], ids=["b32", "b16"])
def test_shared_lists_token_major(shape):
    w, q, k, v = make(*shape)
    assert H.attention_kernel(w) == "128"
    idx, cnt = lists(w, w.n_kv_heads)
    dq, dk, dv = (x.transpose(1, 2).contiguous().transpose(1, 2).to("cuda") for x in (q, k, v))
    out, lse = H.gpu_sparse_shared(w, dq, dk, dv, *dev(idx, cnt))
    check(w, out, lse, q, k, v, *O.expand_shared_lists(idx, cnt, w.n_q_heads), sample(w))


@pytest.mark.parametrize("b", [16, 64])
def test_bad_lists(b):
    """Entries outside the sequence have no tokens, entries behind the count are not read, counts outside the list are clamped."""
    s = 128
    w, q, k, v = make(1, 16, 4, 2950, s, b, 7, 1)
    assert H.attention_kernel(w) == "128"
    idx, cnt = lists(w, w.n_q_heads)
    bad, bad_cnt, ref, ref_cnt = idx.copy(), cnt.copy(), idx.copy(), cnt.copy()
    for h in range(w.n_q_heads):
        for j in range(w.n_segments):
            c = int(cnt[0, h, j])
            bad[0, h, j, c:] = 0
            keep = list(idx[0, h, j, :c])
            if c > 3:
                bad[0, h, j, 1], bad[0, h, j, 2] = (-1 - h, w.n_blocks)[h & 1], (-(1 << 31), (1 << 31) - 1)[j & 1]
                del keep[1:3]
            if (h + j) % 5 == 4:
                bad_cnt[0, h, j], keep = -h, []
            ref[0, h, j] = -1
            ref[0, h, j, :len(keep)] = keep
            ref_cnt[0, h, j] = len(keep)
    out, lse = H.gpu_sparse(w, *dev(q, k, v, bad, bad_cnt))
    o_ref, lse_ref = O.sparse_attention(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), ref, ref_cnt, s, b)
    assert H.max_abs(out.float().cpu().numpy(), o_ref) <= 2e-2
    assert np.array_equal(np.isneginf(lse.cpu().numpy()), np.isneginf(lse_ref))
    again, _ = H.gpu_sparse(w, *dev(q, k, v, bad, bad_cnt))
    assert torch.equal(out, again)
