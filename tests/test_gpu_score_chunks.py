"""The bf16 score kernel at the borders of its forms: rows of one chunk (256 blocks) and of several, one or several groups of 16
segments to a wave, groups shared by several waves, groups of several heads in one workgroup, n2 that no tile or vector store divides.
Both softmax domains, with and without fusion (in place and not), against the fp64 checker with the bar of the other score tests."""
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
    # Hq Hkv    n     s    b
    (1, 1, 40, 16, 16),                # 3 segments, 3 blocks
    (3, 1, 4096, 256, 16),             # 256 blocks: one chunk to the last block, one group shared by eight waves
    (2, 1, 4099, 64, 16),              # 257 blocks: two chunks, most of the second one empty; 65 segments
    (2, 2, 8300, 512, 16),             # 519 blocks, 17 segments: a group of one segment
    (40, 8, 17400, 64, 32),            # 544 blocks, 272 segments, 120 chunks
    (32, 4, 30011, 96, 16),            # 1876 blocks, 313 segments, 256 chunks
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("domain", [0, 1])
def test_scores(shape, domain):
    Hq, Hkv, n, s, b = shape
    w = H.small_workload("chunks", 1, Hq, Hkv, n, s, b, 2, 0, alpha=0.75)
    q, k, _ = synth.make_qkv(w, threads=8)
    heads = sorted({0, Hq - 1})
    G = Hq // Hkv
    qd, kd = q.to(DEV), k.to(DEV)
    p = H.params_for(w, qd, kd, softmax_domain=domain)
    ws = B.alloc_workspace(p)
    plain = B.alloc_scores(p).fill_(float("nan"))
    B.critiprefill_estimate(p, qd, kd, None, plain, ws)
    prev = torch.rand(plain.shape, generator=torch.Generator().manual_seed(n)).to(DEV)
    fused, inplace = torch.full_like(prev, float("nan")), prev.clone()
    B.critiprefill_estimate(p, qd, kd, prev, fused, ws)
    B.critiprefill_estimate(p, qd, kd, inplace, inplace, ws)
    torch.cuda.synchronize()
    assert torch.equal(fused, inplace)
    assert bool(torch.isfinite(plain).all())
    for h in heads:
        S_o = O.estimate(synth.to_f64(q[:, h:h + 1]), synth.to_f64(k[:, h // G:h // G + 1]), s, b, softmax_domain=domain)
        np.testing.assert_allclose(plain[:, h:h + 1].cpu().numpy(), S_o, rtol=2e-4, atol=1e-30)
        S_f = 0.75 * S_o + 0.25 * prev[:, h:h + 1].cpu().numpy().astype(np.float64)
        np.testing.assert_allclose(fused[:, h:h + 1].cpu().numpy(), S_f, rtol=2e-4, atol=1e-30)


# The sixteens of segments of a KV head's query heads are dealt to workgroups, which take eight per round; a last round of at most four, two
# or one is shared by two, four or eight waves each.  Per workgroup here: (40, 8) 9 or 8, (16, 4) 16 or 15, (40, 5) 38, (96, 2) 4,
# (32, 16) 10, (6, 2) 56 or 55.
DEALT = [
    # B  Hq  Hkv   n     s    b
    (1, 40, 8, 17400, 64, 32),         # 17 sixteens a head: most workgroups span two heads
    (2, 16, 4, 17021, 32, 32),         # two rounds, the last with a wave to spare; 532 blocks
    (3, 40, 5, 7001, 24, 8),           # five rounds; an odd number of chunks of (batch, KV head)
    (1, 96, 2, 5003, 64, 16),          # one round, two waves to a group; 313 blocks
    (4, 32, 16, 9003, 128, 16),        # a round and a rest of two, four waves to a group; 563 blocks
    (1, 6, 2, 33003, 16, 8),           # seven rounds and more; 2063 segments, 4126 blocks
]


@pytest.mark.parametrize("shape", DEALT, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("domain", [0, 1])
def test_groups_dealt_to_workgroups(shape, domain):
    """Every row of every head is written, and each position of a query head in its group is compared with the checker."""
    Bt, Hq, Hkv, n, s, b = shape
    w = H.small_workload("dealt", Bt, Hq, Hkv, n, s, b, 2, 0, alpha=0.75)
    q, k, _ = synth.make_qkv(w, threads=8)
    G = Hq // Hkv
    qd, kd = q.to(DEV), k.to(DEV)
    p = H.params_for(w, qd, kd, softmax_domain=domain)
    ws = B.alloc_workspace(p)
    plain = B.alloc_scores(p).fill_(float("nan"))
    B.critiprefill_estimate(p, qd, kd, None, plain, ws)
    prev = torch.rand(plain.shape, generator=torch.Generator().manual_seed(n)).to(DEV)
    fused = prev.clone()
    B.critiprefill_estimate(p, qd, kd, fused, fused, ws)
    torch.cuda.synchronize()
    # an element that a wave did not write is NaN in one and S' in the other
    torch.testing.assert_close(fused, 0.75 * plain + 0.25 * prev, rtol=1e-6, atol=1e-37)
    heads = [(Bt - 1, (Hkv - 1) * G + x) for x in sorted({0, 1, G // 2, G - 1} & set(range(G)))] + [(0, 0)]
    for i, h in heads:
        S_o = O.estimate(synth.to_f64(q[i:i + 1, h:h + 1]), synth.to_f64(k[i:i + 1, h // G:h // G + 1]), s, b, softmax_domain=domain)
        np.testing.assert_allclose(plain[i, h].cpu().numpy(), S_o[0, 0], rtol=2e-4, atol=1e-30)
