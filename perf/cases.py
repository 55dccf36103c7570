"""The work that a user of the library has it do, as cases that can be timed and checked one by one.

A case names an operation (``op``) and its sizes:

``layer``     one attention layer of a prefill: estimate, select, block-sparse attention; with ``fused`` the scores of
              the layer before go in, as in every layer of a model but the first
``estimate``  Algorithm 1 alone (a program that inspects or accumulates the scores)
``select``    the top-k lists alone, from given scores
``sparse``    block-sparse attention alone, with given lists
``shared``    one list per KV head: select_shared and sparse_attn_shared, from given scores
``dense``     dense causal attention: the layers that a program does not prune, and the comparison
``tokens`` = n, ``segment`` = s, ``block`` = b, ``budget`` and ``local`` in blocks.  ``token_major``: Q, K, V and O are
stored [batch, token, head, channel], as a model's projections write them, else [batch, head, token, channel].

Inputs follow the recipe of the package's generator (a random walk over positions plus unit noise per channel, scaled
to unit variance and rounded to bf16, or as drawn in fp32), drawn on the GPU because the largest hold 10^9 values.
"""
import torch

from paper_2409_12490_amd import binding as B

D = 128
DEV = "cuda"


def _case(name, op, dtype, batch, hq, hkv, tokens, segment, block, budget, local, fused=False, domain=0, hot=0.0, lse=False, token_major=False):
    return {"name": name, "op": op, "dtype": dtype, "batch": batch, "hq": hq, "hkv": hkv, "tokens": tokens, "segment": segment, "block": block,
            "budget": budget, "local": local, "fused": fused, "domain": domain, "hot": hot, "lse": lse, "token_major": token_major}


def listed():
    return [
        # the smallest configuration of the benchmark: one fp32 head, where launches and latency are what counts
        _case("layer_fp32_1x2048", "layer", "fp32", 1, 1, 1, 2048, 128, 32, 8, 0),
        # fp32 attention of a few heads at a length that no tile divides: the reference that a bf16 result is compared with
        _case("sparse_fp32_4x4096", "sparse", "fp32", 1, 4, 2, 4096, 256, 64, 6, 1, lse=True),
        _case("dense_fp32_4x2500", "dense", "fp32", 1, 4, 2, 2500, 256, 64, 6, 1, lse=True),
        # a short prompt through a Llama3-8B-shaped layer, of odd length, as the projections lay it out, past its first layer
        _case("layer_bf16_32x2000", "layer", "bf16", 1, 32, 8, 2000, 256, 32, 32, 0, fused=True, token_major=True),
        # the 16K configuration: the pruned attention of a middle-sized prompt
        _case("sparse_bf16_32x16384", "sparse", "bf16", 1, 32, 8, 16384, 512, 64, 16, 1),
        # the layers that stay dense, and prompts too short to prune, with the log-sum-exp that a chunked prefill merges by
        _case("dense_bf16_32x8192", "dense", "bf16", 1, 32, 8, 8192, 512, 64, 16, 1, lse=True),
        # the 4-layer stack at 64K tokens, batch 2, the paper's block of 32: its three steps one by one
        _case("estimate_bf16_2x32x65536", "estimate", "bf16", 2, 32, 8, 65536, 256, 32, 32, 0, fused=True),
        _case("select_2x32x65536", "select", "bf16", 2, 32, 8, 65536, 256, 32, 32, 0),
        _case("sparse_bf16_2x32x65536", "sparse", "bf16", 2, 32, 8, 65536, 256, 32, 32, 0),
        # the headline: one Llama3-8B-shaped layer at 128K tokens
        _case("layer_bf16_32x131072", "layer", "bf16", 1, 32, 8, 131072, 512, 64, 32, 1),
        # a Yi-9B-shaped layer at 128K with hot keys and one list per KV head
        _case("shared_bf16_32x131072", "shared", "bf16", 1, 32, 4, 131072, 512, 64, 32, 1, hot=0.05),
        # dense attention of a long prompt
        _case("dense_bf16_32x32768", "dense", "bf16", 1, 32, 8, 32768, 512, 64, 32, 1),
    ]


def draw(rng):
    while True:
        op = rng.choice(["layer", "layer", "sparse", "sparse", "estimate", "select", "shared", "dense"])
        if rng.random() < 0.25:
            dtype, heads, most = "fp32", [(1, 1), (2, 1), (3, 3), (4, 2), (8, 2)], 8192
        else:
            dtype, heads, most = "bf16", [(32, 8), (32, 8), (32, 4), (8, 2), (4, 4), (2, 1)], 131072
        hq, hkv = rng.choice(heads)
        tokens = int(512 * (most / 512) ** rng.random())
        tokens = tokens if rng.random() < 0.5 else max(512, tokens // 512 * 512)
        segment, block = rng.choice([(512, 64), (512, 64), (512, 32), (256, 32), (256, 64), (128, 32), (512, 128), (128, 16)])
        budget = max(1, int(256 * 16 ** rng.random()) // block)
        case = _case("", op, dtype, rng.choice([1, 1, 2]), hq, hkv, tokens, segment, block, budget, rng.choice([0, 1, 1, 2]),
                     fused=rng.random() < 0.5, domain=rng.choice([0, 0, 0, 1]), hot=rng.choice([0.0, 0.05]), lse=rng.random() < 0.3,
                     token_major=rng.random() < 0.4)
        del case["name"]
        cost = work(case)
        # fp32 has a sixteenth of the matrix rate; the scores of the finest blocks grow with the square of the length
        if cost["flops"] <= (3e10 if dtype == "fp32" else 8e12) and cost["bytes"] <= 3.5e9:
            return case


def _sizes(case):
    n, s, b = case["tokens"], case["segment"], case["block"]
    return n, s, b, s // b, -(-n // s), -(-n // b)


def _pairs(case):
    """(query, key) pairs that one (batch, query head) visits, and the entries of its lists."""
    n, s, b, r, n1, _ = _sizes(case)
    if case["op"] == "dense":
        return n * (n + 1) // 2, 0
    pairs = entries = 0
    for j in range(n1):
        rows = min(n, (j + 1) * s) - j * s
        past = min(case["local"], j * r) + min(case["budget"], max(0, j * r - case["local"]))
        pairs += rows * past * b + rows * (rows + 1) // 2
        entries += past + -(-rows // b)
    return pairs, entries


def work(case):
    n, s, b, r, n1, n2 = _sizes(case)
    bt, hq, hkv, op = case["batch"], case["hq"], case["hkv"], case["op"]
    e = 2 if case["dtype"] == "bf16" else 4
    q, k = bt * hq * n * D * e, bt * hkv * n * D * e
    scores = bt * hq * n1 * n2 * 4
    lists = bt * (hkv if op == "shared" else hq) * n1 * (case["budget"] + case["local"] + r + 1) * 4
    estimate = bt * hq * n1 * n2 * 8 * D
    attention = bt * hq * _pairs(case)[0] * 4 * D
    prev = scores if case["fused"] else 0
    lse = bt * hq * n * 4 if case["lse"] else 0
    return {"layer": {"bytes": 2 * q + 2 * k + prev + scores + lists + lse, "flops": estimate + attention},
            "estimate": {"bytes": q + k + prev + scores, "flops": estimate},
            "select": {"bytes": scores + lists, "flops": 0},
            "sparse": {"bytes": 2 * q + 2 * k + lists + lse, "flops": attention},
            "shared": {"bytes": 2 * q + 2 * k + scores + lists + lse, "flops": attention},
            "dense": {"bytes": 2 * q + 2 * k + lse, "flops": attention}}[op]


# ---- inputs -------------------------------------------------------------------------------------------------------
def _walk(gen, batch, heads, n):
    x = torch.randn((batch, heads, n, D), generator=gen, device=DEV)
    x = x.mul_(0.1).cumsum(2)
    return x.add_(torch.randn((batch, heads, n, D), generator=gen, device=DEV))


def _inputs(case, seed):
    """q, k, v in the storage type and layout of the case, and the scores of the layer before."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n, _, _, _, n1, n2 = _sizes(case)
    out = []
    for name, heads in (("q", case["hq"]), ("k", case["hkv"]), ("v", case["hkv"])):
        x = _walk(gen, case["batch"], heads, n)
        if case["dtype"] == "bf16":
            x.div_(x.std())
        if name == "k" and case["hot"]:
            u = torch.randn((case["batch"], heads, 1, D), generator=gen, device=DEV)
            u *= 3 * D ** 0.5 / u.norm(dim=3, keepdim=True)
            x += u * (torch.rand((case["batch"], heads, n, 1), generator=gen, device=DEV) < case["hot"])
        x = x.to(torch.bfloat16) if case["dtype"] == "bf16" else x
        out.append(x.transpose(1, 2).contiguous().transpose(1, 2) if case["token_major"] else x)
    prev = None
    if case["fused"] and case["op"] in ("layer", "estimate"):
        # a softmax over blocks is what the layer before leaves, most of it far below its largest entries
        prev = torch.randn((case["batch"], case["hq"], n1, n2), generator=gen, device=DEV).mul_(2).softmax(3)
    return (*out, prev)


ALPHA = 0.5


def _scores64(case, q, k, prev):
    """Algorithm 1 in float64."""
    n, s, b, r, n1, n2 = _sizes(case)
    G = case["hq"] // case["hkv"]

    def reps(x, size, groups):
        x = torch.cat([x, x[-1:].expand(groups * size - n, D)]).view(groups, size, D)     # a repeated row changes no max or min
        return x.amax(1).double(), x.amin(1).double()

    future = torch.arange(n2, device=DEV)[None] >= (torch.arange(n1, device=DEV)[:, None] + 1) * r
    out = torch.empty((case["batch"], case["hq"], n1, n2), dtype=torch.float64, device=DEV)
    for i in range(case["batch"]):
        for h in range(case["hq"]):
            qs, ks = reps(q[i, h], s, n1), reps(k[i, h // G], b, n2)
            half = []
            for kr in ks:
                kt = kr.t().contiguous()
                z = [(qr @ kt) * D ** -0.5 for qr in qs]
                if case["domain"] == 1:
                    z = [x.masked_fill(future, float("-inf")) for x in z]
                half.append((z[0].softmax(1) + z[1].softmax(1)) / 2)
            x = torch.maximum(*half).masked_fill(future, 0.0)
            out[i, h] = x if prev is None else ALPHA * x + (1 - ALPHA) * prev[i, h].double()
    return out


def _lists(case, scores):
    """Ascending lists from scores [batch, heads, n1, n2], ties to the smaller block."""
    n, s, b, r, n1, n2 = _sizes(case)
    length = case["budget"] + case["local"] + r
    lists = torch.full((*scores.shape[:3], length), -1, dtype=torch.int32, device=DEV)
    counts = torch.zeros(scores.shape[:3], dtype=torch.int32, device=DEV)
    for j in range(n1):
        first = j * r - min(case["local"], j * r)
        take = min(case["budget"], first)
        if take:
            lists[:, :, j, :take] = scores[:, :, j, :first].sort(dim=2, descending=True, stable=True).indices[..., :take].sort(dim=2).values.int()
        fixed = min(n2, (j + 1) * r) - first
        lists[:, :, j, take:take + fixed] = torch.arange(first, first + fixed, device=DEV).int()
        counts[:, :, j] = take + fixed
    return lists, counts


def _decision(scores):
    """Scores as the library hands them over: fp32, nothing below the smallest normal number."""
    x = scores.float()
    return x.masked_fill_(x.abs() < torch.finfo(torch.float32).tiny, 0.0)


def _given(case, seed):
    """The inputs and, where the operation starts from them, the scores or the lists."""
    q, k, v, prev = _inputs(case, seed)
    scores = lists = None
    if case["op"] in ("select", "sparse", "shared"):
        scores = _decision(_scores64(case, q, k, None))
    if case["op"] == "sparse":
        lists = _lists(case, scores)
    return q, k, v, prev, scores, lists


def prepare(case, seed):
    q, k, v, prev, scores, lists = _given(case, seed)
    out = torch.empty_like(q)                                   # keeps the layout
    p = B.make_params(q, k, case["segment"], case["block"], case["budget"], case["local"], out=out, alpha=ALPHA, softmax_domain=case["domain"])
    st = {"op": case["op"], "p": p, "q": q, "k": k, "v": v, "out": out, "lse": None, "prev": prev, "scores": scores}
    if case["lse"]:
        st["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device=DEV)
    if case["op"] in ("layer", "estimate"):
        st["scores"], st["workspace"] = B.alloc_scores(p), B.alloc_workspace(p)
    if case["op"] in ("layer", "select"):
        st["idx"], st["cnt"] = B.alloc_lists(p)
    if case["op"] == "shared":
        st["idx"], st["cnt"] = B.alloc_shared_lists(p)
    if case["op"] == "sparse":
        st["idx"], st["cnt"] = lists
    torch.cuda.synchronize()
    return st


# ---- one pass -----------------------------------------------------------------------------------------------------
def run(st):
    op, p, q, k, v, out, lse = st["op"], st["p"], st["q"], st["k"], st["v"], st["out"], st["lse"]
    if op == "dense":
        B.critiprefill_dense_causal_attn(p, q, k, v, out, lse)
        return [out] if lse is None else [out, lse]
    found = []
    if op in ("layer", "estimate"):
        B.critiprefill_estimate(p, q, k, st["prev"], st["scores"], st["workspace"])
        found += [st["scores"]]
    if op in ("layer", "select"):
        B.critiprefill_select(p, st["scores"], st["idx"], st["cnt"])
        found += [st["idx"], st["cnt"]]
    if op in ("layer", "sparse"):
        B.critiprefill_sparse_attn(p, q, k, v, st["idx"], st["cnt"], out, lse)
    if op == "shared":
        B.critiprefill_select_shared(p, st["scores"], st["idx"], st["cnt"])
        B.critiprefill_sparse_attn_shared(p, q, k, v, st["idx"], st["cnt"], out, lse)
        found += [st["idx"], st["cnt"]]
    if op in ("layer", "sparse", "shared"):
        found += [out] if lse is None else [out, lse]
    return found


# ---- what is right ------------------------------------------------------------------------------------------------
def tolerance(case):
    op, fp32 = case["op"], case["dtype"] == "fp32"
    if op == "select":
        return "exact"                                          # whole numbers from the same scores
    if op == "estimate" and not fp32:
        return {"rel": 2e-6, "max": 5e-5}                       # exact products, fp32 sums, then an exponential: 1e-7 to 5e-7 seen
    if op in ("estimate", "layer") and fp32:
        # as drawn, the walk grows with the length and the logits z of the representatives with its square, so the error
        # z 2^-24 of an exponent grows in proportion: 8e-6 seen at 2048 tokens
        rel = 3e-5 * max(1.0, case["tokens"] / 2048)
        return {"rel": rel, "max": 40 * rel, "differ": 0.0}
    if fp32:
        return {"rel": 5e-6, "max": 2e-4}                       # 6e-7 to 1.2e-6 seen
    if op == "layer":
        # the lists follow from scores with fp32 rounding: a block or two near the threshold of a few rows may change
        return {"rel": 8e-3, "max": 0.9, "differ": 2e-3}
    return {"rel": 8e-3, "max": 8e-2}                           # P and O rounded to bf16: 1.7e-3 seen against 64 bits


def _attention64(q, k, v, tokens, visible):
    """softmax(q k^T / sqrt(d)) v over the gathered tokens [..., u]; visible [..., rows, u].  Returns O and the log-sum-exp."""
    z = torch.matmul(q.double(), k[tokens].double().transpose(-1, -2).contiguous()).mul_(D ** -0.5)
    z.masked_fill_(~visible, float("-inf"))
    lse = torch.logsumexp(z, -1)
    return torch.matmul(z.sub_(lse.unsqueeze(-1)).exp_(), v[tokens].double()), lse


def exact(case, seed):
    if case["op"] == "select":
        return None
    q, k, v, prev, scores, lists = _given(case, seed)
    n, s, b, r, n1, n2 = _sizes(case)
    if case["op"] == "estimate":
        return [_scores64(case, q, k, prev)]
    if case["op"] == "layer":
        return [_scores64(case, q, k, prev), None, None, None] + ([None] if case["lse"] else [])
    G = case["hq"] // case["hkv"]
    if case["op"] == "shared":
        lists = _lists(case, scores.view(case["batch"], case["hkv"], G, n1, n2).amax(2))
    out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device=DEV)
    for i in range(case["batch"]):
        for h in range(case["hq"]):
            qh, kh, vh = q[i, h], k[i, h // G], v[i, h // G]
            if case["op"] == "dense":
                for t0 in range(0, n, 2048):
                    t1 = min(n, t0 + 2048)
                    u = torch.arange(t1, device=DEV)
                    out[i, h, t0:t1], lse[i, h, t0:t1] = _attention64(qh[t0:t1], kh, vh, u, u[None] <= u[t0:t1, None])
                continue
            idx = lists[0][i, h // G if case["op"] == "shared" else h].long()
            step = max(1, 1 << 27 >> (idx.shape[1] * b * s).bit_length() - 1)           # segments at a time, about 1 GB of weights
            for j0 in range(0, n1, step):
                rows = torch.arange(j0 * s, min(n1, j0 + step) * s, device=DEV).view(-1, s)
                blocks = idx[j0:j0 + step]
                u = (blocks[:, :, None] * b + torch.arange(b, device=DEV)).flatten(1)
                there = (blocks >= 0)[:, :, None].expand(-1, -1, b).flatten(1) & (u < n)
                visible = (u[:, None] <= rows[:, :, None]) & there[:, None]
                o, l = _attention64(qh[rows.clamp(max=n - 1)], kh, vh, u.clamp(0, n - 1), visible)
                keep = rows.flatten() < n
                out[i, h, rows.flatten()[keep]], lse[i, h, rows.flatten()[keep]] = o.flatten(0, 1)[keep], l.flatten()[keep]
    found = [out] + ([lse] if case["lse"] else [])
    return [None, None] + found if case["op"] == "shared" else found
