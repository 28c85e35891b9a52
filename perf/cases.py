"""The work a program has this framework do, as cases that can be timed and compared.

Decoding one token runs the retrieval and the attention once per layer, with one context
shared by the layers and K/V, centroids and codes of each layer's own: a pass of a decode
case walks `layers` layers, so that K/V rows come from HBM and not from the last-level
cache.  Prefill leaves the PQ structures behind (K-Means over all keys of a layer), a
growing cache appends a token's code in every step, and a block cache is refreshed with
what a step retrieved.

Case fields: kind (decode, append, indexed, build, blocks), geometry as in Workload,
`keys` (how the keys are distributed), `layers`, and for single kinds `capacity`,
`iters`, `block`, `slots`, `requests`, `policy`.
"""
import torch

from paper_2407_12820_amd import binding
from paper_2407_12820_amd.workloads import Workload

DEV = "cuda:0"
HEAD_DIM = 128


def _case(name, kind, batch, q_heads, kv_heads, tokens, m, centroids, den, dtype, keys, layers, **more):
    topk = more.pop("topk", tokens // den if den else 0)
    c = dict(kind=kind, batch=batch, q_heads=q_heads, kv_heads=kv_heads, tokens=tokens, m=m, centroids=centroids, topk=topk,
             n_init=4, n_local=64, dtype=dtype, keys=keys, layers=layers, **more)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # one small fp32 head, the smallest call: latency and launches
        _case("decode_tiny_f32", "decode", 1, 1, 1, 4096, 2, 64, 0, "f32", "planted", 1, topk=512),
        # single-sequence decode of an 8B-shaped model (32 query heads, 8 KV heads), a fifth of 32K tokens retrieved
        _case("decode_8b_32k", "decode", 1, 32, 8, 32768, 2, 64, 5, "bf16", "outliers", 8),
        # the same at 128K tokens, a tenth retrieved: long-context chat and document questions
        _case("decode_8b_128k", "decode", 1, 32, 8, 131072, 2, 64, 10, "bf16", "planted", 8),
        # batched serving of eight sequences with the finer PQ (4 partitions of 256 centroids)
        _case("decode_batch8_32k", "decode", 8, 32, 8, 32768, 4, 256, 5, "bf16", "plain", 2),
        # a 70B-shaped layer (64 query heads), four sequences of 128K tokens: the largest decode step
        _case("decode_70b_128k", "decode", 4, 64, 8, 131072, 4, 256, 10, "bf16", "outliers", 2),
        # fp32 caches and a prompt of odd length, a few sequences
        _case("decode_ragged_f32", "decode", 3, 8, 4, 20011, 4, 64, 10, "f32", "plain", 2),
        # a step of the generation loop: the length follows the cache inside larger buffers, the new token gets its code
        _case("append_8b_growing", "append", 1, 32, 8, 49999, 2, 64, 5, "bf16", "outliers", 8, capacity=65536),
        # single-sequence decode with the code-pair statistic kept beside the codes
        _case("indexed_8b_128k", "indexed", 1, 32, 8, 131072, 2, 64, 10, "bf16", "planted", 8),
        # end of prefill: PQ structures of one 8B-shaped layer of 128K tokens
        _case("build_8b_128k", "build", 1, 32, 8, 131072, 2, 64, 10, "bf16", "planted", 1, iters=8),
        # the same for a batch of eight prompts with the finer PQ
        _case("build_batch8_32k", "build", 8, 32, 8, 32768, 4, 256, 5, "bf16", "plain", 1, iters=4),
        # fp32 keys, an odd length, many rounds
        _case("build_ragged_f32", "build", 1, 8, 2, 10007, 2, 64, 5, "f32", "plain", 1, iters=25),
        # refresh of the block cache (32 blocks of 128 tokens) with the tokens a 128K step retrieved
        _case("blocks_8b_128k", "blocks", 1, 32, 8, 131072, 2, 64, 10, "bf16", "plain", 8, block=128, slots=32, requests=32, policy="lfu"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["decode"] * 5 + ["append", "indexed", "build", "build", "blocks"])
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        m, centroids = rng.choice([(2, 64)] * 4 + [(4, 256)] * 4 + [(2, 256), (4, 64), (2, 48)])
        if kind == "indexed":
            m, centroids = 2, rng.choice([64, 64, 48])
        kv_heads = rng.choice([1, 2, 4, 8, 8, 8])
        group = rng.choice([1, 2, 4, 4, 8])
        batch = rng.choice([1, 1, 1, 2, 3, 4, 8])
        tokens = _log_int(rng, 2048, 131072)
        if kind == "indexed":
            tokens -= tokens % 8  # the code-pair path asks for a multiple of eight
        keys = rng.choice(["plain", "outliers", "planted"])
        den = rng.choice([5, 10, 10, 20])
        c = _case("", kind, batch, group * kv_heads, kv_heads, tokens, m, centroids, den, dtype, keys,
                  1 if kind == "build" else rng.choice([1, 2, 4, 8]))
        if kind == "append":
            c["capacity"] = -(-(tokens + rng.randrange(1, 20000)) // 64) * 64
        if kind == "build":
            c["iters"] = rng.choice([2, 4, 8, 10, 25])
        if kind == "blocks":
            c["block"] = rng.choice([64, 128, 256])
            nb = -(-tokens // c["block"])
            c["slots"] = rng.choice([32, 32, 64])
            c["requests"] = min(c["slots"], nb)
            c["policy"] = rng.choice(["lru", "lfu"])
        if _cost(c) <= most and _held(c) <= 12e9:
            return c


# ------------------------------------------------------------------------- inputs
def _workload(c):
    return Workload(name="case", batch=c["batch"], n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"], head_dim=HEAD_DIM,
                    n_tokens=c["tokens"], pq_m=c["m"], pq_centroids=c["centroids"], topk=c["topk"], n_init=c["n_init"],
                    n_local=c["n_local"], dtype=c["dtype"], kmeans_iters=c.get("iters", 1), recipe="plain")


def _rows(c, shape, gen):
    kv = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    return torch.randn(shape, generator=gen, device=DEV, dtype=kv)


def _keys(c, q, room, gen):
    """Keys ~N(0,1) with the features real caches show: a few channels of large magnitude, or tokens that the query attends to."""
    B, H, N = c["batch"], c["kv_heads"], c["tokens"]
    k = _rows(c, (B, H, room, HEAD_DIM), gen)
    if c["keys"] == "outliers":
        ch = torch.rand((B, H, HEAD_DIM), generator=gen, device=DEV).argsort(-1)[..., :4]
        gain = torch.ones((B, H, HEAD_DIM), device=DEV).scatter_(-1, ch, 8.0)
        k.mul_(gain.to(k.dtype).unsqueeze(2))
    elif c["keys"] == "planted":
        mean_q = q.float().view(B, H, -1, HEAD_DIM).mean(2)
        hot = torch.rand((B, H, N, 1), generator=gen, device=DEV) < 0.01
        k[:, :, :N].add_((hot * (2.0 * mean_q).unsqueeze(2)).to(k.dtype))
    return k


def _pq(c, k, gen):
    """Centroids and codes as K-Means leaves them: sampled start, two rounds over a subset of the tokens, every token assigned."""
    B, H, N, M, C = c["batch"], c["kv_heads"], c["tokens"], c["m"], c["centroids"]
    Dm = HEAD_DIM // M
    U = B * H
    pick = torch.rand((N,), generator=gen, device=DEV).argsort()[: min(N, 4096)]
    keys = k.view(U, k.shape[2], HEAD_DIM)

    def split(rows):  # [U', n, D] -> [U' * M, n, Dm]
        return rows.float().view(rows.shape[0], rows.shape[1], M, Dm).transpose(1, 2).reshape(-1, rows.shape[1], Dm).contiguous()

    def nearest(x, cent):
        return (cent.square().sum(-1).unsqueeze(1) - 2.0 * torch.bmm(x, cent.transpose(1, 2).contiguous())).argmin(-1)

    sub = split(keys[:, pick])
    cent = sub[:, :C].contiguous()
    for _ in range(2):
        hit = torch.nn.functional.one_hot(nearest(sub, cent), C).float()
        n = hit.sum(1).unsqueeze(-1)
        cent = torch.where(n > 0, torch.bmm(hit.transpose(1, 2).contiguous(), sub) / n.clamp(min=1.0), cent)
    codes = torch.zeros((U, k.shape[2], M), dtype=torch.uint8, device=DEV)
    step = max(1, (1 << 28) // (M * C * min(N, 32768)))
    for t0 in range(0, N, 32768):
        for u0 in range(0, U, step):
            x = split(keys[u0:u0 + step, t0:min(N, t0 + 32768)])
            a = nearest(x, cent.view(U, M, C, Dm)[u0:u0 + step].reshape(-1, C, Dm))
            codes[u0:u0 + step, t0:t0 + x.shape[1]] = a.view(-1, M, x.shape[1]).transpose(1, 2).to(torch.uint8)
    return cent.view(B, H, M, C, Dm).contiguous(), codes.view(B, H, -1, M)


def prepare(case, seed):
    c = case
    w = _workload(c)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    B, H, N = c["batch"], c["kv_heads"], c["tokens"]
    state = {"case": c, "w": w, "layers": []}
    if c["kind"] == "build":
        q = _rows(c, (B, c["q_heads"], HEAD_DIM), gen)
        init = torch.stack([torch.rand((N,), generator=gen, device=DEV).argsort()[: c["centroids"]] for _ in range(B * H * c["m"])])
        state["keys"] = _keys(c, q, N, gen)
        state["init"] = init.to(torch.int32).view(B, H, c["m"], c["centroids"]).contiguous()
        return state
    if c["kind"] == "blocks":
        for _ in range(c["layers"]):
            # retrieved tokens cluster: some stretches of the text matter to the query, most do not
            heat = torch.rand((B, H, -(-N // 96)), generator=gen, device=DEV).pow(4).repeat_interleave(96, -1)[..., :N]
            score = torch.rand((B, H, N), generator=gen, device=DEV) + heat
            score[..., : c["n_init"]] = 9.0
            score[..., N - c["n_local"]:] = 9.0
            idx = score.topk(w.n_selected, dim=-1).indices.sort(-1).values.to(torch.int32).contiguous()
            slots = [torch.full((B, H, c["slots"]), -1, dtype=torch.int32, device=DEV)]
            slots += [torch.zeros((B, H, c["slots"]), dtype=torch.int32, device=DEV) for _ in range(2)]
            state["layers"].append((idx, slots))
        state["step"] = 0
        return state
    room = c.get("capacity", 0) or N
    ctx = binding.PQCache(w, DEV, capacity=c.get("capacity", 0))
    state["ctx"] = ctx
    for _ in range(c["layers"]):
        q = _rows(c, (B, c["q_heads"], HEAD_DIM), gen)
        k = _keys(c, q, room, gen)
        v = _rows(c, (B, H, room, HEAD_DIM), gen)
        cent, codes = _pq(c, k, gen)
        idx, attn = ctx.empty_outputs()
        layer = dict(q=q, cent=cent, codes=codes, k=k, v=v, idx=idx, attn=attn)
        if c["kind"] == "append":
            layer["new_key"] = k[:, :, N - 1].contiguous()
        if c["kind"] == "indexed":
            pair = codes[..., 0].long() + c["centroids"] * codes[..., 1].long()
            pair += torch.arange(B * H, device=DEV).view(B, H, 1) * c["centroids"] ** 2
            counts = torch.bincount(pair.flatten(), minlength=B * H * c["centroids"] ** 2)
            layer["pairs"] = counts.to(torch.int32).view(B, H, -1).contiguous()
        state["layers"].append(layer)
    return state


def run(state):
    c, w = state["case"], state["w"]
    if c["kind"] == "build":
        cent, codes = binding.pq_build(w, state["keys"], state["init"])
        return {"centroids": cent, "codes": codes}
    out = []
    if c["kind"] == "blocks":
        state["step"] += 1
        for idx, slots in state["layers"]:
            counts, blocks = binding.block_stats(w, idx, c["block"], c["requests"])
            stats = binding.block_cache_update(w, c["block"], c["policy"], state["step"], counts, blocks, *slots)
            out.append([counts, blocks, stats, *slots])
        return out
    ctx = state["ctx"]
    if c["kind"] == "append":
        ctx.set_length(c["tokens"], c["topk"])
    for y in state["layers"]:
        if c["kind"] == "append":
            ctx.decode_append(y["q"], y["cent"], y["codes"], y["k"], y["v"], y["new_key"], c["tokens"] - 1, y["idx"], y["attn"])
            out.append([y["idx"], y["attn"], y["codes"]])
        elif c["kind"] == "indexed":
            ctx.decode_indexed(y["q"], y["cent"], y["codes"], y["pairs"], y["k"], y["v"], y["idx"], y["attn"])
            out.append([y["idx"], y["attn"]])
        else:
            ctx.decode(y["q"], y["cent"], y["codes"], y["k"], y["v"], y["idx"], y["attn"])
            out.append([y["idx"], y["attn"]])
    return out


def work(case):
    c = case
    units = c["batch"] * c["kv_heads"]
    e = 4 if c["dtype"] == "f32" else 2
    n, k, mc = c["tokens"], c["n_init"] + c["topk"] + c["n_local"], c["m"] * c["centroids"]
    cent = units * c["centroids"] * HEAD_DIM * 4
    if c["kind"] == "build":
        # every round looks at every key once (nearest centroid and the sums of the new ones), and once more at the end
        rounds = c["iters"] + 1
        return {"bytes": rounds * units * n * HEAD_DIM * e + units * n * c["m"] + cent,
                "flops": rounds * units * n * c["centroids"] * HEAD_DIM * 2.0}
    if c["kind"] == "blocks":
        nb = -(-n // c["block"])
        return {"bytes": c["layers"] * units * 4 * (k + nb + c["requests"] + 6 * c["slots"]), "flops": 0.0}
    codes = units * n * c["m"] if c["kind"] != "indexed" else units * (n * c["m"] + 4 * c["centroids"] ** 2)
    rows = units * k * HEAD_DIM * 2 * e
    io = c["batch"] * c["q_heads"] * HEAD_DIM * (e + 4) + units * k * 4
    flops = units * (mc * (HEAD_DIM // c["m"]) * 2.0 + n * c["m"]) + c["batch"] * c["q_heads"] * k * HEAD_DIM * 4.0
    return {"bytes": c["layers"] * (codes + rows + io + cent), "flops": c["layers"] * flops}


def _cost(c):
    w = work(c)
    return max(w["bytes"] / 5e12, w["flops"] / 3e14)


def _held(c):
    e = 4 if c["dtype"] == "f32" else 2
    room = c.get("capacity", 0) or c["tokens"]
    return c["batch"] * c["kv_heads"] * room * HEAD_DIM * e * (1 if c["kind"] == "build" else 2 * c["layers"])


def tolerance(case):
    if case["kind"] == "blocks":
        return "exact"
    if case["kind"] == "build":
        # distances are compared in fp32: a token within rounding of two centroids may go to either, and a token that
        # moved shifts two centroids for the next round
        return {"rel": 1e-2, "differ": 1e-2}
    # fp32 accumulation over a few thousand softmax terms; the selected tokens and their order are whole numbers
    return {"rel": 1e-5, "differ": 0.0}
