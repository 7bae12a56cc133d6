"""Workloads on which the speed of this framework is judged: calls of the public entry points as a
serving engine or a training step makes them, over the range of sizes that they are made with.

Nine kinds of call, told apart by the "path" of a case:

    decode      one step over a bf16 key/value cache: contiguous or paged, fixed or ragged lengths,
                one or several query rows, with or without a sliding window
    decode_f32  the same step over an fp32 cache
    mla         one step (or a few rows) over a latent cache shared by all heads
    prompt      RMSNorm + RoPE on q, rho and k, then causal attention: a layer's prefill
    chunk       causal attention of a prompt's next rows over the cache of the rows before them
    train       bf16 forward with the row cache, then the backward pass
    sparse      the same training step under a block mask
    train_f32   the fp32 training step
    prefill_f32 the fp32 forward alone

The 16-query / 8-key-head, d = 128 layer and its compute-matched 32 / 16, d = 64 form are the
layers of the benchmark configurations. Values are N(0, 1): what RMSNorm with unit weights hands
over.
"""
import math

import torch

from paper_2605_29157_amd import binding as plx

D_LATENT, D_ROPE = 512, 64
THETA, EPS = 1.0e6, 1.0e-6


def listed():
    return [
        # the next token of one interactive conversation: launches and latency
        dict(name="decode_single", path="decode", B=1, Hq=16, Hkv=8, d=128, L=2048, page=0, ragged=False, Tq=1,
             window=0),
        # a step of a serving batch: paged cache, every sequence of another length
        dict(name="decode_paged", path="decode", B=24, Hq=16, Hkv=8, d=128, L=6000, page=16, ragged=True, Tq=1,
             window=0),
        # a step over long contexts: the cache is read at the speed of the memory
        dict(name="decode_long", path="decode", B=16, Hq=16, Hkv=8, d=128, L=32768, page=0, ragged=False, Tq=1,
             window=0),
        # a step of a small model kept in fp32
        dict(name="decode_f32", path="decode_f32", B=4, Hq=16, Hkv=8, d=64, L=2048, ragged=True),
        # a latent cache with the heads of one rank of an 8-way head-parallel layer
        dict(name="mla_16_heads", path="mla", B=32, Hq=16, L=8192, ragged=True, Tq=1),
        # a latent cache with all heads on one GPU
        dict(name="mla_128_heads", path="mla", B=8, Hq=128, L=4096, ragged=True, Tq=1),
        # a short prompt of odd length: few workgroups
        dict(name="prompt_short", path="prompt", B=1, Hq=16, Hkv=8, d=128, T=777),
        # the next 512 rows of a long document: few rows, many keys
        dict(name="chunk_512_of_16k", path="chunk", B=1, Hq=16, Hkv=8, d=128, T=512, Tkv=16384),
        # the attention of a training step at the paper's context length
        dict(name="train_d128", path="train", B=4, Hq=16, Hkv=8, d=128, T=4096, window=0),
        # the same for the d = 64 layer, shorter and of odd length
        dict(name="train_d64", path="train", B=3, Hq=32, Hkv=16, d=64, T=1111, window=0),
        # a block-sparse training step: a quarter of the cells and the diagonal
        dict(name="sparse_2048", path="sparse", B=2, Hq=16, Hkv=8, d=128, T=2048, density=0.25),
        # a synthetic-task training step in fp32
        dict(name="train_f32", path="train_f32", B=8, Hq=8, Hkv=8, d=64, T=512),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["decode", "decode", "decode_f32", "mla", "prompt", "chunk", "train", "train", "sparse",
                       "train_f32", "prefill_f32"])
    Hq, Hkv, d = rng.choice([(16, 8, 128), (32, 16, 64), (16, 4, 128), (8, 8, 64)])
    if path == "decode":
        B = _log_uniform(rng, 1, 64)
        L = _log_uniform(rng, 200, min(32768, 524288 // B))
        Tq = rng.choice([1, 1, 1, 2, 4])
        window = rng.choice([0, 0, 0, _log_uniform(rng, 64, 4096)])
        return dict(path=path, B=B, Hq=Hq, Hkv=Hkv, d=d, L=L, page=rng.choice([0, 0, 16, 48, 64]),
                    ragged=rng.random() < 0.5, Tq=Tq, window=window)
    if path == "decode_f32":
        B = _log_uniform(rng, 1, 16)
        return dict(path=path, B=B, Hq=Hq, Hkv=Hkv, d=d, L=_log_uniform(rng, 100, 8192 // B * 2),
                    ragged=rng.random() < 0.5)
    if path == "mla":
        B, heads = _log_uniform(rng, 1, 32), rng.choice([8, 16, 32, 128])
        L = _log_uniform(rng, 200, min(16384, 262144 // B, 8 * 128 * 4096 // (B * heads) * 4))
        return dict(path=path, B=B, Hq=heads, L=L, ragged=rng.random() < 0.5, Tq=rng.choice([1, 1, 2]))
    if path == "prompt":
        B = _log_uniform(rng, 1, 4)
        return dict(path=path, B=B, Hq=Hq, Hkv=Hkv, d=d, T=_log_uniform(rng, 100, 4096))
    if path == "chunk":
        T = _log_uniform(rng, 17, 1024)
        return dict(path=path, B=_log_uniform(rng, 1, 4), Hq=Hq, Hkv=Hkv, d=d, T=T,
                    Tkv=T + _log_uniform(rng, 100, 16384))
    if path == "train":
        return dict(path=path, B=_log_uniform(rng, 1, 4), Hq=Hq, Hkv=Hkv, d=d, T=_log_uniform(rng, 100, 3000),
                    window=rng.choice([0, 0, _log_uniform(rng, 64, 1024)]))
    if path == "sparse":
        return dict(path=path, B=_log_uniform(rng, 1, 3), Hq=Hq, Hkv=Hkv, d=d, T=_log_uniform(rng, 300, 2500),
                    density=rng.choice([0.15, 0.25, 0.5]))
    return dict(path=path, B=_log_uniform(rng, 1, 4), Hq=8, Hkv=rng.choice([4, 8]), d=rng.choice([64, 128]),
                T=_log_uniform(rng, 50, 512))


def _f32(case):
    return case["path"] in ("decode_f32", "train_f32", "prefill_f32")


def _lengths(case, gen):
    """Cached tokens per sequence, uniform in [L/2, L] when ragged (host list)."""
    B, L = case["B"], case["L"]
    if not case["ragged"]:
        return [L] * B
    return torch.randint(max(1, L // 2), L + 1, (B,), generator=gen).tolist()


def _inputs(case, seed):
    dev, path = torch.device("cuda"), case["path"]
    gen = torch.Generator(device=dev).manual_seed(seed)
    host = torch.Generator().manual_seed(seed + 1)
    dtype = torch.float32 if _f32(case) else torch.bfloat16

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=dtype)

    B, Hq = case["B"], case["Hq"]
    s = dict(case=case)
    if path == "mla":
        rows = (case["Tq"],) if case["Tq"] > 1 else ()
        s["q"], s["r"] = normal(B, Hq, *rows, D_LATENT + D_ROPE), normal(B, Hq, *rows, D_LATENT + D_ROPE)
        s["ckv"] = normal(B, case["L"], D_LATENT + D_ROPE)
        s["scale"] = (D_LATENT + D_ROPE) ** -0.5
        s["lens"] = _lengths(case, host)
        s["seq_lens"] = torch.tensor(s["lens"], dtype=torch.int32, device=dev) if case["ragged"] else None
        return s
    Hkv, d = case["Hkv"], case["d"]
    s["scale"] = d ** -0.5
    if path in ("decode", "decode_f32"):
        L, page, rows = case["L"], case.get("page", 0), case.get("Tq", 1)
        shape = (B, Hq, rows, d) if rows > 1 else (B, Hq, d)
        s["q"], s["r"] = normal(*shape), normal(*shape)
        s["lens"] = _lengths(case, host)
        s["seq_lens"] = torch.tensor(s["lens"], dtype=torch.int32, device=dev) if case["ragged"] else None
        if page:
            per_seq = -(-L // page)
            s["k"], s["v"] = normal(B * per_seq, Hkv, page, d), normal(B * per_seq, Hkv, page, d)
            order = torch.randperm(B * per_seq, generator=host)
            s["table"] = order.reshape(B, per_seq).to(torch.int32).to(dev)
        else:
            s["k"], s["v"] = normal(B, Hkv, L, d), normal(B, Hkv, L, d)
        return s
    T, Tkv = case["T"], case.get("Tkv", case["T"])
    s["q"], s["r"] = normal(B, Hq, T, d), normal(B, Hq, T, d)
    s["k"], s["v"] = normal(B, Hkv, Tkv, d), normal(B, Hkv, Tkv, d)
    if path == "prompt":
        s["gamma"] = [1.0 + 0.1 * torch.randn(d, generator=gen, device=dev) for _ in range(3)]
    if path in ("train", "sparse", "train_f32"):
        s["d_o"] = normal(B, Hq, T, d)
    if path == "sparse":
        cells = torch.rand(-(-T // plx.BLOCK_ROWS), -(-T // plx.BLOCK_KEYS), generator=host) < case["density"]
        row = torch.arange(cells.shape[0])[:, None]
        tile = torch.arange(cells.shape[1])[None, :]
        first, last = row * plx.BLOCK_ROWS, row * plx.BLOCK_ROWS + plx.BLOCK_ROWS - 1
        diagonal = (tile * plx.BLOCK_KEYS <= last) & (tile * plx.BLOCK_KEYS + plx.BLOCK_KEYS > first)
        causal = tile * plx.BLOCK_KEYS <= last
        s["mask"] = ((cells & causal) | diagonal).to(dev)
    return s


def prepare(case, seed):
    return _inputs(case, seed)


def run(s):
    case, path, scale = s["case"], s["case"]["path"], s["scale"]
    if path in ("decode", "decode_f32"):
        paged = dict(block_table=s["table"], max_len=case["L"]) if case.get("page") else {}
        return plx.parallax_decode(s["q"], s["r"], s["k"], s["v"], scale, seq_lens=s["seq_lens"],
                                   window=case.get("window", 0), **paged)
    if path == "mla":
        return plx.parallax_decode_mla(s["q"], s["r"], s["ckv"], scale, seq_lens=s["seq_lens"])
    if path == "prompt":
        gq, gr, gk = s["gamma"]
        q, r, k = plx.parallax_norm_rope([(s["q"], gq, True), (s["r"], gr, True), (s["k"], gk, True)], eps=EPS,
                                         theta=THETA)
        return [plx.parallax_prefill(q, r, k, s["v"], scale, causal=True), k]
    if path in ("chunk", "prefill_f32"):
        return plx.parallax_prefill(s["q"], s["r"], s["k"], s["v"], scale, causal=True)
    opts = dict(window=case["window"]) if case.get("window") else {}
    if path == "sparse":
        opts["block_mask"] = s["mask"]
    o, vbar, stats = plx.parallax_prefill(s["q"], s["r"], s["k"], s["v"], scale, causal=True, save_for_backward=True,
                                          **opts)
    grads = plx.parallax_prefill_backward(s["q"], s["r"], s["k"], s["v"], o, vbar, stats, s["d_o"], scale,
                                          causal=True, **opts)
    return [o, *grads]


def _pairs(case):
    """(query row, key) pairs that count, per head and over the batch."""
    path, B = case["path"], case["B"]
    if path in ("decode", "decode_f32", "mla"):
        per = 0.75 * case["L"] if case["ragged"] else case["L"]
        if case.get("window"):
            per = min(per, case["window"])
        return B * case.get("Tq", 1) * per
    T, Tkv = case["T"], case.get("Tkv", case["T"])
    n = T * (Tkv - T) + T * (T + 1) / 2
    if case.get("window") and case["window"] < T:
        W = case["window"]
        n = W * (W + 1) / 2 + (T - W) * W
    if path == "sparse":
        n_rb = -(-T // plx.BLOCK_ROWS)
        diagonal = min(n, n_rb * plx.BLOCK_ROWS * (plx.BLOCK_ROWS + 1) / 2)
        n = diagonal + case["density"] * (n - diagonal)
    return B * n


def work(case):
    path, B, Hq = case["path"], case["B"], case["Hq"]
    pairs = _pairs(case)
    if path == "mla":
        dk = D_LATENT + D_ROPE
        tokens = B * (0.75 * case["L"] if case["ragged"] else case["L"])
        rows = B * Hq * case["Tq"]
        return dict(bytes=2 * (tokens * dk + rows * (2 * dk + D_LATENT)), flops=4 * Hq * pairs * (dk + D_LATENT))
    Hkv, d, size = case["Hkv"], case["d"], 4 if _f32(case) else 2
    if path in ("decode", "decode_f32"):
        tokens = pairs / case.get("Tq", 1)
        rows = B * Hq * case.get("Tq", 1)
        return dict(bytes=size * d * (2 * Hkv * tokens + 3 * rows), flops=8 * d * Hq * pairs)
    rows, keys = B * Hq * case["T"], B * Hkv * case.get("Tkv", case["T"])
    if path in ("prompt", "chunk", "prefill_f32"):
        extra = keys if path == "prompt" else 0  # the prepared keys go to the cache
        return dict(bytes=size * d * (3 * rows + 2 * keys + extra), flops=8 * d * Hq * pairs)
    return dict(bytes=size * d * (6 * rows + 4 * keys), flops=30 * d * Hq * pairs)


def tolerance(case):
    if _f32(case):
        return {"rel": 5e-6}  # 4e-7 to 9e-7 against 64 bits
    return {"rel": 1e-2}  # 2.4e-3 (attention) to 4e-3 (behind rounded q, rho and k) against 64 bits


def _visible(rows, keys, window=0):
    """Rows are the last positions: row i sees keys .. i + (keys - rows), the last `window` of them."""
    i = torch.arange(rows, device="cuda")[:, None] + (keys - rows)
    j = torch.arange(keys, device="cuda")[None, :]
    see = j <= i
    return see & (j > i - window) if window else see


def _attend(q, r, k, v, scale, see, d_o=None):
    """One head in 64 bits: o, and the gradients dq, dr, dk, dv for an upstream d_o."""
    q, r, k, v = (x.double() for x in (q, r, k, v))
    kt = k.t().contiguous()
    p = (scale * (q @ kt)).masked_fill(~see, -math.inf).softmax(dim=1)
    u = r @ kt
    c = 1 + (p * u).sum(dim=1, keepdim=True) - u
    w = p * c
    o = w @ v
    if d_o is None:
        return o
    g = d_o.double()
    a = g @ v.t().contiguous()
    mean_a = (p * a).sum(dim=1, keepdim=True)
    d_u = -p * (a - mean_a)
    d_p = a * c + mean_a * u
    d_s = scale * p * (d_p - (p * d_p).sum(dim=1, keepdim=True))
    d_st, d_ut = d_s.t().contiguous(), d_u.t().contiguous()
    return o, d_s @ k, d_u @ k, d_st @ q + d_ut @ r, w.t().contiguous() @ g


def _norm_rope(x, gamma):
    """RMSNorm over the last dimension, then adjacent pairs rotated by pos * theta^(-2i/d), in 64 bits."""
    x = x.double()
    T, d = x.shape[-2:]
    y = x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + EPS) * gamma.double()
    angle = torch.arange(T, device=x.device, dtype=torch.float64)[:, None] * THETA ** (
        -torch.arange(0, d, 2, device=x.device, dtype=torch.float64) / d)
    c, s = torch.cos(angle), torch.sin(angle)
    even, odd = y[..., 0::2], y[..., 1::2]
    return torch.stack([even * c - odd * s, even * s + odd * c], dim=-1).flatten(-2)


def exact(case, seed):
    s, path = _inputs(case, seed), case["path"]
    B, Hq, scale = case["B"], case["Hq"], s["scale"]
    q, r = s["q"], s["r"]
    if path == "mla":
        rows = case["Tq"]
        out = torch.empty(*q.shape[:-1], D_LATENT, dtype=torch.float64, device=q.device)
        for b in range(B):
            c, n = s["ckv"][b, : s["lens"][b]], s["lens"][b]
            see = _visible(rows, n).repeat(Hq, 1)
            o = _attend(q[b].reshape(Hq * rows, -1), r[b].reshape(Hq * rows, -1), c, c[:, :D_LATENT], scale, see)
            out[b] = o.reshape(out[b].shape)
        return out
    Hkv = case["Hkv"]
    G = Hq // Hkv
    if path in ("decode", "decode_f32"):
        rows, d = case.get("Tq", 1), case["d"]
        out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
        for b in range(B):
            n = s["lens"][b]
            see = _visible(rows, n, case.get("window", 0)).repeat(G, 1)
            if case.get("page"):
                pages = s["table"][b].long()
                k, v = (s[x][pages].transpose(0, 1).reshape(Hkv, -1, d)[:, :n] for x in ("k", "v"))
            else:
                k, v = s["k"][b, :, :n], s["v"][b, :, :n]
            for h in range(Hkv):
                group = slice(h * G, h * G + G)
                o = _attend(q[b, group].reshape(G * rows, d), r[b, group].reshape(G * rows, d), k[h], v[h], scale, see)
                out[b, group] = o.reshape(out[b, group].shape)
        return out
    k, v = s["k"], s["v"]
    if path == "prompt":
        q, r, k = (_norm_rope(x, g) for x, g in zip((q, r, k), s["gamma"]))
    see = _visible(q.shape[2], k.shape[2], case.get("window", 0))
    if path == "sparse":
        cells = s["mask"].repeat_interleave(plx.BLOCK_ROWS, 0).repeat_interleave(plx.BLOCK_KEYS, 1)
        see = see & cells[: see.shape[0], : see.shape[1]]
    o = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    if "d_o" not in s:
        for b in range(B):
            for h in range(Hq):
                o[b, h] = _attend(q[b, h], r[b, h], k[b, h // G], v[b, h // G], scale, see)
        return [o, k] if path == "prompt" else o
    dq, dr = torch.empty_like(o), torch.empty_like(o)
    dk, dv = (torch.zeros(k.shape, dtype=torch.float64, device=k.device) for _ in range(2))
    for b in range(B):
        for h in range(Hq):
            o[b, h], dq[b, h], dr[b, h], gk, gv = _attend(q[b, h], r[b, h], k[b, h // G], v[b, h // G], scale, see,
                                                          s["d_o"][b, h])
            dk[b, h // G] += gk
            dv[b, h // G] += gv
    return [o, dq, dr, dk, dv]
