"""The work this library is used for, as cases that can be timed and compared.

Every case is one dependent chain enqueued through the public entry points (dep_gemm_chain,
dep_conv_chain, dep_conv_chain_n) with the arguments a program leaves at their defaults left there:
the library chooses the macro-tile.  Shapes are the layer shapes of the repository's own workloads
(one 8-way tensor-parallel shard of a GPT-3 / LLaMA block, VGG-19 convolutions) and ragged sizes of
the same kind.
"""
import math

import torch

import paper_2305_13450_amd as ds

KINDS = {"row": ds.ROWSYNC, "tile": ds.TILESYNC, "strided": ds.STRIDEDSYNC, "auto": ds.AUTOSYNC}
# one dispatch for the whole chain, or the two-stream form (the default of the entry points)
MODES = {"fused": ds.MODE_FUSED, "fine": ds.MODE_FINE}
MIDS = {"gelu": ds.MID_GELU, "relu": ds.MID_RELU, "swiglu": ds.MID_SWIGLU}
DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16}

# The largest chain listed, in flops and bytes that count (drawn cases stay below what it costs).
MAX_FLOPS = {"mlp": 6.0e11, "attn": 3.0e11, "conv": 1.2e11}


def _mlp(name, M, K1, N1, N2, mid="gelu", dtype="bf16", policy="auto", mode="fused", packed=False):
    return dict(name=name, kind="mlp", M=M, K1=K1, N1=N1, N2=N2, mid=mid, dtype=dtype, policy=policy, mode=mode, packed=packed)


def _attn(name, batch, seq, cached, heads, K1, N2, dtype="bf16", policy="strided", mode="fused"):
    return dict(name=name, kind="attn", batch=batch, seq=seq, cached=cached, heads=heads, K1=K1, N2=N2, dtype=dtype,
                policy=policy, mode=mode)


def _conv(name, B, H, W, C, K1, K2, K3=0, K4=0, dtype="bf16", policy="strided", mode="fused"):
    return dict(name=name, kind="conv", B=B, H=H, W=W, C=C, K1=K1, K2=K2, K3=K3, K4=K4, dtype=dtype, policy=policy, mode=mode)


def listed():
    return [
        # a small transformer's MLP on one prompt, fp16: a short chain, latency of launch and hand-over
        _mlp("mlp_small_fp16", 256, 1024, 4096, 1024, dtype="fp16", policy="row"),
        # generation, one token at a time: both GeMMs stream their weights
        _mlp("mlp_token_1", 1, 12288, 6144, 12288),
        # generation for a batch of 64 requests, weights packed once when the model was loaded
        _mlp("mlp_tokens_64_packed", 64, 12288, 6144, 12288, packed=True),
        # a prompt of odd length in the two-stream form, the entry point's default
        _mlp("mlp_prompt_333_two_streams", 333, 12288, 6144, 12288, policy="row", mode="fine"),
        # a long prompt or a full prefill batch: the largest chain
        _mlp("mlp_prompt_2048", 2048, 12288, 6144, 12288, policy="row"),
        # the gated MLP of LLaMA on the same number of tokens
        _mlp("swiglu_prompt_2048", 2048, 8192, 2752, 8192, mid="swiglu", policy="tile"),
        # attention block, prompt phase: QKV GeMM, causal attention, output GeMM
        _attn("attn_prompt_2048", 1, 2048, 0, 12, 12288, 12288),
        # the same block continuing a conversation: a ragged chunk of new tokens over cached ones, fp16
        _attn("attn_chunk_300_cached_700_fp16", 1, 300, 700, 12, 12288, 12288, dtype="fp16", policy="row"),
        # attention block, generation: one new token for each of four sequences
        _attn("attn_token_4x2048", 4, 1, 2048, 12, 12288, 12288),
        # convolution pairs of an image network: large images and few channels, ...
        _conv("conv_224x64_b4", 4, 224, 224, 64, 64, 64),
        # ... the middle of the network at a serving batch, ...
        _conv("conv_56x256_b16", 16, 56, 56, 256, 256, 256),
        # ... and a whole layer group of four convolutions on a single image
        _conv("conv_layer_14x512_b1", 1, 14, 14, 512, 512, 512, 512, 512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, m):
    return max(m, _log(rng, lo, hi) // m * m)


def _draw_once(rng):
    kind = rng.choice(["mlp", "mlp", "attn", "conv"])
    dtype = rng.choice(["bf16", "bf16", "fp16"])
    mode = rng.choice(["fused", "fused", "fine"])
    if kind == "mlp":
        c = _mlp("", _log(rng, 1, 2048), _mult(rng, 1024, 12288, 64), _mult(rng, 512, 6144, 64), _mult(rng, 1024, 12288, 8),
                 rng.choice(["gelu", "gelu", "relu", "swiglu"]), dtype, rng.choice(["row", "tile", "auto"]), mode, rng.random() < 0.3)
    elif kind == "attn":
        phase = rng.choice(["prompt", "chunk", "token"])
        heads = rng.randint(4, 16)
        if phase == "prompt":
            batch, seq, cached = 1, _log(rng, 64, 2048), 0
            if rng.random() < 0.3:
                batch, seq = rng.randint(2, 8), rng.choice([100, 128, 256])
        elif phase == "chunk":
            batch, seq, cached = 1, _log(rng, 16, 1024), _log(rng, 16, 2048)
        else:
            batch, seq, cached = _log(rng, 1, 16), 1, _log(rng, 64, 4096)
        c = _attn("", batch, seq, cached, heads, _mult(rng, 2048, 12288, 64), _mult(rng, 2048, 12288, 8), dtype,
                  rng.choice(["row", "tile", "strided", "auto"]), mode)
    else:
        h = _log(rng, 7, 224)
        w = h if rng.random() < 0.5 else max(7, min(224, h + rng.randint(-5, 9)))
        ch = _mult(rng, 64, 512, 64)
        k = [ch] * rng.choice([2, 2, 3, 4])
        if rng.random() < 0.3:
            k[-1] = _mult(rng, 64, 512, 8)
        k += [0] * (4 - len(k))
        c = _conv("", _log(rng, 1, 32), h, w, ch, *k, dtype=dtype, policy=rng.choice(["row", "tile", "strided"]), mode=mode)
    del c["name"]
    return c


def draw(rng):
    """One more case: prompt, chunk and generation sizes over their whole range, odd ones among them."""
    while True:
        c = _draw_once(rng)
        if work(c)["flops"] <= MAX_FLOPS[c["kind"]]:
            return c


def _layers(c):
    return [k for k in (c["K1"], c["K2"], c["K3"], c["K4"]) if k]


def _inputs(case, seed):
    """Activations and weights of a case on the GPU, in the library's layouts, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = DTYPES[case["dtype"]]

    def normal(*shape, std=1.0):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dt)

    if case["kind"] == "conv":
        x = normal(case["B"], case["H"], case["W"], case["C"])
        ws, cin = [], case["C"]
        for k in _layers(case):
            ws.append(normal(k, 3, 3, cin, std=math.sqrt(2.0 / (9 * cin))))
            cin = k
        return dict(x=x, ws=ws)
    K1, N2, kv = case["K1"], case["N2"], {}
    if case["kind"] == "mlp":
        M, k2 = case["M"], case["N1"]
        rows1 = 2 * k2 if case["mid"] == "swiglu" else k2
    else:
        b, k2, cached = case["batch"], case["heads"] * 128, case["cached"]
        M, rows1 = b * case["seq"], 3 * k2
        if cached:
            kv = dict(k_cache=normal(b, cached, k2), v_cache=normal(b, cached, k2))
    X = normal(M, K1)
    W1t = normal(rows1, K1, std=1.0 / math.sqrt(K1))
    W2t = normal(N2, k2, std=1.0 / math.sqrt(k2))
    return dict(X=X, W1t=W1t, W2t=W2t, kv=kv)


def prepare(case, seed):
    """Weights and activations on the GPU, the buffers the chain writes and the policy that owns its semaphores."""
    t = _inputs(case, seed)
    dt = DTYPES[case["dtype"]]

    def empty(*shape):
        return torch.empty(shape, device="cuda", dtype=dt)

    pol = ds.SyncPolicy(KINDS[case["policy"]])
    common = dict(policy=pol, mode=MODES[case["mode"]])
    if case["kind"] == "conv":
        outs = [empty(case["B"], case["H"], case["W"], k) for k in _layers(case)]
        return dict(kind="conv", x=t["x"], ws=t["ws"], outs=outs, common=common)
    X, W1t, W2t = t["X"], t["W1t"], t["W2t"]
    if case["kind"] == "mlp":
        N1, extra = case["N1"], dict(mid=MIDS[case["mid"]])
    else:
        E = case["heads"] * 128
        N1 = 3 * E
        extra = dict(mid=ds.MID_CAUSAL_ATTN, T=empty(X.shape[0], E), batch=case["batch"], seq=case["seq"], heads=case["heads"],
                     head_dim=128, **t["kv"])
    if case.get("packed"):   # static weights: packed once, when a model is loaded
        W1t, W2t = ds.pack_weights_kblocked(W1t), ds.pack_weights_kblocked(W2t)
    return dict(kind="gemm", a=(X, W1t, empty(X.shape[0], N1), W2t, empty(X.shape[0], case["N2"])), extra=extra, common=common)


def run(state):
    """One chain on the current stream; every buffer that it fills."""
    stream = torch.cuda.current_stream()
    if state["kind"] == "conv":
        x, ws, outs = state["x"], state["ws"], state["outs"]
        if len(ws) == 2:
            ds.dep_conv_chain(x, ws[0], outs[0], ws[1], outs[1], stream_producer=stream, **state["common"])
        else:
            ds.dep_conv_chain_n(x, ws, outs, stream_producer=stream, **state["common"])
        return list(outs)
    X, W1t, H, W2t, Y = state["a"]
    ds.dep_gemm_chain(X, W1t, H, W2t, Y, stream_producer=stream, **state["extra"], **state["common"])
    out = [H, Y]
    if "T" in state["extra"]:
        out.append(state["extra"]["T"])
    return out


def work(case):
    """Multiply-adds of the chain; bytes of every input read once and every buffer that comes back written once."""
    if case["kind"] == "conv":
        pix = case["B"] * case["H"] * case["W"]
        flops, nbytes, cin = 0.0, 2.0 * pix * case["C"], case["C"]
        for k in _layers(case):
            flops += 2.0 * pix * k * 9 * cin
            nbytes += 2.0 * (9 * cin * k + pix * k)
            cin = k
        return dict(bytes=nbytes, flops=flops)
    K1, N2 = case["K1"], case["N2"]
    if case["kind"] == "mlp":
        M, N1 = case["M"], case["N1"]
        rows1 = 2 * N1 if case["mid"] == "swiglu" else N1
        return dict(flops=2.0 * M * (rows1 * K1 + N2 * N1), bytes=2.0 * (M * (K1 + N1 + N2) + rows1 * K1 + N2 * N1))
    b, s, cached, E = case["batch"], case["seq"], case["cached"], case["heads"] * 128
    M = b * s
    flops = 2.0 * M * (3 * E * K1 + N2 * E) + 4.0 * b * E * (0.5 * s * (s + 1) + s * cached)
    nbytes = 2.0 * (M * (K1 + 3 * E + E + N2) + 3 * E * K1 + N2 * E + 2 * b * cached * E)
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """About four times the difference from the same chain in 64 bits without the rounding of its intermediates.

    Measured (2-norm / largest): bf16 GeMM chains 2.4e-3 / 1.1e-2, four convolutions 3.3e-3 / 1.9e-2, attention
    3.7e-3 / 7.1e-2 (a sequence's first tokens are rows much larger than the rest); fp16 3.0e-4 / 1.2e-3,
    attention 4.5e-4 / 5.2e-3.
    """
    attn = case["kind"] == "attn"
    if case["dtype"] == "fp16":
        return {"rel": 1.8e-3, "max": 2.0e-2} if attn else {"rel": 1.2e-3, "max": 8.0e-3}
    return {"rel": 1.5e-2, "max": 0.28} if attn else {"rel": 1.2e-2, "max": 6.0e-2}


def _conv64(x, w):
    """3x3 convolution with padding 1, NHWC, as nine shifted products."""
    B, H, W, C = x.shape
    xp = torch.zeros(B, H + 2, W + 2, C, device=x.device, dtype=x.dtype)
    xp[:, 1:-1, 1:-1] = x
    y = torch.zeros(B * H * W, w.shape[0], device=x.device, dtype=x.dtype)
    for r in range(3):
        for q in range(3):
            y += xp[:, r:r + H, q:q + W].reshape(-1, C) @ w[:, r, q].t()
    return y.view(B, H, W, -1)


def _attention64(c, qkv, kv):
    """Causal attention of the new tokens over the cached and the new ones, one head of one sequence at a time."""
    b, s, heads, cached, E = c["batch"], c["seq"], c["heads"], c["cached"], c["heads"] * 128
    T = torch.empty(b * s, E, device=qkv.device, dtype=qkv.dtype)
    hidden = torch.ones(s, cached + s, device=qkv.device, dtype=torch.bool).triu(cached + 1)
    for i in range(b):
        rows = slice(i * s, (i + 1) * s)
        for h in range(heads):
            cols = slice(h * 128, (h + 1) * 128)
            q, k, v = (qkv[rows, j * E + h * 128:j * E + (h + 1) * 128] for j in range(3))
            if cached:
                k, v = torch.cat([kv["k_cache"][i, :, cols].double(), k]), torch.cat([kv["v_cache"][i, :, cols].double(), v])
            p = (q @ k.t() / math.sqrt(128.0)).masked_fill_(hidden, -math.inf)
            T[rows, cols] = torch.softmax(p, dim=1) @ v
    return T


def exact(case, seed):
    """The chain in 64 bits with plain torch, nothing rounded on the way."""
    t = _inputs(case, seed)
    if case["kind"] == "conv":
        x, outs = t["x"].double(), []
        for i, w in enumerate(t["ws"]):
            x = _conv64(x, w.double())
            if i < len(t["ws"]) - 1:
                x = torch.relu_(x)
            outs.append(x)
        return outs
    H = t["X"].double() @ t["W1t"].double().t()
    W2 = t["W2t"].double().t()
    if case["kind"] == "attn":
        T = _attention64(case, H, t["kv"])
        return [H, T @ W2, T]
    if case["mid"] == "swiglu":
        H = torch.nn.functional.silu(H[:, :case["N1"]]) * H[:, case["N1"]:]
    else:
        H = torch.nn.functional.gelu(H) if case["mid"] == "gelu" else torch.relu(H)
    return [H, H @ W2]
