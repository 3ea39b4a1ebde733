"""The work a user of this library has it do, as timed cases.

Users call the C ABI through `paper_2510_02483_amd.lib`: a decoder block forward
and backward in one call, its two sub-layers by themselves (forward only for
evaluation and for hand-rolled pipelines, forward then backward for training),
the language-model head with the cross-entropy, a whole stack of blocks, and the
optimizer step.  Shapes are the presets of `configs.py`, those of the tests, and
generic ones between them; activations are N(0, 1), weights N(0, 0.02^2) and
RMSNorm gains 1 + 0.1 N(0, 1), all rounded to bf16, as everywhere in this
repository.  Buffers (outputs, saved state, workspace) are allocated once, as a
training program does.
"""
from __future__ import annotations

import math

import torch

from paper_2510_02483_amd import inputs, lib
from paper_2510_02483_amd.configs import BlockConfig, StackConfig

BLOCK_KINDS = ("block", "attn_fwd", "attn_train", "mlp_fwd", "mlp_train")
ATTN_W = ("attn_norm", "wq", "wk", "wv", "wo")
MLP_W = ("mlp_norm", "wg", "wu", "wd")


def _shape(kind, batch, seq, hidden, nq, nkv, d, inter, theta=1e4, accumulate=False, **more):
    return dict(kind=kind, batch=batch, seq=seq, hidden=hidden, nq=nq, nkv=nkv, d=d, inter=inter, theta=theta,
                accumulate=accumulate, **more)


def listed():
    llama3b = dict(hidden=3072, nq=24, nkv=8, d=128, inter=8192, theta=5e5)
    report3b = dict(hidden=2048, nq=16, nkv=2, d=128, inter=11008)
    return [
        # the smallest training step in use: a unit-test sized model, where launches and latency count
        dict(name="block_tiny", **_shape("block", 2, 128, 256, 4, 2, 64, 688)),
        # a small model (12 heads of 64) on sequences of odd length with gradient accumulation
        dict(name="block_small_ragged", **_shape("block", 3, 509, 768, 12, 4, 64, 2056, accumulate=True)),
        # the library's benchmark: one 3B-shaped block, micro-batch 4 x 2048
        dict(name="block_3b", **_shape("block", 4, 2048, accumulate=True, **llama3b)),
        # the report's 30B block (64 heads of 104, multi-head) at sequence 4096
        dict(name="block_30b", **_shape("block", 2, 4096, 6656, 64, 64, 104, 17920)),
        # evaluation of one short document: forward of the attention layer, 1 x 500 tokens
        dict(name="attn_fwd_short", **_shape("attn_fwd", 1, 500, **llama3b)),
        # evaluation at long context, where the attention core dominates
        dict(name="attn_fwd_long", **_shape("attn_fwd", 1, 8192, **llama3b)),
        # training of the attention layer of the report's 3B model (few kv heads), 2 x 4096
        dict(name="attn_train_gqa8", **_shape("attn_train", 2, 4096, **report3b)),
        # evaluation of one short document: forward of the MLP layer, 1 x 500 tokens
        dict(name="mlp_fwd_short", **_shape("mlp_fwd", 1, 500, **llama3b)),
        # training of the MLP layer on a micro-batch of odd size
        dict(name="mlp_train_odd", **_shape("mlp_train", 3, 677, **llama3b)),
        # the LM head of a 128k vocabulary: logits, cross-entropy and both gradients, 4096 tokens
        dict(name="head_128k", kind="head", batch=2, seq=2048, hidden=3072, vocab=128256),
        # a whole training pass of four of the report's 3B blocks with embedding and head, with recomputation
        dict(name="stack_4_layers", **_shape("stack", 1, 2048, layers=4, vocab=32000, recompute=True, **report3b)),
        # the optimizer step over one 3B-shaped block's parameters
        dict(name="adamw_block", kind="adamw", n=100_669_440, n_decay=100_663_296, clip=1.0),
    ]


# A drawn case does at most this much: below the largest listed ones.
MAX_FLOPS = 6e12


def _log_int(rng, lo, hi, step=1):
    return max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)


def _draw_once(rng):
    kind = rng.choice(BLOCK_KINDS + ("block", "stack", "head", "adamw"))
    if kind == "adamw":
        n = _log_int(rng, 100_000, 200_000_000)
        return dict(kind=kind, n=n, n_decay=n - min(n, rng.randrange(0, 60_000)), clip=rng.choice([0.0, 1.0]))
    if kind == "head":
        # tokens a multiple of 8, as the matrix products ask
        return dict(kind=kind, batch=1, seq=_log_int(rng, 64, 8192, 8), hidden=_log_int(rng, 256, 4096, 8),
                    vocab=_log_int(rng, 1000, 131_000, 8))
    d = rng.choice([64, 128, 128, 128, 104, 80])
    nkv = rng.choice([1, 2, 4, 8])
    nq = nkv * rng.choice([1, 2, 3, 4, 8])
    while nq * d > 8192 or nq * d < 256:
        nkv = rng.choice([1, 2, 4, 8])
        nq = nkv * rng.choice([1, 2, 3, 4, 8])
    hidden = nq * d if rng.random() < 0.6 else _log_int(rng, 256, 4096, 8)
    inter = int(hidden * rng.uniform(2.6, 5.4)) // 8 * 8
    if rng.random() < 0.5:
        inter = max(64, inter // 64 * 64)
    tokens = _log_int(rng, 64, 16_384)
    batch = min(rng.choice([1, 1, 2, 3, 4, 8]), max(1, tokens // 32))
    seq = max(1, tokens // batch)
    if rng.random() < 0.5:
        seq = max(32, seq // 64 * 64)
    case = _shape(kind, batch, seq, hidden, nq, nkv, d, inter, rng.choice([1e4, 5e5]), rng.random() < 0.4)
    if kind == "stack":
        case.update(layers=rng.randrange(1, 5), vocab=_log_int(rng, 1000, 131_000, 8), recompute=rng.random() < 0.5)
    return case


def draw(rng):
    while True:
        case = _draw_once(rng)
        if work(case)["flops"] <= MAX_FLOPS:
            return case


# ---- state and pass ---------------------------------------------------------------


def _block_config(case):
    return BlockConfig("case", 0, case["batch"], case["seq"], case["hidden"], case["nq"], case["nkv"], case["d"],
                       case["inter"], case["theta"])


def _randn(seed, shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(dtype)


def _block_inputs(case, seed):
    return inputs.make_inputs(_block_config(case), seed_base=1_000_003 * seed, gamma="random", device="cuda")


def _stack_config(case):
    return StackConfig("case", _block_config(case), case["layers"], case["vocab"], case["recompute"])


def _stack_inputs(case, seed):
    sc = _stack_config(case)
    base = 1_000_003 * seed
    g = torch.Generator(device="cuda").manual_seed(base + 90_000)
    ids = torch.randint(0, sc.vocab, (sc.block.batch, sc.block.seq), generator=g, device="cuda", dtype=torch.int32)
    return {"ids": ids, "embed": _randn(base + 90_001, (sc.vocab, sc.block.hidden), 0.02),
            "final_norm": _randn(base + 90_002, (sc.block.hidden,), 0.1, 1.0),
            "layers": [inputs.make_inputs(sc.block, seed_base=base + 100 * (l + 1), gamma="random", activations=False,
                                          device="cuda") for l in range(sc.n_layers)]}


def _head_inputs(case, seed):
    base = 1_000_003 * seed
    T, H, V = case["batch"] * case["seq"], case["hidden"], case["vocab"]
    g = torch.Generator(device="cuda").manual_seed(base)
    ids = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    return {"ids": ids, "h": _randn(base + 1, (T, H)), "embed": _randn(base + 2, (V, H), 0.02)}


def _adamw_inputs(case, seed):
    base = 1_000_003 * seed
    n = case["n"]
    g = torch.Generator(device="cuda").manual_seed(base)
    f = lambda std: torch.randn(n, generator=g, device="cuda").mul_(std)  # noqa: E731
    return {"master": f(0.02), "grad": f(1e-3), "m": f(1e-4), "v": f(1e-3).square_()}


LR, STEP0 = 3e-4, 100


def prepare(case, seed):
    kind = case["kind"]
    u8 = lambda n: torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")  # noqa: E731
    if kind in BLOCK_KINDS:
        c = _block_config(case)
        i = _block_inputs(case, seed)
        sizes = lib.ls_query_sizes(c)
        names = ATTN_W if kind.startswith("attn") else MLP_W if kind.startswith("mlp") else lib.WEIGHTS
        s = {"case": case, "c": c, "x": i["x"].view(c.tokens, c.hidden), "w": {n: i[n] for n in names}}
        s["y"] = torch.empty_like(s["x"])
        if kind == "block":
            s["workspace"] = u8(sizes["block_workspace"])
        else:
            part = kind.split("_")[0]
            s["saved"], s["workspace"] = u8(sizes[part + "_saved"]), u8(sizes[part + "_workspace"])
        if not kind.endswith("fwd"):
            s["dy"] = i["dy"].view(c.tokens, c.hidden)
            s["dx"] = torch.empty_like(s["x"])
            s["grads"] = {n: torch.zeros(s["w"][n].shape, dtype=torch.float32, device="cuda") for n in names}
        return s
    if kind == "stack":
        return {"case": case, "stack": lib.Stack(_stack_config(case), _stack_inputs(case, seed))}
    if kind == "head":
        i = _head_inputs(case, seed)
        T, H = i["h"].shape
        V = case["vocab"]
        return {"case": case, **i, "logits": torch.empty(T, V, dtype=torch.bfloat16, device="cuda"),
                "dh": torch.empty_like(i["h"]), "dE": torch.empty(V, H, dtype=torch.float32, device="cuda"),
                "loss": torch.empty(1, device="cuda"), "row_loss": torch.empty(T, device="cuda"),
                "workspace": u8(lib.ls_cross_entropy_workspace(T))}
    i = _adamw_inputs(case, seed)
    return {"case": case, **i, "step": STEP0, "param": torch.empty(case["n"], dtype=torch.bfloat16, device="cuda"),
            "grad_norm": torch.empty(1, device="cuda"), "workspace": u8(lib.ls_adamw_workspace())}


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "block":
        lib.ls_block_fwd_bwd(s["c"], s["x"], s["w"], s["dy"], s["y"], s["dx"], s["grads"], case["accumulate"],
                             s["workspace"])
        return {"y": s["y"], "dx": s["dx"], "grads": s["grads"]}
    if kind in BLOCK_KINDS:
        if kind.startswith("attn"):
            fwd, bwd = lib.ls_attn_fwd, lib.ls_attn_bwd
        else:
            fwd, bwd = lib.ls_mlp_fwd, lib.ls_mlp_bwd
        fwd(s["c"], s["x"], s["w"], s["y"], s["saved"], s["workspace"])
        if kind.endswith("fwd"):
            return {"y": s["y"]}
        bwd(s["c"], s["x"], s["w"], s["saved"], s["dy"], s["dx"], s["grads"], case["accumulate"], s["workspace"])
        return {"y": s["y"], "dx": s["dx"], "grads": s["grads"]}
    if kind == "stack":
        st = s["stack"]
        st.step(accumulate=case["accumulate"])
        return {"loss": st.loss, "row_loss": st.row_loss, "embed": st.d_embed, "final_norm": st.d_final_norm,
                "layers": st.d_layers}
    if kind == "head":
        lib.ls_gemm_nt(s["h"], s["embed"], s["logits"])
        lib.ls_cross_entropy(s["logits"], case["seq"], s["ids"], None, s["loss"], s["row_loss"], s["workspace"])
        lib.ls_gemm_nn(s["logits"], s["embed"], s["dh"])
        lib.ls_gemm_tn(s["logits"], s["h"], s["dE"])
        return {"loss": s["loss"], "row_loss": s["row_loss"], "dlogits": s["logits"], "dh": s["dh"], "dE": s["dE"]}
    s["step"] += 1
    lib.ls_adamw_step(s["master"], s["param"], s["grad"], s["m"], s["v"], step=s["step"], lr=LR,
                      max_norm=case["clip"], n_decay=case["n_decay"], grad_norm=s["grad_norm"],
                      workspace=s["workspace"])
    return {"master": s["master"], "param": s["param"], "m": s["m"], "v": s["v"], "grad_norm": s["grad_norm"]}


# ---- work and tolerance -------------------------------------------------------------


def _layer_work(case, attn, mlp, train):
    """Matrix products and causal attention of one block's sub-layers (backward twice the forward)."""
    T, S, H, I = case["batch"] * case["seq"], case["seq"], case["hidden"], case["inter"]
    Dq, Dkv = case["nq"] * case["d"], case["nkv"] * case["d"]
    flops = params = 0.0
    if attn:
        params += 2 * H * (Dq + Dkv) + H
        flops += 4 * T * H * (Dq + Dkv) + 4.0 * case["batch"] * Dq * S * (S + 1) / 2
    if mlp:
        params += 3 * H * I + H
        flops += 6.0 * T * H * I
    if not train:
        return flops, 2 * params + 2 * 2 * T * H
    # x, dy in and y, dx out; weights in and their fp32 gradients out (read too when accumulated)
    return 3 * flops, params * (2 + (8 if case["accumulate"] else 4)) + 4 * 2 * T * H


def work(case):
    kind = case["kind"]
    if kind == "adamw":
        return {"bytes": 30.0 * case["n"], "flops": 15.0 * case["n"]}
    if kind == "head":
        T, H, V = case["batch"] * case["seq"], case["hidden"], case["vocab"]
        # h, E in; dlogits, dh, dE out
        return {"bytes": 2.0 * (2 * T * H + V * H + T * V) + 4.0 * V * H, "flops": 6.0 * T * H * V}
    if kind == "stack":
        T, H, V, L = case["batch"] * case["seq"], case["hidden"], case["vocab"], case["layers"]
        flops, nbytes = _layer_work(case, True, True, True)
        return {"bytes": L * nbytes + 10.0 * V * H, "flops": L * flops + 6.0 * T * H * V}
    flops, nbytes = _layer_work(case, not kind.startswith("mlp"), not kind.startswith("attn"), not kind.endswith("fwd"))
    return {"bytes": nbytes, "flops": flops}


# Largest relative error against 64 bits seen over the outputs of listed and drawn cases, bf16 activations
# between fp32 sums: 2.0e-3 attn_fwd, 5.4e-3 attn_train, 3.3e-3 mlp_fwd, 3.7e-3 mlp_train, 1.7e-3 head; a block
# 5.2e-3 up to width 1024, 7.3e-3 up to 4096, 1.1e-2 at 6656; a stack 7.8e-3 with one layer, 2.2e-2 with four;
# the optimizer's fp32 state 2e-7, its bf16 weights one unit in the last place at a few rounding ties in 1e5.
# Each times about four.
TOLERANCE = {"attn_fwd": 8e-3, "attn_train": 2e-2, "mlp_fwd": 1.2e-2, "mlp_train": 1.5e-2, "head": 7e-3,
             "adamw": 1e-4}


def tolerance(case):
    if case["kind"] == "block":
        return {"rel": 2e-2 if case["hidden"] <= 1024 else 3e-2 if case["hidden"] <= 4096 else 4.5e-2}
    if case["kind"] == "stack":
        return {"rel": 2e-2 + 1.7e-2 * case["layers"]}
    return {"rel": TOLERANCE[case["kind"]]}


# ---- the same in 64 bits ----------------------------------------------------------------


class _Attention(torch.autograd.Function):
    """Causal grouped-query attention, one head at a time (its S x S matrices recomputed in the backward pass)."""

    @staticmethod
    def probs(q, k):
        S = q.shape[0]
        s = (q @ k.t()) / math.sqrt(q.shape[1])
        s.masked_fill_(torch.ones(S, S, dtype=torch.bool, device=q.device).triu_(1), -math.inf)
        return torch.softmax(s, dim=1)

    @staticmethod
    def forward(ctx, q, k, v):
        ctx.save_for_backward(q, k, v)
        G = q.shape[1] // k.shape[1]
        o = torch.empty_like(q)
        for b in range(q.shape[0]):
            for h in range(q.shape[1]):
                o[b, h] = _Attention.probs(q[b, h], k[b, h // G]) @ v[b, h // G]
        return o

    @staticmethod
    def backward(ctx, do):
        q, k, v = ctx.saved_tensors
        G = q.shape[1] // k.shape[1]
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        for b in range(q.shape[0]):
            for h in range(q.shape[1]):
                g = h // G
                p = _Attention.probs(q[b, h], k[b, g])
                dp = do[b, h] @ v[b, g].t()
                ds = p * (dp - (p * dp).sum(1, keepdim=True)) / math.sqrt(q.shape[3])
                dq[b, h] = ds @ k[b, g]
                dk[b, g] += ds.t() @ q[b, h]
                dv[b, g] += p.t() @ do[b, h]
        return dq, dk, dv


def _norm64(x, gamma):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * gamma


def _rope64(x, theta):  # [B, heads, S, d]
    half = x.shape[-1] // 2
    dev = x.device
    freq = theta ** (-torch.arange(half, dtype=torch.float64, device=dev) / half)
    a = torch.arange(x.shape[2], dtype=torch.float64, device=dev)[:, None] * freq
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)


def _attn64(case, x, w):
    B, S, d = case["batch"], case["seq"], case["d"]
    h = _norm64(x, w["attn_norm"])
    heads = lambda t: t.view(B, S, -1, d).transpose(1, 2).contiguous()  # noqa: E731
    q, k, v = (heads(h @ w[n].t()) for n in ("wq", "wk", "wv"))
    o = _Attention.apply(_rope64(q, case["theta"]), _rope64(k, case["theta"]), v)
    return x + o.transpose(1, 2).reshape(B * S, -1) @ w["wo"].t()


def _mlp64(case, x, w):
    h = _norm64(x, w["mlp_norm"])
    return x + (torch.nn.functional.silu(h @ w["wg"].t()) * (h @ w["wu"].t())) @ w["wd"].t()


def _head64(h, embed, ids, seq):
    """Logits, row losses (next token within each sequence; the last position has none) and their mean."""
    T = h.shape[0]
    z = h @ embed.t()
    tg = torch.roll(ids.long(), -1)
    has = (torch.arange(T, device=h.device) % seq) != seq - 1
    row = torch.where(has, torch.logsumexp(z, 1) - z.gather(1, tg[:, None])[:, 0], torch.zeros((), dtype=z.dtype,
                                                                                              device=z.device))
    return z, row, row.sum() / has.sum().clamp(min=1)


def _f64(t, grad=True):
    return t.to(torch.float64).requires_grad_(grad)


def exact(case, seed):
    kind = case["kind"]
    if kind == "adamw":
        i = {n: t.double() for n, t in _adamw_inputs(case, seed).items()}
        b1, b2, eps, wd, lr = 0.9, 0.95, 1e-8, 0.01, LR
        t = STEP0 + 1
        norm = i["grad"].norm()
        g = i["grad"] * (torch.clamp(case["clip"] / (norm + 1e-6), max=1.0) if case["clip"] > 0 else 1.0)
        m = b1 * i["m"] + (1 - b1) * g
        v = b2 * i["v"] + (1 - b2) * g * g
        p = i["master"]
        p[:case["n_decay"]] *= 1 - lr * wd
        p -= lr / (1 - b1 ** t) * m / ((v / (1 - b2 ** t)).sqrt() + eps)
        return {"master": p, "param": p.to(torch.bfloat16), "m": m, "v": v, "grad_norm": norm.reshape(1)}
    if kind == "head":
        i = _head_inputs(case, seed)
        h, e = _f64(i["h"], False), _f64(i["embed"], False)
        with torch.no_grad():
            z, row, loss = _head64(h, e, i["ids"], case["seq"])
            T = h.shape[0]
            has = ((torch.arange(T, device=h.device) % case["seq"]) != case["seq"] - 1).double()
            dz = torch.softmax(z, 1)
            del z
            dz[torch.arange(T, device=h.device), torch.roll(i["ids"].long(), -1)] -= 1
            dz *= (has / has.sum().clamp(min=1))[:, None]
            return {"loss": loss.reshape(1), "row_loss": row, "dlogits": dz, "dh": dz @ e, "dE": dz.t() @ h}
    if kind == "stack":
        i = _stack_inputs(case, seed)
        e, f = _f64(i["embed"]), _f64(i["final_norm"])
        layers = [{n: _f64(w[n]) for n in lib.WEIGHTS} for w in i["layers"]]
        ids = i["ids"].view(-1)
        x = e[ids.long()]
        for w in layers:
            x = _mlp64(case, _attn64(case, x, w), w)
        _, row, loss = _head64(_norm64(x, f), e, ids, case["seq"])
        loss.backward()
        return {"loss": loss.detach().reshape(1), "row_loss": row.detach(), "embed": e.grad, "final_norm": f.grad,
                "layers": [{n: w[n].grad for n in w} for w in layers]}
    i = _block_inputs(case, seed)
    train = not kind.endswith("fwd")
    names = ATTN_W if kind.startswith("attn") else MLP_W if kind.startswith("mlp") else lib.WEIGHTS
    w = {n: _f64(i[n], train) for n in names}
    T = case["batch"] * case["seq"]
    x = _f64(i["x"].view(T, -1), train)
    y = x
    if not kind.startswith("mlp"):
        y = _attn64(case, y, w)
    if not kind.startswith("attn"):
        y = _mlp64(case, y, w)
    if not train:
        return {"y": y}
    y.backward(i["dy"].view(T, -1).double())
    return {"y": y.detach(), "dx": x.grad, "grads": {n: w[n].grad for n in names}}
