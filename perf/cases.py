"""Performance cases of the framework: the calls a spatial-temporal transformer
makes, through the public entry points, at the sizes it makes them.

Widths are those of the two models of the paper's experiments: 720M (C = 1152,
16 heads of 72, MLP 4608) and 3B (C = 2048, 32 heads of 64, MLP 8192).  Sequence
sizes are video latents: S tokens of one frame, T frames.  A call keeps its
outputs and workspaces allocated across passes, as a serving or training loop
does.

``listed()`` gives the named cases, ``draw(rng)`` one more of the same ranges,
``prepare(case, seed)`` the inputs on the GPU, ``run(state)`` one pass,
``work(case)`` the bytes and operations it cannot do without, ``tolerance(case)``
the error another correct implementation at the same precision may show, and
``exact(case, seed)`` the pass's results in float64 by plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2403_10266_amd as dsp

WEIGHT_SIGMA = 0.02          # the models' initialisation
MODELS = {"720M": (1152, 16, 4608), "3B": (2048, 32, 8192)}


def listed():
    return [
        # the fp32 projection/attention chain on a tiny latent: a unit check in
        # a user's test suite, and the smallest call there is (launch latency)
        {"name": "chain_f32_tiny", "kind": "chain", "B": 1, "T": 4, "S": 16, "C": 64, "H": 4},
        # the MLP's first layer on one rank's shard when the sequence is cut
        # finely (one 30 x 40 frame): few rows, wide output, bias and GELU
        {"name": "linear_gelu_1200rows", "kind": "linear", "M": 1200, "N": 4608, "K": 1152, "epi": "gelu",
         "bias": True, "dtype": "bf16"},
        # the switch T -> S of one GPU's shard of a 2M-token video over 8 ranks
        {"name": "switch_T64_S4096", "kind": "switch", "dims": "1x64x4096x1152", "from": 1, "to": 2, "n": 8,
         "dtype": "bf16"},
        # spatial attention over 64 x 64 latents, 32 frames in flight
        {"name": "spatial_S4096", "kind": "attn", "layout": "spatial", "B": 2, "X": 16, "L": 4096, "H": 16, "D": 72,
         "dtype": "bf16"},
        # spatial attention read from the packed QKV projection, a few frames
        # of a 30 x 45 latent (neither a tile multiple)
        {"name": "spatial_packed_S1350", "kind": "attn", "layout": "packed", "B": 1, "X": 7, "L": 1350, "H": 16,
         "D": 72, "dtype": "bf16"},
        # temporal attention of a long clip after the switch
        {"name": "temporal_T128", "kind": "attn", "layout": "temporal", "B": 2, "X": 512, "L": 128, "H": 16, "D": 72,
         "dtype": "bf16"},
        # temporal attention of a short clip read straight from (B, T, S, C),
        # as a single-GPU user runs it (no switch)
        {"name": "temporal_unswitched_T49", "kind": "attn", "layout": "unswitched", "B": 1, "X": 1350, "L": 49,
         "H": 16, "D": 72, "dtype": "bf16"},
        # every frame attends to one shared text sequence (keys broadcast)
        {"name": "cross_text_300", "kind": "cross", "B": 2, "X": 16, "Lq": 1024, "Lk": 300, "H": 16, "Hkv": 16,
         "D": 72, "train": False, "dtype": "bf16"},
        # an attention layer of a training step: forward keeping the row
        # statistics, then the gradients of q, k and v
        {"name": "attn_train_S1024", "kind": "attn_train", "B": 1, "X": 32, "L": 1024, "H": 16, "D": 72,
         "dtype": "bf16"},
        # inference through one layer of the 720M model, 32 frames of 32 x 32
        {"name": "block_forward_T32_S1024", "kind": "block", "model": "720M", "B": 1, "T": 32, "S": 1024,
         "train": False, "post_ln": False, "relu": False, "bias": False, "dtype": "bf16"},
        # a training step through one layer (forward, input and weight
        # gradients): a batch of two 17-frame clips of 20 x 20 latents, biases
        {"name": "block_train_T17_S400", "kind": "block", "model": "720M", "B": 2, "T": 17, "S": 400,
         "train": True, "post_ln": False, "relu": False, "bias": True, "dtype": "bf16"},
        # the same step in fp32 on a small clip: the full-precision reference
        # run that a training setup is checked against
        {"name": "block_train_f32_T8_S256", "kind": "block", "model": "720M", "B": 1, "T": 8, "S": 256,
         "train": True, "post_ln": False, "relu": False, "bias": True, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "linear", "switch", "attn", "attn", "cross", "attn_train", "block", "block",
                       "block_f32"])
    limit = 2.4e12  # no more operations than the largest listed case
    while True:
        H, D = rng.choice([(16, 72), (16, 72), (32, 64)])
        if kind == "chain":
            C, heads = rng.choice([(32, 2), (64, 4), (64, 2), (128, 8)])
            c = {"kind": kind, "B": rng.choice([1, 2]), "T": rng.randint(2, 16), "S": rng.randint(4, 64), "C": C,
                 "H": heads}
        elif kind == "linear":
            C, _, F = MODELS[rng.choice(["720M", "720M", "3B"])]
            N, K, epi = rng.choice([(3 * C, C, "none"), (C, C, "resid"), (F, C, "gelu"), (F, C, "relu"),
                                    (C, F, "resid"), (C, C, "f32")])
            dt = rng.choice(["bf16", "bf16", "bf16", "f32"])
            c = {"kind": kind, "M": _log_int(rng, 64, 32768 if dt == "bf16" else 4096), "N": N, "K": K, "epi": epi,
                 "bias": rng.random() < 0.5, "dtype": dt}
        elif kind == "switch":
            n = rng.choice([1, 2, 4, 8])
            dt = rng.choice(["bf16", "bf16", "f32"])
            C = rng.choice([1152, 1152, 2048])
            a, b = _log_int(rng, 4, 256), n * _log_int(rng, 8, 512)
            if rng.random() < 0.3:   # K = 3: T x H x W, T -> H
                c = {"kind": kind, "dims": f"1x{a}x{b}x{rng.randint(5, 64)}x{C}", "from": 1, "to": 2, "n": n,
                     "dtype": dt}
            elif rng.random() < 0.5:
                c = {"kind": kind, "dims": f"{rng.choice([1, 2])}x{a}x{b}x{C}", "from": 1, "to": 2, "n": n,
                     "dtype": dt}
            else:
                c = {"kind": kind, "dims": f"{rng.choice([1, 2])}x{b}x{a}x{C}", "from": 2, "to": 1, "n": n,
                     "dtype": dt}
        elif kind == "attn":
            layout = rng.choice(["spatial", "packed", "temporal", "unswitched"])
            if layout in ("spatial", "packed"):
                X, L = _log_int(rng, 1, 64), _log_int(rng, 100, 4096)
            else:
                X, L = _log_int(rng, 32, 2048), _log_int(rng, 8, 160)
            dt = rng.choice(["bf16"] * 5 + ["f32"])
            if dt == "f32":
                X, L = max(1, X // 16), min(L, 512)
            c = {"kind": kind, "layout": layout, "B": rng.choice([1, 2]), "X": X, "L": L, "H": H, "D": D, "dtype": dt}
        elif kind == "cross":
            c = {"kind": kind, "B": rng.choice([1, 2]), "X": _log_int(rng, 1, 32), "Lq": _log_int(rng, 100, 4096),
                 "Lk": _log_int(rng, 20, 512), "H": H, "Hkv": rng.choice([H, H, H // 4]), "D": D,
                 "train": rng.random() < 0.4, "dtype": "bf16"}
        elif kind == "attn_train":
            if rng.random() < 0.5:
                X, L = _log_int(rng, 1, 64), _log_int(rng, 100, 4096)
            else:
                X, L = _log_int(rng, 32, 2048), _log_int(rng, 8, 128)
            c = {"kind": kind, "B": rng.choice([1, 2]), "X": X, "L": L, "H": H, "D": D, "dtype": "bf16"}
        else:
            f32 = kind == "block_f32"
            train = rng.random() < 0.5
            # ReLU's derivative jumps at 0, so two correct implementations can
            # differ by whole terms of the gradient there: forward only
            c = {"kind": "block", "model": rng.choice(["720M", "720M", "3B"]) if not f32 else "720M",
                 "B": rng.choice([1, 2]), "T": _log_int(rng, 4, 64), "S": _log_int(rng, 64, 2048), "train": train,
                 "post_ln": rng.random() < 0.25, "relu": not train and rng.random() < 0.25,
                 "bias": rng.random() < 0.5, "dtype": "f32" if f32 else "bf16"}
            tokens = c["B"] * c["T"] * c["S"]
            if tokens < 512 or tokens > (2048 if f32 else 32768):
                continue
        w = work(c)
        if w["flops"] <= limit and w["bytes"] <= 1.3e9:
            return c


# --------------------------------------------------------------------------- inputs

def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Draws:
    """Seeded normal tensors, in a fixed order for a case."""

    def __init__(self, seed):
        self.dev = torch.device("cuda:0")
        self.gen = torch.Generator(device=self.dev).manual_seed(int(seed))

    def __call__(self, shape, dtype, sigma=1.0):
        t = torch.randn(shape, generator=self.gen, device=self.dev, dtype=torch.float32)
        return (t * sigma if sigma != 1.0 else t).to(dtype)


def _block_shapes(C, F, attn_only):
    shapes = {"wqkv_s": (3 * C, C), "wo_s": (C, C), "wqkv_t": (3 * C, C), "wo_t": (C, C)}
    if not attn_only:
        shapes.update(w1=(F, C), w2=(C, F))
    return shapes


def _block_weights(d, C, F, dtype, bias, attn_only=False):
    w = {n: d(s, dtype, WEIGHT_SIGMA) for n, s in _block_shapes(C, F, attn_only).items()}
    if bias:
        w.update({"b" + n[1:]: d((s[0],), dtype, WEIGHT_SIGMA) for n, s in _block_shapes(C, F, attn_only).items()})
    return w


def _flags(case):
    return (dsp.DSP_BLOCK_POST_LN if case["post_ln"] else 0) | (dsp.DSP_BLOCK_RELU if case["relu"] else 0)


EPILOGUES = {"none": dsp.DSP_EPI_NONE, "gelu": dsp.DSP_EPI_GELU, "resid": dsp.DSP_EPI_RESID,
             "f32": dsp.DSP_EPI_F32, "relu": dsp.DSP_EPI_RELU}


def _inputs(case, seed):
    """The input tensors of a case, a dict (prepare and exact read the same)."""
    d = _Draws(seed)
    k = case["kind"]
    dt = _dt(case) if "dtype" in case else torch.float32
    if k == "chain":
        C = case["C"]
        return {"x": d((case["B"], case["T"], case["S"], C), torch.float32),
                "w": _block_weights(d, C, 0, torch.float32, False, attn_only=True)}
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"a": d((M, K), dt), "w": d((N, K), dt, WEIGHT_SIGMA),
                "bias": d((N,), dt, WEIGHT_SIGMA) if case["bias"] else None,
                "resid": d((M, N), torch.float32) if case["epi"] == "resid" else None}
    if k == "switch":
        return {"x": d(tuple(int(v) for v in case["dims"].split("x")), dt)}
    if k == "attn":
        B, X, L, C = case["B"], case["X"], case["L"], case["H"] * case["D"]
        if case["layout"] == "packed":
            qkv = d((B, X, L, 3 * C), dt)
            q, kk, v = qkv[..., :C], qkv[..., C:2 * C], qkv[..., 2 * C:]
        elif case["layout"] == "unswitched":   # tensors lie as (B, T = L, S = X, C)
            q, kk, v = (d((B, L, X, C), dt).permute(0, 2, 1, 3) for _ in range(3))
        else:
            q, kk, v = (d((B, X, L, C), dt) for _ in range(3))
        return {"q": q, "k": kk, "v": v}
    if k == "cross":
        B, X, D = case["B"], case["X"], case["D"]
        q = d((B, X, case["Lq"], case["H"] * D), dt)
        xs = X if case["train"] else 1         # gradients need an owner per key: no broadcast
        kv = [d((B, xs, case["Lk"], case["Hkv"] * D), dt).expand(B, X, -1, -1) for _ in range(2)]
        return {"q": q, "k": kv[0], "v": kv[1], "do": d(q.shape, dt) if case["train"] else None}
    if k == "attn_train":
        shape = (case["B"], case["X"], case["L"], case["H"] * case["D"])
        return {n: d(shape, dt) for n in ("q", "k", "v", "do")}
    C, _, F = MODELS[case["model"]]
    x = d((case["B"], case["T"], case["S"], C), torch.float32)
    w = _block_weights(d, C, F, dt, case["bias"])
    dy = d((case["B"], case["S"], case["T"], C), torch.float32) if case["train"] else None
    return {"x": x, "w": w, "dy": dy}


def prepare(case, seed):
    t = _inputs(case, seed)
    k = case["kind"]
    st = {"case": case, **t}
    dev = torch.device("cuda:0")

    def empty(shape, dtype):
        return torch.empty(shape, dtype=dtype, device=dev)

    if k == "chain":
        B, T, S, C = t["x"].shape
        st["out"] = empty((B, S, T, C), torch.float32)
        st["ws"] = empty(dsp.block_workspace_bytes(B, T, S, C, case["H"], 0, dsp.DSP_F32), torch.uint8)
    elif k == "linear":
        st["out"] = empty((case["M"], case["N"]), torch.float32 if case["epi"] in ("resid", "f32") else _dt(case))
    elif k == "switch":
        st["out"] = empty((t["x"].numel(),), t["x"].dtype)
    elif k in ("attn", "cross", "attn_train"):
        q = t["q"]
        if k == "attn" and case["layout"] == "unswitched":
            B, X, L, C = q.shape
            st["out"] = empty((B, L, X, C), q.dtype).permute(0, 2, 1, 3)
        else:
            st["out"] = empty(tuple(q.shape), q.dtype)
        if t.get("do") is not None:
            B, X, L = q.shape[:3]
            st["lse"] = empty((B, X, case["H"], L), torch.float32)
            st["delta"] = empty((B, X, case["H"], L), torch.float32)
            st["grads"] = [empty(tuple(t[n].shape), q.dtype) for n in ("q", "k", "v")]
    else:
        B, T, S, C = t["x"].shape
        _, H, F = MODELS[case["model"]]
        code = dsp.DSP_BF16 if case["dtype"] == "bf16" else dsp.DSP_F32
        st["out"] = empty((B, S, T, C), torch.float32)
        if case["train"]:
            st["saved"] = empty(int(dsp.lib().dsp_st_block_train_saved_bytes(B, T, S, C, H, F, _flags(case), code)),
                                torch.uint8)
            st["ws"] = empty(int(dsp.lib().dsp_st_block_backward_workspace_bytes(B, T, S, C, H, F, code)),
                             torch.uint8)
            st["dx"] = empty((B, T, S, C), torch.float32)
            st["g"] = {n: empty(tuple(v.shape), torch.float32) for n, v in t["w"].items()}
        else:
            st["ws"] = empty(dsp.block_workspace_bytes(B, T, S, C, H, F, code), torch.uint8)
    return st


def run(st):
    case = st["case"]
    k = case["kind"]
    if k == "chain":
        return dsp.dsp_st_block_forward(st["x"], st["w"], case["H"], flags=dsp.DSP_BLOCK_ATTN_ONLY, out=st["out"],
                                        workspace=st["ws"])
    if k == "linear":
        return dsp.dsp_linear(st["a"], st["w"], st["bias"], st["resid"], EPILOGUES[case["epi"]], out=st["out"])
    if k == "switch":
        return dsp.dsp_switch(st["x"], case["from"], case["to"], case["n"], out=st["out"])
    if k == "attn":
        fn = {"spatial": dsp.dsp_spatial_attn, "packed": dsp.dsp_spatial_attn, "temporal": dsp.dsp_temporal_attn,
              "unswitched": dsp.dsp_attn_strided}[case["layout"]]
        return fn(st["q"], st["k"], st["v"], case["H"], out=st["out"])
    if k == "cross":
        if not case["train"]:
            return dsp.dsp_attn_general(st["q"], st["k"], st["v"], case["H"], case["Hkv"], out=st["out"])
        o, lse = dsp.dsp_attn_general(st["q"], st["k"], st["v"], case["H"], case["Hkv"], out=st["out"], lse=st["lse"])
        dq, dk, dv = dsp.dsp_attn_general_bwd(st["q"], st["k"], st["v"], o, st["do"], lse, case["H"], case["Hkv"],
                                              *st["grads"], delta=st["delta"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if k == "attn_train":
        o, lse = dsp.dsp_attn_fwd_lse(st["q"], st["k"], st["v"], case["H"], out=st["out"], lse=st["lse"])
        dq, dk, dv = dsp.dsp_attn_bwd(st["q"], st["k"], st["v"], o, st["do"], lse, case["H"], *st["grads"],
                                      delta=st["delta"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    H = MODELS[case["model"]][1]
    flags = _flags(case)
    if not case["train"]:
        return dsp.dsp_st_block_forward(st["x"], st["w"], H, flags=flags, out=st["out"], workspace=st["ws"])
    y, saved = dsp.dsp_st_block_forward_train(st["x"], st["w"], H, flags=flags, out=st["out"], saved=st["saved"])
    dx, g = dsp.dsp_st_block_backward(st["x"], st["dy"], st["w"], saved, H, flags=flags, dx=st["dx"], grads=st["g"],
                                      workspace=st["ws"])
    return {"y": y, "dx": dx, **{n: g[n] for n in sorted(g)}}


# --------------------------------------------------------------------------- work and tolerance

def work(case):
    """Bytes of every input read once and every output written once, and the
    operations of the definition (no padding, no recomputation)."""
    k = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if k == "switch":
        n = math.prod(int(v) for v in case["dims"].split("x"))
        return {"bytes": 2 * n * es, "flops": 0}
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        out = 4 if case["epi"] in ("resid", "f32") else es
        resid = 4 * M * N if case["epi"] == "resid" else 0
        return {"bytes": (M * K + N * K) * es + M * N * out + resid + (N * es if case["bias"] else 0),
                "flops": 2 * M * N * K}
    if k in ("attn", "attn_train"):
        tok, C = case["B"] * case["X"] * case["L"], case["H"] * case["D"]
        rows = tok * case["H"]
        train = k == "attn_train"
        # training: q, k, v, do in; o, dq, dk, dv and lse out; 4 + 10 L^2 D per unit
        return {"bytes": (8 if train else 4) * tok * C * es + (4 * rows if train else 0),
                "flops": (14 if train else 4) * tok * case["L"] * C}
    if k == "cross":
        tq, C = case["B"] * case["X"] * case["Lq"], case["H"] * case["D"]
        kv = 2 * case["B"] * (case["X"] if case["train"] else 1) * case["Lk"] * case["Hkv"] * case["D"]
        if case["train"]:
            return {"bytes": (4 * tq * C + 2 * kv) * es + 4 * tq * case["H"], "flops": 14 * tq * case["Lk"] * C}
        return {"bytes": (2 * tq * C + kv) * es, "flops": 4 * tq * case["Lk"] * C}
    B, T, S = case["B"], case["T"], case["S"]
    tok = B * T * S
    if k == "chain":
        C, F = case["C"], 0
        train = bias = False
    else:
        C, _, F = MODELS[case["model"]]
        train, bias = case["train"], case["bias"]
    weights = 8 * C * C + 2 * F * C
    nbias = (8 * C + F + C) if bias else 0
    gemm, att = 2 * tok * weights, 4 * tok * (S + T) * C
    by = 8 * tok * C + (weights + nbias) * es
    if not train:
        return {"bytes": by, "flops": gemm + att}
    # x, dy in; y, dx and the fp32 weight gradients out
    return {"bytes": by + 8 * tok * C + 4 * (weights + nbias), "flops": 3 * gemm + att * 14 // 4}


def tolerance(case):
    k = case["kind"]
    if k == "switch":
        return "exact"
    # about four times the distance from exact() measured: 3e-7 to 1.3e-6 in
    # fp32; in bf16 1.7e-3 (a linear map), 1.2e-3 (a block, whose residual
    # stream is fp32), 2.6e-3 to 3.4e-3 (attention and its gradients) and up
    # to 4.8e-3 (a block's weight gradients)
    if case.get("dtype", "f32") == "f32":
        return {"rel": 1e-5}
    if k == "linear":
        return {"rel": 7e-3}
    if k == "block":
        return {"rel": 2e-2 if case["train"] else 5e-3}
    return {"rel": 1.2e-2}


# --------------------------------------------------------------------------- float64 results

def _attn64(q, k, v, H, scale=None, lse=False):
    """q (B, X, Lq, H D), k, v (B, X, Lk, Hkv D), float64; differentiable."""
    B, X, Lq, C = q.shape
    D = C // H
    Hkv = k.shape[3] // D
    Lk = k.shape[2]

    def heads(t, L, n):
        return t.reshape(B * X, L, n, D).permute(0, 2, 1, 3)

    qh = heads(q, Lq, H)
    kh, vh = (heads(t, Lk, Hkv).repeat_interleave(H // Hkv, 1) for t in (k, v))
    per = max(1, int(2.0e8 // max(1, H * Lq * Lk)))
    outs, ls = [], []
    for u in range(0, B * X, per):
        z = torch.matmul(qh[u:u + per], kh[u:u + per].transpose(-1, -2).contiguous()) * (scale or D ** -0.5)
        outs.append(torch.matmul(torch.softmax(z, -1), vh[u:u + per].contiguous()))
        if lse:
            ls.append(torch.logsumexp(z, -1))
    o = torch.cat(outs).permute(0, 2, 1, 3).reshape(B, X, Lq, C)
    return (o, torch.cat(ls).reshape(B, X, H, Lq)) if lse else o


def _block64(x, w, H, attn_only=False, post_ln=False, relu=False, eps=1e-6):
    C = x.shape[-1]

    def ln(v):
        return torch.nn.functional.layer_norm(v, (C,), eps=eps)

    def lin(h, n):
        y = torch.matmul(h, w["w" + n].t())
        return y + w["b" + n] if ("b" + n) in w else y

    def attn(h, side):
        qkv = lin(h, "qkv_" + side)
        return lin(_attn64(qkv[..., :C], qkv[..., C:2 * C], qkv[..., 2 * C:], H), "o_" + side)

    if attn_only:
        return attn(attn(x, "s").permute(0, 2, 1, 3), "t")

    def sub(v, f):
        return ln(v + f(v)) if post_ln else v + f(ln(v))

    act = torch.relu if relu else torch.nn.functional.gelu
    x = sub(x, lambda h: attn(h, "s"))
    y = sub(x.permute(0, 2, 1, 3), lambda h: attn(h, "t"))
    return sub(y, lambda h: lin(act(lin(h, "1")), "2"))


def exact(case, seed):
    t = _inputs(case, seed)
    k = case["kind"]

    def f64(v):
        return None if v is None else v.double()

    if k == "switch":
        x, (fr, to, n) = t["x"], (case["from"], case["to"], case["n"])
        nd = x.dim()
        others = [d for d in range(1, nd - 1) if d != fr]
        y = x.permute(0, *others, fr, nd - 1)                  # from-dim innermost
        at = 1 + others.index(to)
        return torch.stack(y.chunk(n, at)).contiguous().reshape(-1)
    if k == "linear":
        y = torch.matmul(f64(t["a"]), f64(t["w"]).t())
        if t["bias"] is not None:
            y = y + f64(t["bias"])
        if case["epi"] == "gelu":
            y = torch.nn.functional.gelu(y)
        elif case["epi"] == "relu":
            y = torch.relu(y)
        elif case["epi"] == "resid":
            y = y + f64(t["resid"])
        return y
    if k == "attn":
        return _attn64(f64(t["q"]), f64(t["k"]), f64(t["v"]), case["H"])
    if k in ("cross", "attn_train"):
        q, kk, v = (f64(t[n]) for n in ("q", "k", "v"))
        if t["do"] is None:
            return _attn64(q, kk, v, case["H"])
        for a in (q, kk, v):
            a.requires_grad_(True)
        o, lse = _attn64(q, kk, v, case["H"], lse=True)
        dq, dk, dv = torch.autograd.grad(o, (q, kk, v), f64(t["do"]))
        return {"o": o.detach(), "lse": lse.detach(), "dq": dq, "dk": dk, "dv": dv}
    x = f64(t["x"])
    w = {n: f64(v) for n, v in t["w"].items()}
    if k == "chain":
        return _block64(x, w, case["H"], attn_only=True)
    H = MODELS[case["model"]][1]
    opts = {"post_ln": case["post_ln"], "relu": case["relu"]}
    if not case["train"]:
        return _block64(x, w, H, **opts)
    leaves = [x.requires_grad_(True)] + [w[n].requires_grad_(True) for n in sorted(w)]
    y = _block64(x, w, H, **opts)
    grads = torch.autograd.grad(y, leaves, f64(t["dy"]))
    return {"y": y.detach(), "dx": grads[0], **dict(zip(sorted(w), grads[1:]))}
