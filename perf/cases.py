"""The calls that the speed of this library is judged by.

Each case is one pass through the public entry points of
``paper_2609_08443_amd.sa_sketch`` as a serving or training program makes it:
inputs resident in device memory, outputs, workspaces and saved buffers kept by
the caller, nothing read back.  ``listed()`` names the cases, ``draw()`` gives
others of the same ranges, ``exact()`` evaluates a case in float64 with plain
torch operations.

Values: K, V, X, Xs, q, upstream gradients ~ N(0, 1); prototypes ~ N(0, 1/d);
weights ~ N(0, 1/fan-in); norm gains 1 + N(0, 0.01) and biases N(0, 0.01), the
distributions of ``workloads.py``.  User lengths are fixed, log-uniform between
``lo`` and ``hi``, or half of one and half of the other ("empty" makes every
fourth user one without history).

Kinds:
  sketch        sa_sketch_fwd                       serving: refresh of the users' sketches
  sketch_train  sa_sketch_fwd + sa_sketch_bwd       training, R targets per sketch
  tokenwise     sa_sketch_fwd_tokenwise             the token-wise normalised variant
  layer_train   sa_layer_fwd + sa_layer_bwd         the SA layer with its projections
  block         sa_block_fwd                        stacked SA, serving
  block_train   sa_block_fwd (saved) + sa_block_bwd stacked SA, training
  stca          sa_stca_fwd                         targets read the sketch, serving
  stca_train    sa_stca_fwd + sa_stca_bwd           targets read the sketch, training
"""
import math

import numpy as np
import torch

from paper_2609_08443_amd import sa_sketch as sa

DEVICE = "cuda"


def listed():
    return [
        # smallest call: one user's short history in fp32 (the single-user configuration)
        dict(name="serve_1x2048_fp32", kind="sketch", dtype="fp32", B=1, lo=2048, hi=2048, H=1, d=64, M=64, lse=True),
        # one user's recent 10K suffix refreshed on arrival: latency, few tokens per CU
        dict(name="serve_1x10k", kind="sketch", dtype="bf16", B=1, lo=10_000, hi=10_000, H=4, d=128, M=512, lse=False),
        # a uniform batch of recent suffixes (16 x 10K)
        dict(name="uniform_16x10k", kind="sketch", dtype="bf16", B=16, lo=10_000, hi=10_000, H=4, d=64, M=256, lse=True),
        # the largest: full-length histories, 13 GB of K and V
        dict(name="full_64x100k", kind="sketch", dtype="bf16", B=64, lo=100_000, hi=100_000, H=8, d=64, M=1024, lse=True),
        # the training step of the benchmark: ragged 1K..100K histories, four targets per sketch
        dict(name="ragged_train", kind="sketch_train", dtype="bf16", B=32, lo=1_000, hi=100_000, H=4, d=128, M=512, R=4),
        # training at the paper's own width: single head, d = 128, 1024 prototypes
        dict(name="train_M1024", kind="sketch_train", dtype="bf16", B=12, lo=1_000, hi=100_000, H=1, d=128, M=1024, R=4),
        # the paper's serving unit: one 100K history through two stacked layers, d = 128, 1024 prototypes
        dict(name="user_100k_block_M1024", kind="block", dtype="bf16", B=1, lo=100_000, hi=100_000, H=1, d=128, M=1024, L=2),
        # the stacked block trained on a ragged batch
        dict(name="block_train", kind="block_train", dtype="bf16", B=32, lo=1_000, hi=100_000, H=4, d=128, M=512, L=2),
        # the layer in fp32, forward and backward: short ragged histories, reference-precision training
        dict(name="layer_train_fp32", kind="layer_train", dtype="fp32", B=8, lo=500, hi=5_000, H=2, d=64, M=256, R=2),
        # the token-wise variant on the ragged batch
        dict(name="tokenwise_ragged", kind="tokenwise", dtype="bf16", B=32, lo=1_000, hi=100_000, H=4, d=128, M=512),
        # serving: one user's 300 candidate targets against its 1024-row sketch
        dict(name="stca_serve", kind="stca", dtype="bf16", B=1, R=300, k=1024, D=1024, h=16),
        # training: 32 users with 40 targets each
        dict(name="stca_train", kind="stca_train", dtype="bf16", B=32, R=40, k=512, D=1024, h=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sketch", "sketch", "sketch", "sketch_train", "sketch_train", "tokenwise", "layer_train",
                       "block", "block_train", "stca", "stca_train"])
    if kind.startswith("stca"):
        dh = rng.choice([32, 64, 64, 128])
        D = rng.choice([256, 512, 1024, 1024])
        while True:
            c = dict(kind=kind, dtype="bf16", B=_log_int(rng, 1, 48), R=_log_int(rng, 8, 300),
                     k=rng.choice([128, 256, 512, 512, 1024, 1024, 2048, rng.randrange(100, 1500)]), D=D, h=D // dh)
            if c["B"] * c["R"] * c["h"] * c["k"] <= 3e7:
                return c
    fp32 = rng.random() < 0.15
    d = rng.choice([64, 128])
    # prototype counts: the usual multiples of 128, now and then an odd one
    M = rng.choice([64, 200] if rng.random() < 0.15 else [128, 256, 256, 384, 512, 512, 768, 1024, 1024, 1536, 2048])
    most = (1e10 if fp32 else 1.5e12) * (1.0 if kind == "sketch" else 0.4)
    while True:
        c = dict(kind=kind, dtype="fp32" if fp32 else "bf16", B=_log_int(rng, 1, 64), H=rng.choice([1, 1, 2, 4, 8]),
                 d=d, M=M)
        shape = rng.randrange(4)
        hi = _log_int(rng, 1_000, 100_000)
        lo = hi if shape == 0 else max(200, hi // 100)
        c.update(lo=lo, hi=hi, spread=rng.randrange(1000))
        if shape == 1 and c["B"] > 3:
            c["empty"] = True
        if kind == "sketch":
            c["lse"] = rng.random() < 0.6
        if kind in ("sketch_train", "layer_train"):
            c["R"] = rng.choice([1, 2, 4, 8])
        if kind.startswith("block"):
            c["L"] = rng.choice([1, 2, 2, 3])
        T = int(_lengths(c).sum())
        if 4.0 * T * c["H"] * c["d"] * c["M"] * c.get("L", 1) <= most and T * c["H"] * d <= 3e8:
            return c


def _lengths(case):
    B, lo, hi = case["B"], case["lo"], case["hi"]
    if lo == hi:
        n = np.full(B, hi, np.int64)
    else:
        r = np.random.RandomState(8443 + case.get("spread", 0))
        n = np.clip(np.rint(np.exp(r.uniform(math.log(lo), math.log(hi), B))), lo, hi).astype(np.int64)
    if case.get("empty"):
        n[1::4] = 0
    return n


def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _normal(gen, shape, std, dtype):
    x = torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, 1.0, generator=gen)
    return x if std == 1.0 else (x.float() * std).to(dtype)


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(1_000_003 * seed + 8443)
    dt, f32 = _dt(case), torch.float32
    t = {}
    if case["kind"].startswith("stca"):
        B, R, k, D = case["B"], case["R"], case["k"], case["D"]
        t["Xs"], t["q"] = _normal(gen, (B, k, D), 1.0, dt), _normal(gen, (B, R, D), 1.0, dt)
        for w in ("Wq", "Wk", "Wv"):
            t[w] = _normal(gen, (D, D), D ** -0.5, dt)
        if case["kind"] == "stca_train":
            t["dout"] = _normal(gen, (B, R, D), 1.0, f32)
        return t
    n = _lengths(case)
    off = np.zeros(len(n) + 1, np.int64)
    np.cumsum(n, out=off[1:])
    T, H, d, M, B = int(off[-1]), case["H"], case["d"], case["M"], case["B"]
    t["offsets"] = torch.from_numpy(off).to(DEVICE)
    t["P"] = _normal(gen, (H, M, d), d ** -0.5, dt)
    if case["kind"] in ("sketch", "sketch_train", "tokenwise"):
        t["K"], t["V"] = _normal(gen, (T, H, d), 1.0, dt), _normal(gen, (T, H, d), 1.0, dt)
    else:
        t["X"] = _normal(gen, (T, H, d), 1.0, dt)
    if case["kind"] == "layer_train":
        for w in ("Wq", "Wk"):
            t[w] = _normal(gen, (H, d, d), d ** -0.5, dt)
    if case["kind"].startswith("block"):
        L = case["L"]
        for w, shape in (("Wq", (d, d)), ("Wk", (d, d)), ("W1", (d, 2 * d)), ("W3", (d, 2 * d)), ("W2", (2 * d, d))):
            t[w] = _normal(gen, (L, H) + shape, shape[0] ** -0.5, dt)
        ln = _normal(gen, (L, 4, H, d), 0.1, f32)
        ln[:, 0::2] += 1.0
        t["ln"] = ln.to(dt)
    if "R" in case:
        t["dsketch"] = _normal(gen, (B, case["R"], H, M, d), 1.0, f32)
    if case["kind"] == "block_train":
        t["dout"] = _normal(gen, (B, H, M, d), 1.0, f32)
    return t


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device=DEVICE)


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    f32 = dict(dtype=torch.float32, device=DEVICE)
    code = sa.SA_BF16 if case["dtype"] == "bf16" else sa.SA_FP32
    kind = case["kind"]
    if kind.startswith("stca"):
        B, R, k, D, h = (case[n] for n in ("B", "R", "k", "D", "h"))
        s["out"] = torch.empty((B, R, D), **f32)
        s["ws"] = _bytes(sa.stca_fwd_workspace_size(B, R, k, D, h, code))
        if kind == "stca_train":
            s["ws_b"] = _bytes(sa.stca_bwd_workspace_size(B, R, k, D, h, code))
        return s
    B, H, M, d = case["B"], case["H"], case["M"], case["d"]
    T = (s["K"] if "K" in s else s["X"]).shape[0]
    s["sketch"] = torch.empty((B, H, M, d), **f32)
    if kind in ("sketch", "sketch_train"):
        s["ws"] = _bytes(sa.fwd_workspace_size(B, T, H, M, d, code))
        s["lse"] = torch.empty((T, H), **f32) if case.get("lse", True) else None
        if kind == "sketch_train":
            s["dK"], s["dV"], s["dP"] = torch.empty((T, H, d), **f32), torch.empty((T, H, d), **f32), torch.empty((H, M, d), **f32)
            s["ws_b"] = _bytes(sa.bwd_workspace_size(B, T, H, M, d, code, case["R"]))
    elif kind == "tokenwise":
        s["lse"] = torch.empty((B, H, M), **f32)
        s["ws"] = _bytes(sa.tokenwise_workspace_size(B, T, H, M, d, code))
    elif kind == "layer_train":
        s["lse"] = torch.empty((T, H), **f32)
        s["ws"] = _bytes(sa.layer_fwd_workspace_size(B, T, H, M, d, code))
        s["ws_b"] = _bytes(sa.layer_bwd_workspace_size(B, T, H, M, d, code, case["R"]))
    else:
        L = case["L"]
        s["ws"] = _bytes(sa.block_fwd_workspace_size(B, T, H, M, d, L, code))
        if kind == "block_train":
            s["ws_b"] = _bytes(sa.block_bwd_workspace_size(B, T, H, M, d, L, code, True))
            s["saved"] = sa.block_saved_buffer(s["X"], s["P"], s["Wq"], s["offsets"])
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind in ("sketch", "sketch_train"):
        kvp = s["K"], s["V"], s["P"], s["offsets"]
        sketch, lse = sa.sketch_fwd(*kvp, sketch=s["sketch"], lse=s["lse"], want_lse=s["lse"] is not None, workspace=s["ws"])
        if kind == "sketch":
            return sketch, lse
        return (sketch, lse) + tuple(sa.sketch_bwd(*kvp, s["dsketch"], lse, dK=s["dK"], dV=s["dV"], dP=s["dP"], workspace=s["ws_b"]))
    if kind == "tokenwise":
        return sa.sketch_fwd_tokenwise(s["K"], s["V"], s["P"], s["offsets"], sketch=s["sketch"], lse_m=s["lse"], workspace=s["ws"])
    if kind == "layer_train":
        a = s["X"], s["P"], s["Wq"], s["Wk"], s["offsets"]
        sketch, lse = sa.layer_fwd(*a, sketch=s["sketch"], lse=s["lse"], workspace=s["ws"])
        return (sketch, lse) + tuple(sa.layer_bwd(*a, s["dsketch"], lse, workspace=s["ws_b"]))
    if kind.startswith("block"):
        a = tuple(s[n] for n in ("X", "P", "Wq", "Wk", "ln", "W1", "W3", "W2", "offsets"))
        out, _ = sa.block_fwd(*a, out=s["sketch"], saved=s.get("saved"), workspace=s["ws"])
        if kind == "block":
            return out
        return out, sa.block_bwd(*a, s["dout"], saved=s["saved"], workspace=s["ws_b"])
    a = tuple(s[n] for n in ("Xs", "q", "Wq", "Wk", "Wv"))
    out, _ = sa.stca_fwd(*a, case["h"], out=s["out"], workspace=s["ws"])
    if kind == "stca":
        return out
    return out, sa.stca_bwd(*a, case["h"], s["dout"], workspace=s["ws_b"])


def work(case):
    el = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    if kind.startswith("stca"):
        B, R, k, D, h = (case[n] for n in ("B", "R", "k", "D", "h"))
        one = B * R * (4.0 * k * D * h + 6.0 * D * D)  # logits and aggregation per head, three projections
        io = el * (B * k * D + B * R * D + 3 * D * D) + 4 * B * R * D
        if kind == "stca":
            return {"bytes": io, "flops": one}
        return {"bytes": 2 * io + 4 * (B * k * D + B * R * D + 3 * D * D), "flops": 3 * one}
    B, H, M, d, T = case["B"], case["H"], case["M"], case["d"], int(_lengths(case).sum())
    rows, pair = T * H * d, H * M * d
    step = 4.0 * T * H * M * d   # the sketching step's two contractions; its backward has four
    if kind == "tokenwise":
        return {"bytes": 2 * el * rows + el * pair + 4 * B * (pair + H * M), "flops": step}
    if kind in ("sketch", "sketch_train"):
        fwd = 2 * el * rows + el * pair + 4 * B * pair + (4 * T * H if case.get("lse", True) else 0)
        if kind == "sketch":
            return {"bytes": fwd, "flops": step}
        bwd = 2 * el * rows + 4 * T * H + 4 * B * case["R"] * pair + 8 * rows + (el + 4) * pair
        return {"bytes": fwd + bwd, "flops": 3 * step}
    if kind == "layer_train":
        fwd = el * rows + 4 * B * pair + 4 * T * H
        bwd = el * rows + 4 * T * H + 4 * B * case["R"] * pair + 4 * rows
        return {"bytes": fwd + bwd, "flops": 3 * (step + 4.0 * H * M * d * d)}
    L = case["L"]
    refine = 16.0 * B * H * M * d * d  # query projections and the SwiGLU FFN of one layer
    if kind == "block":
        return {"bytes": el * rows + 4 * B * pair + el * L * H * 8 * d * d, "flops": L * (step + refine)}
    return {"bytes": 2 * el * rows + 4 * rows + 8 * B * pair + (el + 4) * L * H * 8 * d * d, "flops": 3 * L * (step + refine)}


def tolerance(case):
    # about four times the distance from float64 that single-precision sums
    # (up to 8e-7), bf16 operands (3e-3), bf16 intermediates in a chain of products
    # (STCA, 5.5e-3) and two stacked layers (6e-3) were measured to have
    if case["dtype"] == "fp32":
        return {"rel": 4e-6}
    if case["kind"].startswith("block"):
        return {"rel": 2.5e-2}
    return {"rel": 2e-2 if case["kind"].startswith("stca") else 1e-2}


# ---------------------------------------------------------------- float64 with plain torch

def _softmax_step(K, V, P, scale, dY=None):
    """One user and head in float64: sketch, lse and, with dY [M,d], dK, dV, dP."""
    sketch, lse = torch.zeros_like(P), torch.empty(K.shape[0], dtype=torch.float64, device=K.device)
    dK, dV, dP = (torch.empty_like(K), torch.empty_like(V), torch.zeros_like(P)) if dY is not None else (None,) * 3
    step = max(1, (1 << 28) // P.shape[0] // 4)
    for i in range(0, K.shape[0], step):
        k, v = K[i:i + step], V[i:i + step]
        s = k @ P.t() * scale
        lse[i:i + step] = torch.logsumexp(s, 1)
        a = torch.exp(s - lse[i:i + step, None])
        sketch += a.t() @ v
        if dY is not None:
            dV[i:i + step] = a @ dY
            da = v @ dY.t()
            ds = a * (da - (a * da).sum(1, keepdim=True)) * scale
            dK[i:i + step] = ds @ P
            dP += ds.t() @ k
    return sketch, lse, dK, dV, dP


class _Sketch(torch.autograd.Function):
    """The step above with K = V = X, for the stacked block's float64 gradients."""

    @staticmethod
    def forward(ctx, X, Kx, P, scale):
        ctx.save_for_backward(X, Kx, P)
        ctx.scale = scale
        return _softmax_step(Kx, X, P, scale)[0]

    @staticmethod
    def backward(ctx, dY):
        X, Kx, P = ctx.saved_tensors
        _, _, dK, dV, dP = _softmax_step(Kx, X, P, ctx.scale, dY)
        return dV, dK, dP, None


def _exact_block(case, t, off):
    H, M, d, L, B = case["H"], case["M"], case["d"], case["L"], case["B"]
    train = case["kind"] == "block_train"
    out = torch.empty((B, H, M, d), dtype=torch.float64, device=DEVICE)
    w = {n: t[n].double() for n in ("P", "Wq", "Wk", "ln", "W1", "W3", "W2")}
    g = {"d" + n: torch.zeros_like(x) for n, x in w.items()}
    dX = torch.zeros(t["X"].shape, dtype=torch.float64, device=DEVICE)
    norm = torch.nn.functional.layer_norm
    for b in range(B):
        for h in range(H):
            X = t["X"][off[b]:off[b + 1], h].double().requires_grad_(train)
            v = {n: (x[h] if n == "P" else x[:, :, h] if n == "ln" else x[:, h]).clone().requires_grad_(train) for n, x in w.items()}
            state = v["P"]
            for l in range(L):
                hat = _Sketch.apply(X, X @ v["Wk"][l], state @ v["Wq"][l], d ** -0.5)
                bar = norm(state + hat, (d,), v["ln"][l, 0], v["ln"][l, 1], 1e-5)
                ffn = (torch.nn.functional.silu(bar @ v["W1"][l]) * (bar @ v["W3"][l])) @ v["W2"][l]
                state = norm(bar + ffn, (d,), v["ln"][l, 2], v["ln"][l, 3], 1e-5)
            out[b, h] = state.detach()
            if train:
                state.backward(t["dout"][b, h].double())
                dX[off[b]:off[b + 1], h] = X.grad
                for n, x in v.items():
                    to = g["d" + n]
                    (to[h] if n == "P" else to[:, :, h] if n == "ln" else to[:, h]).add_(x.grad)
    return (out, dict(g, dX=dX)) if train else out


def _exact_stca(case, t):
    B, R, k, D, h = (case[n] for n in ("B", "R", "k", "D", "h"))
    train, dh = case["kind"] == "stca_train", D // h
    w = {n: t[n].double().requires_grad_(train) for n in ("Wq", "Wk", "Wv")}
    out = torch.empty((B, R, D), dtype=torch.float64, device=DEVICE)
    dXs = torch.empty((B, k, D), dtype=torch.float64, device=DEVICE)
    dq = torch.empty((B, R, D), dtype=torch.float64, device=DEVICE)
    for b in range(B):
        X, q = t["Xs"][b].double().requires_grad_(train), t["q"][b].double().requires_grad_(train)
        Q, K, V = q @ w["Wq"], X @ w["Wk"], X @ w["Wv"]
        o = torch.cat([torch.softmax(Q[:, c:c + dh] @ K[:, c:c + dh].t() * dh ** -0.5, 1) @ V[:, c:c + dh]
                       for c in range(0, D, dh)], 1)
        out[b] = o.detach()
        if train:
            o.backward(t["dout"][b].double())
            dXs[b], dq[b] = X.grad, q.grad
    if not train:
        return out
    return out, dict({"d" + n: x.grad for n, x in w.items()}, dXs=dXs, dq=dq)


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind.startswith("stca"):
        return _exact_stca(case, t)
    off = [int(x) for x in t["offsets"].tolist()]
    if kind.startswith("block"):
        return _exact_block(case, t, off)
    B, H, M, d, T = case["B"], case["H"], case["M"], case["d"], off[-1]
    f64 = dict(dtype=torch.float64, device=DEVICE)
    scale = d ** -0.5
    sketch = torch.zeros((B, H, M, d), **f64)
    if kind == "tokenwise":
        lse = torch.full((B, H, M), -math.inf, **f64)
        for b in range(B):
            for h in range(H):
                k, v = (t[n][off[b]:off[b + 1], h].double() for n in ("K", "V"))
                if k.shape[0]:
                    s = t["P"][h].double() @ k.t() * scale
                    lse[b, h] = torch.logsumexp(s, 1)
                    sketch[b, h] = torch.exp(s - lse[b, h, :, None]) @ v
        return sketch, lse
    layer, train = kind == "layer_train", "R" in case
    lse = torch.empty((T, H), **f64)
    if train:
        dK, dV, dP = torch.empty((T, H, d), **f64), torch.empty((T, H, d), **f64), torch.zeros((H, M, d), **f64)
    if layer:
        dWq, dWk = torch.zeros((H, d, d), **f64), torch.zeros((H, d, d), **f64)
    for h in range(H):
        P = t["P"][h].double()
        if layer:
            Wq, Wk = t["Wq"][h].double(), t["Wk"][h].double()
        for b in range(B):
            a, e = off[b], off[b + 1]
            V = (t["X"] if layer else t["V"])[a:e, h].double()
            K = V @ Wk if layer else t["K"][a:e, h].double()
            dY = t["dsketch"][b, :, h].double().sum(0) if train else None
            sketch[b, h], lse[a:e, h], gk, gv, gp = _softmax_step(K, V, P @ Wq if layer else P, scale, dY)
            if layer:
                dK[a:e, h] = gv + gk @ Wk.t()
                dWk[h] += V.t() @ gk
                dWq[h] += P.t() @ gp
                dP[h] += gp @ Wq.t()
            elif train:
                dK[a:e, h], dV[a:e, h] = gk, gv
                dP[h] += gp
    if layer:
        return sketch, lse, dK, dP, dWq, dWk
    if train:
        return sketch, lse, dK, dV, dP
    return sketch, lse if case["lse"] else None
