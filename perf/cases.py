"""Timed workloads of the group-shared fixed fan-in output layer, one pass each through the public
entry points of ``paper_2606_01117_amd``.

A case is one of these kinds of work:

* ``train``: the training pass of a layer (``haste_tail_step``, and with a dense head
  ``haste_head_fwd_bce`` and ``haste_head_bwd``, whose input gradient adds onto the tail's).
* ``sgd``: the same pass with the momentum step on both weight arrays (``haste_tail_step_sgd``,
  the head's calls, ``haste_sgd_momentum``).
* ``calls``: the separate calls a program makes that wants the logits too (``haste_fwd``,
  ``haste_bce_grad``, ``haste_bwd_w`` with the bias gradient, ``haste_bwd_x``).
* ``predict``: the logits of a small batch, tail and head (``haste_fwd``, ``haste_head_fwd``).
* ``rewire``: one pruning and regrowth of the supports (``haste_rewire``), every few hundred steps.
* ``group``: the semantic grouping of the labels before training (``haste_group_labels``).

Sizes are those of ``synth.WORKLOADS``, of the fan-in and group-size ablations (fan-in 32 to 256,
groups of 1 to 64 labels), and generic odd ones.  Inputs follow the laws of ``synth`` (features
N(0, 1), weights N(0, 1/fan-in), uniform supports, Zipf positives), drawn on the GPU.
"""
from __future__ import annotations

import math

import torch

import paper_2606_01117_amd as hs

DEV = "cuda"
LR, MOMENTUM, DECAY = 0.01, 0.9, 1e-4


def _layer(name, kind, B, F_s, L, G, F_in, H=0, dtype="bf16", P=5, zipf=1.1, bias=False):
    return {"name": name, "kind": kind, "B": B, "F_s": F_s, "L": L, "G": G, "F_in": F_in, "H": H, "dtype": dtype,
            "P": P, "zipf": zipf, "bias": bias}


def listed():
    return [
        # training on the 3M-label set with its 65K-label head: the flagship step
        _layer("train_3m_g32", "train", 512, 768, 2949120, 32, 64, H=65536, P=8, zipf=1.05),
        # training with the optimizer on the 670K-label set, fan-in 128 and a 16K-label head
        _layer("sgd_655k_g32_f128", "sgd", 256, 768, 655360, 32, 128, H=16384),
        # a 131K-label layer without a head, the ordinary small training step
        _layer("train_131k_g16", "train", 128, 768, 131072, 16, 64),
        # the ends of the group-size ablation: standard per-label fixed fan-in, and groups of 4
        _layer("train_655k_g1", "train", 256, 768, 655360, 1, 64),
        _layer("train_655k_g4", "train", 256, 768, 655360, 4, 64),
        # the widest setting of the fan-in ablation
        _layer("train_131k_g32_f256", "train", 256, 768, 131072, 32, 256),
        # fp32 training through the separate calls: the tiny test layer, and a 131K-label one
        _layer("calls_4k_g8_f32", "calls", 32, 256, 4096, 8, 32, dtype="f32", bias=True),
        _layer("calls_131k_g16_f32", "calls", 128, 768, 131072, 16, 64, dtype="f32", bias=True),
        # scoring a handful of requests against every label
        _layer("predict_655k_b8", "predict", 8, 768, 655360, 32, 128, H=16384, bias=True),
        # nothing a power of two: a last batch of an epoch, odd widths, a short head, biases
        _layer("train_ragged", "train", 77, 500, 65544, 24, 48, H=1003, P=7, bias=True),
        # rewiring the 3M-label layer, with its momentum, at the usual tenth
        {**_layer("rewire_3m_g32", "rewire", 0, 768, 2949120, 32, 64), "rho": 0.1},
        # grouping 131K labels by 768-dimensional embeddings, bucket factor 16
        {"name": "group_131k", "kind": "group", "N": 131072, "D": 768, "G": 32, "beta": 16, "iters": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train"] * 6 + ["sgd"] * 3 + ["calls"] * 4 + ["predict"] * 3 + ["rewire"] * 2 + ["group"])
    if kind == "group":
        return {"kind": "group", "N": _log(rng, 8192, 131072), "D": 64 * rng.randint(1, 12), "G": rng.choice([8, 16, 32, 64]),
                "beta": 16, "iters": rng.randint(4, 10)}
    dtype = "f32" if kind in ("calls", "train", "sgd") and rng.random() < 0.25 else "bf16"
    G = rng.choice([1, 2, 4, 8, 16, 16, 32, 32, 32, 64, rng.randint(3, 60)])
    F_s = rng.choice([256, 384, 512, 768, 768, 768, 2 * rng.randint(150, 440), rng.randint(300, 900)])
    F_in = rng.choice([32, 64, 64, 128, 256, rng.randint(20, 200)])
    F_in = min(F_in, F_s)
    B = _log(rng, 1, 48) if kind == "predict" else _log(rng, 16, 512)
    B = 8 * max(2, B // 8) if kind != "predict" and rng.random() < 0.5 else B
    most = min(655360, 32_000_000 // B * 2 if dtype == "f32" else 655360, 3_000_000_000 // (B * F_in))
    L = G * max(1, _log(rng, 4096, max(8192, most)) // G)
    H = rng.choice([0, 0, 1024, 4096, 16384, rng.randint(500, 9000)])
    c = _layer("", kind, 0 if kind == "rewire" else B, F_s, L, G, F_in, H=0 if kind in ("calls", "rewire") else H,
               dtype=dtype, P=rng.choice([5, 5, 8, rng.randint(1, 40)]), bias=rng.random() < 0.5)
    del c["name"]
    if kind == "rewire":
        c["rho"] = rng.choice([0.05, 0.1, 0.2, 0.3])
    return c


# ---- inputs -----------------------------------------------------------------------------------
def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _code(c):
    return hs.HASTE_DTYPE_F32 if c["dtype"] == "f32" else hs.HASTE_DTYPE_BF16


def _supports(K, F_s, F_in, gen):
    idx = torch.empty((K, F_in), dtype=torch.int32, device=DEV)
    for k in range(0, K, 65536):
        n = min(65536, K - k)
        keys = torch.rand((n, F_s), device=DEV, generator=gen)
        idx[k:k + n] = keys.argsort(1)[:, :F_in].sort(1).values.int()
    return idx


def _normal(shape, scale, dtype, gen):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    for r in range(0, shape[0], 1 << 20):
        n = min(1 << 20, shape[0] - r)
        out[r:r + n] = (torch.randn((n, shape[1]), device=DEV, generator=gen) * scale).to(dtype)
    return out


def _positives(c, gen):
    """Tail and head positives [B, P] (-1 where a positive belongs to the other): Zipf ranks over
    head and tail labels, the tail's stored in a random order."""
    B, P, L, H = c["B"], c["P"], c["L"], c["H"]
    cdf = torch.arange(1, H + L + 1, dtype=torch.float64, device=DEV).pow(-c["zipf"]).cumsum(0)
    u = torch.rand((B, P), dtype=torch.float64, device=DEV, generator=gen) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=H + L - 1)
    place = torch.randperm(L, device=DEV, generator=gen)
    tail = torch.where(rank >= H, place[(rank - H).clamp_(min=0)], -1)
    return tail.int().contiguous(), torch.where(rank < H, rank, -1).int().contiguous()


def _inputs(c, seed):
    """What a pass reads, from the seed alone."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    if c["kind"] == "group":
        N, D = c["N"], c["D"]
        topics = torch.randn((max(16, N // 160), D), device=DEV, generator=gen)
        topics /= topics.norm(dim=1, keepdim=True)
        e = topics[torch.randint(0, topics.shape[0], (N,), device=DEV, generator=gen)]
        e = e + 0.3 / D ** 0.5 * torch.randn((N, D), device=DEV, generator=gen)
        return {"E": torch.round(127 * e / e.norm(dim=1, keepdim=True)).to(torch.int8)}
    B, F_s, L, G, F_in, H, dt = c["B"], c["F_s"], c["L"], c["G"], c["F_in"], c["H"], _dt(c)
    s = {"idx": _supports(L // G, F_s, F_in, gen), "W": _normal((L, F_in), F_in ** -0.5, dt, gen)}
    if c["kind"] in ("rewire", "sgd"):
        s["m"] = _normal((L, F_in), 0.01, torch.float32, gen)
    if c["kind"] == "rewire":
        return s
    s["X"] = _normal((B, F_s), 1.0, dt, gen)
    s["bias"] = 0.1 * torch.randn(L, device=DEV, generator=gen) if c["bias"] else None
    s["pos"], s["pos_h"] = _positives(c, gen)
    if H:
        s["W_h"] = _normal((H, F_s), F_s ** -0.5, dt, gen)
        s["bias_h"] = 0.1 * torch.randn(H, device=DEV, generator=gen) if c["bias"] else None
        if c["kind"] == "sgd":
            s["m_h"] = _normal((H, F_s), 0.01, torch.float32, gen)
    return s


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    s["case"], s["seed"] = c, seed
    if c["kind"] == "group":
        s["opts"] = hs.group_opts(c["G"], c["beta"], c["iters"], 5)
        s["ws"] = hs.workspace(hs.haste_group_workspace_bytes(c["N"], c["D"], s["opts"]))
        s["order"], s["gsize"], s["cluster"] = (torch.zeros(c["N"], dtype=torch.int32, device=DEV) for _ in range(3))
        s["n_groups"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        return s
    B, F_s, L, F_in, H, dt, code = c["B"], c["F_s"], c["L"], c["F_in"], c["H"], _dt(c), _code(c)
    desc = s["desc"] = hs.make_desc(B, F_s, L, c["G"], F_in, code)
    op = {"train": hs.HASTE_OP_TAIL_STEP, "sgd": hs.HASTE_OP_TAIL_STEP_SGD, "rewire": hs.HASTE_OP_REWIRE,
          "calls": hs.HASTE_OP_BWD_W, "predict": hs.HASTE_OP_FWD}[c["kind"]]
    s["ws"] = hs.workspace(hs.haste_workspace_bytes(desc, op))
    if c["kind"] == "rewire":
        return s

    def new(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device=DEV)

    if c["kind"] in ("predict", "calls"):
        s["Y"] = new(B, L, dtype=dt)
        if H:
            s["Y_h"] = new(B, H, dtype=dt)
    if c["kind"] == "predict":
        return s
    s["dY"], s["dX"] = new(B, L, dtype=dt), new(B, F_s)
    s["dbias"] = new(L) if c["bias"] else None
    if c["kind"] == "sgd":
        s["opt"], s["W_next"] = hs.sgd_opts(LR, MOMENTUM, DECAY), new(L, F_in, dtype=dt)
    else:
        s["dW"] = new(L, F_in)
    if c["kind"] == "calls":
        s["ws_x"] = hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_X))
    if H:
        s["dY_h"], s["dW_h"] = new(B, H, dtype=dt), new(H, F_s)
        s["ws_h"] = hs.workspace(hs.haste_head_workspace_bytes(B, F_s, H, code))
        if c["kind"] == "sgd":
            s["W_h_next"] = new(H, F_s, dtype=dt)
    return s


# ---- one pass ---------------------------------------------------------------------------------
def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "group":
        hs.haste_group_labels(s["E"], s["opts"], s["order"], s["gsize"], s["n_groups"], s["cluster"], s["ws"])
        return {k: s[k] for k in ("order", "gsize", "n_groups", "cluster")}
    desc, B, F_s, H, code = s["desc"], c["B"], c["F_s"], c["H"], _code(c)
    if kind == "rewire":
        n = hs.haste_rewire(desc, s["idx"], s["W"], s["m"], c["rho"], 1, s["seed"] & 0xffff, s["ws"])
        return {"idx": s["idx"], "W": s["W"], "m": s["m"], "pruned": n}
    if kind == "predict":
        hs.haste_fwd(desc, s["X"], s["idx"], s["W"], s["bias"], s["Y"], s["ws"])
        if H:
            hs.haste_head_fwd(B, F_s, H, code, s["X"], s["W_h"], s["bias_h"], s["Y_h"])
        return {k: s[k] for k in ("Y", "Y_h") if k in s}
    if kind == "calls":
        hs.haste_fwd(desc, s["X"], s["idx"], s["W"], s["bias"], s["Y"])
        hs.haste_bce_grad(B, c["L"], code, s["Y"], s["pos"], s["dY"])
        hs.haste_bwd_w(desc, s["X"], s["idx"], s["dY"], s["dW"], s["dbias"], 0, s["ws"])
        hs.haste_bwd_x(desc, s["idx"], s["W"], s["dY"], s["dX"], 0, s["ws_x"])
        return {k: s[k] for k in ("Y", "dY", "dW", "dbias", "dX")}
    if kind == "train":
        hs.haste_tail_step(desc, s["X"], s["idx"], s["W"], s["bias"], s["pos"], s["dY"], s["dW"], s["dbias"], 0,
                           s["dX"], 0, s["ws"])
    else:
        hs.haste_tail_step_sgd(desc, s["X"], s["idx"], s["W"], s["bias"], s["pos"], s["dY"], s["dbias"], s["opt"],
                               s["m"], s["W_next"], s["dX"], 0, s["ws"])
    if H:
        hs.haste_head_fwd_bce(B, F_s, H, code, s["X"], s["W_h"], s["bias_h"], s["pos_h"], s["dY_h"])
        hs.haste_head_bwd(B, F_s, H, code, s["X"], s["W_h"], s["dY_h"], s["dW_h"], s["dX"], 1, s["ws_h"])
        if kind == "sgd":
            hs.haste_sgd_momentum(H * F_s, code, s["W_h"], s["dW_h"], s["m_h"], s["opt"], s["W_h_next"])
    names = ("dY", "dW", "dbias", "m", "W_next", "dX", "dY_h", "dW_h", "m_h", "W_h_next")
    return {k: s[k] for k in names if s.get(k) is not None}


# ---- what a pass cannot do without, and what it may differ by ------------------------------------
def work(case):
    c = case
    if c["kind"] == "group":
        clusters = max(1, c["N"] // (c["beta"] * c["G"]))
        return {"bytes": c["N"] * (c["D"] + 12), "flops": 2 * c["N"] * c["D"] * clusters * (c["iters"] + 1)}
    B, F_s, L, F_in, H = c["B"], c["F_s"], c["L"], c["F_in"], c["H"]
    e = 4 if c["dtype"] == "f32" else 2
    w, idx, wh = L * F_in, L // c["G"] * F_in * 4, H * F_s
    if c["kind"] == "rewire":
        return {"bytes": 2 * (w * (e + 4) + idx), "flops": w}
    x, pos, bias = B * F_s * e, B * c["P"] * 4, (L + H) * 4 if c["bias"] else 0
    n = x + idx + w * e + wh * e + bias
    if c["kind"] == "predict":
        return {"bytes": n + B * (L + H) * e, "flops": 2 * B * (w + wh)}
    n += pos + B * (L + H) * e + B * F_s * 4 + (bias if c["bias"] else 0)
    if c["kind"] == "sgd":
        n += (w + wh) * (8 + e)          # the velocity in and out, the next weights
    else:
        n += (w + wh) * 4
    if c["kind"] == "calls":
        n += B * L * e                   # the logits beside their gradient
    return {"bytes": n, "flops": 6 * B * (w + wh)}


def tolerance(case):
    if case["kind"] in ("rewire", "group"):
        return "exact"
    # four times what the outputs differ by from the 64-bit pass (fp32: 3.7e-7 and 1.3e-6 over sums of
    # up to 335K labels, longer ones differ by more; bf16: 2.3e-3 and 1.1e-2, of the stored weights)
    return {"rel": 2e-6, "max": 2e-5} if case["dtype"] == "f32" else {"rel": 9e-3, "max": 4.5e-2}


# ---- the same pass in 64 bits -----------------------------------------------------------------------
def exact(case, seed):
    """Dense fp64 products over zero-filled weight rows, 32768 labels at a time."""
    c = case
    if c["kind"] in ("rewire", "group"):
        return None
    s = _inputs(c, seed)
    B, F_s, L, G, H = c["B"], c["F_s"], c["L"], c["G"], c["H"]
    X = s["X"].double()

    def grad(z, pos, first, n):
        rows, at = torch.arange(B, device=DEV)[:, None].expand_as(pos), pos.long() - first
        ok = (at >= 0) & (at < n)
        t = torch.zeros_like(z)
        t[rows[ok], at[ok]] = 1.0
        return torch.sigmoid(z) - t

    def step(w, g, m):
        m = MOMENTUM * m.double() + (g + DECAY * w)
        return m, w - LR * m

    Y = torch.empty((B, L), dtype=torch.float64, device=DEV)
    dY = torch.empty_like(Y) if c["kind"] != "predict" else None
    dW = torch.empty(s["W"].shape, dtype=torch.float64, device=DEV) if dY is not None else None
    dX = torch.zeros((B, F_s), dtype=torch.float64, device=DEV)
    for l0 in range(0, L, 32768):
        l1 = min(L, l0 + 32768)
        sup = s["idx"][torch.arange(l0, l1, device=DEV) // G].long()
        dense = torch.zeros((l1 - l0, F_s), dtype=torch.float64, device=DEV).scatter_(1, sup, s["W"][l0:l1].double())
        z = X @ dense.t()
        if s["bias"] is not None:
            z += s["bias"][l0:l1].double()
        Y[:, l0:l1] = z
        if dY is not None:
            d = grad(z, s["pos"], l0, l1 - l0)
            dY[:, l0:l1] = d
            dW[l0:l1] = (d.t() @ X).gather(1, sup)
            dX += d @ dense
    out = {"Y": Y, "dY": dY, "dW": dW, "dX": dX}
    if dY is not None and s["bias"] is not None:
        out["dbias"] = dY.sum(0)
    if H:
        Wh = s["W_h"].double()
        z = X @ Wh.t()
        if s["bias_h"] is not None:
            z += s["bias_h"].double()
        out["Y_h"] = z
        if dY is not None:
            out["dY_h"] = grad(z, s["pos_h"], 0, H)
            out["dW_h"] = out["dY_h"].t() @ X
            dX += out["dY_h"] @ Wh
    if c["kind"] == "sgd":
        out["m"], out["W_next"] = step(s["W"].double(), dW, s["m"])
        if H:
            out["m_h"], out["W_h_next"] = step(Wh, out["dW_h"], s["m_h"])
    names = {"predict": ("Y", "Y_h"), "calls": ("Y", "dY", "dW", "dbias", "dX"),
             "train": ("dY", "dW", "dbias", "dX", "dY_h", "dW_h"),
             "sgd": ("dY", "dbias", "m", "W_next", "dX", "dY_h", "dW_h", "m_h", "W_h_next")}[c["kind"]]
    return {k: out[k] for k in names if k in out}
