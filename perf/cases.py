"""Workloads by which the speed of this library is measured.

A case is one call, or one training step, of the entry points in
``paper_2502_10940_amd.cola``, at sizes that programs built on them use:

  infer    ``infer`` / ``group_infer``: decode (a few tokens, where latency
           counts) and prefill (hundreds to thousands of tokens)
  layer    ``fwd`` then ``bwd`` of one projection, CoLA or CoLA-M, fp32 or bf16
  group    ``group_fwd`` then ``group_bwd``: projections that read one input
  outer    ``fwd_outer`` then ``bwd_outer``: the variant with a sigma on top
  block    ``block_fwd`` then ``block_bwd``: a LLaMA decoder block

Widths are those of the LLaMA shapes in ``paper_2502_10940_amd/inputs.py``
(512/1376, 1024/2736, 2048/5461, 4096/11008, rank a quarter of the width).
Rows are either tight or padded to whole 128-byte lines ("pad").  Inputs follow
the same file's recipe: X, dY ~ N(0, 1), A ~ N(0, 1/d_in), B ~ N(0, 1/r),
RMSNorm gains 1 + N(0, 0.1^2).
"""
import math

import torch

from paper_2502_10940_amd import cola

DEV = "cuda:0"
FFN = {512: 1376, 1024: 2736, 2048: 5461, 4096: 11008}


def _infer(T, d_in, d_out, r, n=1, act="silu", dtype="bf16", pad=True):
    return dict(kind="infer", T=T, d_in=d_in, d_out=d_out, r=r, n=n, act=act, dtype=dtype, pad=pad)


def _train(kind, T, d_in, d_out, r, n=1, act="silu", dtype="bf16", recompute=False, pad=True, outer="silu"):
    return dict(kind=kind, T=T, d_in=d_in, d_out=d_out, r=r, n=n, act=act, dtype=dtype, recompute=recompute, pad=pad,
                outer=outer)


def _block(n_seq, seq_len, d, ffn, heads, r, act="silu", recompute=False):
    return dict(kind="block", n_seq=n_seq, seq_len=seq_len, d=d, ffn=ffn, heads=heads, r=r, act=act,
                recompute=recompute)


def listed():
    cases = [
        # one token of one sequence through an attention projection of the 1B shape: serving latency
        ("decode_1b_one_token", _infer(1, 2048, 2048, 512)),
        # a batch of 32 sequences, one token each, through q, k and v of the 7B shape
        ("decode_7b_qkv_batch", _infer(32, 4096, 4096, 1024, n=3)),
        # a prompt of ordinary length through gate and up of the 1B shape (rows of 5461: odd, padded by the caller)
        ("prefill_1b_gate_up", _infer(1000, 2048, 5461, 512, n=2)),
        # the single layer in fp32 that small experiments and gradient checks train
        ("layer_fp32", _train("layer", 256, 512, 512, 128, dtype="f32")),
        # a fine-tuning micro-batch of the 1B shape: four sequences of 256 tokens
        ("layer_1b_small_batch", _train("layer", 1024, 2048, 2048, 512)),
        # the down projection on tight rows of 5461 bf16 values, an odd token count, GeLU: a caller who pads nothing
        ("layer_1b_down_tight_odd", _train("layer", 4095, 5461, 2048, 512, act="gelu", pad=False)),
        # pre-training layers at the full token batches: memory-bound rank 128, then the large ones
        ("layer_60m_gate", _train("layer", 65536, 512, 1376, 128)),
        ("group_350m_gate_up", _train("group", 32768, 1024, 2736, 256, n=2)),
        ("layer_7b_q_colam", _train("layer", 16384, 4096, 4096, 1024, recompute=True)),
        # the ablation's layer that keeps the original SiLU on top of gate
        ("outer_350m_gate", _train("outer", 8192, 1024, 2736, 256)),
        # whole decoder blocks: the 1B shape on sequences of 256, and heads of 128 on long sequences in CoLA-M
        ("block_1b", _block(128, 256, 2048, 5461, 32, 512)),
        ("block_7b_long_colam", _block(2, 2048, 4096, 11008, 32, 1024, recompute=True)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "f32", "layer", "layer", "group", "outer", "block"])
    d = rng.choice([512, 1024, 2048, 4096])
    ffn, r = FFN[d], d // 4
    act = rng.choice(["silu", "silu", "gelu", "identity"])
    pad = rng.random() < 0.7
    if rng.random() < 0.25:                                   # widths off the usual grid
        ffn, r = _log(rng, d, 2.75 * d), _log(rng, 16, d // 4)
    d_in, d_out = rng.choice([(d, d), (d, ffn), (ffn, d)])
    n = rng.choice([1, 2, 3])
    # at most the work of a 16384-token 7B attention projection
    top = min(65536, int(16384 * 1024 * 8192 / (r * (d_in + d_out))))
    if kind == "decode":
        return _infer(_log(rng, 1, 64), d_in, d_out, r, n, act, pad=pad)
    if kind == "prefill":
        return _infer(_log(rng, 100, 8192), d_in, d_out, r, n, act, pad=pad)
    if kind == "f32":
        w = [_log(rng, 64, 1024) for _ in range(2)]
        return _train("layer", _log(rng, 32, 2048), w[0], w[1], _log(rng, 16, 256), act=act, dtype="f32",
                      recompute=rng.random() < 0.5, pad=pad)
    if kind == "block":
        d = rng.choice([512, 1024, 2048])
        seq_len = _log(rng, 64, 2048)
        n_seq = max(1, _log(rng, 256, 65536 * 512 // d) // seq_len)
        return _block(n_seq, seq_len, d, FFN[d], d // rng.choice([64, 128]), d // 4, rng.choice(["silu", "gelu"]),
                      rng.random() < 0.5)
    T = _log(rng, 256, top)
    if kind == "group":
        T = max(1, T // n)
    return _train(kind, T, d_in, d_out, r, n if kind == "group" else 1, act, recompute=rng.random() < 0.5, pad=pad,
                  outer=rng.choice(["silu", "gelu"]))


# ---------------------------------------------------------------------------
# inputs and plans
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype, mean=0.0):
    x = torch.empty(shape, dtype=torch.float32, device=DEV).normal_(mean, std, generator=g)
    return x.to(dtype)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _ld(case, width):
    if not case["pad"]:
        return width
    per = 32 if case["dtype"] == "f32" else 64
    return -(-width // per) * per


def _rows(case, width, ld=None, src=None):
    """[T][width] with the case's pitch: the values of `src`, or room for an output."""
    ld = _ld(case, width) if ld is None else ld
    x = torch.zeros((case["T"], ld), dtype=_dtype(case), device=DEV)[:, :width]
    if src is not None:
        x.copy_(src)
    return x


def _layer_values(case, seed):
    """The seeded values of a layer's (or group's) inputs, before any layout."""
    g, dt = _gen(seed), _dtype(case)
    T, d_in, d_out, r, n = (case[k] for k in ("T", "d_in", "d_out", "r", "n"))
    v = {"X": _normal(g, (T, d_in), 1.0, dt), "A": _normal(g, (n * r, d_in), d_in ** -0.5, dt)}
    v["B"] = [_normal(g, (d_out, r), r ** -0.5, dt) for _ in range(n)]
    if case["kind"] != "infer":
        v["dY"] = [_normal(g, (T, d_out), 1.0, dt) for _ in range(n)]
    return v


def _block_values(case, seed):
    g, bf = _gen(seed), torch.bfloat16
    d, ffn, r = case["d"], case["ffn"], case["r"]
    T = case["n_seq"] * case["seq_len"]
    v = {"x0": _normal(g, (T, d), 1.0, bf), "dx2": _normal(g, (T, d), 1.0, bf)}
    shapes = {"g1": (d,), "g2": (d,), "A_qkv": (3 * r, d), "B_q": (d, r), "B_k": (d, r), "B_v": (d, r),
              "A_o": (r, d), "B_o": (d, r), "A_gu": (2 * r, d), "B_g": (ffn, r), "B_u": (ffn, r), "A_d": (r, ffn),
              "B_d": (d, r)}
    for name, shape in shapes.items():
        v[name] = (_normal(g, shape, 0.1, bf, mean=1.0) if len(shape) == 1 else
                   _normal(g, shape, shape[1] ** -0.5, bf))
    return v


def _ws(sizes):
    return torch.empty(max(1, *sizes), dtype=torch.uint8, device=DEV)


def _f32(shape):
    return torch.empty(shape, dtype=torch.float32, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "block":
        v = _block_values(case, seed)
        d = cola.block_desc(case["n_seq"], case["seq_len"], case["d"], case["ffn"], case["heads"], case["r"],
                            case["act"], case["recompute"])
        w = {k: v[k] for k in cola.BLOCK_PARAMS}
        return dict(kind=kind, d=d, w=w, x0=v["x0"], dx2=v["dx2"], x2=torch.empty_like(v["x0"]),
                    dx0=torch.empty_like(v["x0"]), grads={k: _f32(t.shape) for k, t in w.items()},
                    saved=_ws([cola.block_saved_bytes(d)]), ws=_ws([cola.block_workspace_bytes(d, p) for p in (0, 1)]))

    v = _layer_values(case, seed)
    T, d_in, d_out, r, n = (case[k] for k in ("T", "d_in", "d_out", "r", "n"))
    recompute = case.get("recompute", False)
    ldx, ldy, ldz = _ld(case, d_in), _ld(case, d_out), _ld(case, n * r)
    grouped = kind == "group" or (kind == "infer" and n > 1)
    s = dict(kind=kind, grouped=grouped, X=_rows(case, d_in, src=v["X"]), A=v["A"], B=v["B"],
             Y=[_rows(case, d_out) for _ in range(n)])
    if grouped:
        s["d"] = d = cola.group_desc(T, d_in, [r] * n, [d_out] * n, case["dtype"], case["act"], recompute, ldx, ldz,
                                     [ldy] * n)
        size, phases = cola.group_workspace_bytes, (2,) if kind == "infer" else (0, 1)
    else:
        s["d"] = d = cola.desc(T, d_in, d_out, r, case["dtype"], case["act"], recompute, ldx, ldy, ldz)
        size, phases = cola.workspace_bytes, {"infer": (2,), "layer": (0, 1), "outer": (0, 3)}[kind]
    s["ws"] = _ws([size(d, p) for p in phases])
    if kind != "infer":
        s.update(Z=_rows(case, n * r), H=None if recompute else _rows(case, n * r), dX=_rows(case, d_in),
                 dY=[_rows(case, d_out, src=y) for y in v["dY"]], dA=_f32((n * r, d_in)),
                 dB=[_f32((d_out, r)) for _ in range(n)])
    if kind == "outer":
        s.update(P=_rows(case, d_out), outer=case["outer"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "block":
        cola.block_fwd(s["d"], s["w"], s["x0"], s["x2"], s["saved"], s["ws"])
        cola.block_bwd(s["d"], s["w"], s["x0"], s["saved"], s["dx2"], s["dx0"], s["grads"], s["ws"])
        return {"x2": s["x2"], "dx0": s["dx0"], "grads": s["grads"]}
    d, X, A, B, Y, ws = (s[k] for k in ("d", "X", "A", "B", "Y", "ws"))
    if kind == "infer":
        if s["grouped"]:
            cola.group_infer(d, X, A, B, Y, ws)
        else:
            cola.infer(d, X, A, B[0], Y[0], ws)
        return {"Y": Y}
    Z, H, dY, dX, dA, dB = (s[k] for k in ("Z", "H", "dY", "dX", "dA", "dB"))
    out = {"Y": Y, "Z": Z, "dX": dX, "dA": dA, "dB": dB}
    if H is not None:
        out["H"] = H
    if kind == "group":
        cola.group_fwd(d, X, A, B, Y, Z, H, ws)
        cola.group_bwd(d, dY, X, Z, H, A, B, dX, dA, dB, ws)
    elif kind == "outer":
        cola.fwd_outer(d, s["outer"], X, A, B[0], Y[0], s["P"], Z, H, ws)
        cola.bwd_outer(d, s["outer"], dY[0], s["P"], X, Z, H, A, B[0], dX, dA, dB[0], ws)
        out["P"] = s["P"]
    else:
        cola.fwd(d, X, A, B[0], Y[0], Z, H, ws)
        cola.bwd(d, dY[0], X, Z, H, A, B[0], dX, dA, dB[0], ws)
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what its results are held to
# ---------------------------------------------------------------------------

def work(case):
    if case["kind"] == "block":
        d, ffn, r, L = case["d"], case["ffn"], case["r"], case["seq_len"]
        T = case["n_seq"] * L
        weights = 2 * d + 8 * d * r + 3 * (d * r + r * ffn)
        # forward and backward: the input and output of each, the weights, their fp32 gradients; x1 and the
        # pre-activations Z at least cross from one call to the other
        byts = 2 * (4 * T * d + weights) + 4 * weights + 2 * 2 * (T * d + 7 * T * r)
        proj = 6 * T * r * (4 * 2 * d + 3 * (d + ffn))
        attn = 3 * 4 * T * (L + 1) // 2 * d
        return {"bytes": byts, "flops": proj + attn}
    T, d_in, d_out, r, n = (case[k] for k in ("T", "d_in", "d_out", "r", "n"))
    es = 4 if case["dtype"] == "f32" else 2
    weights = n * r * (d_in + d_out)
    fwd = 2 * T * weights
    if case["kind"] == "infer":
        return {"bytes": es * (T * d_in + weights + n * T * d_out), "flops": fwd}
    rows = 2 * T * d_in + 2 * n * T * d_out + n * T * r
    if not case["recompute"]:
        rows += n * T * r
    if case["kind"] == "outer":
        rows += T * d_out
    return {"bytes": es * (rows + weights) + 4 * weights, "flops": 3 * fwd}


def tolerance(case):
    if case["kind"] == "block":
        # bf16 tensors between a block's kernels: up to 8e-3 from 64 bits
        return {"rel": 3e-2}
    if case["dtype"] == "f32":
        return {"rel": 3e-6}                                    # up to 5e-7 from 64 bits
    # Z, H, dZ (and P, dP) rounded to bf16 between the products: 2e-3 to 4e-3 from 64 bits
    return {"rel": 1.2e-2}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def _sigma(name, z):
    if name == "silu":
        return z * torch.sigmoid(z)
    if name == "gelu":
        return 0.5 * z * (1.0 + torch.erf(z * 0.5 ** 0.5))
    return z


def _sigma_prime(name, z):
    if name == "silu":
        s = torch.sigmoid(z)
        return s * (1.0 + z * (1.0 - s))
    if name == "gelu":
        return 0.5 * (1.0 + torch.erf(z * 0.5 ** 0.5)) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)
    return torch.ones_like(z)


def _exact_layer(case, seed):
    v = _layer_values(case, seed)
    act, r, n, kind = case["act"], case["r"], case["n"], case["kind"]
    X, A = v["X"].double(), v["A"].double()
    Z = X @ A.T
    H = _sigma(act, Z)
    cols = [slice(p * r, (p + 1) * r) for p in range(n)]
    B = [b.double() for b in v["B"]]
    Y = [H[:, c] @ b.T for c, b in zip(cols, B)]
    if kind == "infer":
        return {"Y": Y}
    dY = [y.double() for y in v["dY"]]
    out = {"Y": Y, "Z": Z}
    if kind == "outer":
        out["P"] = Y[0]
        out["Y"] = [_sigma(case["outer"], Y[0])]
        dY = [dY[0] * _sigma_prime(case["outer"], Y[0])]
    dZ = torch.cat([y @ b for y, b in zip(dY, B)], 1) * _sigma_prime(act, Z)
    out.update(dX=dZ @ A, dA=dZ.T @ X, dB=[y.T @ H[:, c] for y, c in zip(dY, cols)])
    if not case["recompute"]:
        out["H"] = H
    return out


def _exact_block(case, seed):
    d, ffn, r, heads, L, act = (case[k] for k in ("d", "ffn", "r", "heads", "seq_len", "act"))
    hd, n_seq = d // heads, case["n_seq"]
    v = {k: t.double().requires_grad_(k != "dx2") for k, t in _block_values(case, seed).items()}
    pos = torch.arange(L, device=DEV, dtype=torch.float64)
    freq = 10000.0 ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)
    cos, sin = torch.cos(pos[:, None] * freq), torch.sin(pos[:, None] * freq)

    def norm(x, gain):
        return x * torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-6) * gain

    def proj(x, A, B):
        return _sigma(act, x @ A.T) @ B.T

    def split(x):
        return x.view(n_seq, L, heads, hd).transpose(1, 2).contiguous()

    def rope(x):
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    a = norm(v["x0"], v["g1"])
    q, k, u = (split(proj(a, v["A_qkv"][i * r:(i + 1) * r], v[name])) for i, name in enumerate(("B_q", "B_k", "B_v")))
    q, k = rope(q), rope(k)
    mask = torch.ones((L, L), dtype=torch.bool, device=DEV).triu(1)
    p = torch.softmax((q @ k.transpose(-1, -2).contiguous() / math.sqrt(hd)).masked_fill(mask, -math.inf), -1)
    att = (p @ u).transpose(1, 2).reshape(n_seq * L, d)
    x1 = v["x0"] + proj(att, v["A_o"], v["B_o"])
    b = norm(x1, v["g2"])
    m = proj(b, v["A_gu"][:r], v["B_g"]) * proj(b, v["A_gu"][r:], v["B_u"])
    x2 = x1 + proj(m, v["A_d"], v["B_d"])
    names = ["x0"] + list(cola.BLOCK_PARAMS)
    grads = dict(zip(names, torch.autograd.grad(x2, [v[k] for k in names], v["dx2"])))
    return {"x2": x2.detach(), "dx0": grads.pop("x0"), "grads": grads}


def exact(case, seed):
    return _exact_block(case, seed) if case["kind"] == "block" else _exact_layer(case, seed)
