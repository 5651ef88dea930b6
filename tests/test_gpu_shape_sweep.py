"""Seeded sweeps of shapes around the kernels' decision points: single
layers, grouped projections and the dense layer.

Each of T, d_in, d_out and r is drawn from one of three bands -- below one
32-wide MFMA tile, around the 128 / 256 tile edges (where the
ragged-edge paths start; at these sizes the launcher takes the small tiles,
test_gpu_tiles.py asks for the others), and several tiles wide -- together with the storage
dtype, the activation, CoLA or CoLA-M, and tight or cache-line row pitches
(tight pitches with odd widths take the guarded, unaligned paths).  Every
draw runs forward and backward through the C ABI (and the inference
forward, whose Y must be the training forward's bit for bit, and the other
of CoLA / CoLA-M, whose outputs must be the same bits) and is compared
with the fp64 oracle (1e-2 bf16, 1e-5 fp32); bf16 draws are also held to the
reference that applies the path's bf16 storage policy (1e-3, Z and H equal
bit for bit except for the rare element next to a rounding boundary).  Pad
columns must keep their NaN fill.  The draws are fixed by the seed, so a
failure names a reproducible shape."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_10940_amd import cola
from paper_2502_10940_amd import inputs as I

from layer_runner import LayerRun, relerr
from test_gpu_rounding import TOL as ROUNDED_TOL, rounded_layer

SEED = 25021094
N_DRAWS = 96
# oracle cost bound: T r (d_in + d_out) multiply-adds per GEMM pass
MAX_WORK = 3.0e8
TOL = {"f32": 1e-5, "bf16": 1e-2}
EDGES = (32, 64, 127, 128, 129, 255, 256, 257)


def _dim(rng, lo_band, hi_band):
    band = int(rng.integers(0, 3))
    if band == 0:
        return int(rng.integers(1, 41))
    if band == 1:
        return max(1, int(EDGES[int(rng.integers(0, len(EDGES)))] + rng.integers(-1, 2)))
    return int(rng.integers(lo_band, hi_band + 1))


def draws(seed=SEED, n=N_DRAWS):
    """The sweep's cases: (T, d_in, d_out, r, dtype, act, recompute, padded)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    while len(out) < n:
        T = _dim(rng, 300, 3000)
        d_in = _dim(rng, 300, 1500)
        d_out = _dim(rng, 300, 1500)
        r = _dim(rng, 260, 520)
        if T * r * (d_in + d_out) > MAX_WORK:
            continue
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        act = ("silu", "gelu", "identity")[int(rng.choice(3, p=[0.6, 0.25, 0.15]))]
        out.append((T, d_in, d_out, r, dtype, act, bool(rng.random() < 0.5), bool(rng.random() < 0.5)))
    return out


CASES = draws()


def _id(c):
    T, d_in, d_out, r, dtype, act, rec, padded = c
    return f"T{T}-{d_in}x{d_out}-r{r}-{dtype}-{act}-{'colam' if rec else 'cola'}-{'pad' if padded else 'tight'}"


def test_draws_cover_the_bands():
    """The sweep is what it claims (no GPU): deterministic, within the oracle
    budget, and reaching both sides of the family switch (an output
    dimension of at most 128 against both above 128), ragged and exact tile
    edges, both dtypes, every activation, both modes and both pitch kinds."""
    assert draws() == CASES
    assert all(T * r * (di + do) <= MAX_WORK for T, di, do, r, *_ in CASES)
    dims = [d for T, di, do, r, *_ in CASES for d in (T, di, do, r)]
    assert min(dims) >= 1
    assert any(d <= 40 for d in dims) and any(d > 300 for d in dims)
    assert any(d % 256 == 0 for d in dims) and any(d % 128 == 0 and d % 256 for d in dims)
    assert any(d % 32 for d in dims)
    # K1 / K3 outputs are T x r, K2 / K4 outputs T x d_out / T x d_in
    assert any(c[3] <= 128 for c in CASES)
    assert any(T > 128 and r > 128 for T, _, _, r, *_ in CASES)
    assert any(T > 128 and do > 128 for T, _, do, *_ in CASES)
    assert {c[4] for c in CASES} == {"bf16", "f32"}
    assert {c[5] for c in CASES} == {"silu", "gelu", "identity"}
    assert {c[6] for c in CASES} == {False, True}
    assert {c[7] for c in CASES} == {False, True}


@pytest.fixture(scope="module")
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cola.lib()
    yield


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)), ids=[_id(c) for c in CASES])
def test_shape_sweep(case, _device):
    T, d_in, d_out, r, dtype, act, recompute, padded = CASES[case]
    print(f"\n[sweep] case {case}: {_id(CASES[case])}", flush=True)
    ins = I.layer_inputs(500 + case, 0, d_in, d_out, r, T, dtype)
    pitch = (lambda w: I.padded_ld(w, dtype)) if padded else (lambda w: w)
    run = LayerRun(ins, T, d_in, d_out, r, dtype, act, recompute,
                   ldx=pitch(d_in), ldy=pitch(d_out), ldz=pitch(r)).run()
    got = run.outputs()
    assert run.padding_untouched()
    # the inference forward (K1 keeps only H) gives the training forward's Y bit for bit
    from layer_runner import DEV, NAN_BITS, empty
    di = cola.desc(T, d_in, d_out, r, dtype, act, False, pitch(d_in), pitch(d_out), pitch(r))
    Yi = empty(T, pitch(d_out), dtype, NAN_BITS[dtype])
    cola.infer(di, run.X, run.A, run.B, Yi,
               torch.empty(max(1, cola.workspace_bytes(di, 2)), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    bits = (lambda t: t.view(torch.int16)) if dtype == "bf16" else (lambda t: t.view(torch.int32))
    assert torch.equal(bits(Yi[:, :d_out].contiguous()), bits(run.Y[:, :d_out].contiguous())), "inference Y"
    if pitch(d_out) > d_out:
        assert torch.isnan(Yi[:, d_out:].float()).all(), "inference wrote pad columns"
    # the other mode (CoLA-M recomputes H) gives the same bits
    other_run = LayerRun(ins, T, d_in, d_out, r, dtype, act, not recompute,
                         ldx=pitch(d_in), ldy=pitch(d_out), ldz=pitch(r)).run()
    other, mine = other_run.raw(), run.raw()
    for k in mine:
        assert np.array_equal(mine[k], other[k]), f"{k}: CoLA and CoLA-M differ"

    X, A, B, dY = (ins[k].f64 for k in ("X", "A", "B", "dY"))
    Z, H, Y = oracle.cola_fwd(X, A, B, act)
    _, dX, dA, dB = oracle.cola_bwd(X, Z, A, B, dY, act)
    ref = {"Z": Z, "H": H, "Y": Y, "dX": dX, "dA": dA, "dB": dB}
    for k, g in got.items():
        assert np.all(np.isfinite(g)), f"{k}: non-finite values"
        e = relerr(g, ref[k])
        assert e <= TOL[dtype], f"{k}: {e:.3e} against the oracle"

    if dtype == "bf16":
        rr = rounded_layer(X, A, B, dY, act)
        for k, g in got.items():
            e = relerr(g, rr[k])
            assert e <= ROUNDED_TOL, f"{k}: {e:.3e} against the storage-policy reference"
            if k in ("Z", "H"):
                differ = int(np.sum(g != rr[k]))
                assert differ <= 2 + 0.001 * g.size, f"{k}: {differ} of {g.size} elements differ"


# ---- grouped projections (one X, several CoLA layers) and the dense layer ----

def group_draws(seed=SEED + 1, n=24):
    """(T, d_in, ranks, widths, dtype, act) with 1-4 projections."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    while len(out) < n:
        T = _dim(rng, 300, 2000)
        d_in = _dim(rng, 300, 1200)
        k = int(rng.integers(1, 5))
        ranks = [_dim(rng, 260, 400) for _ in range(k)]
        widths = [_dim(rng, 300, 1200) for _ in range(k)]
        if sum(T * r * (d_in + w) for r, w in zip(ranks, widths)) > MAX_WORK:
            continue
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        act = ("silu", "gelu", "identity")[int(rng.choice(3, p=[0.6, 0.25, 0.15]))]
        out.append((T, d_in, ranks, widths, dtype, act, bool(rng.random() < 0.5)))
    return out


def dense_draws(seed=SEED + 2, n=24):
    """(T, d_in, d_out, dtype, padded)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    while len(out) < n:
        T, d_in, d_out = _dim(rng, 300, 3000), _dim(rng, 300, 1500), _dim(rng, 300, 1500)
        if T * d_in * d_out > MAX_WORK:
            continue
        out.append((T, d_in, d_out, "f32" if rng.random() < 0.2 else "bf16", bool(rng.random() < 0.5)))
    return out


GROUP_CASES = group_draws()
DENSE_CASES = dense_draws()


def test_group_and_dense_draws():
    """Deterministic, within budget, and reaching one to four projections
    (one to the limit of eight the ABI takes) and both dtypes (no GPU)."""
    assert group_draws() == GROUP_CASES and dense_draws() == DENSE_CASES
    assert {len(c[2]) for c in GROUP_CASES} == {1, 2, 3, 4}
    assert {c[4] for c in GROUP_CASES} == {"bf16", "f32"} and {c[3] for c in DENSE_CASES} == {"bf16", "f32"}
    assert {c[4] for c in DENSE_CASES} == {False, True}
    assert all(T * di * do <= MAX_WORK for T, di, do, *_ in DENSE_CASES)


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(GROUP_CASES)),
                         ids=[f"T{c[0]}-in{c[1]}-r{'_'.join(map(str, c[2]))}-out{'_'.join(map(str, c[3]))}-{c[4]}"
                              f"-{c[5]}-{'colam' if c[6] else 'cola'}" for c in GROUP_CASES])
def test_group_shape_sweep(case, _device):
    from test_gpu_group import GroupRun, group_inputs, oracle_group
    T, d_in, ranks, widths, dtype, act, recompute = GROUP_CASES[case]
    print(f"\n[group sweep] case {case}: T={T} d_in={d_in} r={ranks} d_out={widths} {dtype} {act} "
          f"recompute={recompute}", flush=True)
    X, As, Bs, dYs = group_inputs(600 + case, T, d_in, ranks, widths, dtype)
    ref = oracle_group(X, As, Bs, dYs, act)
    got = GroupRun(X, As, Bs, dYs, T, d_in, ranks, widths, dtype, act, recompute).run().results()
    for k, g in got.items():
        gl = g if isinstance(g, list) else [g]
        rl = ref[k] if isinstance(ref[k], list) else [ref[k]]
        for p, (gp, rp) in enumerate(zip(gl, rl)):
            assert np.all(np.isfinite(gp)), f"{k}[{p}]: non-finite values"
            e = relerr(gp, rp)
            assert e <= TOL[dtype], f"{k}[{p}]: {e:.3e} against the oracle"


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(DENSE_CASES)),
                         ids=[f"T{c[0]}-{c[1]}x{c[2]}-{c[3]}-{'pad' if c[4] else 'tight'}" for c in DENSE_CASES])
def test_dense_shape_sweep(case, _device):
    from layer_runner import NAN_BITS, empty, to_device
    T, d_in, d_out, dtype, padded = DENSE_CASES[case]
    print(f"\n[dense sweep] case {case}: T={T} {d_in}->{d_out} {dtype} padded={padded}", flush=True)
    ins = I.layer_inputs(700 + case, 0, d_in, d_out, 1, T, dtype, with_dense=True)
    ldx = I.padded_ld(d_in, dtype) if padded else d_in
    ldy = I.padded_ld(d_out, dtype) if padded else d_out
    d = cola.dense_desc(T, d_in, d_out, dtype, ldx, ldy)
    Xd = to_device(ins["X"].store, dtype, ldx)
    Wd = to_device(ins["W"].store, dtype)
    dYd = to_device(ins["dY"].store, dtype, ldy)
    Y = empty(T, ldy, dtype, NAN_BITS[dtype])
    dX = empty(T, ldx, dtype, NAN_BITS[dtype])
    dW = torch.full((d_out, d_in), float("nan"), dtype=torch.float32, device=Xd.device)
    ws = torch.empty(max(1, cola.dense_workspace_bytes(d, 0), cola.dense_workspace_bytes(d, 1)),
                     dtype=torch.uint8, device=Xd.device)
    cola.dense_fwd(d, Xd, Wd, Y, ws)
    cola.dense_bwd(d, dYd, Xd, Wd, dX, dW, ws)
    torch.cuda.synchronize()
    for t, w in ((Y, d_out), (dX, d_in)):
        if t.shape[1] > w:
            assert torch.isnan(t[:, w:].float()).all(), "pad columns written"
    X, W, dY = ins["X"].f64, ins["W"].f64, ins["dY"].f64
    ref_Y = oracle.dense_fwd(X, W)
    ref_dX, ref_dW = oracle.dense_bwd(X, W, dY)
    for name, g, ref in (("Y", Y[:, :d_out], ref_Y), ("dX", dX[:, :d_in], ref_dX), ("dW", dW, ref_dW)):
        a = g.double().cpu().numpy()
        assert np.all(np.isfinite(a)), f"{name}: non-finite values"
        e = relerr(a, ref)
        assert e <= TOL[dtype], f"{name}: {e:.3e} against the oracle"


# ---- the decoder block ----

def block_draws(seed=SEED + 3, n=32):
    """(n_seq, L, d, ffn, heads, r, act, recompute): head size 64 or 128,
    sequence lengths from three bands (short, across the 64 / 128 attention
    tiles, beyond what the whole-sequence attention kernels hold)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    while len(out) < n:
        hd = (64, 128)[int(rng.integers(0, 2))]
        heads = int(rng.integers(1, 5))
        d = hd * heads
        band = int(rng.integers(0, 3))
        L = (int(rng.integers(1, 41)), int(rng.integers(56, 141)), int(rng.integers(250, 321)))[band]
        n_seq = int(rng.integers(1, 4))
        ffn = int(rng.integers(16, 101)) if rng.random() < 0.5 else int(rng.integers(200, 601))
        # the block takes ranks that are multiples of 8
        r = 8 * (int(rng.integers(1, 6)) if rng.random() < 0.5 else int(rng.integers(12, 19)))
        T = n_seq * L
        if T * (14 * r * d + 2 * r * (d + ffn)) + n_seq * heads * L * L * hd > MAX_WORK:
            continue
        act = "gelu" if rng.random() < 0.25 else "silu"
        out.append((n_seq, L, d, ffn, heads, r, act, bool(rng.random() < 0.5)))
    return out


BLOCK_CASES = block_draws()
# The storage policy alone puts the block up to about 1e-2 from the fp64
# oracle (tests/test_block_rounding.py computes that on the CPU for the worst
# draw here); two valid bf16 evaluations of the block, the path and the
# storage-policy reference, differ by rounding flips that cascade through the
# chain of stored tensors (observed up to 5.1e-3 over these draws).
BLOCK_TOL = 2e-2
BLOCK_ROUNDED_TOL = 7.5e-3


def test_block_draws():
    """Deterministic, both head sizes, every sequence-length band (the long
    one at both head sizes), both activations and both modes (no GPU)."""
    assert block_draws() == BLOCK_CASES
    assert all(c[5] % 8 == 0 for c in BLOCK_CASES)
    hd = lambda c: c[2] // c[4]
    assert {hd(c) for c in BLOCK_CASES} == {64, 128}
    assert any(c[1] <= 40 for c in BLOCK_CASES) and any(56 <= c[1] <= 140 for c in BLOCK_CASES)
    assert {hd(c) for c in BLOCK_CASES if c[1] >= 250} == {64, 128}
    assert {c[6] for c in BLOCK_CASES} == {"silu", "gelu"} and {c[7] for c in BLOCK_CASES} == {False, True}


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(BLOCK_CASES)),
                         ids=[f"seq{c[0]}x{c[1]}-d{c[2]}-ffn{c[3]}-h{c[4]}-r{c[5]}-{c[6]}-{'colam' if c[7] else 'cola'}"
                              for c in BLOCK_CASES])
def test_block_shape_sweep(case, _device):
    from oracle import block as OB
    from block_runner import BlockRun
    from block_rounding import rounded_block
    from test_gpu_rounding import round_bf16
    n_seq, L, d, ffn, heads, r, act, recompute = BLOCK_CASES[case]
    print(f"\n[block sweep] case {case}: n_seq={n_seq} L={L} d={d} ffn={ffn} heads={heads} r={r} {act} "
          f"recompute={recompute}", flush=True)
    ins = I.block_inputs(60 + case, n_seq, L, d, ffn, r)
    got = BlockRun(ins, n_seq, L, d, ffn, heads, r, act, recompute).run().results()
    c = OB.Cfg(n_seq, L, d, ffn, heads, r, act=act)
    p = {k: v.f64 for k, v in ins.items()}
    x2, saved = OB.block_forward(c, p, p["x0"], recompute)
    dx0, g = OB.block_backward(c, p, p["x0"], saved, p["dx2"], recompute)
    ref = {"x2": x2, "dx0": dx0, **{"d" + k: v for k, v in g.items()}}
    rx2, rdx0, rg = rounded_block(c, p, p["x0"], p["dx2"], round_bf16)
    rr = {"x2": rx2, "dx0": rdx0, **{"d" + k: v for k, v in rg.items()}}
    errs = {k: (relerr(got[k], rv), relerr(got[k], rr[k])) for k, rv in ref.items() if rv.any()}
    print("oracle: " + " ".join(f"{k}={e[0]:.2e}" for k, e in sorted(errs.items(), key=lambda kv: -kv[1][0])[:4]),
          flush=True)
    print("rounded: " + " ".join(f"{k}={e[1]:.2e}" for k, e in sorted(errs.items(), key=lambda kv: -kv[1][1])[:4]),
          flush=True)
    for k, rv in ref.items():
        assert np.isfinite(got[k]).all(), f"{k}: non-finite values"
        if not rv.any():
            # zero by the method's structure: one-token sequences give q and k
            # no gradient (constant softmax); the kernels leave rounding noise
            assert L == 1 and k in ("dB_q", "dB_k"), k
            assert np.linalg.norm(got[k]) <= 1e-4 * np.linalg.norm(got["dB_v"]), k
            continue
        e_oracle, e_rounded = errs[k]
        assert e_oracle <= BLOCK_TOL, f"{k}: {e_oracle:.3e} against the block oracle"
        assert e_rounded <= BLOCK_ROUNDED_TOL, f"{k}: {e_rounded:.3e} against the storage-policy reference"
