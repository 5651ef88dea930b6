"""Every tile of the bf16 products (COLA_OPT_TILE: 256 x 256, 128 x 128, 128 x 64,
64 x 64) at ragged edges: layers, the both-sigma variant, groups of up to eight
projections (whose products share launches four at a time) and the decoder block's
gated epilogues.  Left to itself the library gives shapes that the oracle can check
64 x 64 tiles mostly.  Against the fp64 oracle (1e-2) and the reference that applies
the storage policy (1e-3, as in the shape sweep); and since every kernel sums over k
in order, outputs that are not split have the same bits with every tile."""
import functools

import numpy as np
import pytest
import torch

import bench
import oracle
from paper_2502_10940_amd import cola
from paper_2502_10940_amd import inputs as I

from block_runner import BlockRun
from layer_runner import LayerRun, empty, NAN_BITS, relerr
from test_gpu_block import CASES as BLOCK_CASES
from test_gpu_group import GroupRun, check, group_inputs, oracle_group
from test_gpu_outer import OuterRun
from test_gpu_rounding import TOL as ROUNDED_TOL, rounded_layer

pytestmark = pytest.mark.gpu

TILES = {"256x256": 1, "128x128": 2, "128x64": 3, "64x64": 4}

# (T, d_in, d_out, r, padded): widths, tokens and K below, at and past the edges of
# 64, 128 and 256, whole and partial K tiles, one to several tiles
CASES = [(255, 136, 257, 129, True), (257, 392, 1000, 136, False), (513, 904, 640, 128, False),
         (1030, 520, 333, 200, True), (4099, 264, 392, 136, True), (6044, 300, 3000, 128, True)]


class tile:
    def __init__(self, value):
        self.value = value

    def __enter__(self):
        cola.set_option(cola.OPT_TILE, self.value)

    def __exit__(self, *_):
        cola.set_option(cola.OPT_TILE, 0)


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@functools.lru_cache(maxsize=1)
def _layer(case):
    T, d_in, d_out, r, _ = case
    ins = I.layer_inputs(2000 + T, 0, d_in, d_out, r, T, "bf16")
    X, A, B, dY = (ins[k].f64 for k in ("X", "A", "B", "dY"))
    Z, H, Y = oracle.cola_fwd(X, A, B, "silu")
    _, dX, dA, dB = oracle.cola_bwd(X, Z, A, B, dY, "silu")
    return ins, {"Z": Z, "H": H, "Y": Y, "dX": dX, "dA": dA, "dB": dB}, rounded_layer(X, A, B, dY, "silu")


def _kernels(fn):
    """Names of the GEMM kernels that fn launches."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    names = [e.name for e in p.events() if "gemm_" in e.name]
    if not names:
        pytest.skip("the profiler reports no kernels here")
    return names


@pytest.mark.parametrize("name", TILES)
def test_the_tile_asked_for_runs(name):
    ins = I.layer_inputs(2000, 0, 264, 392, 136, 300, "bf16")
    with tile(TILES[name]):
        run = LayerRun(ins, 300, 264, 392, 136, "bf16", "silu", False)
        names = _kernels(lambda: (run.forward(), run.backward()))
    part = "gemm_pp_" if name == "256x256" else "<" + name.replace("x", ", ") + ","
    assert all(part in n for n in names), names


# (T, d_in, d_out, r): kernels of the forward's products and of dZ, dX as chosen by
# size: 256 x 256 tiles on half the CUs stay unless another gains more than the
# model's error (K of 512 or more), else the tile that the model prefers
CHOSEN = [((32768, 1024, 1024, 256), {"fwd_z_sigma": "gemm_pp_", "bwd_dz": "gemm_pp_"}),
          ((32768, 2048, 2048, 512), {"fwd_z_sigma": "gemm_pp_", "fwd_y": "gemm_pp_", "bwd_dz": "gemm_pp_",
                                      "bwd_dx": "gemm_pp_"}),
          ((8192, 1024, 2736, 256), {"bwd_dx": "gemm_mid_"}),
          ((1024, 2048, 2048, 512), {"fwd_z_sigma": "gemm_mid_", "fwd_y": "gemm_mid_", "bwd_dz": "gemm_mid_"}),
          ((33, 2048, 2048, 512), {"fwd_z_sigma": "gemm_mid_", "fwd_y": "gemm_mid_"}),
          ((32, 2048, 2048, 512), {"fwd_z_sigma": "gemm_skinny_", "fwd_y": "gemm_skinny_"})]


@pytest.mark.parametrize("case", CHOSEN, ids=["T%d-%dx%d-r%d" % c[0] for c in CHOSEN])
def test_the_kernel_chosen_by_size(case):
    (T, d_in, d_out, r), want = case
    rows = lambda n, w: torch.zeros((n, w), dtype=torch.bfloat16, device="cuda:0")
    d = cola.desc(T, d_in, d_out, r)
    X, Y, Z, H, A, B = rows(T, d_in), rows(T, d_out), rows(T, r), rows(T, r), rows(r, d_in), rows(d_out, r)
    dA, dB = (torch.empty(s, device="cuda:0") for s in ((r, d_in), (d_out, r)))
    ws = torch.empty(max(1, cola.workspace_bytes(d, 1)), dtype=torch.uint8, device="cuda:0")

    def step():
        cola.fwd(d, X, A, B, Y, Z, H)
        cola.bwd(d, Y, X, Z, H, A, B, rows(T, d_in), dA, dB, ws)
    ran = {bench.gemm_class(n)[0]: n for n in _kernels(step)}
    for step_name, kernel in want.items():
        assert kernel in ran[step_name], (step_name, ran[step_name])


@pytest.mark.parametrize("name", TILES)
@pytest.mark.parametrize("case", CASES, ids=["T%d-%dx%d-r%d-%s" % (*c[:4], "pad" if c[4] else "tight") for c in CASES])
def test_layer(case, name):
    T, d_in, d_out, r, padded = case
    ins, ref, rounded = _layer(case)
    ld = [I.padded_ld(w, "bf16") if padded else w for w in (d_in, d_out, r)]
    raw = {}
    for t in (TILES[name], 0):
        with tile(t):
            run = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", False, *ld).run()
            got = run.outputs()
            assert run.padding_untouched()
            raw[t] = run.raw()
            Yi = empty(T, ld[1], "bf16", NAN_BITS["bf16"])
            cola.infer(run.desc, run.X, run.A, run.B, Yi,
                       torch.empty(cola.workspace_bytes(run.desc, 2), dtype=torch.uint8, device="cuda:0"))
            assert torch.equal(Yi[:, :d_out], run.Y[:, :d_out])
            m = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", True, *ld).run().raw()
            for k in m:
                assert np.array_equal(m[k], raw[t][k]), f"CoLA-M {k}"
        for k, g in got.items():
            assert np.all(np.isfinite(g)), k
            assert relerr(g, ref[k]) <= 1e-2, k
            assert relerr(g, rounded[k]) <= ROUNDED_TOL, k
    for k in ("Y", "Z", "dX"):
        assert np.array_equal(raw[TILES[name]][k], raw[0][k]), k


def test_outer():
    T, d_in, d_out, r = 700, 264, 333, 136
    ins = I.layer_inputs(2001, 0, d_in, d_out, r, T, "bf16")
    first = None
    for t in range(5):
        with tile(t):
            run = OuterRun(ins, T, d_in, d_out, r, "bf16", "silu", "gelu", False, ldy=384).run()
        got = dict(run.raw(), P=run.P[:, :d_out].contiguous().view(torch.int16).cpu().numpy())
        first = got if first is None else first
        for k in ("P", "Y", "Z", "dX"):
            assert np.array_equal(got[k], first[k]), (t, k)


RANKS = [136, 128, 144, 129, 200, 64, 136, 40]
WIDTHS = [264, 300, 136, 257, 130, 512, 129, 200]


@pytest.mark.parametrize("n", (2, 4, 5, 8))
def test_group(n):
    T, d_in, ranks, widths = 519, 264, RANKS[:n], WIDTHS[:n]
    X, As, Bs, dYs = group_inputs(95 + n, T, d_in, ranks, widths, "bf16")
    ref = oracle_group(X, As, Bs, dYs, "silu")
    first = None
    for t in range(5):
        with tile(t):
            for recompute in (False, True):
                run = GroupRun(X, As, Bs, dYs, T, d_in, ranks, widths, "bf16", "silu", recompute).run()
                got = run.results()
                check(got, {k: v for k, v in ref.items() if k in got}, "bf16", f"tile {t} recompute={recompute}")
                flat = {k: np.concatenate([g.ravel() for g in got[k]]) for k in ("Z", "Y", "dX", "dA", "dB")}
                if recompute:
                    for k in flat:
                        assert np.array_equal(flat[k], stored[k]), f"tile {t}: CoLA-M {k}"
                stored = flat
            first = flat if first is None else first
            for k in ("Z", "Y", "dX"):
                assert np.array_equal(flat[k], first[k]), f"tile {t}: {k}"
            Yi = [empty(T, w, "bf16", NAN_BITS["bf16"]) for w in widths]
            cola.group_infer(run.desc, run.X, run.A_all, run.B, Yi,
                             torch.empty(cola.group_workspace_bytes(run.desc, 2), dtype=torch.uint8, device="cuda:0"))
            torch.cuda.synchronize()
            for a, b in zip(Yi, run.Y):
                assert torch.equal(a, b), f"tile {t}: infer"


@pytest.mark.parametrize("n", (5, 8))
def test_group_fp32(n):
    T, d_in, ranks, widths = 131, 70, [9 + 3 * p for p in range(n)], [40 + 7 * p for p in range(n)]
    X, As, Bs, dYs = group_inputs(105 + n, T, d_in, ranks, widths, "f32")
    ref = oracle_group(X, As, Bs, dYs, "gelu")
    for recompute in (False, True):
        got = GroupRun(X, As, Bs, dYs, T, d_in, ranks, widths, "f32", "gelu", recompute).run().results()
        check(got, {k: v for k, v in ref.items() if k in got}, "f32", f"recompute={recompute}")


@pytest.mark.parametrize("recompute", (False, True), ids=["cola", "colam"])
@pytest.mark.parametrize("case", [BLOCK_CASES[1], BLOCK_CASES[3]], ids=[BLOCK_CASES[1][0], BLOCK_CASES[3][0]])
def test_gated_epilogues(case, recompute):
    """Fused and elementwise, with every tile: the same bits but for the token
    splits of the weight gradients, which are the tile's."""
    _, n_seq, L, d, ffn, heads, r, act = case
    ins = I.block_inputs(9, n_seq, L, d, ffn, r)
    first = None
    for t in range(5):
        raw = {}
        with tile(t):
            for fuse in (1, 0):
                cola.set_option(cola.OPT_FUSE_GATE, fuse)
                try:
                    raw[fuse] = BlockRun(ins, n_seq, L, d, ffn, heads, r, act, recompute).run().raw()
                finally:
                    cola.set_option(cola.OPT_FUSE_GATE, 1)
        for k in raw[1]:
            assert np.array_equal(raw[1][k], raw[0][k]), f"tile {t}: {k}"
        first = raw[1] if first is None else first
        for k in ("x2", "dx0"):
            assert np.array_equal(raw[1][k], first[k]), f"tile {t}: {k}"
        for k in raw[1]:
            if k not in ("x2", "dx0"):
                a, b = raw[1][k].view(np.float32), first[k].view(np.float32)
                assert relerr(a.astype(np.float64), b.astype(np.float64)) <= 1e-5, f"tile {t}: {k}"
