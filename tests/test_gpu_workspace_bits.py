"""The bits of a layer's results do not depend on how much workspace the caller
brings: with room for the aligned copies of unaligned rows, for some of them (one
byte less than cola_workspace_bytes) or none (the lean size), and in
cola_bwd_scratch's array; nor on whether H
was stored (CoLA) or is made again (CoLA-M) in any of them.  Bitwise: one plan of
the weight gradients' splits, and every kernel sums a split in order."""
import numpy as np
import pytest
import torch

from paper_2502_10940_amd import cola
from paper_2502_10940_amd import inputs as I

from layer_runner import LayerRun
from test_gpu_group import GroupRun, group_inputs
from test_gpu_outer import OuterRun

pytestmark = pytest.mark.gpu

# (T, d_in, d_out, r): rows of X, of dY and Y, of Z and H unaligned, alone and together
CASES = [(33, 1369, 512, 64), (700, 512, 1369, 64), (513, 264, 272, 129), (1030, 341, 333, 65),
         (4095, 1365, 512, 128), (5000, 1024, 1021, 256), (3000, 512, 512, 129)]


def _same(a, b, what):
    for k in b:
        if k in a:
            assert np.array_equal(a[k], b[k]), f"{what}: {k} differs in {(a[k] != b[k]).sum()} of {a[k].size} values"


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("case", CASES, ids=["T%d-%dx%d-r%d" % c for c in CASES])
@pytest.mark.parametrize("outer", (False, True), ids=["plain", "outer"])
def test_layer(case, outer):
    _gpu()
    T, d_in, d_out, r = case
    ins = I.layer_inputs(1800, 0, d_in, d_out, r, T, "bf16")
    first = None
    for recompute in (False, True):
        for lean in (0, 1, 2):
            if outer:
                run = OuterRun(ins, T, d_in, d_out, r, "bf16", "silu", "silu", recompute)
            else:
                run = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", recompute)
            wf, wb = cola.workspace_bytes(run.desc, 0), cola.workspace_bytes(run.desc, 3 if outer else 1)
            if lean == 2:
                wf = cola.workspace_bytes(run.desc, 0 + cola.WS_LEAN)
                wb = cola.workspace_bytes(run.desc, (3 if outer else 1) + cola.WS_LEAN)
            elif lean:
                # less by a byte wherever that only costs the copies
                wf -= 1 if d_in % 8 or (r % 8 and not recompute) else 0
                wb -= 1 if d_in % 8 or (d_out % 8 and not outer) or (r % 8 and not recompute) else 0
            ws = run.ws
            run.ws = ws[:wf]
            run.forward()
            run.ws = ws[:wb]
            run.backward()
            torch.cuda.synchronize()
            got = run.raw()
            first = got if first is None else first
            _same(got, first, f"recompute={recompute} lean={lean}")


def test_group():
    _gpu()
    T, d_in, ranks, widths = 1111, 133, [33, 65, 40], [200, 77, 129]
    X, As, Bs, dYs = group_inputs(91, T, d_in, ranks, widths, "bf16")
    first = None
    for recompute in (False, True):
        for lean in (0, 1, 2):
            run = GroupRun(X, As, Bs, dYs, T, d_in, ranks, widths, "bf16", "silu", recompute)
            if lean == 2:
                wf, wb = (cola.group_workspace_bytes(run.desc, p + cola.WS_LEAN) for p in (0, 1))
            else:
                wf, wb = (cola.group_workspace_bytes(run.desc, p) - lean for p in (0, 1))
            cola.group_fwd(run.desc, run.X, run.A_all, run.B, run.Y, run.Z, run.H, run.ws, ws_bytes=wf)
            cola.group_bwd(run.desc, run.dY, run.X, run.Z, run.H, run.A_all, run.B, run.dX, run.dA, run.dB, run.ws,
                           ws_bytes=wb)
            torch.cuda.synchronize()
            got = {"dX": run.dX, "dA": run.dA, "Z": run.Z[:, :run.R]}
            got.update({f"dB{p}": t for p, t in enumerate(run.dB)})
            got.update({f"Y{p}": t for p, t in enumerate(run.Y)})
            got = {k: t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32).cpu().numpy()
                   for k, t in got.items()}
            first = got if first is None else first
            _same(got, first, f"recompute={recompute} lean={lean}")


# 40 MB of copies beside 30 MB of dZ and partials; splits that just fit; fp32
SCRATCH = [(40000, 257, 255, 129, "bf16"), (9913, 824, 4848, 1016, "bf16"), (2000, 1365, 500, 127, "bf16"),
           (10522, 304, 7896, 16, "f32")]


@pytest.mark.parametrize("case", SCRATCH, ids=["T%d-%dx%d-r%d-%s" % c for c in SCRATCH])
def test_scratch(case):
    _gpu()
    T, d_in, d_out, r, dtype = case
    ins = I.layer_inputs(1801, 0, d_in, d_out, r, T, dtype)
    first = None
    for recompute in (False, True):
        run = LayerRun(ins, T, d_in, d_out, r, dtype, "silu", recompute).run()
        got = run.raw()
        first = got if first is None else first
        _same(got, first, f"cola_bwd recompute={recompute}")
        for t in (run.dX, run.dA, run.dB):
            t.fill_(float("nan"))
        try:
            cola.bwd_scratch(run.desc, run.dY, run.X, run.Z, run.H, run.A, run.B, run.dX, run.dA, run.dB)
        except cola.ColaError as e:
            # CoLA-M's H may be what exceeds the array
            assert recompute and e.status == cola.ERR_SCRATCH
            continue
        torch.cuda.synchronize()
        _same(run.raw(), first, f"scratch recompute={recompute}")
