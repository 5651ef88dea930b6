"""bf16 token rows that do not start on 16-byte boundaries (odd pitches, odd
column offsets in a group): the path that copies them to aligned rows, and the
one taken when the workspace has no room for the copies (one byte less than
cola_workspace_bytes), against the fp64 oracle (1e-2) and, with the copies, bit
for bit the same layer on aligned rows (same kernels, same sums); and
cola_bwd_scratch where the copies alone exceed its static array."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_10940_amd import cola
from paper_2502_10940_amd import inputs as I

from layer_runner import DEV, LayerRun, relerr

pytestmark = pytest.mark.gpu

# (T, d_in, d_out, r): X, dY or H unaligned, alone and together
CASES = [(33, 1369, 512, 64), (300, 512, 1369, 64), (513, 264, 272, 129), (1030, 341, 333, 65)]


def _refs(ins, act="silu"):
    X, A, B, dY = (ins[k].f64 for k in ("X", "A", "B", "dY"))
    Z, H, Y = oracle.cola_fwd(X, A, B, act)
    _, dX, dA, dB = oracle.cola_bwd(X, Z, A, B, dY, act)
    return {"Z": Z, "H": H, "Y": Y, "dX": dX, "dA": dA, "dB": dB}


def _check(run, ins):
    got = run.outputs()
    for k, ref in _refs(ins).items():
        if k in got:
            assert np.all(np.isfinite(got[k])), k
            e = relerr(got[k], ref)
            assert e <= 1e-2, f"{k}: {e:.2e}"


@pytest.mark.parametrize("recompute", (False, True))
@pytest.mark.parametrize("case", range(len(CASES)), ids=["T%d-%dx%d-r%d" % c for c in CASES])
def test_tight_rows(case, recompute):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    T, d_in, d_out, r = CASES[case]
    ins = I.layer_inputs(1500 + case, 0, d_in, d_out, r, T, "bf16")
    tight = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", recompute).run()
    _check(tight, ins)
    pad = lambda w: I.padded_ld(w, "bf16")
    padded = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", recompute, ldx=pad(d_in), ldy=pad(d_out),
                      ldz=pad(r)).run()
    a, b = tight.raw(), padded.raw()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    # no room for the copies
    lean = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", recompute)
    d = lean.desc
    odd_h = not recompute and r % 8 != 0
    wf = cola.workspace_bytes(d, 0) - (1 if d_in % 8 or odd_h else 0)
    wb = cola.workspace_bytes(d, 1) - (1 if d_in % 8 or d_out % 8 else 0)   # a copy of H alone is less than the splits
    cola.fwd(d, lean.X, lean.A, lean.B, lean.Y, lean.Z, lean.H, lean.ws, ws_bytes=wf)
    cola.bwd(d, lean.dY, lean.X, lean.Z, lean.H, lean.A, lean.B, lean.dX, lean.dA, lean.dB, lean.ws, ws_bytes=wb)
    torch.cuda.synchronize()
    _check(lean, ins)


def test_group_of_odd_ranks():
    from test_gpu_group import GroupRun, check, group_inputs, oracle_group
    T, d_in, ranks, widths = 411, 133, [33, 65, 40], [200, 77, 129]
    X, As, Bs, dYs = group_inputs(90, T, d_in, ranks, widths, "bf16")
    ref = oracle_group(X, As, Bs, dYs, "silu")
    for recompute in (False, True):
        got = GroupRun(X, As, Bs, dYs, T, d_in, ranks, widths, "bf16", "silu", recompute).run().results()
        check(got, {k: v for k, v in ref.items() if k in got}, "bf16", f"odd ranks recompute={recompute}")


def test_scratch_backward_without_room_for_copies():
    # 40 MB of copies of X and dY beside 30 MB of dZ and partials
    T, d_in, d_out, r = 40000, 257, 255, 129
    ins = I.layer_inputs(1590, 0, d_in, d_out, r, T, "bf16")
    run = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", True)
    assert cola.workspace_bytes(run.desc, 1) > cola.SCRATCH_BYTES
    run.forward()
    cola.bwd_scratch(run.desc, run.dY, run.X, run.Z, None, run.A, run.B, run.dX, run.dA, run.dB)
    torch.cuda.synchronize()
    _check(run, ins)
