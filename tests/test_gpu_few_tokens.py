"""Forward products of a few tokens: token counts around the 16 / 32 row tiles of
the kernel for at most 32 and the 64 row tiles past it, K around 64-deep tiles,
odd and tight widths, one layer and groups, against the fp64
oracle (1e-2) and the storage-policy reference (1e-3, as in the shape sweep);
the inference forward's Y bit for bit the training forward's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_10940_amd import cola
from paper_2502_10940_amd import inputs as I

from layer_runner import DEV, LayerRun, empty, relerr, to_f64
from test_gpu_rounding import TOL as ROUNDED_TOL, rounded_layer

pytestmark = pytest.mark.gpu

TOKENS = (1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65)
# (d_in, d_out, r, padded rows)
SHAPES = [(2048, 512, 64, True), (65, 33, 9, False), (1369, 520, 65, False), (512, 1369, 1024, True)]


@pytest.mark.parametrize("act", ("silu", "gelu"))
@pytest.mark.parametrize("shape", range(len(SHAPES)), ids=["%dx%d-r%d-%s" % (*s[:3], "pad" if s[3] else "tight")
                                                           for s in SHAPES])
@pytest.mark.parametrize("T", TOKENS)
def test_few_tokens(T, shape, act):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d_in, d_out, r, padded = SHAPES[shape]
    ins = I.layer_inputs(1600 + 20 * shape, 0, d_in, d_out, r, T, "bf16")
    pitch = (lambda w: I.padded_ld(w, "bf16")) if padded else (lambda w: w)
    run = LayerRun(ins, T, d_in, d_out, r, "bf16", act, False, ldx=pitch(d_in), ldy=pitch(d_out), ldz=pitch(r))
    run.forward()
    torch.cuda.synchronize()
    got = {"Y": to_f64(run.Y, d_out), "Z": to_f64(run.Z, r), "H": to_f64(run.H, r)}
    X, A, B, dY = (ins[k].f64 for k in ("X", "A", "B", "dY"))
    ref = dict(zip(("Z", "H", "Y"), oracle.cola_fwd(X, A, B, act)))
    rounded = rounded_layer(X, A, B, dY, act)
    for k, g in got.items():
        assert np.all(np.isfinite(g)), k
        assert relerr(g, ref[k]) <= 1e-2, k
        assert relerr(g, rounded[k]) <= ROUNDED_TOL, k
    for t, w in ((run.Y, d_out), (run.Z, r), (run.H, r)):
        assert t.shape[1] == w or torch.isnan(t[:, w:].float()).all(), "pad columns written"
    # inference: alone, and as the second of a group whose first has another width
    Y = empty(T, pitch(d_out), "bf16")
    cola.infer(run.desc, run.X, run.A, run.B, Y,
               torch.empty(max(1, cola.workspace_bytes(run.desc, 2)), dtype=torch.uint8, device=DEV))
    gd = cola.group_desc(T, d_in, [3, r], [41, d_out], "bf16", act, ldx=pitch(d_in), ldy=[41, pitch(d_out)])
    A2 = torch.cat([torch.zeros((3, d_in), dtype=torch.bfloat16, device=DEV), run.A])
    B2 = [torch.ones((41, 3), dtype=torch.bfloat16, device=DEV), run.B]
    Y2 = [empty(T, 41, "bf16"), empty(T, pitch(d_out), "bf16")]
    cola.group_infer(gd, run.X, A2, B2, Y2,
                     torch.empty(max(1, cola.group_workspace_bytes(gd, 2)), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    assert torch.equal(Y[:, :d_out].view(torch.int16), run.Y[:, :d_out].view(torch.int16))
    assert relerr(to_f64(Y2[1], d_out), got["Y"]) <= ROUNDED_TOL
    assert not Y2[0].float().abs().max().item() > 0.0
