"""Layers whose products run on the small tiles, as the library chooses them (64 x 64,
for some 128 x 64; test_gpu_tiles.py asks for each tile): token counts and widths one below, at and one above tile edges, K of one
partial tile up to more K tiles than LDS slots, and splits of the weight
gradients, against the fp64 oracle (1e-2) and the reference that applies the
path's bf16 storage policy (1e-3, as in the shape sweep)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_10940_amd import inputs as I

from layer_runner import LayerRun, relerr
from test_gpu_rounding import TOL as ROUNDED_TOL, rounded_layer

pytestmark = pytest.mark.gpu

# (T, d_in, d_out, r, padded rows)
CASES = [
    (65, 64, 72, 24, True), (127, 200, 129, 65, True), (129, 320, 64, 128, False), (255, 1096, 264, 63, True),
    (256, 512, 512, 128, False), (257, 136, 1000, 129, True), (511, 904, 640, 72, False), (1030, 264, 1096, 136, True),
    (1030, 520, 333, 136, False), (4099, 136, 136, 24, True), (4096, 128, 256, 64, False),
]


@pytest.mark.parametrize("recompute", (False, True))
@pytest.mark.parametrize("case", range(len(CASES)), ids=["T%d-%dx%d-r%d-%s" % (*c[:4], "pad" if c[4] else "tight")
                                                         for c in CASES])
def test_small_tiles(case, recompute):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    T, d_in, d_out, r, padded = CASES[case]
    ins = I.layer_inputs(1300 + case, 0, d_in, d_out, r, T, "bf16")
    pitch = (lambda w: I.padded_ld(w, "bf16")) if padded else (lambda w: w)
    run = LayerRun(ins, T, d_in, d_out, r, "bf16", "silu", recompute, ldx=pitch(d_in), ldy=pitch(d_out),
                   ldz=pitch(r)).run()
    got = run.outputs()
    assert run.padding_untouched()
    X, A, B, dY = (ins[k].f64 for k in ("X", "A", "B", "dY"))
    Z, H, Y = oracle.cola_fwd(X, A, B, "silu")
    _, dX, dA, dB = oracle.cola_bwd(X, Z, A, B, dY, "silu")
    ref = {"Z": Z, "H": H, "Y": Y, "dX": dX, "dA": dA, "dB": dB}
    rounded = rounded_layer(X, A, B, dY, "silu")
    for k, g in got.items():
        assert np.all(np.isfinite(g)), k
        assert relerr(g, ref[k]) <= 1e-2, k
        assert relerr(g, rounded[k]) <= ROUNDED_TOL, k
