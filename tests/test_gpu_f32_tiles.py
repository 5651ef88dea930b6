"""fp32 layers around the edges of the fp32 kernel's tiles: K below, at and one
past a 32-deep K tile and past the eight K tiles its waves share, ragged rows and
columns at any alignment, outputs on both sides of the switch from 32 x 32 to
64 x 64 tiles (256 of the latter), and split weight gradients.  Against the fp64
oracle: a dot product of n fp32 terms summed in any order is within n 2^-24 of
the sum of its terms' magnitudes; random signs leave about sqrt(n) of that, so
1e-6 covers every K here (up to 9001) with room."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_10940_amd import inputs as I

from layer_runner import LayerRun, relerr

pytestmark = pytest.mark.gpu

# (T, d_in, d_out, r, padded rows)
CASES = [
    (1, 1, 1, 1, False), (31, 33, 31, 5, False), (32, 32, 32, 32, True), (33, 129, 65, 31, False),
    (65, 127, 128, 33, True), (97, 161, 64, 129, False), (1023, 1031, 257, 17, False), (1024, 1024, 1024, 64, True),
    (1025, 260, 1025, 70, True), (9001, 40, 70, 12, False),
]


@pytest.mark.parametrize("act", ("silu", "gelu"))
@pytest.mark.parametrize("case", range(len(CASES)), ids=["T%d-%dx%d-r%d-%s" % (*c[:4], "pad" if c[4] else "tight")
                                                         for c in CASES])
def test_f32_tiles(case, act):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    T, d_in, d_out, r, padded = CASES[case]
    ins = I.layer_inputs(1400 + case, 0, d_in, d_out, r, T, "f32")
    pitch = (lambda w: I.padded_ld(w, "f32")) if padded else (lambda w: w)
    run = LayerRun(ins, T, d_in, d_out, r, "f32", act, case % 2 == 1, ldx=pitch(d_in), ldy=pitch(d_out),
                   ldz=pitch(r)).run()
    got = run.outputs()
    assert run.padding_untouched()
    X, A, B, dY = (ins[k].f64 for k in ("X", "A", "B", "dY"))
    Z, H, Y = oracle.cola_fwd(X, A, B, act)
    _, dX, dA, dB = oracle.cola_bwd(X, Z, A, B, dY, act)
    for k, ref in {"Z": Z, "H": H, "Y": Y, "dX": dX, "dA": dA, "dB": dB}.items():
        if k not in got:
            continue
        assert np.all(np.isfinite(got[k])), k
        e = relerr(got[k], ref)
        assert e <= (1e-6 if T > 1 else 1e-5), f"{k}: {e:.2e}"
