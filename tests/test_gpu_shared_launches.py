"""COLA_OPT_WGRAD_PAIR: 1 shares launches (dA with dB, in small layers dX with
both), 0 gives every product of a backward one of its own.  Counted by the
library's kernel timing, in a small layer that shares all three and a larger one,
bf16 and fp32; dX has the same bits either way (its sums are never split)."""
import pytest
import torch

from paper_2502_10940_amd import cola
from paper_2502_10940_amd import inputs as I

from layer_runner import LayerRun

pytestmark = pytest.mark.gpu

# (T, d_in, d_out, r, dtype, dX joins)
CASES = [(300, 264, 200, 72, "bf16", True), (1024, 520, 512, 128, "bf16", True), (130, 70, 90, 20, "f32", True),
         (20000, 1024, 1024, 256, "bf16", False), (4096, 512, 512, 128, "f32", False)]


def _launches(run):
    cola.timing_reset()
    cola.timing_enable(True)
    try:
        run.backward()
        torch.cuda.synchronize()
        return {k: cola.timing_read(i)[0] for i, k in enumerate(cola.KERNEL_CLASSES)}
    finally:
        cola.timing_enable(False)
        cola.timing_reset()


@pytest.mark.parametrize("case", CASES, ids=["T%d-%dx%d-r%d-%s" % c[:5] for c in CASES])
def test_launches_and_bits(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    T, d_in, d_out, r, dtype, joins = case
    ins = I.layer_inputs(1900, 0, d_in, d_out, r, T, dtype)
    dX = {}
    for pair in (1, 0):
        cola.set_option(cola.OPT_WGRAD_PAIR, pair)
        try:
            run = LayerRun(ins, T, d_in, d_out, r, dtype, "silu", False)
            run.forward()
            n = _launches(run)
        finally:
            cola.set_option(cola.OPT_WGRAD_PAIR, 1)
        dX[pair] = run.raw()["dX"]
        got = tuple(n[k] for k in ("bwd_dz", "bwd_dx", "bwd_da", "bwd_db", "bwd_da_db"))
        assert got == ((1, 0 if joins else 1, 0, 0, 1) if pair else (1, 1, 1, 1, 0)), (pair, got)
    assert (dX[0] == dX[1]).all()
