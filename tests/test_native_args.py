"""The native checks of cola.py's layer and group calls (_torch_args): whatever
the Python checks refuse, they hand back (None) instead of calling the library;
plain calls run."""
import pytest
import torch

from paper_2502_10940_amd import cola

T, D_IN, D_OUT, R = 5, 24, 16, 8
BF = torch.bfloat16


def _args(dev):
    z = lambda *s, dt=BF: torch.zeros(s, dtype=dt, device=dev)
    return {"X": z(T, D_IN), "A": z(R, D_IN), "B": z(D_OUT, R), "Y": z(T, D_OUT), "Z": z(T, R), "H": z(T, R),
            "ws": z(1 << 16, dt=torch.uint8)}


def _fwd(a, d=None, n=None):
    d = d or cola.desc(T, D_IN, D_OUT, R)
    return cola._native_calls().fwd(d, a["X"], a["A"], a["B"], a["Y"], a["Z"], a["H"], a["ws"], n, 0)


def test_cpu_tensors_and_wrong_calls_are_handed_back():
    m = cola._native_calls()
    assert m, "the extension is built with the library"
    a = _args("cpu")
    assert _fwd(a) is None
    assert m.fwd() is None and m.fwd(*range(10)) is None
    assert m.group_infer(cola.desc(T, D_IN, D_OUT, R), a["X"], a["A"], [a["B"]], [a["Y"]], a["ws"], None, 0) is None


@pytest.mark.gpu
def test_refusals_are_handed_back():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert _fwd(_args("cuda:0")) == 0
    z = lambda *s, dt=BF: torch.zeros(s, dtype=dt, device="cuda:0")
    bad = [("X", z(T, D_IN, dt=torch.float32)), ("X", z(T - 1, D_IN)), ("X", z(T, D_IN - 1)), ("X", z(D_IN, T).t()),
           ("X", z(T, D_IN + 8)[:, :D_IN]), ("Y", z(T * D_OUT)), ("Z", None), ("A", 4096), ("B", z(D_OUT, R).cpu()),
           ("H", z(T, R, 1)), ("ws", z(64, 64, dt=torch.uint8).t()), ("ws", 4096)]
    for key, t in bad:
        a = _args("cuda:0")
        a[key] = t
        assert _fwd(a) is None, key
    a = _args("cuda:0")
    assert _fwd(a, n=(1 << 16) + 1) is None
    # a padded view whose last row's pad lies outside the storage
    d = cola.desc(T, D_IN, D_OUT, R, ldx=32)
    a["X"] = torch.zeros(T * 32 - 8, dtype=BF, device="cuda:0").as_strided((T, D_IN), (32, 1))
    assert _fwd(a, d) is None
    with pytest.raises(ValueError):
        cola.fwd(d, a["X"], a["A"], a["B"], a["Y"], a["Z"], a["H"], a["ws"])
    # library errors come back as a status
    assert _fwd(_args("cuda:0"), cola.desc(T, D_IN, D_OUT, R, recompute=True)) == cola.ERR_INVALID_ARG
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_streams_and_parameters():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = cola.desc(T, D_IN, D_OUT, R, act="identity")
    a = _args("cuda:0")
    a["A"] = torch.nn.Parameter(torch.ones((R, D_IN), dtype=BF, device="cuda:0"))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a["X"].fill_(0.5)
        cola.fwd(d, a["X"], a["A"], a["B"], a["Y"], a["Z"], a["H"], a["ws"])
    s.synchronize()
    assert torch.all(a["Z"].float() == 0.5 * D_IN)
    a["Z"].zero_()
    torch.cuda.synchronize()
    cola.fwd(d, a["X"], a["A"], a["B"], a["Y"], a["Z"], a["H"], a["ws"], stream=s)
    s.synchronize()
    assert torch.all(a["Z"].float() == 0.5 * D_IN)
