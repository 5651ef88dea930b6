"""The C ABI on the CPU: libcola.so loads without a GPU, exports every function
include/cola.h declares, and rejects every invalid argument with its documented
status before touching the GPU (only failing calls are made here)."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2502_10940_amd import cola

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "cola.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"^\s*(?:const\s+)?[A-Za-z_][\w\s]*?[\s\*]+([a-z_][a-z0-9_]*)\s*\(",
                       text, flags=re.M)
    return sorted(set(n for n in names if not n.startswith("typedef")))


def test_header_declares_expected_calls():
    names = declared_functions()
    for n in ("cola_fwd", "cola_bwd", "cola_workspace_bytes", "cola_strerror", "cola_abi_version",
              "dense_fwd", "dense_bwd", "dense_workspace_bytes", "cola_timing_enable",
              "cola_timing_read", "cola_timing_reset", "cola_kernel_name",
              "cola_group_fwd", "cola_group_bwd", "cola_group_workspace_bytes", "cola_infer",
              "cola_group_infer", "cola_fwd_outer", "cola_bwd_outer", "cola_set_option",
              "cola_get_option"):
        assert n in names


def test_library_exports_every_declared_symbol():
    L = cola.lib()
    for n in declared_functions():
        assert hasattr(L, n), n
    out = subprocess.run(["nm", "-D", "--defined-only", cola.LIB_PATH], capture_output=True,
                         text=True, check=True).stdout
    exported = set(line.split()[-1] for line in out.splitlines() if line.strip())
    for n in declared_functions():
        assert n in exported, n
    assert set(declared_functions()) == set(cola.EXPORTS)


def test_abi_version_and_strerror():
    L = cola.lib()
    assert L.cola_abi_version() == 2
    for s in range(6):
        assert L.cola_strerror(s)
    assert L.cola_strerror(99) == b"unknown status"
    for k in range(len(cola.KERNEL_CLASSES)):
        assert cola.kernel_name(k) == cola.KERNEL_CLASSES[k]
    assert cola.kernel_name(-1) == "invalid"


FAKE = 0x1000  # never dereferenced: every call below fails validation first


def fwd_status(d, X=FAKE, A=FAKE, B=FAKE, Y=FAKE, Z=FAKE, H=FAKE, ws=None, ws_bytes=0):
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_fwd(p, X, A, B, Y, Z, H, ws, ws_bytes, None)


def bwd_status(d, dY=FAKE, X=FAKE, Z=FAKE, H=FAKE, A=FAKE, B=FAKE, dX=FAKE, dA=FAKE, dB=FAKE,
               ws=None, ws_bytes=0):
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_bwd(p, dY, X, Z, H, A, B, dX, dA, dB, ws, ws_bytes, None)


def test_invalid_descriptors():
    assert fwd_status(None) == cola.ERR_INVALID_ARG
    assert bwd_status(None) == cola.ERR_INVALID_ARG
    for kw, code in ((dict(dtype=7), cola.ERR_INVALID_ARG), (dict(act=3), cola.ERR_INVALID_ARG),
                     (dict(recompute=True), None)):
        d = cola.desc(16, 32, 32, 8, **{k: v for k, v in kw.items() if k != "recompute"})
        if "recompute" in kw:
            d.recompute = 2
            code = cola.ERR_INVALID_ARG
        assert fwd_status(d) == code
        assert bwd_status(d) == code
    for shape in ((16, 0, 32, 8), (16, 32, 0, 8), (16, 32, 32, 0), (-1, 32, 32, 8)):
        d = cola.desc(*shape)
        assert fwd_status(d) == cola.ERR_BAD_SHAPE
        assert bwd_status(d) == cola.ERR_BAD_SHAPE
        assert cola.workspace_bytes(d, 0) == 0 and cola.workspace_bytes(d, 1) == 0
    for ld in (dict(ldx=31), dict(ldy=30), dict(ldz=7)):
        d = cola.desc(16, 32, 32, 8, **ld)
        assert fwd_status(d) == cola.ERR_BAD_SHAPE
        assert bwd_status(d) == cola.ERR_BAD_SHAPE
    d = cola.desc(1 << 41, 32, 32, 8)
    assert fwd_status(d) == cola.ERR_BAD_SHAPE


def test_row_pitch_limit():
    """Row pitches up to COLA_MAX_PITCH (2^22 elements, what the 256 x 256
    family's buffer descriptors reach) are taken; wider ones, and widths
    beyond it, are refused before anything is enqueued."""
    maxp = 1 << 22
    hdr = open(os.path.join(ROOT, "include", "cola.h")).read()
    assert "#define COLA_MAX_PITCH (1LL << 22)" in hdr
    for ld in (dict(ldx=maxp), dict(ldy=maxp), dict(ldz=maxp)):
        assert cola.workspace_bytes(cola.desc(16, 32, 32, 8, **ld), 1) > 0
    for ld in (dict(ldx=maxp + 1), dict(ldy=maxp + 8), dict(ldz=maxp + 64)):
        d = cola.desc(16, 32, 32, 8, **ld)
        assert fwd_status(d) == cola.ERR_BAD_SHAPE
        assert bwd_status(d) == cola.ERR_BAD_SHAPE
        assert cola.workspace_bytes(d, 0) == 0 and cola.workspace_bytes(d, 1) == 0
    assert cola.workspace_bytes(cola.desc(16, maxp + 8, 32, 8), 1) == 0
    assert cola.group_workspace_bytes(cola.group_desc(16, 32, [8, 8], [32, 32], ldz=maxp + 64), 1) == 0
    assert cola.group_workspace_bytes(cola.group_desc(16, 32, [8, 8], [32, 32], ldz=maxp), 1) > 0
    assert cola.dense_workspace_bytes(cola.dense_desc(16, 32, 32, "bf16", maxp + 8, 32), 1) == 0
    assert cola.block_saved_bytes(cola.block_desc(2, 64, 128, maxp + 1, 2, 8)) == 0
    assert cola.block_saved_bytes(cola.block_desc(2, 64, 128, maxp - 64, 2, 8)) > 0


def test_h_must_match_recompute():
    d = cola.desc(16, 32, 32, 8, recompute=False)
    assert fwd_status(d, H=None) == cola.ERR_INVALID_ARG
    assert bwd_status(d, H=None) == cola.ERR_INVALID_ARG
    d = cola.desc(16, 32, 32, 8, recompute=True)
    assert fwd_status(d, H=FAKE) == cola.ERR_INVALID_ARG
    assert bwd_status(d, H=FAKE) == cola.ERR_INVALID_ARG


@pytest.mark.parametrize("name", ["X", "A", "B", "Y", "Z"])
def test_null_forward_pointers(name):
    d = cola.desc(16, 32, 32, 8)
    assert fwd_status(d, **{name: None}) == cola.ERR_INVALID_ARG


@pytest.mark.parametrize("name", ["dY", "X", "Z", "A", "B", "dX", "dA", "dB"])
def test_null_backward_pointers(name):
    d = cola.desc(16, 32, 32, 8)
    need = cola.workspace_bytes(d, 1)
    assert bwd_status(d, ws=FAKE, ws_bytes=need, **{name: None}) == cola.ERR_INVALID_ARG


def test_workspace_too_small():
    d = cola.desc(64, 32, 48, 8, recompute=True)
    need = cola.workspace_bytes(d, 0)
    assert need >= 64 * 8 * 2
    assert fwd_status(d, H=None, ws=FAKE, ws_bytes=need - 1) == cola.ERR_WORKSPACE
    assert fwd_status(d, H=None, ws=None, ws_bytes=need) == cola.ERR_WORKSPACE
    need_b = cola.workspace_bytes(d, 1)
    assert need_b >= 2 * 64 * 8 * 2          # dZ and the recomputed H
    assert bwd_status(d, H=None, ws=FAKE, ws_bytes=need_b - 1) == cola.ERR_WORKSPACE


def test_workspace_sizes():
    for dtype, es in (("bf16", 2), ("f32", 4)):
        d = cola.desc(1000, 96, 80, 24, dtype=dtype)
        assert cola.workspace_bytes(d, 0) == 0                       # CoLA: H is an output
        dm = cola.desc(1000, 96, 80, 24, dtype=dtype, recompute=True)
        assert cola.workspace_bytes(dm, 0) >= 1000 * 24 * es         # CoLA-M keeps H here
        assert cola.workspace_bytes(dm, 1) >= cola.workspace_bytes(d, 1) + 1000 * 24 * es
        assert cola.workspace_bytes(d, 2) == cola.workspace_bytes(dm, 0)  # inference keeps H there too
        assert cola.workspace_bytes(d, 3) >= cola.workspace_bytes(d, 1) + 1000 * 80 * es  # both-sigma: + dP
        assert cola.workspace_bytes(d, 4) == 0
    empty = cola.desc(0, 96, 80, 24)
    assert cola.workspace_bytes(empty, 0) == 0 and cola.workspace_bytes(empty, 1) == 0


@pytest.mark.parametrize("T,d_in,d_out,r", [(65536, 2048, 5461, 512), (1000, 77, 40, 9), (300, 512, 333, 65)])
def test_lean_workspace_sizes(T, d_in, d_out, r):
    """Tight odd rows: the lean size is that of the same layer on padded rows (no
    copies of token rows), less than the full one, and the least accepted."""
    pad = lambda w: -(-w // 8) * 8
    for rc in (False, True):
        tight = cola.desc(T, d_in, d_out, r, recompute=rc)
        padded = cola.desc(T, d_in, d_out, r, "bf16", "silu", rc, pad(d_in), pad(d_out), pad(r))
        for phase in range(4):
            lean = cola.workspace_bytes(tight, phase + cola.WS_LEAN)
            assert lean == cola.workspace_bytes(padded, phase) == cola.workspace_bytes(padded, phase + cola.WS_LEAN)
            assert lean <= cola.workspace_bytes(tight, phase)
        lean = cola.workspace_bytes(tight, 1 + cola.WS_LEAN)
        assert lean < cola.workspace_bytes(tight, 1)
        H = None if rc else FAKE
        assert bwd_status(tight, H=H, ws=FAKE, ws_bytes=lean - 1) == cola.ERR_WORKSPACE
        g = cola.group_desc(T, d_in, [r, r], [d_out, d_out], recompute=rc)
        for phase in range(3):
            assert cola.group_workspace_bytes(g, phase + cola.WS_LEAN) <= cola.group_workspace_bytes(g, phase)
        assert 0 < cola.group_workspace_bytes(g, 1 + cola.WS_LEAN) < cola.group_workspace_bytes(g, 1)
    for phase in (4, 15, 4 + cola.WS_LEAN, 2 * cola.WS_LEAN, -1, -cola.WS_LEAN):
        assert cola.workspace_bytes(tight, phase) == 0
    assert cola.group_workspace_bytes(g, 3 + cola.WS_LEAN) == 0
    # 129 MB where the full size is 850
    if T == 65536:
        d = cola.desc(T, d_in, d_out, r)
        assert cola.workspace_bytes(d, 1 + cola.WS_LEAN) < 160 << 20 < cola.workspace_bytes(d, 1)


def test_empty_forward_is_a_noop():
    # T = 0 is an empty batch: nothing to compute, nothing enqueued
    d = cola.desc(0, 32, 32, 8)
    assert fwd_status(d, X=None, A=None, B=None, Y=None, Z=None) == cola.OK
    assert fwd_status(d, X=None, A=None, B=None, Y=None, Z=None, H=None) == cola.OK
    dm = cola.desc(0, 32, 32, 8, recompute=True)
    assert fwd_status(dm, X=None, A=None, B=None, Y=None, Z=None, H=None) == cola.OK
    assert fwd_status(dm, H=FAKE) == cola.ERR_INVALID_ARG


def test_dense_validation():
    L = cola.lib()
    d = cola.dense_desc(16, 0, 8)
    assert L.dense_fwd(ctypes.byref(d), FAKE, FAKE, FAKE, None, 0, None) == cola.ERR_BAD_SHAPE
    d = cola.dense_desc(16, 32, 8, dtype=3)
    assert L.dense_fwd(ctypes.byref(d), FAKE, FAKE, FAKE, None, 0, None) == cola.ERR_INVALID_ARG
    d = cola.dense_desc(16, 32, 8)
    assert L.dense_fwd(ctypes.byref(d), None, FAKE, FAKE, None, 0, None) == cola.ERR_INVALID_ARG
    assert L.dense_bwd(ctypes.byref(d), FAKE, FAKE, FAKE, FAKE, None, None, 0, None) == cola.ERR_INVALID_ARG
    big = cola.dense_desc(100000, 512, 512)
    need = cola.dense_workspace_bytes(big, 1)
    assert need > 0
    assert L.dense_bwd(ctypes.byref(big), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, need - 1, None) == cola.ERR_WORKSPACE


def test_timing_api_validation():
    L = cola.lib()
    n = ctypes.c_int64(); x = ctypes.c_double()
    assert L.cola_timing_read(99, ctypes.byref(n), ctypes.byref(x), ctypes.byref(x),
                              ctypes.byref(x)) == cola.ERR_INVALID_ARG
    assert L.cola_timing_read(0, None, ctypes.byref(x), ctypes.byref(x), ctypes.byref(x)) == cola.ERR_INVALID_ARG
    # enable/disable touch no GPU state
    assert L.cola_timing_enable(0) == cola.OK


def test_binding_raises_on_error():
    d = cola.desc(16, 0, 32, 8)
    with pytest.raises(cola.ColaError) as e:
        cola.fwd(d, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, stream=0)
    assert e.value.status == cola.ERR_BAD_SHAPE


# --------------------------------------------------------------------------
# grouped projections (shared input): validation before any GPU work
# --------------------------------------------------------------------------

def group_fwd_status(d, X=FAKE, A=FAKE, B=FAKE, Y=FAKE, Z=FAKE, H=FAKE, ws=None, ws_bytes=0, n=None):
    n = d.n if (d is not None and n is None) else (n or 1)
    arr = lambda v: None if v is None else ctypes.cast((ctypes.c_void_p * max(n, 1))(*([v] * max(n, 1))),
                                                      ctypes.c_void_p)
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_group_fwd(p, X, A, arr(B), arr(Y), Z, H, ws, ws_bytes, None)


def test_group_struct_layout_matches_header():
    # offsets of the C struct (compiled from include/cola.h) against the binding's
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "_sz.c")
    exe = os.path.join(os.path.dirname(os.path.abspath(__file__)), "_sz")
    code = ('#include "cola.h"\n#include <stdio.h>\n#include <stddef.h>\n'
            'int main(void){printf("%zu %zu %zu %zu %zu\\n", sizeof(cola_group_desc),'
            'offsetof(cola_group_desc, r), offsetof(cola_group_desc, d_out),'
            'offsetof(cola_group_desc, ldy), offsetof(cola_group_desc, ldz)); return 0;}\n')
    try:
        open(src, "w").write(code)
        subprocess.run(["gcc", "-I", os.path.join(ROOT, "include"), src, "-o", exe], check=True)
        got = [int(v) for v in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()]
    finally:
        for f in (src, exe):
            if os.path.exists(f):
                os.remove(f)
    G = cola.GroupDesc
    assert got == [ctypes.sizeof(G), G.r.offset, G.d_out.offset, G.ldy.offset, G.ldz.offset]


def test_group_invalid_descriptors():
    ok = cola.group_desc(64, 32, [8, 16, 8], [32, 32, 16])
    assert cola.group_workspace_bytes(ok, 1) > 0
    bad = [
        cola.group_desc(64, 32, [8], [32], dtype=7),
        cola.group_desc(64, 32, [8], [32], act=3),
        cola.group_desc(64, 0, [8], [32]),
        cola.group_desc(64, 32, [8, 0], [32, 32]),
        cola.group_desc(64, 32, [8, 8], [32, 0]),
        cola.group_desc(-1, 32, [8], [32]),
        cola.group_desc(64, 32, [8, 8], [32, 32], ldz=15),       # ldz < R = 16
        cola.group_desc(64, 32, [8], [32], ldx=31),
        cola.group_desc(64, 32, [8], [32], ldy=[31]),
    ]
    for d in bad:
        assert cola.group_workspace_bytes(d, 0) == 0
        assert cola.group_workspace_bytes(d, 1) == 0
        assert group_fwd_status(d) in (cola.ERR_INVALID_ARG, cola.ERR_BAD_SHAPE)
    for n in (0, 9):
        d = cola.group_desc(64, 32, [8], [32])
        d.n = n
        assert cola.group_workspace_bytes(d, 0) == 0
        assert group_fwd_status(d, n=1) == cola.ERR_INVALID_ARG
    assert group_fwd_status(None) == cola.ERR_INVALID_ARG


def test_group_pointer_and_workspace_checks():
    d = cola.group_desc(64, 32, [8, 16], [32, 24])
    assert group_fwd_status(d, H=None) == cola.ERR_INVALID_ARG          # CoLA needs H
    assert group_fwd_status(d, X=None) == cola.ERR_INVALID_ARG
    assert group_fwd_status(d, B=None) == cola.ERR_INVALID_ARG
    assert group_fwd_status(d, Y=None) == cola.ERR_INVALID_ARG
    m = cola.group_desc(64, 32, [8, 16], [32, 24], recompute=True)
    assert group_fwd_status(m) == cola.ERR_INVALID_ARG                  # CoLA-M takes no H
    assert group_fwd_status(m, H=None) == cola.ERR_WORKSPACE            # H_all copy needs workspace
    # an empty batch enqueues nothing
    e = cola.group_desc(0, 32, [8, 16], [32, 24])
    assert group_fwd_status(e, X=None, A=None, B=None, Y=None, Z=None, H=None) == cola.OK


def infer_status(d, X=FAKE, A=FAKE, B=FAKE, Y=FAKE, ws=None, ws_bytes=0):
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_infer(p, X, A, B, Y, ws, ws_bytes, None)


def group_infer_status(d, X=FAKE, A=FAKE, B=FAKE, Y=FAKE, ws=None, ws_bytes=0, n=None):
    n = d.n if (d is not None and n is None) else (n or 1)
    arr = lambda v: None if v is None else ctypes.cast((ctypes.c_void_p * max(n, 1))(*([v] * max(n, 1))),
                                                      ctypes.c_void_p)
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_group_infer(p, X, A, arr(B), arr(Y), ws, ws_bytes, None)


def test_infer_checks():
    d = cola.desc(64, 32, 48, 8)
    # H lives in the workspace whatever recompute says: the CoLA-M forward's size
    need = cola.workspace_bytes(d, 2)
    assert need == cola.workspace_bytes(cola.desc(64, 32, 48, 8, recompute=True), 0) > 0
    assert cola.workspace_bytes(d, 4) == 0
    assert infer_status(None) == cola.ERR_INVALID_ARG
    for kw in (dict(dtype=7), dict(act=3)):
        assert infer_status(cola.desc(64, 32, 48, 8, **kw)) == cola.ERR_INVALID_ARG
    assert infer_status(cola.desc(64, 0, 48, 8)) == cola.ERR_BAD_SHAPE
    assert infer_status(cola.desc(64, 32, 48, 8, ldx=31)) == cola.ERR_BAD_SHAPE
    for k in ("X", "A", "B", "Y"):
        assert infer_status(d, **{k: None}) == cola.ERR_INVALID_ARG
    assert infer_status(d) == cola.ERR_WORKSPACE
    assert infer_status(d, ws=FAKE, ws_bytes=need - 1) == cola.ERR_WORKSPACE
    assert infer_status(cola.desc(0, 32, 48, 8), X=None, A=None, B=None, Y=None) == cola.OK


def test_group_infer_checks():
    d = cola.group_desc(64, 32, [8, 16], [32, 24])
    need = cola.group_workspace_bytes(d, 2)
    assert need == cola.group_workspace_bytes(cola.group_desc(64, 32, [8, 16], [32, 24], recompute=True), 0)
    assert cola.group_workspace_bytes(d, 3) == 0
    assert group_infer_status(None) == cola.ERR_INVALID_ARG
    assert group_infer_status(cola.group_desc(64, 32, [8, 0], [32, 32])) == cola.ERR_BAD_SHAPE
    assert group_infer_status(cola.group_desc(64, 32, [8], [32], act=3)) == cola.ERR_INVALID_ARG
    for k in ("X", "A", "B", "Y"):
        assert group_infer_status(d, **{k: None}) == cola.ERR_INVALID_ARG
    assert group_infer_status(d) == cola.ERR_WORKSPACE
    assert group_infer_status(d, ws=FAKE, ws_bytes=need - 1) == cola.ERR_WORKSPACE
    e = cola.group_desc(0, 32, [8, 16], [32, 24])
    assert group_infer_status(e, X=None, A=None, B=None, Y=None) == cola.OK


def fwd_outer_status(d, outer=1, X=FAKE, A=FAKE, B=FAKE, Y=FAKE, P=FAKE, Z=FAKE, H=FAKE, ws=None, ws_bytes=0):
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_fwd_outer(p, outer, X, A, B, Y, P, Z, H, ws, ws_bytes, None)


def bwd_outer_status(d, outer=1, dY=FAKE, P=FAKE, X=FAKE, Z=FAKE, H=FAKE, A=FAKE, B=FAKE, dX=FAKE, dA=FAKE,
                     dB=FAKE, ws=None, ws_bytes=0):
    p = ctypes.byref(d) if d is not None else None
    return cola.lib().cola_bwd_outer(p, outer, dY, P, X, Z, H, A, B, dX, dA, dB, ws, ws_bytes, None)


def test_outer_checks():
    d = cola.desc(64, 32, 48, 8)
    assert fwd_outer_status(None) == cola.ERR_INVALID_ARG
    assert bwd_outer_status(None) == cola.ERR_INVALID_ARG
    for bad in (-1, 3, 99):
        assert fwd_outer_status(d, outer=bad) == cola.ERR_INVALID_ARG
        assert bwd_outer_status(d, outer=bad) == cola.ERR_INVALID_ARG
    assert fwd_outer_status(cola.desc(64, 32, 48, 8, act=3)) == cola.ERR_INVALID_ARG
    assert fwd_outer_status(cola.desc(64, 32, 48, 8, ldy=47)) == cola.ERR_BAD_SHAPE
    for k in ("X", "A", "B", "Y", "P", "Z"):
        assert fwd_outer_status(d, **{k: None}) == cola.ERR_INVALID_ARG
    assert fwd_outer_status(d, H=None) == cola.ERR_INVALID_ARG                       # CoLA needs H
    m = cola.desc(64, 32, 48, 8, recompute=True)
    assert fwd_outer_status(m) == cola.ERR_INVALID_ARG                               # CoLA-M takes no H
    assert fwd_outer_status(m, H=None) == cola.ERR_WORKSPACE
    # backward: the layer's workspace plus T*d_out elements of dP
    need = cola.workspace_bytes(d, 3)
    assert need >= cola.workspace_bytes(d, 1) + 64 * 48 * 2
    for k in ("dY", "P", "X", "Z", "A", "B", "dX", "dA", "dB"):
        assert bwd_outer_status(d, ws=FAKE, ws_bytes=need, **{k: None}) == cola.ERR_INVALID_ARG
    assert bwd_outer_status(d, ws=FAKE, ws_bytes=need - 1) == cola.ERR_WORKSPACE
    e = cola.desc(0, 32, 48, 8)
    assert cola.workspace_bytes(e, 3) == 0
    assert fwd_outer_status(e, X=None, A=None, B=None, Y=None, P=None, Z=None) == cola.OK


# --------------------------------------------------------------------------
# the binding refuses tensors that do not match the descriptor before the
# library sees a pointer (CPU: every check but the device one runs first, so
# a well-formed CPU tensor is refused only for being on the CPU)
# --------------------------------------------------------------------------

def _layer_tensors(T=64, d_in=32, d_out=24, r=8, dt=None):
    import torch
    dt = dt or torch.bfloat16
    return dict(X=torch.zeros(T, d_in, dtype=dt), A=torch.zeros(r, d_in, dtype=dt),
                B=torch.zeros(d_out, r, dtype=dt), Y=torch.zeros(T, d_out, dtype=dt),
                Z=torch.zeros(T, r, dtype=dt), H=torch.zeros(T, r, dtype=dt),
                dY=torch.zeros(T, d_out, dtype=dt), dX=torch.zeros(T, d_in, dtype=dt),
                dA=torch.zeros(r, d_in, dtype=torch.float32), dB=torch.zeros(d_out, r, dtype=torch.float32))


def _refused(match, fn, *args, **kw):
    with pytest.raises(ValueError, match=match):
        fn(*args, **kw)


def test_binding_refuses_mismatched_tensors():
    import torch
    d = cola.desc(64, 32, 24, 8, "bf16", "silu", False)
    t = _layer_tensors()
    bwd_args = lambda **o: [o.get(k, t[k]) for k in ("dY", "X", "Z", "H", "A", "B", "dX", "dA", "dB")]
    # dA allocated in bf16: the kernels write fp32
    _refused("dA: dtype", cola.bwd, d, *bwd_args(dA=torch.zeros(8, 32, dtype=torch.bfloat16)))
    # fp32 activations under a bf16 descriptor
    _refused("X: dtype", cola.fwd, d, torch.zeros(64, 32), t["A"], t["B"], t["Y"], t["Z"], t["H"])
    # too few rows, too narrow, 1-D
    _refused("Y: shape", cola.fwd, d, t["X"], t["A"], t["B"], torch.zeros(63, 24, dtype=torch.bfloat16),
             t["Z"], t["H"])
    _refused("B: shape", cola.fwd, d, t["X"], t["A"], torch.zeros(24, 7, dtype=torch.bfloat16), t["Y"],
             t["Z"], t["H"])
    _refused("Z: expected a 2-D", cola.fwd, d, t["X"], t["A"], t["B"], t["Y"],
             torch.zeros(64 * 8, dtype=torch.bfloat16), t["H"])
    # a non-contiguous view (a transposed weight) and a strided column slice
    _refused("A: strides", cola.fwd, d, t["X"], torch.zeros(32, 8, dtype=torch.bfloat16).t(), t["B"], t["Y"],
             t["Z"], t["H"])
    _refused("X: strides", cola.fwd, d, torch.zeros(64, 40, dtype=torch.bfloat16)[:, :32], t["A"], t["B"],
             t["Y"], t["Z"], t["H"])
    # a padded pitch that the tensor's storage does not cover
    dp = cola.desc(64, 32, 24, 8, "bf16", "silu", False, ldx=40)
    _refused("X: storage", cola.fwd, dp, torch.zeros(64 * 40 - 8, dtype=torch.bfloat16)[: 63 * 40 + 32]
             .as_strided((64, 32), (40, 1)), t["A"], t["B"], t["Y"], t["Z"], t["H"])
    # the same padded view, with storage for all 64 x 40 elements, passes every check but the device
    x = torch.zeros(64, 40, dtype=torch.bfloat16)[:, :32]
    _refused("X: tensor is on cpu", cola.fwd, dp, x, t["A"], t["B"], t["Y"], t["Z"], t["H"])
    # workspace: more bytes claimed than the tensor holds
    _refused("ws: ws_bytes", cola.fwd, d, t["X"], t["A"], t["B"], t["Y"], t["Z"], t["H"],
             ws=torch.zeros(16, dtype=torch.uint8), ws_bytes=17)
    # fp32 descriptor: dB must still be fp32, activations fp32
    d32 = cola.desc(64, 32, 24, 8, "f32", "silu", False)
    t32 = _layer_tensors(dt=torch.float32)
    _refused("dY: tensor is on cpu", cola.bwd, d32, *[t32[k] for k in ("dY", "X", "Z", "H", "A", "B", "dX", "dA",
                                                                        "dB")])


def test_binding_refuses_mismatched_group_and_dense_tensors():
    import torch
    bf = torch.bfloat16
    g = cola.group_desc(64, 32, [8, 16], [24, 40])
    X = torch.zeros(64, 32, dtype=bf)
    A_all = torch.zeros(24, 32, dtype=bf)
    B = [torch.zeros(24, 8, dtype=bf), torch.zeros(40, 16, dtype=bf)]
    Y = [torch.zeros(64, 24, dtype=bf), torch.zeros(64, 40, dtype=bf)]
    Z = torch.zeros(64, 24, dtype=bf)
    _refused("B\\[1\\]: shape", cola.group_fwd, g, X, A_all, [B[0], torch.zeros(40, 8, dtype=bf)], Y, Z, Z)
    _refused("Y: 1 entries", cola.group_fwd, g, X, A_all, B, Y[:1], Z, Z)
    _refused("A_all: shape", cola.group_fwd, g, X, torch.zeros(16, 32, dtype=bf), B, Y, Z, Z)
    _refused("dB\\[0\\]: dtype", cola.group_bwd, g, Y, X, Z, Z, A_all, B, X, torch.zeros(24, 32),
             [torch.zeros(24, 8, dtype=bf), torch.zeros(40, 16)])
    dd = cola.dense_desc(64, 32, 24)
    W = torch.zeros(24, 32, dtype=bf)
    _refused("dW: dtype", cola.dense_bwd, dd, Y[0], X, W, X, torch.zeros(24, 32, dtype=bf))
    _refused("W: shape", cola.dense_fwd, dd, X, torch.zeros(24, 31, dtype=bf), Y[0])
    _refused("X: tensor is on cpu", cola.dense_fwd, dd, X, W, Y[0])


def test_tuning_options():
    L = cola.lib()
    assert cola.get_option(cola.OPT_STREAM_ONLY) == 0
    assert cola.get_option(cola.OPT_WGRAD_PAIR) == 1
    assert cola.get_option(cola.OPT_FUSE_GATE) == 1
    assert cola.get_option(cola.OPT_TILE) == 0
    for v in (-1, 5):
        assert L.cola_set_option(cola.OPT_TILE, v) == cola.ERR_INVALID_ARG
    assert L.cola_get_option(7) == -1
    assert L.cola_set_option(7, 0) == cola.ERR_INVALID_ARG
    assert L.cola_set_option(cola.OPT_WGRAD_PAIR, 2) == cola.ERR_INVALID_ARG
    assert cola.get_option(cola.OPT_WGRAD_PAIR) == 1
    # the workspace plan follows the setting: one split for both weight
    # gradients when paired, one each when not
    d = cola.desc(32768, 2048, 2048, 512)
    paired = cola.workspace_bytes(d, 1)
    cola.set_option(cola.OPT_WGRAD_PAIR, 0)
    try:
        assert cola.get_option(cola.OPT_WGRAD_PAIR) == 0
        assert cola.workspace_bytes(d, 1) != paired
    finally:
        cola.set_option(cola.OPT_WGRAD_PAIR, 1)
    assert cola.workspace_bytes(d, 1) == paired


# --------------------------------------------------------------------------
# decoder block entry points: descriptor validation and the saved set (host
# only; every call here is refused before anything is enqueued)
# --------------------------------------------------------------------------

def test_block_descriptor_validation():
    L = cola.lib()
    ok = cola.block_desc(2, 256, 512, 1376, 8, 128)
    assert cola.block_saved_bytes(ok) > 0
    assert cola.block_workspace_bytes(ok, 0) > 0 and cola.block_workspace_bytes(ok, 1) > 0
    assert cola.block_workspace_bytes(ok, 2) == 0
    bad = [cola.block_desc(2, 256, 512, 1376, 16, 128),      # head dim 32: not compiled in
           cola.block_desc(2, 256, 500, 1376, 5, 128),       # d not a multiple of 8
           cola.block_desc(2, 256, 512, 1376, 8, 100),       # r not a multiple of 8
           cola.block_desc(2, 0, 512, 1376, 8, 128),         # empty sequences
           cola.block_desc(-1, 256, 512, 1376, 8, 128),
           cola.block_desc(2, 256, 512, 1376, 7, 128),       # heads do not divide d
           cola.block_desc(2, 256, 512, 1376, 8, 128, act=5),
           cola.block_desc(2, 256, 512, 1376, 8, 128, rope_base=0.0),
           cola.block_desc(70000, 1, 512, 1376, 8, 128)]     # beyond the attention grid
    for d in bad:
        assert cola.block_saved_bytes(d) == 0
        assert cola.block_workspace_bytes(d, 1) == 0
    W = cola.BlockWeights(*([FAKE] * len(cola.BLOCK_PARAMS)))
    G = cola.BlockGrads(*([FAKE] * len(cola.BLOCK_PARAMS)))
    st = L.cola_block_fwd(ctypes.byref(bad[0]), ctypes.byref(W), FAKE, FAKE, FAKE, 1 << 40, FAKE, 1 << 40, None)
    assert st == cola.ERR_UNSUPPORTED
    st = L.cola_block_fwd(ctypes.byref(bad[1]), ctypes.byref(W), FAKE, FAKE, FAKE, 1 << 40, FAKE, 1 << 40, None)
    assert st == cola.ERR_BAD_SHAPE
    # a NULL weight, a misaligned input, a short saved buffer, a short workspace
    W0 = cola.BlockWeights(*([FAKE] * (len(cola.BLOCK_PARAMS) - 1) + [None]))
    assert L.cola_block_fwd(ctypes.byref(ok), ctypes.byref(W0), FAKE, FAKE, FAKE, 1 << 40, FAKE, 1 << 40,
                            None) == cola.ERR_INVALID_ARG
    assert L.cola_block_fwd(ctypes.byref(ok), ctypes.byref(W), FAKE + 2, FAKE, FAKE, 1 << 40, FAKE, 1 << 40,
                            None) == cola.ERR_INVALID_ARG
    need_s = cola.block_saved_bytes(ok)
    need_w = cola.block_workspace_bytes(ok, 0)
    assert L.cola_block_fwd(ctypes.byref(ok), ctypes.byref(W), FAKE, FAKE, FAKE, need_s - 1, FAKE, need_w,
                            None) == cola.ERR_WORKSPACE
    assert L.cola_block_fwd(ctypes.byref(ok), ctypes.byref(W), FAKE, FAKE, FAKE, need_s, FAKE, need_w - 1,
                            None) == cola.ERR_WORKSPACE
    assert L.cola_block_bwd(ctypes.byref(ok), ctypes.byref(W), FAKE, FAKE, need_s, FAKE, FAKE, None, FAKE,
                            1 << 40, None) == cola.ERR_INVALID_ARG
    need_b = cola.block_workspace_bytes(ok, 1)
    assert L.cola_block_bwd(ctypes.byref(ok), ctypes.byref(W), FAKE, FAKE, need_s, FAKE, FAKE, ctypes.byref(G),
                            FAKE, need_b - 1, None) == cola.ERR_WORKSPACE


@pytest.mark.parametrize("shape", [(2, 256, 512, 1376, 8, 128), (128, 256, 2048, 5461, 32, 512),
                                   (64, 256, 4096, 11008, 32, 1024)])
def test_block_cola_m_saved_set_is_2nd_plus_7nr(shape):
    # App. C: CoLA-M keeps 2nd + 7nr values per block: the block input (the
    # caller's x0), the mid-block residual x1 and the seven r-wide
    # pre-activations; bf16, so 2 bytes each (r a multiple of 64 and an even T:
    # no row or alignment padding)
    n_seq, L, d, ffn, heads, r = shape
    n = n_seq * L
    dm = cola.block_desc(n_seq, L, d, ffn, heads, r, recompute=True)
    saved_m = cola.block_saved_bytes(dm)
    assert saved_m + 2 * n * d == 2 * (2 * n * d + 7 * n * r)
    # CoLA keeps the 14 nr of the low-rank activations (Z and H of the seven)
    # and, besides x1, the n x d norms, q, k, v, att and the n x ffn gate, up, product
    dc = cola.block_desc(n_seq, L, d, ffn, heads, r, recompute=False)
    ffn_pitch = (ffn + 63) // 64 * 64
    lse = (n * heads * 4 + 255) // 256 * 256
    assert cola.block_saved_bytes(dc) == 2 * (7 * n * d + 14 * n * r + 3 * n * ffn_pitch) + lse
    # the slots tile the buffer without overlap; CoLA-M has no CoLA-only slot
    spans = []
    for i, name in enumerate(cola.BLOCK_SLOTS):
        off, ld = cola.block_saved_slot(dc, name)
        rows = heads if name == "lse" else n
        spans.append((off, off + rows * ld * (4 if name == "lse" else 2)))
        if i >= 5:
            with pytest.raises(cola.ColaError):
                cola.block_saved_slot(dm, name)
    spans.sort()
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
    assert spans[-1][1] <= cola.block_saved_bytes(dc)


def _no_gpu_here():
    """True only where no GPU can be reached: no kernel driver node and no
    device visible to the runtime.  The test below hands the library fake
    addresses, which a real device would fault on."""
    if os.path.exists("/dev/kfd"):
        return False
    import torch
    return torch.cuda.device_count() == 0


@pytest.mark.skipif(not _no_gpu_here(), reason="forces a launch failure; runs only where no GPU exists")
def test_launch_failure_reports_hip_error():
    """A call that passes validation but whose first launch fails (here: no
    device at all) returns COLA_ERR_HIP, and cola_strerror names the step
    and carries HIP's own text; the failure handling of SURVEY's status-code
    contract, forced from the host."""
    L = cola.lib()
    fake = lambda k: ctypes.c_void_p(0x100000 * k)
    d = cola.desc(256, 512, 512, 128, "bf16", "silu", False)
    ws = L.cola_workspace_bytes(ctypes.byref(d), 0) + L.cola_workspace_bytes(ctypes.byref(d), 1)
    st = L.cola_fwd(ctypes.byref(d), fake(1), fake(2), fake(3), fake(4), fake(5), fake(6), fake(7), ws, None)
    assert st == cola.ERR_HIP
    text = L.cola_strerror(st).decode()
    assert text.startswith("fwd_z_sigma:") and len(text) > len("fwd_z_sigma: ")
    st = L.cola_bwd(ctypes.byref(d), *(fake(k) for k in range(1, 11)), ws, None)
    assert st == cola.ERR_HIP
    assert L.cola_strerror(st).decode().split(":")[0] in ("bwd_dz", "pack_rows")
    dd = cola.DenseDesc(256, 512, 512, 0, 0, cola.BF16)
    wsd = L.dense_workspace_bytes(ctypes.byref(dd), 1)
    st = L.dense_fwd(ctypes.byref(dd), fake(1), fake(2), fake(3), fake(4), wsd, None)
    assert st == cola.ERR_HIP
    # the status text of a later validation error is its own, not the old HIP text
    st = L.cola_fwd(None, fake(1), fake(2), fake(3), fake(4), fake(5), fake(6), fake(7), ws, None)
    assert st == cola.ERR_INVALID_ARG
