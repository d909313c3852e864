"""The C-ABI library loads, exports every declared symbol, and rejects bad
arguments with status codes before any launch (CPU only: no kernel runs)."""

import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2608_30386_amd import _lib
from paper_2608_30386_amd._lib import LIB, Shape, PlanDesc, PlanOut

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = [os.path.join(ROOT, "include", f) for f in sorted(os.listdir(os.path.join(ROOT, "include")))
           if f.endswith(".h")]

FAKE = C.c_void_p(0x10000)       # aligned, never dereferenced: validation fails first
FAKE_ODD = C.c_void_p(0x10004)   # not 16-byte aligned


def declared_functions():
    names = set()
    for h in HEADERS:
        text = open(h).read()
        names |= set(re.findall(r"^(?:int|const char \*)\s*(dasc_\w+)\s*\(", text, re.M))
    return sorted(names)


def test_every_declared_symbol_is_exported():
    names = declared_functions()
    assert len(names) == 16
    assert set(names) == set(_lib.EXPORTED)
    lib = C.CDLL(_lib.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n


def restore_refresh(shape, layer=0, W=8, n_req=1, init=0, ptrs=None, n_rows=4, n_slots=1, T=1,
                    slice_rows=4, n_pool=1, ws=None, ws_bytes=0):
    p = dict(ckpt=FAKE, src=FAKE, inv=FAKE, states=FAKE, dst=FAKE, k=FAKE, v=FAKE, g=FAKE,
             beta=FAKE)
    p.update(ptrs or {})
    return LIB.dasc_restore_refresh(C.byref(shape) if shape is not None else None, layer,
                                    p["ckpt"], n_slots, p["src"], T, slice_rows, n_rows, p["inv"],
                                    p["states"], n_pool, p["dst"], p["k"], p["v"], p["g"],
                                    p["beta"], n_req, W, init, ws, ws_bytes, None)


def test_restore_refresh_argument_errors():
    E = _lib
    assert restore_refresh(None) == E.DASC_E_INVAL
    assert restore_refresh(kda(dv=6)) == E.DASC_E_SHAPE
    assert restore_refresh(kda(), layer=2) == E.DASC_E_INVAL
    assert restore_refresh(kda(), W=0) == E.DASC_E_INVAL
    assert restore_refresh(kda(), W=E.DASC_MAX_WINDOW + 1) == E.DASC_E_INVAL
    assert restore_refresh(kda(), n_req=0) == E.DASC_E_INVAL
    assert restore_refresh(kda(), init=5) == E.DASC_E_INVAL
    assert restore_refresh(kda(), n_slots=0) == E.DASC_E_INVAL
    assert restore_refresh(kda(), T=0) == E.DASC_E_INVAL
    assert restore_refresh(kda(), n_pool=0) == E.DASC_E_INVAL
    assert restore_refresh(kda(), n_rows=9, T=2, slice_rows=4) == E.DASC_E_INVAL
    assert restore_refresh(kda(L=1, H=1, dk=4, dv=4), n_rows=5) == E.DASC_E_SHAPE
    for name in ("ckpt", "src", "inv", "states", "dst", "k", "v", "g", "beta"):
        assert restore_refresh(kda(), ptrs={name: None}) == E.DASC_E_INVAL, name
    assert restore_refresh(kda(), ptrs={"ckpt": None}, n_rows=0) == E.DASC_E_UNSUPPORTED
    for name in ("ckpt", "states", "k", "v"):
        assert restore_refresh(kda(), ptrs={name: FAKE_ODD}) == E.DASC_E_INVAL, name
    # every argument valid: only dk = dv = 128 has a fused kernel
    assert restore_refresh(kda()) == E.DASC_E_UNSUPPORTED
    assert restore_refresh(kda(dk=128, dv=64)) == E.DASC_E_UNSUPPORTED


def test_tp_permutation_argument_errors():
    E = _lib
    uc = np.zeros(8, np.int32)
    out = np.zeros(8, np.int32)
    r1, r2 = np.zeros(4, np.int64), np.zeros(4, np.int64)
    ptr = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    call = lambda sh, T, u=uc: LIB.dasc_tp_permutation(  # noqa: E731
        C.byref(sh) if sh is not None else None, ptr(u), T, ptr(out), ptr(r1), ptr(r2))
    assert call(None, 2) == E.DASC_E_SHAPE
    assert call(Shape(E.DASC_ARCH_GDN, 2, 4, 3, 16, 16), 1) == E.DASC_E_SHAPE   # H % Hqk
    assert call(kda(L=2, H=4), 0) == E.DASC_E_INVAL
    assert call(kda(L=2, H=4), 3) == E.DASC_E_INVAL                            # Hqk % T
    assert call(kda(L=2, H=4), 2, np.full(8, 17, np.int32)) == E.DASC_E_INVAL   # > dk
    assert call(Shape(E.DASC_ARCH_GDN, 2, 4, 2, 16, 16), 2, np.full(8, 2, np.int32)) == E.DASC_E_INVAL
    assert LIB.dasc_tp_permutation(C.byref(kda(L=2, H=4)), None, 2, ptr(out), ptr(r1),
                                   ptr(r2)) == E.DASC_E_INVAL
    assert call(kda(L=2, H=4), 2) == E.DASC_OK


def test_padded_argument_errors():
    E = _lib
    sh = kda()

    def pp(shape=sh, n=1, r_max=4, n_rows=4, ptrs=None, n_pool=1, n_slots=1):
        p = dict(states=FAKE, src=FAKE, unit=FAKE, off=FAKE, ckpt=FAKE, dst=FAKE)
        p.update(ptrs or {})
        return LIB.dasc_pack_padded(C.byref(shape) if shape is not None else None, p["states"],
                                    n_pool, p["src"], p["unit"], n_rows, p["off"], r_max,
                                    p["ckpt"], n_slots, p["dst"], n, None)

    def rp(shape=sh, n=1, r_max=4, n_rows=4, ptrs=None, n_pool=1, n_slots=1):
        p = dict(ckpt=FAKE, src=FAKE, off=FAKE, inv=FAKE, states=FAKE, dst=FAKE)
        p.update(ptrs or {})
        return LIB.dasc_restore_padded(C.byref(shape) if shape is not None else None, p["ckpt"],
                                       n_slots, p["src"], p["off"], r_max, n_rows, p["inv"],
                                       p["states"], n_pool, p["dst"], n, None)

    for f in (pp, rp):
        assert f(shape=None) == E.DASC_E_SHAPE
        assert f(shape=kda(dv=6)) == E.DASC_E_SHAPE
        assert f(n=-1) == E.DASC_E_INVAL
        assert f(r_max=0) == E.DASC_E_INVAL
        assert f(r_max=1 << 31) == E.DASC_E_INVAL
        assert f(n_pool=0) == E.DASC_E_INVAL
        assert f(n_slots=0) == E.DASC_E_INVAL
        assert f(n_rows=10**6) == E.DASC_E_SHAPE
        assert f(n=0) == E.DASC_OK                                     # nothing to do
    for name in ("states", "src", "unit", "off", "ckpt", "dst"):
        assert pp(ptrs={name: None}) == E.DASC_E_INVAL, name
    for name in ("ckpt", "src", "off", "inv", "states", "dst"):
        assert rp(ptrs={name: None}) == E.DASC_E_INVAL, name
    assert pp(ptrs={"ckpt": FAKE_ODD}) == E.DASC_E_INVAL
    assert rp(ptrs={"states": FAKE_ODD}) == E.DASC_E_INVAL


def test_strerror_total():
    for code in (0, -1, -2, -3, -4, -5, -6, 7, -99):
        assert LIB.dasc_strerror(code)


def kda(L=2, H=4, Hqk=4, dk=16, dv=16):
    return Shape(_lib.DASC_ARCH_KDA, L, H, Hqk, dk, dv)


def pack(shape, n=1, states=FAKE, src=FAKE, unit_row=FAKE, n_rows=4, ckpt=FAKE, dst=FAKE,
         n_pool=1, n_slots=1, T=1, slice_rows=4):
    return LIB.dasc_pack(C.byref(shape) if shape is not None else None, states, n_pool, src,
                         unit_row, n_rows, ckpt, n_slots, dst, T, slice_rows, n, None)


def restore(shape, n=1, ckpt=FAKE, src=FAKE, inv=FAKE, states=FAKE, dst=FAKE, n_rows=4,
            n_pool=1, n_slots=1, T=1, slice_rows=4):
    return LIB.dasc_restore(C.byref(shape) if shape is not None else None, ckpt, n_slots, src, T,
                            slice_rows, n_rows, inv, states, n_pool, dst, n, None)


def test_pack_restore_argument_errors():
    E = _lib
    assert pack(None) == E.DASC_E_SHAPE
    assert pack(kda(dv=6)) == E.DASC_E_SHAPE                     # dv % 4
    assert pack(Shape(7, 1, 1, 1, 4, 4)) == E.DASC_E_SHAPE       # bad arch
    assert pack(kda(H=4, Hqk=3)) == E.DASC_E_SHAPE               # H % Hqk
    assert pack(kda(L=0)) == E.DASC_E_SHAPE
    assert pack(kda(), n=-1) == E.DASC_E_INVAL
    assert pack(kda(), n_pool=0) == E.DASC_E_INVAL
    assert pack(kda(), n_rows=2 * 4 * 16 + 1) == E.DASC_E_SHAPE  # more rows than a state has
    assert pack(kda(), T=2, slice_rows=1) == E.DASC_E_INVAL      # slices do not cover R
    assert pack(kda(), states=None) == E.DASC_E_INVAL
    assert pack(kda(), unit_row=None) == E.DASC_E_INVAL
    assert pack(kda(), states=FAKE_ODD) == E.DASC_E_INVAL
    assert pack(kda(), ckpt=FAKE_ODD) == E.DASC_E_INVAL
    assert pack(kda(), n=0) == E.DASC_OK                         # nothing to do, no launch
    assert pack(kda(), n_rows=0) == E.DASC_OK
    assert restore(None) == E.DASC_E_SHAPE
    assert restore(kda(), inv=None) == E.DASC_E_INVAL
    assert restore(kda(), states=FAKE_ODD) == E.DASC_E_INVAL
    assert restore(kda(), n_slots=0) == E.DASC_E_INVAL
    assert restore(kda(), n=0) == E.DASC_OK


def refresh(shape, layer=0, W=8, n_req=1, init=0, ptrs=None, ws=None, ws_bytes=0, n_pool=1):
    p = dict(inv=FAKE, states=FAKE, slot=FAKE, k=FAKE, v=FAKE, g=FAKE, beta=FAKE)
    p.update(ptrs or {})
    return LIB.dasc_refresh(C.byref(shape) if shape is not None else None, layer, p["inv"],
                            p["states"], n_pool, p["slot"], p["k"], p["v"], p["g"], p["beta"],
                            n_req, W, init, ws, ws_bytes, None)


def test_refresh_argument_errors():
    E = _lib
    assert refresh(None) == E.DASC_E_INVAL
    assert refresh(kda(dv=6)) == E.DASC_E_SHAPE
    assert refresh(kda(), W=0) == E.DASC_E_INVAL
    assert refresh(kda(), W=-3) == E.DASC_E_INVAL
    assert refresh(kda(), W=E.DASC_MAX_WINDOW + 1) == E.DASC_E_INVAL
    assert refresh(kda(), layer=2) == E.DASC_E_INVAL
    assert refresh(kda(), layer=-1) == E.DASC_E_INVAL
    assert refresh(kda(), n_req=0) == E.DASC_E_INVAL
    assert refresh(kda(), init=5) == E.DASC_E_INVAL
    assert refresh(kda(), n_pool=0) == E.DASC_E_INVAL
    for name in ("inv", "states", "slot", "k", "v", "g", "beta"):
        assert refresh(kda(), ptrs={name: None}) == E.DASC_E_INVAL, name
    assert refresh(kda(), ptrs={"states": FAKE_ODD}) == E.DASC_E_INVAL
    assert refresh(kda(dk=8)) == E.DASC_E_UNSUPPORTED            # no kernel for dk = 8
    assert refresh(kda(dv=512)) == E.DASC_E_UNSUPPORTED
    gdn_bad = Shape(_lib.DASC_ARCH_GDN, 1, 4, 3, 16, 16)
    assert refresh(gdn_bad) == E.DASC_E_SHAPE
    need = C.c_size_t(99)
    assert LIB.dasc_refresh_workspace_bytes(C.byref(kda()), 1, 0, C.byref(need)) == E.DASC_E_INVAL
    assert LIB.dasc_refresh_workspace_bytes(C.byref(kda()), 2, 64, C.byref(need)) == E.DASC_OK
    assert need.value == 0


def select(shape, kernel, **kw):
    p = dict(inv=FAKE, states=FAKE, slot=FAKE, k=FAKE, v=FAKE, g=FAKE, beta=FAKE)
    p.update(kw.pop("ptrs", {}))
    ws, ws_bytes = kw.pop("ws", None), kw.pop("ws_bytes", 0)
    W, n_req = kw.pop("W", 8), kw.pop("n_req", 1)
    return LIB.dasc_refresh_select(C.byref(shape) if shape is not None else None, 0, p["inv"],
                                   p["states"], 1, p["slot"], p["k"], p["v"], p["g"], p["beta"],
                                   n_req, W, 0, ws, ws_bytes, kernel, None)


def test_refresh_select_argument_errors():
    # the kernel choice is an explicit argument (no process-wide switch)
    E = _lib
    assert select(kda(), 3) == E.DASC_E_INVAL                          # unknown kernel
    assert select(kda(), -1) == E.DASC_E_INVAL
    assert select(None, E.DASC_REFRESH_KERNEL_COLUMN) == E.DASC_E_INVAL
    # the channel-wise chunked kernel exists for dk = dv = 128 only
    assert select(kda(dk=16, dv=16), E.DASC_REFRESH_KERNEL_CHANNEL_WY) == E.DASC_E_UNSUPPORTED
    assert select(kda(dk=64, dv=128), E.DASC_REFRESH_KERNEL_CHANNEL_WY) == E.DASC_E_UNSUPPORTED
    # AUTO on GDN heads at 128 asks for the workspace, like dasc_refresh
    gdn = Shape(_lib.DASC_ARCH_GDN, 1, 4, 2, 128, 128)
    assert select(gdn, E.DASC_REFRESH_KERNEL_AUTO, W=64, n_req=2) == E.DASC_E_WORKSPACE
    for name in ("inv", "states", "slot", "k", "v", "g", "beta"):
        assert select(kda(), E.DASC_REFRESH_KERNEL_COLUMN, ptrs={name: None}) == E.DASC_E_INVAL
    assert os.path.basename(HEADERS[0]) == "dasc.h" and len(HEADERS) >= 2
    for src in ("refresh.hip", "refresh_wy.hip", "refresh_wy_gdn.hip"):
        text = open(os.path.join(ROOT, "paper_2608_30386_amd", "csrc", src)).read()
        assert "getenv" not in text, src


def test_refresh_noalloc_argument_errors():
    # host-side checks of the entry point that allocates nothing: arguments are those of
    # dasc_refresh, and a request whose workspace would exceed the limit that the interface
    # states is refused before anything touches the device
    E = _lib

    def na(shape, n_req=1, W=8, ptrs=None):
        p = dict(inv=FAKE, states=FAKE, slot=FAKE, k=FAKE, v=FAKE, g=FAKE, beta=FAKE)
        p.update(ptrs or {})
        return LIB.dasc_refresh_noalloc(C.byref(shape) if shape is not None else None, 0,
                                        p["inv"], p["states"], 1, p["slot"], p["k"], p["v"],
                                        p["g"], p["beta"], n_req, W, 0, None)

    assert na(None) == E.DASC_E_INVAL
    assert na(kda(), W=0) == E.DASC_E_INVAL
    assert na(kda(), n_req=0) == E.DASC_E_INVAL
    assert na(kda(dv=6)) == E.DASC_E_SHAPE
    for name in ("inv", "states", "slot", "k", "v", "g", "beta"):
        assert na(kda(), ptrs={name: None}) == E.DASC_E_INVAL, name
    gdn = Shape(_lib.DASC_ARCH_GDN, 1, 32, 16, 128, 128)
    need = C.c_size_t(0)
    assert LIB.dasc_refresh_workspace_bytes(C.byref(gdn), 3, 8192, C.byref(need)) == E.DASC_OK
    assert need.value > E.DASC_NOALLOC_SCRATCH_BYTES
    assert na(gdn, n_req=3, W=8192) == E.DASC_E_SCRATCH
    assert b"scratch" in LIB.dasc_strerror(E.DASC_E_SCRATCH)
    # the largest request that fits: 16 requests x 32 heads x 32 chunks x 4 KiB = 64 MiB
    assert LIB.dasc_refresh_workspace_bytes(C.byref(gdn), 16, 1024, C.byref(need)) == E.DASC_OK
    assert need.value == E.DASC_NOALLOC_SCRATCH_BYTES


def test_plan_padded_geometry_fields():
    # App. B Scheme 1 geometry comes out of the planner: per-layer offsets in rows and
    # the rows every layer reserves; a NULL layer_off_rows member is skipped
    E = _lib
    sh = Shape(_lib.DASC_ARCH_GDN, 3, 4, 2, 8, 4)
    keep = np.array([[1, 0, 0, 1], [0, 0, 0, 0], [1, 1, 1, 0]], bool)
    g = np.where(keep, np.log(1e-3) / 1000.0, np.log(1e-3) / 2.0).reshape(-1)
    out = PlanOut()
    rows = np.full(4, -9, np.int32)
    out.layer_off_rows = rows.ctypes.data_as(C.POINTER(C.c_int32))
    desc = PlanDesc(sh, 0, 0, 16, 1, 1e-3, 0)
    assert LIB.dasc_plan(C.byref(desc), g.ctypes.data, C.byref(out)) == E.DASC_OK
    np.testing.assert_array_equal(rows, [0, 16, 16, 40])                 # 2, 0, 3 heads of 8 rows
    assert out.r_max_rows == 24 and out.n_rows == 40
    out2 = PlanOut()
    assert LIB.dasc_plan(C.byref(desc), g.ctypes.data, C.byref(out2)) == E.DASC_OK
    assert out2.r_max_rows == 24


def test_gdn_refresh_workspace():
    # GDN heads at dk = dv = 128 are asked for 4 KiB per (request, head, 32-token chunk), which
    # the interface states and the kernels leave untouched
    E = _lib
    gdn = Shape(_lib.DASC_ARCH_GDN, 2, 32, 16, 128, 128)
    need = C.c_size_t(0)
    for n_req, W in ((8, 1024), (1, 1), (3, 33), (2, 2048)):
        assert LIB.dasc_refresh_workspace_bytes(C.byref(gdn), n_req, W, C.byref(need)) == E.DASC_OK
        assert need.value == n_req * 32 * (-(-W // 32)) * 4096
    # other shapes need none
    for sh in (Shape(_lib.DASC_ARCH_GDN, 1, 4, 2, 64, 64), kda(dk=128, dv=128)):
        assert LIB.dasc_refresh_workspace_bytes(C.byref(sh), 4, 256, C.byref(need)) == E.DASC_OK
        assert need.value == 0
    W, n_req = 64, 2
    full = n_req * 32 * 2 * 4096
    assert refresh(gdn, W=W, n_req=n_req) == E.DASC_E_WORKSPACE                       # none
    assert refresh(gdn, W=W, n_req=n_req, ws=FAKE, ws_bytes=full - 1) == E.DASC_E_WORKSPACE
    assert refresh(gdn, W=W, n_req=n_req, ws=None, ws_bytes=full) == E.DASC_E_WORKSPACE
    assert refresh(gdn, W=W, n_req=n_req, ws=FAKE_ODD, ws_bytes=full) == E.DASC_E_INVAL
    assert restore_refresh(gdn, W=W, n_req=n_req) == E.DASC_E_WORKSPACE
    assert restore_refresh(gdn, W=W, n_req=n_req, ws=FAKE_ODD, ws_bytes=full) == E.DASC_E_INVAL


def test_plan_argument_errors():
    E = _lib
    sh = kda(L=1, H=2, Hqk=2, dk=4, dv=4)
    g = np.full(8, -0.5)
    out = PlanOut()

    def plan(desc, gg=g):
        return LIB.dasc_plan(C.byref(desc), gg.ctypes.data, C.byref(out))

    ok = PlanDesc(sh, 0, 0, 16, 1, 1e-3, 0)
    assert plan(ok) == E.DASC_OK
    assert LIB.dasc_plan(None, g.ctypes.data, C.byref(out)) == E.DASC_E_INVAL
    assert LIB.dasc_plan(C.byref(ok), None, C.byref(out)) == E.DASC_E_INVAL
    assert plan(PlanDesc(sh, 0, 0, 16, 1, 0.0, 0)) == E.DASC_E_INVAL        # eps
    assert plan(PlanDesc(sh, 0, 0, 16, 1, 1.0, 0)) == E.DASC_E_INVAL
    assert plan(PlanDesc(sh, 0, 0, -1, 1, 1e-3, 0)) == E.DASC_E_INVAL       # w_max
    assert plan(PlanDesc(sh, 0, 0, 16, 0, 1e-3, 0)) == E.DASC_E_INVAL       # n_ranks
    assert plan(PlanDesc(sh, 9, 0, 16, 1, 1e-3, 0)) == E.DASC_E_INVAL       # keep mode
    assert plan(PlanDesc(sh, 1, 5, 16, 1, 1e-3, 0)) == E.DASC_E_INVAL       # k > dk
    assert plan(PlanDesc(sh, 0, 0, 16, 1, 1e-3, -1)) == E.DASC_E_INVAL      # conv bytes
    gdn = Shape(_lib.DASC_ARCH_GDN, 1, 2, 2, 4, 4)
    assert plan(PlanDesc(gdn, 1, 1, 16, 1, 1e-3, 0), np.full(2, -0.5)) == E.DASC_E_SHAPE
    for bad in (0.0, 0.3, np.inf, -np.inf, np.nan):
        gb = g.copy()
        gb[3] = bad
        assert plan(ok, gb) == E.DASC_E_INVAL, bad
    slots = C.c_int64()
    assert LIB.dasc_matched_slots(100, 0, C.byref(slots)) == E.DASC_E_INVAL
    assert LIB.dasc_matched_slots(-1, 10, C.byref(slots)) == E.DASC_E_INVAL
    assert LIB.dasc_static_log_decay(None, None, -0.3, 1, g.ctypes.data) == E.DASC_E_INVAL


def test_binding_rejects_host_tensors():
    import torch
    import paper_2608_30386_amd as D

    sh = D.Shape("kda", 1, 2, 2, 16, 16)
    x = torch.zeros(4)
    with pytest.raises((TypeError, ValueError)):
        D.dasc_pack(sh, x, x, x, x, x)
    st = torch.zeros(1, 1, 2, 16, 16)
    ck = torch.zeros(1, 1, 16)
    idx = torch.zeros(1, dtype=torch.int32)
    with pytest.raises(TypeError, match="device tensor"):
        D.dasc_pack(sh, st, idx, idx, ck, idx)


def test_code_independence():
    """The library package and the oracle never import each other."""
    pkg = os.path.join(ROOT, "paper_2608_30386_amd")
    orc = os.path.join(ROOT, "oracle")
    for d, bad in ((pkg, r"^\s*(from|import)\s+oracle\b"), (orc, r"paper_2608_30386_amd")):
        for base, _, files in os.walk(d):
            for f in files:
                if f.endswith((".py", ".hip", ".cpp", ".h")):
                    text = open(os.path.join(base, f)).read()
                    assert not re.search(bad, text, re.M), (f, bad)
    wl = os.path.join(ROOT, "workloads")
    for f in os.listdir(wl):
        if f.endswith(".py"):
            text = open(os.path.join(wl, f)).read()
            assert not re.search(r"^\s*(from|import)\s+(oracle|paper_2608_30386_amd)\b", text, re.M)


def test_shape_copies_and_pickles_after_use():
    # a Shape keeps its C struct once a call has used it; copies and pickles carry the fields only
    import copy
    import dataclasses
    import pickle

    import paper_2608_30386_amd as D

    a = D.Shape("gdn", 2, 4, 2, 16, 32)
    assert a.rows == 128 and a._ref is a._ref
    for b in (copy.copy(a), copy.deepcopy(a), pickle.loads(pickle.dumps(a))):
        assert b == a and hash(b) == hash(a) and b.rows == 128
    assert dataclasses.replace(a, dk=32).rows == 256
