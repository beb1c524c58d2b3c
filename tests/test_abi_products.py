"""The shared-launch products of the C ABI reject bad arguments on the host, before anything is
launched, with the codes of the calls they stand for."""

import ctypes
import math
import os

import pytest

import paper_2608_15473_amd as qf
from paper_2608_15473_amd.binding import DecodeDesc, LinearArgs, load_library

pytestmark = pytest.mark.skipif(not os.path.exists(qf.LIB_PATH), reason="libqfattn.so not built")
A = ctypes.c_void_p(4096)


def _args(rows=1, n=64, k=512, pro=0, x=4096, gain=4096, out=4096):
    return LinearArgs(rows, n, k, pro, x, 4096, gain, 1e-6, None, out, n, None)


def test_linear_pair():
    f = load_library().qf_linear_pair
    ok, none = _args(), _args(rows=0)
    assert f(None, ctypes.byref(ok), None) == qf.QF_EINVAL
    assert f(ctypes.byref(ok), None, None) == qf.QF_EINVAL
    assert f(ctypes.byref(_args(rows=9)), ctypes.byref(ok), None) == qf.QF_EUNSUPPORTED
    assert f(ctypes.byref(ok), ctypes.byref(_args(out=None)), None) == qf.QF_EINVAL
    assert f(ctypes.byref(_args(x=4104)), ctypes.byref(ok), None) == qf.QF_EALIGN
    assert f(ctypes.byref(none), ctypes.byref(none), None) == qf.QF_OK


def test_linear_beside_merge():
    f = load_library().qf_linear_beside_merge
    ok, none = _args(), _args(rows=0)

    def call(p=ok, batch=1, hq=4, d=128, shards=2, po=A, pl=A, mo=A, ml=A):
        return f(None if p is None else ctypes.byref(p), batch, hq, d, shards, po, pl, mo, ml, None)

    assert call(p=None) == qf.QF_EINVAL
    assert call(p=_args(k=60)) == qf.QF_EUNSUPPORTED
    assert call(batch=-1) == qf.QF_EINVAL and call(hq=0) == qf.QF_EINVAL
    assert call(hq=4097) == qf.QF_EINVAL and call(shards=0) == qf.QF_EINVAL
    assert call(d=64) == qf.QF_EUNSUPPORTED
    assert call(mo=None) == qf.QF_EINVAL and call(ml=None) == qf.QF_EINVAL
    assert call(mo=ctypes.c_void_p(4104)) == qf.QF_EALIGN
    assert call(p=none, batch=0, po=None, pl=None, mo=None, ml=None) == qf.QF_OK


def test_linear_attn_current():
    f = load_library().qf_linear_attn_current

    def call(batch=1, hq=4, hkv=2, p=None, num_pages=8, over=()):
        d = DecodeDesc(batch, hq, hkv, 128, 16, 8, num_pages, 1, 1 / math.sqrt(128))
        a = dict(mo=A, ml=A, q=A, k=A, v=A, attn=A, lse=None, kc=A, vc=A, bt=A, ctx=A, st=None)
        a.update(over)
        p = _args(rows=batch) if p is None else p
        return f(ctypes.byref(d), *a.values(), ctypes.byref(p), None)

    assert call(batch=2) == qf.QF_EUNSUPPORTED
    assert call(hq=3, hkv=2) == qf.QF_EINVAL
    assert call(p=_args(k=1024)) == qf.QF_EINVAL                  # not Hq * D inputs
    assert call(p=_args(rows=2)) == qf.QF_EINVAL
    assert call(p=_args(pro=qf.QF_LINEAR_RMS_NORM)) == qf.QF_EINVAL
    assert call(p=_args(x=8192)) == qf.QF_EINVAL                  # not the attention
    for name in ("mo", "ml", "q", "k", "v", "kc", "vc", "ctx"):
        assert call(over={name: None}) == qf.QF_EINVAL, name
    assert call(over={"q": ctypes.c_void_p(4104)}) == qf.QF_EALIGN
    assert call(over={"ctx": ctypes.c_void_p(4098)}) == qf.QF_EALIGN
    assert call(over={"bt": None}, num_pages=7) == qf.QF_EINVAL
    assert call(batch=0) == qf.QF_OK
