"""The marshalling module of the Python binding (csrc/kvc_call.c): every argument of every entry point arrives in its place, as the
ctypes signature of the library function has it; refusals and odd forms of arguments.  Host only: the library's functions are
replaced by recorders."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2605_16439_amd import kvcapsule as kv

SHAPE = kv.make_shape(2, 4, 2, 128, 16, 3, 5, torch.bfloat16)


@pytest.fixture
def recorded():
    """kv's entry points bound to recorders; yields the list of (name, arguments) they saw."""
    L, seen, keep = kv.lib(), [], []
    for name in kv._BOUND:
        types = [ctypes.c_void_p if hasattr(t, "_type_") and not isinstance(t._type_, str) else t for t in getattr(L, name).argtypes]
        proto = ctypes.CFUNCTYPE(ctypes.c_int, *types)
        keep.append(proto(lambda *a, name=name: (seen.append((name, a)), -2)[1]))
    native = kv._call()
    native.bind(*(ctypes.cast(f, ctypes.c_void_p).value for f in keep))
    yield seen
    kv._native = None
    kv._call()


class Stream:
    cuda_stream = 0x7f0000001230


def tensors(*names):
    return {n: torch.zeros(2, 2, 3, 8, 128, dtype=torch.bfloat16) for n in names}


def params():
    t = [torch.zeros(8) for _ in range(6)]
    return kv.make_params(*t), t


def ptr(t):
    return None if t is None else t.data_ptr()


@pytest.mark.parametrize("lse,new", [(False, True), (True, False)])
def test_decode_calls_pass_every_argument(lse, new, recorded):
    a = tensors("q", "Kc", "Vc", "Kt", "Vt", "kn", "vn", "out")
    p, keep = params()
    if not new:
        a["kn"] = a["vn"] = a["Kt"] = None
    L = torch.zeros(8) if lse else None
    ws = torch.zeros(1024, dtype=torch.uint8)[3:]
    off = -ws.data_ptr() % 256
    ni, tl = torch.zeros(2, dtype=torch.int32), torch.ones(2, dtype=torch.int32)
    common = dict(softmax_scale=0.25, out=a["out"], lse_out=L, stream=Stream, check=False)
    A = [a[k] for k in ("q", "Kc", "Vc", "Kt", "Vt")]
    w = (ws.data_ptr() + off, ws.numel() - off, Stream.cuda_stream)
    for generic in (False, True):
        assert kv.kvc_reconstruct_attend_decode(SHAPE, p, *A, 7, 9, a["kn"], a["vn"], workspace=ws, generic=generic, **common) == -2
    kv.kvc_reconstruct_attend_decode_ragged(SHAPE, p, *A, ni, tl, np.int64(9), a["kn"], a["vn"], workspace=ws, **common)
    kv.kvc_reconstruct_attend_decode_static(SHAPE, p, *A, torch.tensor(7), 9.0, a["kn"], a["vn"], **common)
    kv.kvc_static_attend_decode(SHAPE, *A, 7, 9, a["kn"], a["vn"], workspace=ws, **common)
    s, pp = ctypes.addressof(SHAPE), ctypes.addressof(p)
    t5, new2, o = tuple(ptr(x) for x in A), (ptr(a["kn"]), ptr(a["vn"])), (0.25, ptr(a["out"]), ptr(L))
    assert recorded == [
        ("kvc_reconstruct_attend_decode", (s, pp) + t5 + (7, 9) + new2 + o + w),
        ("kvc_reconstruct_attend_decode_generic", (s, pp) + t5 + (7, 9) + new2 + o + w),
        ("kvc_reconstruct_attend_decode_ragged", (s, pp) + t5 + (ni.data_ptr(), tl.data_ptr(), 9) + new2 + o + w),
        ("kvc_reconstruct_attend_decode_static", (s, pp) + t5 + (7, 9) + new2 + o + w[2:]),
        ("kvc_static_attend_decode", (s,) + t5 + (7, 9) + new2 + o + w)]


def test_prefill_and_full_cache_calls_pass_every_argument(recorded):
    p, keep = params()
    K, V = (torch.zeros(2, 40, 2, 128, dtype=torch.bfloat16).transpose(1, 2) for _ in range(2))
    Kc, Vc, W, q, kn, vn, out = (torch.zeros(2, 4, 128, dtype=torch.bfloat16) for _ in range(7))
    ws = torch.zeros(777, dtype=torch.uint8)
    off = -ws.data_ptr() % 256
    w = (ws.data_ptr() + off, 777 - off, Stream.cuda_stream)
    st = (40 * 256, 128, 256)
    for generic in (False, True):
        kv.kvc_compress(SHAPE, p, K, V, 13, Kc, Vc, ws, stream=Stream, generic=generic, check=False)
    kv.kvc_mlp_hidden(SHAPE, W, 2, Kc, Vc, stream=Stream, check=False)
    kv.kvc_attend_full_decode(q, K, V, 31, kn, vn, 0.5, out, None, ws, stream=Stream, check=False)
    s, pp = ctypes.addressof(SHAPE), ctypes.addressof(p)
    body = (s, pp, K.data_ptr(), V.data_ptr()) + st + (13, 40, Kc.data_ptr(), Vc.data_ptr()) + w
    assert recorded == [
        ("kvc_compress", body), ("kvc_compress_generic", body),
        ("kvc_mlp_hidden", (s, W.data_ptr(), 2, Kc.data_ptr(), Vc.data_ptr(), Stream.cuda_stream)),
        ("kvc_attend_full_decode", (2, 4, 2, 128, kv.KVC_BF16, q.data_ptr(), K.data_ptr(), V.data_ptr()) + st +
         (31, 40, kn.data_ptr(), vn.data_ptr(), 0.5, out.data_ptr(), None) + w)]


def test_refusals(recorded):
    p, keep = params()
    K = torch.zeros(2, 2, 40, 128, dtype=torch.bfloat16)
    x, ws = torch.zeros(8), torch.zeros(512, dtype=torch.uint8)
    with pytest.raises(AssertionError):
        kv.kvc_compress(SHAPE, p, K, K.transpose(1, 2), 0, x, x, ws, stream=Stream)
    with pytest.raises(AssertionError):
        kv.kvc_compress(SHAPE, p, K.transpose(2, 3), K.transpose(2, 3), 0, x, x, ws, stream=Stream)
    with pytest.raises(TypeError):
        kv.kvc_mlp_hidden(p, x, 0, x, x, stream=Stream)                  # a structure of another size
    with pytest.raises(AttributeError):
        kv.kvc_mlp_hidden(SHAPE, 1234, 0, x, x, stream=Stream)           # not a tensor
    with pytest.raises(ValueError):
        kv.kvc_static_attend_decode(SHAPE, x, x, x, x, x, "seven", 9, x, x, 0.0, x, None, ws, stream=Stream)
    with pytest.raises(TypeError):
        kv.kvc_static_attend_decode(SHAPE, x, x, x, x, x, 7, 9, x, x, "0.0", x, None, ws, stream=Stream)
    assert recorded == []
    with pytest.raises(kv.KvcError) as e:
        kv.kvc_compress(SHAPE, p, K, K, 0, x, x, ws, stream=Stream)
    assert e.value.status == -2
