"""csrc/py_calls.cpp hands every argument to the C function in its place and width, and its status back."""
import ctypes
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
I, P, Z = ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t
FORMS = {"biq_gemm": [P] * 4 + [I] * 5 + [P, Z, P], "biq_query": [P] * 4 + [I] * 5 + [P, Z, P],
         "biq_gemm_noalloc": [P] * 4 + [I] * 5 + [P], "biq_pack": [P] * 2 + [I] * 4 + [P],
         "biq_quantize": [P] * 3 + [I] * 3 + [P], "biq_build_lut": [P] * 2 + [I] * 3 + [P],
         "biq_gemm_grouped": [P, I, I, P], "biq_lstm_cell": [P] * 7 + [I] * 5 + [P]}


class Stream:
    cuda_stream = 0x7654321012345670


@pytest.fixture()
def recorded(monkeypatch):
    from paper_2005_09904_amd import binding
    from paper_2005_09904_amd.build import build_library, is_stale

    if is_stale():
        build_library()
    lib = binding.load_library()
    seen, status, keep = [], [0], []

    def recorder(name, form):
        def f(*args):
            seen.append((name, [a or 0 for a in args]))
            return status[0]
        keep.append(ctypes.CFUNCTYPE(I, *form)(f))
        return ctypes.cast(keep[-1], P).value

    for name, form in FORMS.items():
        assert getattr(lib, name).restype is I and len(getattr(lib, name).argtypes) == len(form)
    from paper_2005_09904_amd._calls import Calls

    monkeypatch.setattr(binding, "_calls", Calls({n: recorder(n, f) for n, f in FORMS.items()}, binding._check,
                                                 binding._as_int, lambda: 0x1122334455667788))
    return binding, seen, status, keep


def test_every_argument_arrives(recorded):
    b, seen, status, _ = recorded
    t = [torch.zeros(i + 3) for i in range(7)]
    p = [x.data_ptr() for x in t]
    ws = torch.zeros(5, 7, dtype=torch.float64)
    S, D = Stream.cuda_stream, 0x1122334455667788
    ints = [3, -5, 2**31 - 1, np.int64(11), True]     # (an int keeps its low 32 bits, as with ctypes)
    want = [3, -5, 2**31 - 1, 11, 1]
    calls = [
        ("biq_gemm", lambda: b.biq_gemm(*t[:4], *ints, workspace=ws, stream=Stream()), p[:4] + want + [ws.data_ptr(), 280, S]),
        ("biq_gemm", lambda: b.biq_gemm(*t[:4], *ints), p[:4] + want + [0, 0, D]),
        ("biq_query", lambda: b.biq_query(*t[:4], *ints, ws), p[:4] + want + [ws.data_ptr(), 280, D]),
        ("biq_gemm_noalloc", lambda: b.biq_gemm_noalloc(*t[:4], *ints), p[:4] + want + [D]),
        ("biq_pack", lambda: b.biq_pack(*t[:2], *ints[:4], stream=Stream()), p[:2] + want[:4] + [S]),
        ("biq_quantize", lambda: b.biq_quantize(*t[:3], 2**32 + 9, *ints[1:3]), p[:3] + [9] + want[1:3] + [D]),
        ("biq_build_lut", lambda: b.biq_build_lut(None, t[1], *ints[:3]), [0, p[1]] + want[:3] + [D]),
        ("biq_lstm_cell", lambda: b.biq_lstm_cell(*t, *ints), p + want + [D]),
        ("biq_gemm", b.PreparedGemm(*t[:4], *ints, workspace=ws), p[:4] + want + [ws.data_ptr(), 280, D]),
        ("biq_lstm_cell", b.PreparedLstmCell(*t, *ints, stream=Stream()), p + want + [S]),
    ]
    for name, call, args in calls:
        for status[0] in (0, -2):
            del seen[:]
            if status[0]:
                with pytest.raises(b.BiqError, match=name) as e:
                    call()
                assert e.value.status == -2
            else:
                assert call() is None
            assert seen == [(name, args)]
    status[0] = 0
    group = b.PreparedGroup([(*t[:4], 1, 2, 3, 4)] * 3, 8)
    group()
    assert seen[-1] == ("biq_gemm_grouped", [ctypes.addressof(group._array), 3, 8, D])


def test_what_is_no_integer_or_tensor_is_refused(recorded):
    b, seen, _, _ = recorded
    t = torch.zeros(3)
    for bad in (1.5, "1", None):
        with pytest.raises(ctypes.ArgumentError):
            b.biq_pack(t, t, bad, 1, 1, 8)
    with pytest.raises(AttributeError):
        b.biq_pack(5, t, 1, 1, 1, 8)
    with pytest.raises(TypeError):
        b.PreparedGemm(t, t, t, t, 1, 1, 1, 1, 8)._call(1)
    assert not seen


def test_the_module_is_the_running_interpreters(recorded, monkeypatch):
    """Its file name carries the interpreter's tag, so that another interpreter builds its own."""
    import sysconfig

    import paper_2005_09904_amd._calls as calls
    from paper_2005_09904_amd import build

    b, _, _, _ = recorded
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.samefile(calls.__file__, build.CALLS_PATH) and build.CALLS_PATH.endswith("_calls" + suffix)
    assert sys.implementation.cache_tag.replace("-", "") in suffix.replace("-", "") and not build.is_stale()
    other = build.CALLS_PATH[:-len(suffix)] + ".cpython-399-x86_64-linux-gnu.so"      # what another one looks for
    monkeypatch.setattr(build, "CALLS_PATH", other)
    monkeypatch.setattr(b, "CALLS_PATH", other)
    assert build.is_stale()
    with pytest.raises(FileNotFoundError, match="cpython-399"):
        b.load_library(build.LIB_PATH)
