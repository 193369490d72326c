"""The marshalling of GEMM calls in C (csrc/pycall.cpp): every argument of every form arrives at the entry point as ctypes
delivers it, and what it does not take is left to ctypes."""
import ctypes
import os
import sysconfig

import numpy as np
import pytest

import paper_2003_06795_amd.binding as ks

HEAD = ks._GEMM[:13]
TYPES = {0: ks._GEMM, 1: [ks._i] + ks._GEMM, 2: [ks._i, ks._i] + ks._GEMM, 3: [ks._i, ks._i] + HEAD + [ks._p] + ks._GEMM[13:],
         4: [ks._i, ks._i] + ks._GEMM[:-1] + [ks._p, ctypes.c_size_t, ks._p]}
ARGS = (1, 0, 5, 6, 2 ** 40, 1.5, 4096, 7, 8192, 8, -0.25, 12288, 9, 3, 11, -12, 13)      # transA .. strideC


class Operand:
    def data_ptr(self):
        return 4096


@pytest.fixture()
def module():
    ks.lib()
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        pytest.skip("the module is not built without Python's C headers")
    from paper_2003_06795_amd import _pycall
    return _pycall


@pytest.mark.parametrize("form", sorted(TYPES))
def test_every_argument_arrives(module, form):
    got = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int, *TYPES[form])(lambda *a: got.append(a) or -7)
    address = ctypes.cast(entry, ctypes.c_void_p).value
    args = list(ARGS)
    args[6] = Operand()
    rc = module.gemm(address, form, 2, 33, *args, 77, 555 if form >= 3 else None, 666 if form == 4 else 0)
    want = list(ARGS) + [77]
    if form == 3:
        want.insert(13, 555)
    if form == 4:
        want[-1:-1] = [555, 666]
    want = {0: [], 1: [33]}.get(form, [2, 33]) + want
    assert rc == -7 and list(got[0]) == want


@pytest.mark.parametrize("at,value", [(0, 1.0), (0, 2 ** 40), (2, np.int64(5)), (2, 2 ** 70), (5, True), (5, 2 ** 2000), (5, np.float64(1.0)),
                                      (6, -1), (6, 2 ** 64), (6, object()), (11, np.int64(8)), (12, None), (16, "1")])
def test_what_is_left_to_ctypes(module, at, value):
    entry = ctypes.CFUNCTYPE(ctypes.c_int, *TYPES[0])(lambda *a: 0)
    args = list(ARGS)
    args[at] = value
    assert module.gemm(ctypes.cast(entry, ctypes.c_void_p).value, 0, 0, 0, *args, 77, None, 0) is NotImplemented


class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


def test_whole_scalars_and_stream_objects_are_taken(module):
    """alpha = 1, beta = 0 and a stream object are what many programs pass."""
    got = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int, *TYPES[0])(lambda *a: got.append(a) or 0)
    args = list(ARGS)
    args[5], args[10] = 2, 0
    assert module.gemm(ctypes.cast(entry, ctypes.c_void_p).value, 0, 0, 0, *args, Stream(77), None, 0) == 0
    assert list(got[0]) == args + [77]
    args[5], args[10] = -(2 ** 53 + 1), 2 ** 24 + 1                       # rounded as ctypes rounds them
    assert module.gemm(ctypes.cast(entry, ctypes.c_void_p).value, 0, 0, 0, *args, 77, None, 0) == 0
    assert got[1][5] == ctypes.c_float(args[5]).value and got[1][10] == ctypes.c_float(args[10]).value


@pytest.mark.parametrize("stream", [object(), Stream(None), Stream(-1), Stream(np.int64(5)), "1", True])
def test_an_unusual_stream_is_seen_before_the_operands(module, stream):
    class Counted(Operand):
        asked = 0

        def data_ptr(self):
            Counted.asked += 1
            return 4096
    entry = ctypes.CFUNCTYPE(ctypes.c_int, *TYPES[0])(lambda *a: 0)
    args = list(ARGS)
    args[6] = Counted()
    assert module.gemm(ctypes.cast(entry, ctypes.c_void_p).value, 0, 0, 0, *args, stream, None, 0) is NotImplemented
    assert Counted.asked == 0


def test_errors_of_an_operand_and_unusual_calls(module):
    class Broken:
        def data_ptr(self):
            raise KeyError("gone")
    with pytest.raises(KeyError):
        ks.gemm_f32(0, 0, 4, 4, 4, 1.0, Broken(), 4, 4096, 4, 0.0, 4096, 4)
    with pytest.raises(ctypes.ArgumentError):
        ks.gemm_f32(0, 0, 4.0, 4, 4, 1.0, 4096, 4, 4096, 4, 0.0, 4096, 4, stream=0)
    with pytest.raises(TypeError):
        ks.gemm_f32_with_kernel(None, 0, 0, 4, 4, 4, 1.0, 4096, 4, 4096, 4, 0.0, 4096, 4, stream=0)
    for kid in (0, np.int32(0), 0.0):                                         # nothing to do: no device needed
        ks.gemm_f32_with_kernel(kid, 0, 0, 0, 4, 4, 1, None, 4, None, 4, 0, None, 4, stream=0)
    with pytest.raises(ks.KsError):
        ks.gemm_bias(ks.F32, -1, 0, 0, 4, 4, 4, 1.0, None, 4, None, 4, 0.0, None, 4, None, stream=0)


@pytest.mark.parametrize("missing", ["headers", "compiler"])
def test_the_library_builds_without_the_module(monkeypatch, tmp_path, capsys, missing):
    """No Python.h or no g++: the build goes on, and no module of an older source stays behind."""
    from paper_2003_06795_amd import build as lib_build
    stale = tmp_path / "_pycall.so"
    stale.write_bytes(b"older")
    monkeypatch.setattr(lib_build, "PYCALL", str(stale))
    if missing == "headers":
        monkeypatch.setattr(lib_build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    else:
        monkeypatch.setenv("PATH", str(tmp_path))
    assert lib_build.build_pycall(force=True) is None
    assert os.listdir(tmp_path) == [] and "ctypes" in capsys.readouterr().out
