"""The extension that marshals the calls of every step (csrc/bns_call.cpp): what the library's functions receive, argument by
argument, against the values that the binding was given; what is accepted and what is refused, and how, as by ctypes, which the extension
leaves unusual arguments to."""
import ctypes as C
import importlib.machinery
import inspect
import os
import subprocess
import sys
import types

import numpy as np
import pytest

from paper_1810_10962_amd import bns

NAMES = ("forward", "backward", "forward_mixed", "backward_mixed", "inference")
SHAPE = bns.make_shape(5, 6, 7, 8, "bf16", "nhwc")
SPEC = bns.make_spec(bns.BNS_FS, 1, 2, 3, 0, 2 ** 32 - 2, 9)


class Tensor:
    def __init__(self, address, nbytes=0):
        self.address, self.nbytes = address, nbytes

    def data_ptr(self):
        return self.address


@pytest.fixture(params=["extension", "ctypes"])
def received(request, monkeypatch):
    """Calls received by stand-ins for the five functions, which answer with the status in `received.status`: through the extension, and
    with everything left to ctypes."""
    class Calls(list):
        status = 0
    calls = Calls()

    def stand_in(name):
        restype, argtypes = bns._PROTOS["bns_" + name]

        def fn(*args):
            plain = [bytes(a.contents) if isinstance(a, C._Pointer) else a for a in args]
            calls.append((name, plain))
            return calls.status
        return C.CFUNCTYPE(restype, *argtypes)(fn)

    bns.load()
    keep = [stand_in(n) for n in NAMES]
    bns._call.bind(bns.bns_shape, bns.bns_spec, *(C.cast(f, C.c_void_p).value for f in keep))
    monkeypatch.setattr(bns, "_lib", types.SimpleNamespace(bns_status_string=bns._lib.bns_status_string,
                                                            **{"bns_" + n: f for n, f in zip(NAMES, keep)}))
    if request.param == "ctypes":
        monkeypatch.setattr(bns, "_call", types.SimpleNamespace(**{n: lambda *args: None for n in NAMES}))
    monkeypatch.setattr(bns, "_stream", lambda t: 0x7fff12345678)
    yield calls
    monkeypatch.undo()
    bns.load(reload=True)


def _arguments(name):
    """One value for each parameter of the Python function and what the C function has to receive, in its order."""
    given, wanted = {}, []
    reals = {"eps": 1e-5, "momentum": 1, "mix_beta": 0.25}
    for i, p in enumerate(inspect.signature(getattr(bns, "bns_" + name)).parameters):
        if p == "shape":
            given[p], w = SHAPE, bytes(SHAPE)
        elif p == "spec":
            given[p], w = SPEC, bytes(SPEC)
        elif p == "seed":
            given[p], w = -3, 2 ** 64 - 3                   # (modulo 2^64, as through ctypes)
        elif p == "n_v":
            given[p], w = 2, 2
        elif p in reals:
            given[p], w = reals[p], C.c_float(reals[p]).value
        elif p in ("running_mean", "running_var") and name != "inference":
            given[p], w = None, None
        else:
            given[p], w = Tensor(2 ** 47 + 4096 * i, 12345), 2 ** 47 + 4096 * i
        wanted.append(w)
        if p == "workspace":
            wanted.append(12345)
    return given, wanted + [0x7fff12345678]


@pytest.mark.parametrize("name", NAMES)
def test_arguments_reach_the_library(received, name):
    given, wanted = _arguments(name)
    getattr(bns, "bns_" + name)(*given.values())
    getattr(bns, "bns_" + name)(**given)
    assert received == [(name, wanted)] * 2
    received.status = bns.BNS_EWORKSPACE
    with pytest.raises(bns.BnsError) as e:
        getattr(bns, "bns_" + name)(**given)
    assert e.value.status == bns.BNS_EWORKSPACE


class AsParameter:
    def __init__(self, value):
        self._as_parameter_ = value


@pytest.mark.parametrize("name", NAMES)
def test_what_ctypes_converts_is_accepted(received, name):
    given, _ = _arguments(name)
    f32 = C.c_float(0.1).value
    values = {"seed": [(C.c_uint64(2 ** 64 - 3), 2 ** 64 - 3), (AsParameter(7), 7), (True, 1), (np.int64(9), 9)],
              "n_v": [(C.c_int32(-2), -2), (AsParameter(C.c_int32(3)), 3), (2 ** 32 + 1, 1)],
              "eps": [(C.c_float(0.1), f32), (AsParameter(0.1), f32), (np.float32(0.1), f32), (np.float64(0.1), f32), (1e300, float("inf"))],
              "momentum": [(C.c_float(0.1), f32)], "mix_beta": [(C.c_float(0.1), f32)],
              "x": [(Tensor(None), None), (Tensor(C.c_void_p(4096)), 4096), (Tensor(-16), 2 ** 64 - 16)], "beta": [(None, None)]}
    for p, pairs in values.items():
        for i, (value, want) in enumerate(pairs if p in given else []):
            received.clear()
            getattr(bns, "bns_" + name)(**{**given, p: value})
            assert received[0][1][list(given).index(p)] == want, (p, i)


@pytest.mark.parametrize("name", NAMES)
def test_refused_arguments(received, name):
    given, _ = _arguments(name)
    bad = C.ArgumentError                                   # (which is no TypeError)
    wrong = {"shape": [(None, TypeError), (SPEC, bad), (b"0" * 24, TypeError)], "spec": [(None, TypeError), (SHAPE, bad)],
             "seed": [(1.0, bad), ("1", bad), (None, bad), (C.c_int64(1), bad)], "n_v": [(2.0, bad), (None, bad)],
             "eps": [("1", bad), (None, bad), (C.c_double(1.0), bad)], "momentum": [(None, bad)], "mix_beta": [(None, bad)],
             "x": [(17, AttributeError), ("x", AttributeError), (Tensor(1.5), bad)], "y": [(object(), AttributeError)],
             "dx": [(3.5, AttributeError)], "workspace": [(None, AttributeError)]}
    for p, values in wrong.items():
        for value, kind in values if p in given else []:
            with pytest.raises(Exception) as e:
                getattr(bns, "bns_" + name)(**{**given, p: value})
            assert e.type is kind, (p, value, e.type)
    assert received == []


@pytest.mark.parametrize("name", NAMES)
def test_the_extension_leaves_other_numbers_of_arguments_alone(name):
    bns.load()
    assert getattr(bns._call, name)(SHAPE) is None


class Broken(Tensor):
    def data_ptr(self):
        raise RuntimeError("no storage")


def test_exceptions_of_a_tensor_pass_through(received):
    given, _ = _arguments("inference")
    with pytest.raises(RuntimeError, match="no storage"):
        bns.bns_inference(**{**given, "gamma": Broken(0)})
    assert received == []


def test_another_interpreter_marshals_through_ctypes():
    """The extension carries the interpreter's tag; one that finds none of its own loads the library all the same."""
    assert os.path.basename(bns.CALL_PATH) == "_bnscall" + importlib.machinery.EXTENSION_SUFFIXES[0]
    assert "cpython-3" in bns.CALL_PATH
    code = ("import importlib.machinery as m; m.EXTENSION_SUFFIXES[0] = '.cpython-399-none.so'\n"
            "from paper_1810_10962_amd import bns\n"
            "assert bns.bns_status_string(1) and bns.bns_moving_average_weight(1, 0.5) == 1.0\n"
            "assert bns._call.__name__ == '_NoExtension'\n"
            "class T:\n"
            "    nbytes = 0\n"
            "    def data_ptr(self): return None\n"
            "bns._stream = lambda t: 0\n"
            "try: bns.bns_inference(bns.make_shape(2, 3, 4, 5), T(), T(), T(), T(), T(), 1e-5, T())\n"
            "except bns.BnsError as e: assert e.status == bns.BNS_EINVAL\n"
            "else: raise SystemExit('null pointers were taken')\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
