"""The extension that marshals the calls of every step (csrc/bns_call.cpp): what the library's functions receive, argument by
argument, against the values that the binding was given; what it refuses; the exceptions of bad calls."""
import ctypes as C
import inspect

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


@pytest.fixture
def received(monkeypatch):
    """Calls received by stand-ins for the five functions, which answer with the status in `received.status`."""
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
    monkeypatch.setattr(bns, "_stream", lambda t: 0x7fff12345678)
    yield calls
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


@pytest.mark.parametrize("name", NAMES)
def test_refused_arguments(received, name):
    given, _ = _arguments(name)
    wrong = {"shape": [None, SPEC, b"0" * 24], "spec": [None, SHAPE], "seed": [1.0, "1", None], "n_v": [2.0, None],
             "eps": ["1", None], "momentum": [None], "mix_beta": [None], "x": [17, "x"], "y": [object()], "dx": [3.5],
             "workspace": [None]}
    for p, values in wrong.items():
        for v in values if p in given else []:
            with pytest.raises((TypeError, AttributeError)):
                getattr(bns, "bns_" + name)(**{**given, p: v})
    assert received == []
    with pytest.raises(TypeError):
        getattr(bns._call, name)(SHAPE)


class Broken(Tensor):
    def data_ptr(self):
        raise RuntimeError("no storage")


def test_exceptions_of_a_tensor_pass_through(received):
    given, _ = _arguments("inference")
    with pytest.raises(RuntimeError, match="no storage"):
        bns.bns_inference(**{**given, "gamma": Broken(0)})
    assert received == []
