"""The binding's native calls: which calls an entry makes itself, with which arguments, and which it leaves to the Python code.  Stand-ins for torch and for the C functions, no GPU."""
import ctypes
import inspect

import numpy as np
import pytest

from paper_2407_13726_amd import dastac

calls = pytest.importorskip("paper_2407_13726_amd._calls")


class Tensor:
    def __init__(self, at, dtype="f", cuda=True):
        self.at, self.dtype, self.is_cuda = at, dtype, cuda

    def data_ptr(self):
        return self.at


class Other(Tensor):
    pass


@pytest.fixture
def seen():
    """Arguments of the calls that a fake C function (i, f, d, i and the stream) got; it returns 7 times the first."""
    got = []
    proto = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_int64] * 5)
    fn = proto(lambda *a: got.append(a) or 7 * a[0])
    calls.torch(Tensor, "f", "d", lambda device: 1000 + device, lambda: 3)
    e = calls.entry("ifdi")
    assert e(1, Tensor(8), Tensor(16, "d"), 2, None) == -1 and not got  # not bound yet
    calls.bind(e, ctypes.cast(fn, ctypes.c_void_p).value)
    yield e, got
    calls.bind(e, 0)
    assert e(1, Tensor(8), Tensor(16, "d"), 2, None) == -1
    import torch

    calls.torch(torch.Tensor, torch.float32, torch.float64, torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice)


def test_ordinary_calls_are_made(seen):
    e, got = seen
    assert e(0, Tensor(8), Tensor(2 ** 63 + 16, "d"), -5, None) == 0
    assert e(2, None, Tensor(16, "d"), 2 ** 63 - 1, None) == 14
    assert got == [(0, 8, 16 - 2 ** 63, -5, 1003), (2, 0, 16, 2 ** 63 - 1, 1003)]


@pytest.mark.parametrize("args", [
    (1, Tensor(8, cuda=False), Tensor(16, "d"), 2, None), (1, Tensor(8, "d"), Tensor(16, "d"), 2, None), (1, Tensor(8), Tensor(16), 2, None), (1, Other(8), Tensor(16, "d"), 2, None),
    (1, 8, Tensor(16, "d"), 2, None), (True, Tensor(8), Tensor(16, "d"), 2, None), (1.0, Tensor(8), Tensor(16, "d"), 2, None), (2 ** 63, Tensor(8), Tensor(16, "d"), 2, None),
    (1, Tensor(8), Tensor(16, "d"), 2, "a stream"), (1, Tensor(8), Tensor(16, "d"), 2), (1, Tensor(8), Tensor(16, "d"), 2, None, None), (1, None, None, 2, None),
    (1, Tensor("text"), Tensor(16, "d"), 2, None)])
def test_other_calls_are_left_to_python(seen, args):
    e, got = seen
    assert e(*args) == -1 and not got


def test_keywords_are_left_to_python(seen):
    e, got = seen
    assert e(1, Tensor(8), Tensor(16, "d"), 2, stream=None) == -1 and not got


def test_every_entry_has_its_functions_arguments():
    ints, ptrs = ctypes.c_int64, ctypes.c_void_p
    assert len(dastac._entries) == sum(1 for _, a in dastac.SIGNATURES.values() if a and a[-1] is ptrs)
    for name, entry in dastac._entries.items():
        args = dastac.SIGNATURES["dastac_" + name][1]
        params = list(inspect.signature(getattr(dastac, name)).parameters.values())
        assert [p.name for p in params][-1] == "stream" and params[-1].default is None and len(params) == len(args)
        kinds = "".join("i" if a is ints else "d" if name.endswith("f64") else "f" for a in args[:-1])
        assert set(args) <= {ints, ptrs}
        assert dastac._kinds(name) == kinds


def test_numpy_integers_are_integers(seen):
    e, got = seen
    assert e(np.int64(2), None, Tensor(16, "d"), np.uint8(5), None) == 14 and got == [(2, 0, 16, 5, 1003)]
    assert e(1, None, Tensor(16, "d"), np.uint64(2 ** 63), None) == -1 and e(1, None, Tensor(16, "d"), np.float64(2), None) == -1 and len(got) == 1


class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


def test_a_given_stream_is_handed_on(seen):
    e, got = seen
    assert e(1, Tensor(8), Tensor(16, "d"), 2, Stream(77)) == 7 and got == [(1, 8, 16, 2, 77)]


@pytest.mark.parametrize("handle", [None, "text", 1.0, -1, 2 ** 64])
def test_handles_that_are_no_addresses_are_left_to_python(seen, handle):
    e, got = seen
    assert e(1, Tensor(8), Tensor(16, "d"), 2, Stream(handle)) == -1 and not got


@pytest.mark.parametrize("name,args", [("trmv_f32", (3, Tensor(8, "f"), None, Tensor(24, "f"))), ("tet_mttkrp_f64", (3, 2, Tensor(8, "d"), Tensor(16, "d"), 5, None, 6, Tensor(24, "d"), 7))])
def test_every_call_can_go_through_ctypes(monkeypatch, name, args):
    """What an entry leaves gets the same arguments, in the order of the C function, and its complaints the function's name."""
    got = []
    fn = lambda *a: got.append(a) or 4
    monkeypatch.setitem(dastac._ctypes_calls, name, (fn, [None if k == "i" else (lambda t: None if t is None else t.data_ptr()) for k in dastac._kinds(name)]))
    monkeypatch.setattr(dastac, "_" + name, lambda *a: -1)
    with pytest.raises(dastac.DastacError, match=name) as error:
        getattr(dastac, name)(*args, stream=Stream(99))
    assert error.value.status == 4
    assert got == [(*[a.at if isinstance(a, Tensor) else a for a in args], 99)]
