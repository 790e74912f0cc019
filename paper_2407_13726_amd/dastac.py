"""Binding over libdastac_hip.so -- argument marshalling only.

Every function has the name and argument order of the C entry point in
``include/dastac.h`` (minus the ``dastac_`` prefix and ``_f32`` suffix kept as
is).  Device operands are ``torch`` tensors on a HIP device (used for their
memory and for the current stream, nothing else); outputs are passed in by the
caller.  A non-zero status raises ``DastacError``.  There is no fallback: if
the library is not built, importing this module's functions raises.
"""
from __future__ import annotations

import ctypes
import os

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libdastac_hip.so")

OK, EINVAL, ENULL, EOVERFLOW, EALIAS, EHIP = 0, 1, 2, 3, 4, 5

_i64 = ctypes.c_int64
_vp = ctypes.c_void_p

# name -> (restype, argtypes); this table is also what the symbol-export test walks.
SIGNATURES = {
    "dastac_strerror": (ctypes.c_char_p, [ctypes.c_int]),
    "dastac_tri_count": (_i64, [_i64]),
    "dastac_tet_count": (_i64, [_i64]),
    "dastac_band_count": (_i64, [_i64, _i64]),
    "dastac_tri_offset": (_i64, [_i64, _i64, _i64]),
    "dastac_tet_offset": (_i64, [_i64, _i64, _i64, _i64]),
    "dastac_band_offset": (_i64, [_i64, _i64, _i64, _i64]),
    "dastac_tri_inverse": (ctypes.c_int, [_i64, _i64, ctypes.POINTER(_i64), ctypes.POINTER(_i64)]),
    "dastac_tet_inverse": (ctypes.c_int, [_i64, _i64, ctypes.POINTER(_i64), ctypes.POINTER(_i64),
                                          ctypes.POINTER(_i64)]),
    "dastac_pack_triu_f32": (ctypes.c_int, [_i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_triu_f32": (ctypes.c_int, [_i64, _vp, _vp, _i64, _vp]),
    "dastac_pack_tet_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp]),
    "dastac_unpack_tet_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp]),
    "dastac_pack_band_f32": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_band_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp]),
    "dastac_trmv_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmm_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp, _i64, _vp]),
    "dastac_band_spmv_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp, _vp]),
    "dastac_tet_ttv_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_tet_mttkrp_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp, _i64, _vp, _i64, _vp]),
    "dastac_symv_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmv_t_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmv_lower_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmv_lower_t_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_symv_lower_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_tril_offset": (_i64, [_i64, _i64, _i64]),
    "dastac_pack_tril_f32": (ctypes.c_int, [_i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_tril_f32": (ctypes.c_int, [_i64, _vp, _vp, _i64, _vp]),
    "dastac_uhc_count": (_i64, [_i64, _i64]),
    "dastac_uhc_offset": (_i64, [_i64, _i64, _i64, _i64, _i64]),
    "dastac_pack_uhc_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp]),
    "dastac_unpack_uhc_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp]),
    "dastac_ttm_ut_f32": (ctypes.c_int, [_i64, _i64, _i64, _vp, _vp, _i64, _vp, _vp]),
    "dastac_symm_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp, _i64, _vp]),
    "dastac_pr_a2_f32": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_pr_a3_f32": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_pack_triu_f64": (ctypes.c_int, [_i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_triu_f64": (ctypes.c_int, [_i64, _vp, _vp, _i64, _vp]),
    "dastac_pack_tet_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp]),
    "dastac_unpack_tet_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp]),
    "dastac_pack_band_f64": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_band_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp]),
    "dastac_trmv_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_band_spmv_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp, _vp]),
    "dastac_tet_ttv_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmm_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp, _i64, _vp]),
    "dastac_symm_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp, _i64, _vp]),
    "dastac_pack_uhc_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp]),
    "dastac_unpack_uhc_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp]),
    "dastac_ttm_ut_f64": (ctypes.c_int, [_i64, _i64, _i64, _vp, _vp, _i64, _vp, _vp]),
    "dastac_pr_a2_f64": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_pr_a3_f64": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_tet_mttkrp_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp, _i64, _vp, _i64, _vp]),
    "dastac_pack_tril_f64": (ctypes.c_int, [_i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_tril_f64": (ctypes.c_int, [_i64, _vp, _vp, _i64, _vp]),
    "dastac_symv_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmv_t_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_symv_lower_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmv_lower_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_trmv_lower_t_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp]),
    "dastac_pack_sband_f64": (ctypes.c_int, [_i64, _i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_sband_f64": (ctypes.c_int, [_i64, _i64, _i64, _vp, _vp, _i64, _vp]),
    "dastac_sband_spmv_f64": (ctypes.c_int, [_i64, _i64, _i64, _vp, _vp, _vp, _vp]),
    "dastac_pack_subtri_f64": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_subtri_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp]),
    "dastac_subtri_spmv_f64": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp, _vp]),
    "dastac_pack_leslie_f64": (ctypes.c_int, [_i64, _vp, _i64, _vp, _vp, _vp]),
    "dastac_unpack_leslie_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _i64, _vp]),
    "dastac_leslie_spmv_f64": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp, _vp]),
    "dastac_subtri_offset": (_i64, [_i64, _i64, _i64, _i64]),
    "dastac_pack_sband_f32": (ctypes.c_int, [_i64, _i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_sband_f32": (ctypes.c_int, [_i64, _i64, _i64, _vp, _vp, _i64, _vp]),
    "dastac_pack_subtri_f32": (ctypes.c_int, [_i64, _i64, _vp, _i64, _vp, _vp]),
    "dastac_unpack_subtri_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _i64, _vp]),
    "dastac_pack_leslie_f32": (ctypes.c_int, [_i64, _vp, _i64, _vp, _vp, _vp]),
    "dastac_unpack_leslie_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _i64, _vp]),
    "dastac_sband_spmv_f32": (ctypes.c_int, [_i64, _i64, _i64, _vp, _vp, _vp, _vp]),
    "dastac_subtri_spmv_f32": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp, _vp]),
    "dastac_leslie_spmv_f32": (ctypes.c_int, [_i64, _vp, _vp, _vp, _vp, _vp]),
    "dastac_stream_sum_f32": (ctypes.c_int, [_i64, _vp, _vp, _i64, _vp]),
}


class DastacError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__("%s: status %d (%s)" % (where, status, strerror(status)))


_lib = None


def lib() -> ctypes.CDLL:
    """Load the built library; raise if it is missing (no CPU fallback exists)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                "libdastac_hip.so is not built: run `python -c 'import __graft_entry__ as g; g.build()'`")
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


# ---- calls without ctypes ----------------------------------------------------
# The functions below try an entry of the native module first.  It makes the ordinary call itself (csrc/calls.cpp says
# which) and returns its status; for any other call, and for the first, it returns -1, and _settle makes it through ctypes.
try:
    from . import _calls
except ImportError:  # not built: everything goes through ctypes
    _calls = None
_entries = {}


def _kinds(name):
    """One letter for each argument before the stream: i, an integer; f or d, a float32 or float64 tensor."""
    real = "d" if name.endswith("f64") else "f"
    return "".join("i" if kind is _i64 else real for kind in SIGNATURES["dastac_" + name][1][:-1])


def _entry(name):
    if _calls is None:
        return lambda *args: -1
    _entries[name] = _calls.entry(_kinds(name))
    return _entries[name]


def _bind(L, torch, raw, device):
    """Gives the entries the library's functions and what they ask torch with."""
    if _calls is None or raw is None or device is None:
        return
    _calls.torch(torch.Tensor, torch.float32, torch.float64, raw, device)
    for name, entry in _entries.items():
        _calls.bind(entry, ctypes.cast(getattr(L, "dastac_" + name), ctypes.c_void_p).value)


def _unbind():
    for entry in _entries.values():
        _calls.bind(entry, 0)


if _calls is not None:  # a forked child may not use its parent's device: torch says so in the calls below
    os.register_at_fork(after_in_child=_unbind)


def strerror(status: int) -> str:
    return lib().dastac_strerror(int(status)).decode()


def _check(status: int, where: str) -> None:
    if status != OK:
        raise DastacError(status, where)


_ctypes_calls = {}  # name -> the C function, and how each argument before the stream is handed to it (None: as it is)


def _settle(status, name, *args):
    """The outcome of a call whose entry did not return OK: an error, or a call that the entry left, made through ctypes."""
    if status < 0:
        if name not in _ctypes_calls:
            _ctypes_calls[name] = getattr(lib(), "dastac_" + name), [{"i": None, "f": _ptr, "d": _ptr64}[k] for k in _kinds(name)]
        call, hand = _ctypes_calls[name]
        status = call(*[a if h is None else h(a) for h, a in zip(hand, args)], _stream(args[-1]))
    _check(status, name)


def _ptr(t):
    """Device address of a float32 tensor (None -> NULL)."""
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("device tensor expected")
    if t.dtype is not _dtypes()[0]:
        raise ValueError("float32 tensor expected")
    return t.data_ptr()


def _ptr64(t):
    """Device address of a float64 tensor (None -> NULL)."""
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("device tensor expected")
    if t.dtype is not _dtypes()[1]:
        raise ValueError("float64 tensor expected")
    return t.data_ptr()


# torch is imported at the first call that needs it (the index polynomials do not) and looked up once: its dtypes, and
# the raw handle of a device's current stream, which costs a call a tenth of what building a Stream object does (a
# small product is called in 4 us; through the object it was 7).
_torch_parts = None


def _dtypes():
    global _torch_parts
    if _torch_parts is None:
        import torch

        raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
        device = getattr(torch._C, "_cuda_getDevice", None)
        _torch_parts = (torch.float32, torch.float64, torch.cuda, raw if device is not None else None, device)
        _bind(lib(), torch, raw, device)
    return _torch_parts


def _stream(stream=None):
    """Handle of `stream`, or of the current device's current stream, asked anew at every call."""
    if stream is not None:
        return stream.cuda_stream
    _, _, cuda, raw, device = _dtypes()
    if raw is not None and cuda.is_initialized():
        return raw(device())
    return cuda.current_stream().cuda_stream


# ---- index polynomials (host) -------------------------------------------------

def tri_count(n): return int(lib().dastac_tri_count(n))
def tet_count(n): return int(lib().dastac_tet_count(n))
def band_count(n, w): return int(lib().dastac_band_count(n, w))
def tri_offset(n, i, j): return int(lib().dastac_tri_offset(n, i, j))
def tet_offset(n, i, j, k): return int(lib().dastac_tet_offset(n, i, j, k))
def band_offset(n, w, d, i): return int(lib().dastac_band_offset(n, w, d, i))


def tri_inverse(n, p):
    i, j = _i64(), _i64()
    _check(lib().dastac_tri_inverse(n, p, ctypes.byref(i), ctypes.byref(j)), "tri_inverse")
    return i.value, j.value


def tet_inverse(n, p):
    i, j, k = _i64(), _i64(), _i64()
    _check(lib().dastac_tet_inverse(n, p, ctypes.byref(i), ctypes.byref(j), ctypes.byref(k)), "tet_inverse")
    return i.value, j.value, k.value


# ---- device operations -----------------------------------------------------------

_pack_triu_f32 = _entry("pack_triu_f32")


def pack_triu_f32(n, dense, ld, packed, stream=None):
    status = _pack_triu_f32(n, dense, ld, packed, stream)
    if status:
        _settle(status, "pack_triu_f32", n, dense, ld, packed, stream)


_unpack_triu_f32 = _entry("unpack_triu_f32")


def unpack_triu_f32(n, packed, dense, ld, stream=None):
    status = _unpack_triu_f32(n, packed, dense, ld, stream)
    if status:
        _settle(status, "unpack_triu_f32", n, packed, dense, ld, stream)


_pack_tet_f32 = _entry("pack_tet_f32")


def pack_tet_f32(n, dense, packed, stream=None):
    status = _pack_tet_f32(n, dense, packed, stream)
    if status:
        _settle(status, "pack_tet_f32", n, dense, packed, stream)


_unpack_tet_f32 = _entry("unpack_tet_f32")


def unpack_tet_f32(n, packed, dense, stream=None):
    status = _unpack_tet_f32(n, packed, dense, stream)
    if status:
        _settle(status, "unpack_tet_f32", n, packed, dense, stream)


_pack_band_f32 = _entry("pack_band_f32")


def pack_band_f32(n, w, dense, ld, diag_major, stream=None):
    status = _pack_band_f32(n, w, dense, ld, diag_major, stream)
    if status:
        _settle(status, "pack_band_f32", n, w, dense, ld, diag_major, stream)


_unpack_band_f32 = _entry("unpack_band_f32")


def unpack_band_f32(n, w, diag_major, dense, ld, stream=None):
    status = _unpack_band_f32(n, w, diag_major, dense, ld, stream)
    if status:
        _settle(status, "unpack_band_f32", n, w, diag_major, dense, ld, stream)


_trmv_f32 = _entry("trmv_f32")


def trmv_f32(n, Up, x, y, stream=None):
    status = _trmv_f32(n, Up, x, y, stream)
    if status:
        _settle(status, "trmv_f32", n, Up, x, y, stream)


_trmm_f32 = _entry("trmm_f32")


def trmm_f32(n, m, Up, B, ldb, C, ldc, stream=None):
    status = _trmm_f32(n, m, Up, B, ldb, C, ldc, stream)
    if status:
        _settle(status, "trmm_f32", n, m, Up, B, ldb, C, ldc, stream)


_band_spmv_f32 = _entry("band_spmv_f32")


def band_spmv_f32(n, w, D, x, y, stream=None):
    status = _band_spmv_f32(n, w, D, x, y, stream)
    if status:
        _settle(status, "band_spmv_f32", n, w, D, x, y, stream)


_tet_ttv_f32 = _entry("tet_ttv_f32")


def tet_ttv_f32(n, Ap, v, Mp, stream=None):
    status = _tet_ttv_f32(n, Ap, v, Mp, stream)
    if status:
        _settle(status, "tet_ttv_f32", n, Ap, v, Mp, stream)


_tet_mttkrp_f32 = _entry("tet_mttkrp_f32")


def tet_mttkrp_f32(n, R, Ap, B, ldb, C, ldc, M, ldm, stream=None):
    status = _tet_mttkrp_f32(n, R, Ap, B, ldb, C, ldc, M, ldm, stream)
    if status:
        _settle(status, "tet_mttkrp_f32", n, R, Ap, B, ldb, C, ldc, M, ldm, stream)


def uhc_count(n, Q): return int(lib().dastac_uhc_count(n, Q))
def uhc_offset(n, Q, i, j, l): return int(lib().dastac_uhc_offset(n, Q, i, j, l))


_pack_uhc_f32 = _entry("pack_uhc_f32")


def pack_uhc_f32(n, Q, dense, packed, stream=None):
    status = _pack_uhc_f32(n, Q, dense, packed, stream)
    if status:
        _settle(status, "pack_uhc_f32", n, Q, dense, packed, stream)


_unpack_uhc_f32 = _entry("unpack_uhc_f32")


def unpack_uhc_f32(n, Q, packed, dense, stream=None):
    status = _unpack_uhc_f32(n, Q, packed, dense, stream)
    if status:
        _settle(status, "unpack_uhc_f32", n, Q, packed, dense, stream)


_ttm_ut_f32 = _entry("ttm_ut_f32")


def ttm_ut_f32(n, Q, K, Bp, C, ldc, Ap, stream=None):
    status = _ttm_ut_f32(n, Q, K, Bp, C, ldc, Ap, stream)
    if status:
        _settle(status, "ttm_ut_f32", n, Q, K, Bp, C, ldc, Ap, stream)


_symv_f32 = _entry("symv_f32")


def symv_f32(n, Up, x, y, stream=None):
    status = _symv_f32(n, Up, x, y, stream)
    if status:
        _settle(status, "symv_f32", n, Up, x, y, stream)


_trmv_t_f32 = _entry("trmv_t_f32")


def trmv_t_f32(n, Up, x, y, stream=None):
    status = _trmv_t_f32(n, Up, x, y, stream)
    if status:
        _settle(status, "trmv_t_f32", n, Up, x, y, stream)


_trmv_lower_f32 = _entry("trmv_lower_f32")


def trmv_lower_f32(n, Lp, x, y, stream=None):
    status = _trmv_lower_f32(n, Lp, x, y, stream)
    if status:
        _settle(status, "trmv_lower_f32", n, Lp, x, y, stream)


_trmv_lower_t_f32 = _entry("trmv_lower_t_f32")


def trmv_lower_t_f32(n, Lp, x, y, stream=None):
    status = _trmv_lower_t_f32(n, Lp, x, y, stream)
    if status:
        _settle(status, "trmv_lower_t_f32", n, Lp, x, y, stream)


_symv_lower_f32 = _entry("symv_lower_f32")


def symv_lower_f32(n, Lp, x, y, stream=None):
    status = _symv_lower_f32(n, Lp, x, y, stream)
    if status:
        _settle(status, "symv_lower_f32", n, Lp, x, y, stream)


def tril_offset(n, i, j): return int(lib().dastac_tril_offset(n, i, j))


_pack_tril_f32 = _entry("pack_tril_f32")


def pack_tril_f32(n, dense, ld, packed, stream=None):
    status = _pack_tril_f32(n, dense, ld, packed, stream)
    if status:
        _settle(status, "pack_tril_f32", n, dense, ld, packed, stream)


_unpack_tril_f32 = _entry("unpack_tril_f32")


def unpack_tril_f32(n, packed, dense, ld, stream=None):
    status = _unpack_tril_f32(n, packed, dense, ld, stream)
    if status:
        _settle(status, "unpack_tril_f32", n, packed, dense, ld, stream)



def subtri_offset(N, k, i, j): return int(lib().dastac_subtri_offset(N, k, i, j))


_pack_sband_f32 = _entry("pack_sband_f32")


def pack_sband_f32(n, w, s, dense, ld, diag_major, stream=None):
    status = _pack_sband_f32(n, w, s, dense, ld, diag_major, stream)
    if status:
        _settle(status, "pack_sband_f32", n, w, s, dense, ld, diag_major, stream)


_unpack_sband_f32 = _entry("unpack_sband_f32")


def unpack_sband_f32(n, w, s, diag_major, dense, ld, stream=None):
    status = _unpack_sband_f32(n, w, s, diag_major, dense, ld, stream)
    if status:
        _settle(status, "unpack_sband_f32", n, w, s, diag_major, dense, ld, stream)


_pack_subtri_f32 = _entry("pack_subtri_f32")


def pack_subtri_f32(N, k, dense, ld, packed, stream=None):
    status = _pack_subtri_f32(N, k, dense, ld, packed, stream)
    if status:
        _settle(status, "pack_subtri_f32", N, k, dense, ld, packed, stream)


_unpack_subtri_f32 = _entry("unpack_subtri_f32")


def unpack_subtri_f32(N, k, packed, dense, ld, stream=None):
    status = _unpack_subtri_f32(N, k, packed, dense, ld, stream)
    if status:
        _settle(status, "unpack_subtri_f32", N, k, packed, dense, ld, stream)


_pack_leslie_f32 = _entry("pack_leslie_f32")


def pack_leslie_f32(n, dense, ld, R, S, stream=None):
    status = _pack_leslie_f32(n, dense, ld, R, S, stream)
    if status:
        _settle(status, "pack_leslie_f32", n, dense, ld, R, S, stream)


_unpack_leslie_f32 = _entry("unpack_leslie_f32")


def unpack_leslie_f32(n, R, S, dense, ld, stream=None):
    status = _unpack_leslie_f32(n, R, S, dense, ld, stream)
    if status:
        _settle(status, "unpack_leslie_f32", n, R, S, dense, ld, stream)


_sband_spmv_f32 = _entry("sband_spmv_f32")


def sband_spmv_f32(n, w, s, D, x, y, stream=None):
    status = _sband_spmv_f32(n, w, s, D, x, y, stream)
    if status:
        _settle(status, "sband_spmv_f32", n, w, s, D, x, y, stream)


_subtri_spmv_f32 = _entry("subtri_spmv_f32")


def subtri_spmv_f32(N, k, Ap, x, y, stream=None):
    status = _subtri_spmv_f32(N, k, Ap, x, y, stream)
    if status:
        _settle(status, "subtri_spmv_f32", N, k, Ap, x, y, stream)


_leslie_spmv_f32 = _entry("leslie_spmv_f32")


def leslie_spmv_f32(n, R, S, x, y, stream=None):
    status = _leslie_spmv_f32(n, R, S, x, y, stream)
    if status:
        _settle(status, "leslie_spmv_f32", n, R, S, x, y, stream)


_stream_sum_f32 = _entry("stream_sum_f32")


def stream_sum_f32(count, src, partial, npartial, stream=None):
    status = _stream_sum_f32(count, src, partial, npartial, stream)
    if status:
        _settle(status, "stream_sum_f32", count, src, partial, npartial, stream)


_symm_f32 = _entry("symm_f32")


def symm_f32(n, m, Up, B, ldb, C, ldc, stream=None):
    status = _symm_f32(n, m, Up, B, ldb, C, ldc, stream)
    if status:
        _settle(status, "symm_f32", n, m, Up, B, ldb, C, ldc, stream)


_pr_a2_f32 = _entry("pr_a2_f32")


def pr_a2_f32(N, d, B, ldb, A2p, stream=None):
    status = _pr_a2_f32(N, d, B, ldb, A2p, stream)
    if status:
        _settle(status, "pr_a2_f32", N, d, B, ldb, A2p, stream)


_pr_a3_f32 = _entry("pr_a3_f32")


def pr_a3_f32(N, d, B, ldb, A3p, stream=None):
    status = _pr_a3_f32(N, d, B, ldb, A3p, stream)
    if status:
        _settle(status, "pr_a3_f32", N, d, B, ldb, A3p, stream)


# ---- double precision ---------------------------------------------------------

_pack_triu_f64 = _entry("pack_triu_f64")


def pack_triu_f64(n, dense, ld, packed, stream=None):
    status = _pack_triu_f64(n, dense, ld, packed, stream)
    if status:
        _settle(status, "pack_triu_f64", n, dense, ld, packed, stream)


_unpack_triu_f64 = _entry("unpack_triu_f64")


def unpack_triu_f64(n, packed, dense, ld, stream=None):
    status = _unpack_triu_f64(n, packed, dense, ld, stream)
    if status:
        _settle(status, "unpack_triu_f64", n, packed, dense, ld, stream)


_pack_tet_f64 = _entry("pack_tet_f64")


def pack_tet_f64(n, dense, packed, stream=None):
    status = _pack_tet_f64(n, dense, packed, stream)
    if status:
        _settle(status, "pack_tet_f64", n, dense, packed, stream)


_unpack_tet_f64 = _entry("unpack_tet_f64")


def unpack_tet_f64(n, packed, dense, stream=None):
    status = _unpack_tet_f64(n, packed, dense, stream)
    if status:
        _settle(status, "unpack_tet_f64", n, packed, dense, stream)


_pack_band_f64 = _entry("pack_band_f64")


def pack_band_f64(n, w, dense, ld, diag_major, stream=None):
    status = _pack_band_f64(n, w, dense, ld, diag_major, stream)
    if status:
        _settle(status, "pack_band_f64", n, w, dense, ld, diag_major, stream)


_unpack_band_f64 = _entry("unpack_band_f64")


def unpack_band_f64(n, w, diag_major, dense, ld, stream=None):
    status = _unpack_band_f64(n, w, diag_major, dense, ld, stream)
    if status:
        _settle(status, "unpack_band_f64", n, w, diag_major, dense, ld, stream)


_trmv_f64 = _entry("trmv_f64")


def trmv_f64(n, Up, x, y, stream=None):
    status = _trmv_f64(n, Up, x, y, stream)
    if status:
        _settle(status, "trmv_f64", n, Up, x, y, stream)


_band_spmv_f64 = _entry("band_spmv_f64")


def band_spmv_f64(n, w, D, x, y, stream=None):
    status = _band_spmv_f64(n, w, D, x, y, stream)
    if status:
        _settle(status, "band_spmv_f64", n, w, D, x, y, stream)


_tet_ttv_f64 = _entry("tet_ttv_f64")


def tet_ttv_f64(n, Ap, v, Mp, stream=None):
    status = _tet_ttv_f64(n, Ap, v, Mp, stream)
    if status:
        _settle(status, "tet_ttv_f64", n, Ap, v, Mp, stream)


_trmm_f64 = _entry("trmm_f64")


def trmm_f64(n, m, Up, B, ldb, C, ldc, stream=None):
    status = _trmm_f64(n, m, Up, B, ldb, C, ldc, stream)
    if status:
        _settle(status, "trmm_f64", n, m, Up, B, ldb, C, ldc, stream)


_symm_f64 = _entry("symm_f64")


def symm_f64(n, m, Up, B, ldb, C, ldc, stream=None):
    status = _symm_f64(n, m, Up, B, ldb, C, ldc, stream)
    if status:
        _settle(status, "symm_f64", n, m, Up, B, ldb, C, ldc, stream)


_pack_uhc_f64 = _entry("pack_uhc_f64")


def pack_uhc_f64(n, Q, dense, packed, stream=None):
    status = _pack_uhc_f64(n, Q, dense, packed, stream)
    if status:
        _settle(status, "pack_uhc_f64", n, Q, dense, packed, stream)


_unpack_uhc_f64 = _entry("unpack_uhc_f64")


def unpack_uhc_f64(n, Q, packed, dense, stream=None):
    status = _unpack_uhc_f64(n, Q, packed, dense, stream)
    if status:
        _settle(status, "unpack_uhc_f64", n, Q, packed, dense, stream)


_ttm_ut_f64 = _entry("ttm_ut_f64")


def ttm_ut_f64(n, Q, K, Bp, C, ldc, Ap, stream=None):
    status = _ttm_ut_f64(n, Q, K, Bp, C, ldc, Ap, stream)
    if status:
        _settle(status, "ttm_ut_f64", n, Q, K, Bp, C, ldc, Ap, stream)


_pr_a2_f64 = _entry("pr_a2_f64")


def pr_a2_f64(N, d, B, ldb, A2p, stream=None):
    status = _pr_a2_f64(N, d, B, ldb, A2p, stream)
    if status:
        _settle(status, "pr_a2_f64", N, d, B, ldb, A2p, stream)


_pr_a3_f64 = _entry("pr_a3_f64")


def pr_a3_f64(N, d, B, ldb, A3p, stream=None):
    status = _pr_a3_f64(N, d, B, ldb, A3p, stream)
    if status:
        _settle(status, "pr_a3_f64", N, d, B, ldb, A3p, stream)


_tet_mttkrp_f64 = _entry("tet_mttkrp_f64")


def tet_mttkrp_f64(n, R, Ap, B, ldb, C, ldc, M, ldm, stream=None):
    status = _tet_mttkrp_f64(n, R, Ap, B, ldb, C, ldc, M, ldm, stream)
    if status:
        _settle(status, "tet_mttkrp_f64", n, R, Ap, B, ldb, C, ldc, M, ldm, stream)


_pack_tril_f64 = _entry("pack_tril_f64")


def pack_tril_f64(n, dense, ld, packed, stream=None):
    status = _pack_tril_f64(n, dense, ld, packed, stream)
    if status:
        _settle(status, "pack_tril_f64", n, dense, ld, packed, stream)


_unpack_tril_f64 = _entry("unpack_tril_f64")


def unpack_tril_f64(n, packed, dense, ld, stream=None):
    status = _unpack_tril_f64(n, packed, dense, ld, stream)
    if status:
        _settle(status, "unpack_tril_f64", n, packed, dense, ld, stream)


_symv_f64 = _entry("symv_f64")


def symv_f64(n, Up, x, y, stream=None):
    status = _symv_f64(n, Up, x, y, stream)
    if status:
        _settle(status, "symv_f64", n, Up, x, y, stream)


_trmv_t_f64 = _entry("trmv_t_f64")


def trmv_t_f64(n, Up, x, y, stream=None):
    status = _trmv_t_f64(n, Up, x, y, stream)
    if status:
        _settle(status, "trmv_t_f64", n, Up, x, y, stream)


_symv_lower_f64 = _entry("symv_lower_f64")


def symv_lower_f64(n, Lp, x, y, stream=None):
    status = _symv_lower_f64(n, Lp, x, y, stream)
    if status:
        _settle(status, "symv_lower_f64", n, Lp, x, y, stream)


_trmv_lower_f64 = _entry("trmv_lower_f64")


def trmv_lower_f64(n, Lp, x, y, stream=None):
    status = _trmv_lower_f64(n, Lp, x, y, stream)
    if status:
        _settle(status, "trmv_lower_f64", n, Lp, x, y, stream)


_trmv_lower_t_f64 = _entry("trmv_lower_t_f64")


def trmv_lower_t_f64(n, Lp, x, y, stream=None):
    status = _trmv_lower_t_f64(n, Lp, x, y, stream)
    if status:
        _settle(status, "trmv_lower_t_f64", n, Lp, x, y, stream)


_pack_sband_f64 = _entry("pack_sband_f64")


def pack_sband_f64(n, w, s, dense, ld, diag_major, stream=None):
    status = _pack_sband_f64(n, w, s, dense, ld, diag_major, stream)
    if status:
        _settle(status, "pack_sband_f64", n, w, s, dense, ld, diag_major, stream)


_unpack_sband_f64 = _entry("unpack_sband_f64")


def unpack_sband_f64(n, w, s, diag_major, dense, ld, stream=None):
    status = _unpack_sband_f64(n, w, s, diag_major, dense, ld, stream)
    if status:
        _settle(status, "unpack_sband_f64", n, w, s, diag_major, dense, ld, stream)


_sband_spmv_f64 = _entry("sband_spmv_f64")


def sband_spmv_f64(n, w, s, D, x, y, stream=None):
    status = _sband_spmv_f64(n, w, s, D, x, y, stream)
    if status:
        _settle(status, "sband_spmv_f64", n, w, s, D, x, y, stream)


_pack_subtri_f64 = _entry("pack_subtri_f64")


def pack_subtri_f64(N, k, dense, ld, packed, stream=None):
    status = _pack_subtri_f64(N, k, dense, ld, packed, stream)
    if status:
        _settle(status, "pack_subtri_f64", N, k, dense, ld, packed, stream)


_unpack_subtri_f64 = _entry("unpack_subtri_f64")


def unpack_subtri_f64(N, k, packed, dense, ld, stream=None):
    status = _unpack_subtri_f64(N, k, packed, dense, ld, stream)
    if status:
        _settle(status, "unpack_subtri_f64", N, k, packed, dense, ld, stream)


_subtri_spmv_f64 = _entry("subtri_spmv_f64")


def subtri_spmv_f64(N, k, Ap, x, y, stream=None):
    status = _subtri_spmv_f64(N, k, Ap, x, y, stream)
    if status:
        _settle(status, "subtri_spmv_f64", N, k, Ap, x, y, stream)


_pack_leslie_f64 = _entry("pack_leslie_f64")


def pack_leslie_f64(n, dense, ld, R, S, stream=None):
    status = _pack_leslie_f64(n, dense, ld, R, S, stream)
    if status:
        _settle(status, "pack_leslie_f64", n, dense, ld, R, S, stream)


_unpack_leslie_f64 = _entry("unpack_leslie_f64")


def unpack_leslie_f64(n, R, S, dense, ld, stream=None):
    status = _unpack_leslie_f64(n, R, S, dense, ld, stream)
    if status:
        _settle(status, "unpack_leslie_f64", n, R, S, dense, ld, stream)


_leslie_spmv_f64 = _entry("leslie_spmv_f64")


def leslie_spmv_f64(n, R, S, x, y, stream=None):
    status = _leslie_spmv_f64(n, R, S, x, y, stream)
    if status:
        _settle(status, "leslie_spmv_f64", n, R, S, x, y, stream)
