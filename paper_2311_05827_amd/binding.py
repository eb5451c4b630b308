"""Binding of libaccept.so (ctypes, and native code for the frequent calls): argument marshalling only.

Every step of the compression path runs in the library's HIP kernels; this module turns
PyTorch device tensors into pointers, allocates the output buffers with ``torch.empty`` and
passes the current HIP stream.  Function names follow the C ABI (include/accept.h).  There
is no CPU fallback: if the shared library is missing, importing this module raises.
"""
from __future__ import annotations

import ctypes
import os
import warnings

# PyTorch first: it brings its own copy of the HIP runtime, and the library and PyTorch must
# share one (they exchange stream handles and device pointers).  The dynamic loader gives
# the library whichever copy is already in the process, so the order of the two loads decides.
import torch

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libaccept.so")

UNIFORM, MBQ = 0, 1
F32, BF16 = 0, 1
ROUND_NEAREST_EVEN, ROUND_STOCHASTIC = 0, 1
LAYOUT_PACKED, LAYOUT_BATCH, LAYOUT_UNENCODED = 0, 1, 2
MAX_STAGES = 8

STATUS_NAMES = {0: "ACCEPT_OK", 1: "ACCEPT_ERR_INVALID_ARG", 2: "ACCEPT_ERR_UNSUPPORTED",
                3: "ACCEPT_ERR_BUFFER_TOO_SMALL", 4: "ACCEPT_ERR_HIP"}


class AcceptError(RuntimeError):
    def __init__(self, status, where):
        self.status = int(status)
        super().__init__("%s: %s (%s)" % (where, STATUS_NAMES.get(self.status, self.status),
                                          status_string(self.status)))


class Desc(ctypes.Structure):
    """Mirror of accept_desc."""
    _fields_ = [
        ("scheme", ctypes.c_int32), ("bits", ctypes.c_int32),
        ("in_dtype", ctypes.c_int32), ("out_dtype", ctypes.c_int32),
        ("n", ctypes.c_int64), ("m", ctypes.c_int64), ("channels", ctypes.c_int64),
        ("rounding", ctypes.c_int32), ("layout", ctypes.c_int32),
        ("seed", ctypes.c_uint64), ("t", ctypes.c_int64),
    ]


def _load():
    if not os.path.exists(LIB_PATH):
        raise ImportError(
            "libaccept.so is not built (%s). Run `python -m paper_2311_05827_amd.build`; "
            "there is no CPU fallback." % LIB_PATH)
    lib = ctypes.CDLL(LIB_PATH)
    P, V, I = ctypes.POINTER, ctypes.c_void_p, ctypes.c_int
    sz = P(ctypes.c_size_t)
    lib.accept_packed_size.argtypes = [P(Desc), sz, sz]
    lib.accept_workspace_size.argtypes = [P(Desc), sz]
    lib.accept_compress.argtypes = [P(Desc), V, V, V, V, V, V]
    lib.accept_decompress.argtypes = [P(Desc), V, V, V, V]
    lib.accept_compress_noalloc.argtypes = [P(Desc), V, V, V, V, V]
    lib.accept_mbq_init.argtypes = [P(Desc), V, V, V, V]
    lib.accept_mbq_compress_first.argtypes = [P(Desc), V, V, V, V, V]
    lib.accept_compress_timed.argtypes = [P(Desc), V, V, V, V, V, V, P(ctypes.c_float), P(I)]
    lib.accept_decompress_timed.argtypes = [P(Desc), V, V, V, V, P(ctypes.c_float), P(I)]
    lib.accept_compress_polls.argtypes = [P(Desc), V, V, V, V, V, V, I]
    lib.accept_stage_name.argtypes = [P(Desc), I, I]
    lib.accept_stage_name.restype = ctypes.c_char_p
    lib.accept_bits_schedule.argtypes = [I, I]
    lib.accept_bits_schedule.restype = I
    lib.accept_status_string.argtypes = [I]
    lib.accept_status_string.restype = ctypes.c_char_p
    lib.accept_version.argtypes = []
    lib.accept_version.restype = ctypes.c_char_p
    for name in ("accept_packed_size", "accept_workspace_size", "accept_compress", "accept_decompress",
                 "accept_compress_noalloc", "accept_mbq_init", "accept_mbq_compress_first", "accept_compress_timed", "accept_decompress_timed",
                 "accept_compress_polls"):
        getattr(lib, name).restype = I
    return lib


lib = _load()
try:
    from . import _native   # the calls below for plain tensors, without the interpreter
except ImportError as e:    # not built, or for another PyTorch: ctypes serves every call, in more host time
    warnings.warn("%s: calls go through ctypes; rebuild with `python -m paper_2311_05827_amd.build`" % e, RuntimeWarning)

    class _native:
        compress = decompress = staticmethod(lambda *args: -1)


def status_string(status):
    return lib.accept_status_string(int(status)).decode()


def version():
    return lib.accept_version().decode()


def _check(st, where):
    if st != 0:
        raise AcceptError(st, where)


def make_desc(scheme, bits, n, m, channels=0, in_dtype=F32, out_dtype=F32, rounding=0, seed=0, t=0,
              layout=LAYOUT_PACKED):
    return Desc(int(scheme), int(bits), int(in_dtype), int(out_dtype), int(n), int(m), int(channels),
                int(rounding), int(layout), int(seed), int(t))


def accept_packed_size(desc):
    h, p = ctypes.c_size_t(0), ctypes.c_size_t(0)
    _check(lib.accept_packed_size(ctypes.byref(desc), ctypes.byref(h), ctypes.byref(p)), "accept_packed_size")
    return h.value, p.value


def accept_workspace_size(desc):
    b = ctypes.c_size_t(0)
    _check(lib.accept_workspace_size(ctypes.byref(desc), ctypes.byref(b)), "accept_workspace_size")
    return b.value


def accept_bits_schedule(direction, lr_changes_so_far):
    return lib.accept_bits_schedule(int(direction), int(lr_changes_so_far))


def accept_stage_name(desc, is_decompress, i):
    s = lib.accept_stage_name(ctypes.byref(desc), int(is_decompress), int(i))
    return s.decode() if s else None


# ---------------------------------------------------------------------- device-side calls
# A small tensor's call is host time.  accept_compress, accept_decompress and accept_mbq_compress_first go
# through csrc/native.cpp, which makes the checks below and the call in one step; whatever it does not
# take (its answer is negative then, and nothing has been done) comes here.  It reads a descriptor's bytes, so it
# is given none but Desc: other objects of 64 bytes go the way on which they are refused.
# Here sizes are asked for once per geometry, tensors are looked at with a handful of
# attribute reads, and pointers and the stream travel as plain integers: 6-8 us.
_DTYPES = (torch.float32, torch.bfloat16)   # by F32 / BF16
_GEOMETRY_BYTES = Desc.seed.offset          # the fields before seed and t: all that sizes depend on
_SIZES = {}                                 # geometry -> (header, payload, workspace) bytes
_MAX_SIZES = 1024


def _sizes(desc):
    """(header, payload, workspace) bytes of a descriptor; raises on a bad one."""
    key = bytes(desc)[:_GEOMETRY_BYTES]
    got = _SIZES.get(key)
    if got is None or desc.t < 0:  # (a negative t is the one other thing that makes a descriptor bad)
        hb, pb = accept_packed_size(desc)
        got = (hb, pb, accept_workspace_size(desc))
        if len(_SIZES) >= _MAX_SIZES:
            _SIZES.clear()
        _SIZES[key] = got
    return got


_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream_handle():
    if _raw_stream is not None:  # the current stream's handle without building a Stream object
        return _raw_stream(torch.cuda.current_device())
    return torch.cuda.current_stream().cuda_stream


def _ptr(t):
    return t.data_ptr() if t is not None else None


def dtype_code(t):
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise TypeError("unsupported dtype %s (float32 or bfloat16)" % t.dtype)


def alloc_outputs(desc, device):
    """header (uint8, 4-byte sized), payload (uint8) and workspace (uint8, zero-filled as the
    library asks of a fresh workspace) device buffers."""
    hb, pb, wb = _sizes(desc)
    header = torch.empty(hb, dtype=torch.uint8, device=device)
    payload = torch.empty(max(pb, 1), dtype=torch.uint8, device=device)[:pb]
    workspace = torch.zeros(wb, dtype=torch.uint8, device=device)
    return header, payload, workspace


# ---- argument checks before any pointer reaches the library --------------------------------
# The C functions take no capacities: a tensor that is smaller than the descriptor says, or of
# another element type, would make a kernel read or write outside it.  Everything is checked
# here, on the host, and refused with the status code the C header reserves for it.
INVALID_ARG, BUFFER_TOO_SMALL = 1, 3


def _nbytes(t):
    return t.numel() * t.element_size()


def _check_tensor(t, where, what, dtype_is=None, min_elems=None, min_bytes=None):
    if t is None:
        raise AcceptError(INVALID_ARG, "%s: %s is missing" % (where, what))
    if not t.is_cuda:
        raise AcceptError(INVALID_ARG, "%s: %s is not a device tensor" % (where, what))
    if not t.is_contiguous():
        raise AcceptError(INVALID_ARG, "%s: %s is not contiguous" % (where, what))
    if dtype_is is not None and dtype_code(t) != dtype_is:
        raise AcceptError(INVALID_ARG, "%s: %s has dtype %s, the descriptor says %s"
                          % (where, what, t.dtype, "bfloat16" if dtype_is == BF16 else "float32"))
    if min_elems is not None and t.numel() < min_elems:
        raise AcceptError(BUFFER_TOO_SMALL, "%s: %s has %d elements, %d needed" % (where, what, t.numel(), min_elems))
    if min_bytes is not None and _nbytes(t) < min_bytes:
        raise AcceptError(BUFFER_TOO_SMALL, "%s: %s has %d bytes, %d needed" % (where, what, _nbytes(t), min_bytes))


# The checks' quick form: true if a tensor is fine; whatever is not goes through _check_tensor, which
# says what is wrong.
def _holds_bytes(t, nbytes):
    return t is not None and t.is_cuda and t.numel() * t.element_size() >= nbytes and t.is_contiguous()


def _holds_elems(t, dtype, elems):
    return t is not None and t.dtype is dtype and t.is_cuda and t.numel() >= elems and t.is_contiguous()


def _check_compress_args(where, desc, x, alpha_prev, header, payload, workspace, need_alpha):
    hb, pb, wb = _sizes(desc)  # raises on a bad descriptor
    if not _holds_elems(x, _DTYPES[desc.in_dtype], desc.n * desc.m):
        _check_tensor(x, where, "x", dtype_is=desc.in_dtype, min_elems=desc.n * desc.m)
    if not _holds_bytes(header, hb):
        _check_tensor(header, where, "header", min_bytes=hb)
    if not _holds_bytes(payload, pb):
        _check_tensor(payload, where, "payload", min_bytes=pb)
    if workspace is not None and not _holds_bytes(workspace, wb):
        _check_tensor(workspace, where, "workspace", min_bytes=wb)
    if need_alpha and desc.scheme == MBQ and not _holds_elems(alpha_prev, torch.float32, desc.bits):
        _check_tensor(alpha_prev, where, "alpha_prev", dtype_is=F32, min_elems=desc.bits)


def _check_decompress_args(where, desc, header, payload):
    hb, pb, _ = _sizes(desc)
    if not _holds_bytes(header, hb):
        _check_tensor(header, where, "header", min_bytes=hb)
    if not _holds_bytes(payload, pb):
        _check_tensor(payload, where, "payload", min_bytes=pb)


def _check_out(where, desc, out):
    if not _holds_elems(out, _DTYPES[desc.out_dtype], desc.n * desc.m):
        _check_tensor(out, where, "out", dtype_is=desc.out_dtype, min_elems=desc.n * desc.m)


def accept_compress(desc, x, alpha_prev=None, header=None, payload=None, workspace=None):
    """Enqueue compression of the device tensor x on the current stream.

    Returns (header, payload) uint8 device tensors (allocated here unless passed in)."""
    if header is None or payload is None or workspace is None:
        h, p, w = alloc_outputs(desc, x.device)
        header = h if header is None else header
        payload = p if payload is None else payload
        workspace = w if workspace is None else workspace
    st = _native.compress(desc, x, alpha_prev, header, payload, workspace, False) if type(desc) is Desc else -1
    if st < 0:
        _check_compress_args("accept_compress", desc, x, alpha_prev, header, payload, workspace, True)
        st = lib.accept_compress(ctypes.byref(desc), _ptr(x), _ptr(alpha_prev), _ptr(header), _ptr(payload),
                                 _ptr(workspace), _stream_handle())
    if st != 0:
        _check(st, "accept_compress")
    return header, payload


def accept_compress_noalloc(desc, x, alpha_prev, header, payload):
    """accept_compress on the library's built-in scratch: the caller passes every buffer and
    nothing is allocated, here or in the library."""
    _check_compress_args("accept_compress_noalloc", desc, x, alpha_prev, header, payload, None, True)
    st = lib.accept_compress_noalloc(ctypes.byref(desc), _ptr(x), _ptr(alpha_prev), _ptr(header), _ptr(payload),
                                     _stream_handle())
    _check(st, "accept_compress_noalloc")
    return header, payload


def accept_decompress(desc, header, payload, out=None):
    """Enqueue decompression on the current stream; returns the flat x_hat device tensor."""
    st = _native.decompress(desc, header, payload, out) if type(desc) is Desc else -1
    if type(st) is torch.Tensor:  # made there, in place of the `out` that was not given
        return st
    if st < 0:
        if out is None:
            _check_decompress_args("accept_decompress", desc, header, payload)
            out = torch.empty(desc.n * desc.m, dtype=_DTYPES[desc.out_dtype], device=payload.device)
        _check_decompress_args("accept_decompress", desc, header, payload)
        _check_out("accept_decompress", desc, out)
        st = lib.accept_decompress(ctypes.byref(desc), _ptr(header), _ptr(payload), _ptr(out), _stream_handle())
    if st != 0:
        _check(st, "accept_decompress")
    return out


def accept_mbq_init(desc, x, alpha0=None, workspace=None):
    accept_packed_size(desc)
    _check_tensor(x, "accept_mbq_init", "x", dtype_is=desc.in_dtype, min_elems=desc.n * desc.m)
    if alpha0 is None:
        alpha0 = torch.empty(desc.bits, dtype=torch.float32, device=x.device)
    if workspace is None:
        workspace = torch.zeros(accept_workspace_size(desc), dtype=torch.uint8, device=x.device)
    _check_tensor(alpha0, "accept_mbq_init", "alpha0", dtype_is=F32, min_elems=desc.bits)
    _check_tensor(workspace, "accept_mbq_init", "workspace", min_bytes=accept_workspace_size(desc))
    st = lib.accept_mbq_init(ctypes.byref(desc), _ptr(x), _ptr(alpha0), _ptr(workspace), _stream_handle())
    _check(st, "accept_mbq_init")
    return alpha0


def accept_mbq_compress_first(desc, x, header=None, payload=None, workspace=None):
    """Batch 0 of an epoch: residue initialisation; returns (header, payload) like accept_compress."""
    if header is None or payload is None or workspace is None:
        h, p, w = alloc_outputs(desc, x.device)
        header = h if header is None else header
        payload = p if payload is None else payload
        workspace = w if workspace is None else workspace
    st = _native.compress(desc, x, None, header, payload, workspace, True) if type(desc) is Desc else -1
    if st < 0:
        _check_compress_args("accept_mbq_compress_first", desc, x, None, header, payload, workspace, False)
        st = lib.accept_mbq_compress_first(ctypes.byref(desc), _ptr(x), _ptr(header), _ptr(payload), _ptr(workspace),
                                           _stream_handle())
    if st != 0:
        _check(st, "accept_mbq_compress_first")
    return header, payload


def accept_compress_timed(desc, x, alpha_prev, header, payload, workspace):
    """Measurement variant: returns {stage name: milliseconds}; synchronises."""
    _check_compress_args("accept_compress_timed", desc, x, alpha_prev, header, payload, workspace, True)
    ms = (ctypes.c_float * MAX_STAGES)()
    ns = ctypes.c_int(0)
    st = lib.accept_compress_timed(ctypes.byref(desc), _ptr(x), _ptr(alpha_prev), _ptr(header), _ptr(payload),
                                   _ptr(workspace), _stream_handle(), ms, ctypes.byref(ns))
    _check(st, "accept_compress_timed")
    return [(accept_stage_name(desc, 0, i), float(ms[i])) for i in range(ns.value)]


def accept_compress_polls(desc, x, header, payload, workspace, polls):
    """accept_compress (scheme M: accept_mbq_compress_first) with fewer looks at other workgroups (see accept_profile.h)."""
    _check_compress_args("accept_compress_polls", desc, x, None, header, payload, workspace, False)
    st = lib.accept_compress_polls(ctypes.byref(desc), _ptr(x), _ptr(None), _ptr(header), _ptr(payload),
                                   _ptr(workspace), _stream_handle(), int(polls))
    _check(st, "accept_compress_polls")
    return header, payload


def accept_decompress_timed(desc, header, payload, out):
    _check_decompress_args("accept_decompress_timed", desc, header, payload)
    _check_out("accept_decompress_timed", desc, out)
    ms = (ctypes.c_float * MAX_STAGES)()
    ns = ctypes.c_int(0)
    st = lib.accept_decompress_timed(ctypes.byref(desc), _ptr(header), _ptr(payload), _ptr(out), _stream_handle(),
                                     ms, ctypes.byref(ns))
    _check(st, "accept_decompress_timed")
    return [(accept_stage_name(desc, 1, i), float(ms[i])) for i in range(ns.value)]
