"""Binding of libspin.so (include/spin.h).  Argument marshalling only: every step of the protocol runs in the library's kernels.
The frequent calls first go through a compiled binding (csrc/binding.cpp); whatever that does not take is done here with ctypes.

Ring tensors are torch.int64 CUDA tensors (the bit pattern of a uint64 ring
element), party-major ([n, ...]).  Calls are enqueued on torch's current
stream.  The library must have been built (python -m paper_2402_02320_amd.build);
there is no fallback: a missing library raises.
"""
import ctypes
import importlib.util
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libspin.so")

LIMB_MFMA, VALU = 0, 1
MAX_PARTIES = 8

_lib = None
# The compiled binding (csrc/binding.cpp), there once lib() has loaded the library.  Its functions return None for every call that is not
# well formed, or not theirs; the code below each of them then says what is wrong, or does it.
BINDING_PATH = os.path.join(_HERE, "_binding.so")
_fast = None


class SpinError(RuntimeError):
    pass


def lib():
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise SpinError("%s not found: build it with `python -m paper_2402_02320_amd.build`" % LIB_PATH)
        L = ctypes.CDLL(LIB_PATH)
        u64, sz, i32, p = ctypes.c_uint64, ctypes.c_size_t, ctypes.c_int, ctypes.c_void_p
        L.spin_random.argtypes = [p, sz, u64, u64, u64, u64, p]
        L.spin_share.argtypes = [p, sz, i32, u64, u64, p, p]
        L.spin_open.argtypes = [p, p, sz, i32, p, p]
        L.spin_beaver_matmul.argtypes = [i32] * 5 + [p] * 6 + [i32, p, sz, p]
        L.spin_beaver_matmul_nt.argtypes = L.spin_beaver_matmul.argtypes
        L.spin_beaver_matmul_nt.restype = i32
        L.spin_beaver_matmul_static.argtypes = [i32] * 5 + [p] * 6 + [i32, p]
        L.spin_beaver_matmul_static.restype = i32
        L.spin_beaver_matmul_grouped.argtypes = [i32, i32, p, i32, p, sz, p]
        L.spin_beaver_matmul_grouped.restype = i32
        L.spin_beaver_matmul_grouped_workspace_bytes.argtypes = [i32, i32, p, i32]
        L.spin_beaver_matmul_grouped_workspace_bytes.restype = sz
        L.spin_beaver_matmul_workspace_bytes.argtypes = [i32] * 5 + [i32]
        L.spin_beaver_matmul_workspace_bytes.restype = sz
        L.spin_beaver_matmul_preferred_workspace_bytes.argtypes = [i32] * 5 + [i32]
        L.spin_beaver_matmul_preferred_workspace_bytes.restype = sz
        L.spin128_beaver_matmul_preferred_workspace_bytes.argtypes = [i32] * 5 + [i32]
        L.spin128_beaver_matmul_preferred_workspace_bytes.restype = sz
        L.spin_beaver_mul.argtypes = [i32, sz] + [p] * 6 + [p]
        L.spin_beaver_mul_trunc.argtypes = [i32, sz, i32] + [p] * 9 + [p]
        L.spin_beaver_mul_trunc.restype = i32
        L.spin_beaver_mul_bcast.argtypes = [i32, sz, sz, sz, i32] + [p] * 6 + [p]
        L.spin_beaver_mul_bcast.restype = i32
        L.spin_trunc.argtypes = [i32, sz, i32] + [p] * 5 + [p]
        L.spin_lincomb_trunc.argtypes = [i32, sz, i32, p, p, u64, i32, p, p, p, p, p]
        L.spin_lincomb_trunc.restype = i32
        L.spin_completed_square_trunc.argtypes = [i32, sz, p, u64, u64, u64, u64, p, p, p, p, p]
        L.spin_completed_square_trunc.restype = i32
        L.spin_bshare.argtypes = [p, sz, i32, u64, u64, p, p]
        L.spin_bopen.argtypes = [p, p, sz, i32, p, p]
        L.spin_beaver_and.argtypes = [i32, sz] + [p] * 6 + [p]
        for name in ("spin_bshare", "spin_bopen", "spin_beaver_and"):
            getattr(L, name).restype = i32
        for name in ("spin_random", "spin_share", "spin_open", "spin_beaver_matmul", "spin_beaver_mul", "spin_trunc"):
            getattr(L, name).restype = i32
        L.spin_profile_enable.argtypes = [i32]
        L.spin_profile_enable.restype = None
        L.spin_profile_reset.restype = None
        L.spin_profile_read.argtypes = [i32, ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_uint)]
        L.spin_profile_read.restype = i32
        L.spin128_share.argtypes = L.spin_share.argtypes
        L.spin128_open.argtypes = L.spin_open.argtypes
        L.spin128_beaver_matmul.argtypes = L.spin_beaver_matmul.argtypes
        L.spin128_beaver_matmul_workspace_bytes.argtypes = L.spin_beaver_matmul_workspace_bytes.argtypes
        L.spin128_beaver_matmul_workspace_bytes.restype = sz
        L.spin128_beaver_mul.argtypes = L.spin_beaver_mul.argtypes
        L.spin128_trunc.argtypes = L.spin_trunc.argtypes
        for name in ("spin128_share", "spin128_open", "spin128_beaver_matmul", "spin128_beaver_mul", "spin128_trunc"):
            getattr(L, name).restype = i32
        L.spin32_share.argtypes = L.spin_share.argtypes
        L.spin32_open.argtypes = L.spin_open.argtypes
        L.spin32_beaver_matmul.argtypes = L.spin_beaver_matmul.argtypes
        L.spin32_beaver_matmul_workspace_bytes.argtypes = L.spin_beaver_matmul_workspace_bytes.argtypes
        L.spin32_beaver_matmul_workspace_bytes.restype = sz
        L.spin32_beaver_matmul_preferred_workspace_bytes.argtypes = L.spin_beaver_matmul_workspace_bytes.argtypes
        L.spin32_beaver_matmul_preferred_workspace_bytes.restype = sz
        L.spin32_beaver_mul.argtypes = L.spin_beaver_mul.argtypes
        L.spin32_trunc.argtypes = L.spin_trunc.argtypes
        L.spin_cast_64_to_32.argtypes = [p, sz, p, p]
        for name in ("spin32_share", "spin32_open", "spin32_beaver_matmul", "spin32_beaver_mul", "spin32_trunc",
                     "spin_cast_64_to_32"):
            getattr(L, name).restype = i32
        L.spin_matmul_way_of.argtypes = [i32] * 6 + [ctypes.POINTER(_MatmulWay)]
        L.spin_matmul_grouped_way_of.argtypes = [i32, i32, p, ctypes.POINTER(_MatmulWay)]
        L.spin_matmul_by.argtypes = [_MatmulWay] + [i32] * 6 + [p] * 6 + [i32, p, sz, p]
        L.spin_matmul_grouped_by.argtypes = [_MatmulWay, i32, i32, p, p, sz, p]
        for name in ("spin_matmul_way_of", "spin_matmul_grouped_way_of", "spin_matmul_by", "spin_matmul_grouped_by"):
            getattr(L, name).restype = i32
        L.spin_probe_mfma.argtypes = [p, i32, i32, p, p]
        L.spin_probe_mfma.restype = i32
        L.spin_status_string.argtypes = [i32]
        L.spin_status_string.restype = ctypes.c_char_p
        L.spin_last_hip_error.restype = ctypes.c_char_p
        _load_binding(L)
        _lib = L                                         # last: a binding that does not load raises on every call
    return _lib


def _load_binding(L):
    global _fast
    if not os.path.exists(BINDING_PATH):
        raise SpinError("%s not found: build it with `python -m paper_2402_02320_amd.build`" % BINDING_PATH)
    spec = importlib.util.spec_from_file_location("_binding", BINDING_PATH)
    try:
        binding = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(binding)
    except ImportError as e:                             # built against another torch, above all
        raise SpinError("%s does not load (build it anew with `python -m paper_2402_02320_amd.build`): %s" % (BINDING_PATH, e)) from e
    entries = ("share", "bshare", "open", "bopen", "beaver_mul", "beaver_and", "trunc", "beaver_matmul", "beaver_matmul_nt",
               "beaver_matmul_preferred_workspace_bytes", "beaver_matmul_grouped", "beaver_matmul_grouped_workspace_bytes",
               "completed_square_trunc")
    binding.bind(tuple(ctypes.cast(getattr(L, "spin_" + e), ctypes.c_void_p).value for e in entries), _UNASKED_BYTES)
    _fast = binding


def _done(result):
    """What the compiled binding answered with: the result, or a status of the library."""
    if type(result) is int:
        _check(result)
    return result


def _check(status):
    if status != 0:
        L = lib()
        msg = L.spin_status_string(status).decode()
        if status == 4:
            msg += ": " + L.spin_last_hip_error().decode()
        raise SpinError(msg)


def _check_matmul(status, workspace_bytes_of, *dims):
    """_check, with the dimensions' own message.  Asked for after the call, not before: the query takes a microsecond."""
    if status != 0:
        if workspace_bytes_of(*dims) == 0:
            raise SpinError("invalid matmul dimensions")
        _check(status)


def _dev(t, name):
    if not (isinstance(t, torch.Tensor) and t.is_cuda and t.dtype == torch.int64 and t.is_contiguous()):
        raise SpinError("%s must be a contiguous torch.int64 CUDA tensor" % name)
    return t.data_ptr()


def _enough(out, words, exactly=False):
    """Raises where the caller's `out` is not the size of the result: the kernels write that many words wherever it points.  A longer
    one holds the result in front, except where the library reads the number of elements off it."""
    if out.numel() < words or (exactly and out.numel() != words):
        raise SpinError("out has %d words, the result %d" % (out.numel(), words))


def _dev_out(t, name, words, exactly=False):
    ptr = _dev(t, name)
    _enough(t, words, exactly)
    return ptr


def _workspace_ptr(t):
    if not (t.is_cuda and t.is_contiguous()):
        raise SpinError("workspace must be a contiguous CUDA tensor")
    return t.data_ptr()


def _same_words(x, *others):
    """Raises where an operand of an elementwise call has another number of words than the first: the library takes one count for all."""
    for t in others:
        if t is not None and t.numel() != x.numel():
            raise SpinError("inconsistent operand shapes")


# The handle of torch's current stream.  torch.cuda.current_stream() builds a Stream object around it, 2.6 us of the 6 to 9
# a call takes on the host; the raw query takes 0.3 us.  Every call asks anew: streams are the caller's to change.
if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    def _stream():
        return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())
else:
    def _stream():
        return torch.cuda.current_stream().cuda_stream


def random(count, seed, stream_id, party, first_idx=0, device="cuda"):
    out = torch.empty(count, dtype=torch.int64, device=device)
    _check(lib().spin_random(_dev(out, "out"), count, seed, stream_id, party, first_idx, _stream()))
    return out


def share(x, n, seed, stream_id, out=None):
    if _fast is not None:
        r = _fast.share(x, n, seed, stream_id, out)
        if r is not None:
            return _done(r)
    if out is None:
        out = torch.empty((n,) + tuple(x.shape), dtype=torch.int64, device=x.device)
    _check(lib().spin_share(_dev(x, "x"), x.numel(), n, seed, stream_id, _dev_out(out, "shares", n * x.numel()), _stream()))
    return out


def open(shares, mask=None, out=None):  # noqa: A001 - named after the C entry point
    if _fast is not None:
        r = _fast.open(shares, mask, out)
        if r is not None:
            return _done(r)
    n = shares.shape[0]
    if out is None:
        out = torch.empty(tuple(shares.shape[1:]), dtype=torch.int64, device=shares.device)
    if mask is not None and mask.shape != shares.shape:
        raise SpinError("mask must have the shape of shares")
    _check(lib().spin_open(_dev(shares, "shares"), None if mask is None else _dev(mask, "mask"),
                           out.numel(), n, _dev_out(out, "out", shares.numel() // (n or 1), True), _stream()))
    return out


def beaver_matmul_workspace_bytes(n, batch, M, N, K, path=LIMB_MFMA):
    return int(lib().spin_beaver_matmul_workspace_bytes(n, batch, M, N, K, path))


def beaver_matmul_preferred_workspace_bytes(n, batch, M, N, K, path=LIMB_MFMA):
    """The size with which beaver_matmul is fastest; never below beaver_matmul_workspace_bytes."""
    return int(lib().spin_beaver_matmul_preferred_workspace_bytes(n, batch, M, N, K, path))


# Workspace beyond what a call needs that is taken without a look at the device's memory (0.02 % of it): the look takes 5 to 50 us on
# the host, as much as a call takes whose workspaces differ by less.
_UNASKED_BYTES = 64 << 20


def _has_room(size, device):
    """Whether `size` bytes are at most a quarter of the memory this process can still get on the device.  Asking torch for more
    than there is makes it synchronise and give its whole cache back before it fails, on every call."""
    free, total = torch.cuda.mem_get_info(device)
    share = torch.cuda.get_per_process_memory_fraction(device)
    if share == 1.0 and 4 * size <= free:
        return True
    if torch.cuda.is_current_stream_capturing():
        return False                                     # a graph's own pool has no use for what torch has cached
    stats = torch.cuda.memory_stats(device)
    reserved = stats.get("reserved_bytes.all.current", 0)
    cached = reserved - stats.get("allocated_bytes.all.current", 0) - stats.get("inactive_split_bytes.all.current", 0)
    return 4 * size <= min(free, int(share * total) - reserved) + cached


def _matmul_workspace(dims, path, need_of, preferred_of, device):
    """A workspace of the preferred size, or, where memory is short, of the size needed."""
    size = int(preferred_of(*dims, path))
    if size == 0:
        raise SpinError("invalid matmul dimensions")
    if size > _UNASKED_BYTES and device.type == "cuda":      # smaller ones are not worth the second query
        need = int(need_of(*dims, path))
        if size > need + _UNASKED_BYTES and not _has_room(size, device):
            size = need
    try:
        return torch.empty(size, dtype=torch.uint8, device=device)
    except torch.OutOfMemoryError:
        need = int(need_of(*dims, path))
        if size == need:
            raise
        return torch.empty(need, dtype=torch.uint8, device=device)


def beaver_matmul(X, Y, A, B, C, path=LIMB_MFMA, out=None, workspace=None, y_transposed=False):
    """X, A: [n,batch,M,K]; Y, B: [n,batch,K,N] (or [n,batch,N,K] with y_transposed, for X . Y^T);
    C: [n,batch,M,N] -> Z [n,batch,M,N]."""
    if _fast is not None:
        r = _fast.matmul(X, Y, A, B, C, path, out, workspace, y_transposed)
        if r is not None:
            if type(r) is int:                           # never called again: a launch that failed may have added a part onto out
                _check_matmul(r, beaver_matmul_workspace_bytes, *X.shape[:3], C.shape[3], X.shape[3], path)
            return r
    n, batch, M, K = X.shape
    N = Y.shape[2] if y_transposed else Y.shape[3]
    yshape = (n, batch, N, K) if y_transposed else (n, batch, K, N)
    if tuple(Y.shape) != yshape or A.shape != X.shape or B.shape != Y.shape or tuple(C.shape) != (n, batch, M, N):
        raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(C)
    if workspace is None:
        workspace = _matmul_workspace((n, batch, M, N, K), path, lib().spin_beaver_matmul_workspace_bytes,
                                      lib().spin_beaver_matmul_preferred_workspace_bytes, X.device)
    call = lib().spin_beaver_matmul_nt if y_transposed else lib().spin_beaver_matmul
    _check_matmul(call(n, batch, M, N, K, _dev(X, "X"), _dev(Y, "Y"), _dev(A, "A"), _dev(B, "B"), _dev(C, "C"),
                       _dev_out(out, "Z", C.numel()), path, _workspace_ptr(workspace), workspace.numel() * workspace.element_size(), _stream()),
                  beaver_matmul_workspace_bytes, n, batch, M, N, K, path)
    return out


STATIC_WORKSPACE_BYTES = 64 << 20


def beaver_matmul_static(X, Y, A, B, C, out, path=LIMB_MFMA):
    """spin_beaver_matmul_static: the Beaver matmul on the library's built-in workspace.  The entry point
    allocates nothing, so the binding does not either: the caller passes `out`."""
    n, batch, M, K = X.shape
    N = Y.shape[3]
    if tuple(Y.shape) != (n, batch, K, N) or A.shape != X.shape or B.shape != Y.shape \
            or tuple(C.shape) != (n, batch, M, N) or out.shape != C.shape:
        raise SpinError("inconsistent operand shapes")
    _check(lib().spin_beaver_matmul_static(n, batch, M, N, K, _dev(X, "X"), _dev(Y, "Y"), _dev(A, "A"), _dev(B, "B"),
                                           _dev(C, "C"), _dev(out, "Z"), path, _stream()))
    return out


class _MatmulWay(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int), ("parts", ctypes.c_int)]


class _MatmulGroup(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int), ("M", ctypes.c_int), ("N", ctypes.c_int), ("K", ctypes.c_int),
                ("X", ctypes.c_void_p), ("Y", ctypes.c_void_p), ("A", ctypes.c_void_p), ("B", ctypes.c_void_p),
                ("C", ctypes.c_void_p), ("Z", ctypes.c_void_p), ("y_transposed", ctypes.c_int)]


def beaver_matmul_grouped(groups, path=LIMB_MFMA, workspace=None):
    """groups: list of dicts with X, Y, A, B, C (as for beaver_matmul), optional out and y_transposed; shapes may
    differ between groups, the party count may not.  Returns the list of Z tensors."""
    if _fast is not None:
        r = _fast.grouped(groups, path, workspace)
        if r is not None:
            return _done(r)
    n, desc, outs = _descriptors(groups)
    L = lib()
    need = int(L.spin_beaver_matmul_grouped_workspace_bytes(n, len(groups), desc, path))
    if need == 0:
        raise SpinError("invalid matmul dimensions")
    if workspace is None:
        workspace = torch.empty(need, dtype=torch.uint8, device=outs[0].device)
    _check(L.spin_beaver_matmul_grouped(n, len(groups), desc, path, _workspace_ptr(workspace),
                                        workspace.numel() * workspace.element_size(), _stream()))
    return outs


def _descriptors(groups):
    """The party count, the library's description of the groups and their results."""
    n = groups[0]["X"].shape[0]
    desc = (_MatmulGroup * len(groups))()
    outs = []
    for d, g in zip(desc, groups):
        X, Y, A, B, C = g["X"], g["Y"], g["A"], g["B"], g["C"]
        yt = bool(g.get("y_transposed", False))
        nn, batch, M, K = X.shape
        N = Y.shape[2] if yt else Y.shape[3]
        yshape = (n, batch, N, K) if yt else (n, batch, K, N)
        if nn != n or tuple(Y.shape) != yshape or A.shape != X.shape or B.shape != Y.shape \
                or tuple(C.shape) != (n, batch, M, N):
            raise SpinError("inconsistent operand shapes")
        out = g.get("out")
        if out is None:
            out = torch.empty_like(C)
        outs.append(out)
        d.batch, d.M, d.N, d.K = batch, M, N, K
        d.X, d.Y, d.A, d.B, d.C, d.Z = (_dev(t, k) for t, k in ((X, "X"), (Y, "Y"), (A, "A"), (B, "B"), (C, "C"), (out, "Z")))
        _enough(out, C.numel())
        d.y_transposed = 1 if yt else 0
    return n, desc, outs


def beaver_mul(x, y, a, b, c, out=None):
    if _fast is not None:
        r = _fast.beaver_mul(x, y, a, b, c, out)
        if r is not None:
            return _done(r)
    n = x.shape[0]
    shape = x.shape
    for t in (y, a, b, c):
        if t.shape != shape:
            raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(x)
    _check(lib().spin_beaver_mul(n, x.numel() // (n or 1), _dev(x, "x"), _dev(y, "y"), _dev(a, "a"), _dev(b, "b"),
                                 _dev(c, "c"), _dev_out(out, "z", x.numel()), _stream()))
    return out


def beaver_mul_trunc(x, y, a, b, c, r, r_top, r_msb, f, out=None):
    """Mul then Truncate by f bits in one pass; all operands [n, count]."""
    n = x.shape[0]
    shape = x.shape
    for t in (y, a, b, c, r, r_top, r_msb):
        if t.shape != shape:
            raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(x)
    _check(lib().spin_beaver_mul_trunc(n, x.numel() // (n or 1), f, _dev(x, "x"), _dev(y, "y"), _dev(a, "a"), _dev(b, "b"),
                                       _dev(c, "c"), _dev(r, "r"), _dev(r_top, "r_top"), _dev(r_msb, "r_msb"),
                                       _dev_out(out, "out", x.numel()), _stream()))
    return out


def beaver_mul_bcast(x, y, a, b, c, over_inner, out=None):
    """Batch multiplication with the small factor tiled (Section 7.3).  y, b, c: [n, outer, mid, inner];
    x, a: [n, outer, mid] (over_inner, one factor per row) or [n, outer, inner] (one per column)."""
    n, outer, mid, inner = y.shape
    small = (n, outer, mid) if over_inner else (n, outer, inner)
    if tuple(x.shape) != small or a.shape != x.shape or b.shape != y.shape or c.shape != y.shape:
        raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(y)
    _check(lib().spin_beaver_mul_bcast(n, outer, mid, inner, 1 if over_inner else 0, _dev(x, "x"), _dev(y, "y"),
                                       _dev(a, "a"), _dev(b, "b"), _dev(c, "c"), _dev_out(out, "z", y.numel()), _stream()))
    return out


def trunc(x, r, r_top, r_msb, f, out=None):
    if _fast is not None:
        t = _fast.trunc(x, r, r_top, r_msb, f, out)
        if t is not None:
            return _done(t)
    n = x.shape[0]
    shape = x.shape
    for t in (r, r_top, r_msb):
        if t.shape != shape:
            raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(x)
    _check(lib().spin_trunc(n, x.numel() // (n or 1), f, _dev(x, "x"), _dev(r, "r"), _dev(r_top, "r_top"),
                            _dev(r_msb, "r_msb"), _dev_out(out, "out", x.numel()), _stream()))
    return out


def bshare(x, n, seed, stream_id, out=None):
    if _fast is not None:
        r = _fast.bshare(x, n, seed, stream_id, out)
        if r is not None:
            return _done(r)
    if out is None:
        out = torch.empty((n,) + tuple(x.shape), dtype=torch.int64, device=x.device)
    _check(lib().spin_bshare(_dev(x, "x"), x.numel(), n, seed, stream_id, _dev_out(out, "shares", n * x.numel()), _stream()))
    return out


def bopen(shares, mask=None, out=None):
    if _fast is not None:
        r = _fast.bopen(shares, mask, out)
        if r is not None:
            return _done(r)
    n = shares.shape[0]
    if out is None:
        out = torch.empty(tuple(shares.shape[1:]), dtype=torch.int64, device=shares.device)
    if mask is not None and mask.shape != shares.shape:
        raise SpinError("mask must have the shape of shares")
    _check(lib().spin_bopen(_dev(shares, "shares"), None if mask is None else _dev(mask, "mask"),
                            out.numel(), n, _dev_out(out, "out", shares.numel() // (n or 1), True), _stream()))
    return out


def beaver_and(x, y, a, b, c, out=None):
    if _fast is not None:
        r = _fast.beaver_and(x, y, a, b, c, out)
        if r is not None:
            return _done(r)
    n = x.shape[0]
    shape = x.shape
    for t in (y, a, b, c):
        if t.shape != shape:
            raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(x)
    _check(lib().spin_beaver_and(n, x.numel() // (n or 1), _dev(x, "x"), _dev(y, "y"), _dev(a, "a"), _dev(b, "b"),
                                 _dev(c, "c"), _dev_out(out, "z", x.numel()), _stream()))
    return out


def lincomb_trunc(terms, coefs, constant=0, f=0, tuple_=None, out=None):
    """out = Truncate(sum_j coefs[j] * terms[j] + constant, f); f = 0 leaves the sum untruncated."""
    n = terms[0].shape[0]
    for t in terms:
        if t.shape != terms[0].shape:
            raise SpinError("inconsistent operand shapes")
    if out is None:
        out = torch.empty_like(terms[0])
    ptrs = (ctypes.c_void_p * len(terms))(*[_dev(t, "term") for t in terms])
    cf = (ctypes.c_uint64 * len(terms))(*[int(c) % (1 << 64) for c in coefs])
    r = rt = rm = None
    if f > 0:
        r, rt, rm = (_dev(t, "tuple") for t in tuple_)
        for t in tuple_:
            if t.numel() != terms[0].numel():
                raise SpinError("truncation tuple must have the shape of the terms")
    _check(lib().spin_lincomb_trunc(n, terms[0].numel() // (n or 1), len(terms), ptrs, cf, int(constant) % (1 << 64), f,
                                    r, rt, rm, _dev_out(out, "out", terms[0].numel()), _stream()))
    return out


def completed_square_trunc(x, t3, t2, lin, t0, triples, tuples, f, out=None):
    """((x + t3)^2 truncated by f[0], + t2)^2 + lin x + t0, truncated by f[1], in one pass.  t3, t2, lin, t0: public ring
    elements; triples, tuples: two (a, b, c) and two (r, r_top, r_msb) of x's shape."""
    if _fast is not None:
        r = _fast.completed_square(x, t3, t2, lin, t0, triples, tuples, f, out)
        if r is not None:
            return _done(r)
    for t in tuple(triples[0]) + tuple(tuples[0]) + tuple(triples[1]):
        if t.shape != x.shape:
            raise SpinError("inconsistent operand shapes")
    for t in tuples[1]:
        if t.numel() != x.numel():
            raise SpinError("truncation tuple must have the shape of the terms")
    if out is None:
        out = torch.empty_like(x)
    six = ctypes.c_void_p * 6
    (a0, b0, c0), (a1, b1, c1) = triples
    (r0, rt0, rm0), (r1, rt1, rm1) = tuples
    t_ptr = six(*[_dev(t, "triple") for t in (a0, b0, c0, a1, b1, c1)])
    u_ptr = six(*[_dev(t, "tuple") for t in (r0, rt0, rm0, r1, rt1, rm1)])
    const = [int(v) % (1 << 64) for v in (t3, t2, lin, t0)]
    _check(lib().spin_completed_square_trunc(x.shape[0], x.numel() // (x.shape[0] or 1), _dev(x, "x"), *const, t_ptr, u_ptr,
                                             (ctypes.c_int * 2)(*f), _dev_out(out, "out", x.numel()), _stream()))
    return out


class ring128:
    """The same calls over Z_2^128.  A ring tensor of shape S is a torch.int64 tensor of shape S + (2,):
    two 64-bit words per element, low word first."""

    @staticmethod
    def _elems(t):
        if t.shape[-1] != 2:
            raise SpinError("128-bit ring tensors carry a trailing axis of 2 words")
        return t.numel() // 2

    @staticmethod
    def share(x, n, seed, stream_id, out=None):
        if out is None:
            out = torch.empty((n,) + tuple(x.shape), dtype=torch.int64, device=x.device)
        _check(lib().spin128_share(_dev(x, "x"), ring128._elems(x), n, seed, stream_id, _dev_out(out, "shares", n * x.numel()), _stream()))
        return out

    @staticmethod
    def open(shares, mask=None, out=None):  # noqa: A003
        n = shares.shape[0]
        _same_words(shares, mask)
        if out is None:
            out = torch.empty(tuple(shares.shape[1:]), dtype=torch.int64, device=shares.device)
        _check(lib().spin128_open(_dev(shares, "shares"), None if mask is None else _dev(mask, "mask"),
                                  ring128._elems(out), n, _dev_out(out, "out", shares.numel() // (n or 1), True), _stream()))
        return out

    @staticmethod
    def beaver_matmul_workspace_bytes(n, batch, M, N, K, path=LIMB_MFMA):
        return int(lib().spin128_beaver_matmul_workspace_bytes(n, batch, M, N, K, path))

    @staticmethod
    def beaver_matmul_preferred_workspace_bytes(n, batch, M, N, K, path=LIMB_MFMA):
        return int(lib().spin128_beaver_matmul_preferred_workspace_bytes(n, batch, M, N, K, path))

    @staticmethod
    def beaver_matmul(X, Y, A, B, C, path=LIMB_MFMA, out=None, workspace=None):
        n, batch, M, K, _ = X.shape
        N = Y.shape[3]
        if tuple(Y.shape) != (n, batch, K, N, 2) or A.shape != X.shape or B.shape != Y.shape \
                or tuple(C.shape) != (n, batch, M, N, 2):
            raise SpinError("inconsistent operand shapes")
        if out is None:
            out = torch.empty_like(C)
        if workspace is None:
            workspace = _matmul_workspace((n, batch, M, N, K), path, lib().spin128_beaver_matmul_workspace_bytes,
                                          lib().spin128_beaver_matmul_preferred_workspace_bytes, X.device)
        _check_matmul(lib().spin128_beaver_matmul(n, batch, M, N, K, _dev(X, "X"), _dev(Y, "Y"), _dev(A, "A"), _dev(B, "B"),
                                                  _dev(C, "C"), _dev_out(out, "Z", C.numel()), path, _workspace_ptr(workspace),
                                                  workspace.numel() * workspace.element_size(), _stream()),
                      ring128.beaver_matmul_workspace_bytes, n, batch, M, N, K, path)
        return out

    @staticmethod
    def beaver_mul(x, y, a, b, c, out=None):
        n = x.shape[0]
        _same_words(x, y, a, b, c)
        if out is None:
            out = torch.empty_like(x)
        _check(lib().spin128_beaver_mul(n, ring128._elems(x) // (n or 1), _dev(x, "x"), _dev(y, "y"), _dev(a, "a"),
                                        _dev(b, "b"), _dev(c, "c"), _dev_out(out, "z", x.numel()), _stream()))
        return out

    @staticmethod
    def trunc(x, r, r_top, r_msb, f, out=None):
        n = x.shape[0]
        _same_words(x, r, r_top, r_msb)
        if out is None:
            out = torch.empty_like(x)
        _check(lib().spin128_trunc(n, ring128._elems(x) // (n or 1), f, _dev(x, "x"), _dev(r, "r"), _dev(r_top, "r_top"),
                                   _dev(r_msb, "r_msb"), _dev_out(out, "out", x.numel()), _stream()))
        return out


def _dev32_out(t, name, words, exactly=False):
    ptr = _dev32(t, name)
    _enough(t, words, exactly)
    return ptr


def _dev32(t, name):
    if not (isinstance(t, torch.Tensor) and t.is_cuda and t.dtype == torch.int32 and t.is_contiguous()):
        raise SpinError("%s must be a contiguous torch.int32 CUDA tensor" % name)
    return t.data_ptr()


class ring32:
    """The same calls over Z_2^32 (the Fixed32 representation of Section 7.1).  Ring tensors are
    torch.int32 CUDA tensors (the bit pattern of a uint32 ring element), party-major."""

    @staticmethod
    def cast_from_64(shares, out=None):
        """Local Fixed64 -> Fixed32 cast: every party keeps the low half of its own share."""
        if out is None:
            out = torch.empty(tuple(shares.shape), dtype=torch.int32, device=shares.device)
        _check(lib().spin_cast_64_to_32(_dev(shares, "shares"), shares.numel(), _dev32_out(out, "out", shares.numel()), _stream()))
        return out

    @staticmethod
    def share(x, n, seed, stream_id, out=None):
        if out is None:
            out = torch.empty((n,) + tuple(x.shape), dtype=torch.int32, device=x.device)
        _check(lib().spin32_share(_dev32(x, "x"), x.numel(), n, seed, stream_id, _dev32_out(out, "shares", n * x.numel()), _stream()))
        return out

    @staticmethod
    def open(shares, mask=None, out=None):  # noqa: A003
        n = shares.shape[0]
        if out is None:
            out = torch.empty(tuple(shares.shape[1:]), dtype=torch.int32, device=shares.device)
        if mask is not None and mask.shape != shares.shape:
            raise SpinError("mask must have the shape of shares")
        _check(lib().spin32_open(_dev32(shares, "shares"), None if mask is None else _dev32(mask, "mask"),
                                 out.numel(), n, _dev32_out(out, "out", shares.numel() // (n or 1), True), _stream()))
        return out

    @staticmethod
    def beaver_matmul_workspace_bytes(n, batch, M, N, K, path=LIMB_MFMA):
        return int(lib().spin32_beaver_matmul_workspace_bytes(n, batch, M, N, K, path))

    @staticmethod
    def beaver_matmul_preferred_workspace_bytes(n, batch, M, N, K, path=LIMB_MFMA):
        return int(lib().spin32_beaver_matmul_preferred_workspace_bytes(n, batch, M, N, K, path))

    @staticmethod
    def beaver_matmul(X, Y, A, B, C, path=LIMB_MFMA, out=None, workspace=None):
        n, batch, M, K = X.shape
        N = Y.shape[3]
        if tuple(Y.shape) != (n, batch, K, N) or A.shape != X.shape or B.shape != Y.shape \
                or tuple(C.shape) != (n, batch, M, N):
            raise SpinError("inconsistent operand shapes")
        if out is None:
            out = torch.empty_like(C)
        if workspace is None:
            L = lib()
            workspace = _matmul_workspace((n, batch, M, N, K), path, L.spin32_beaver_matmul_workspace_bytes,
                                          L.spin32_beaver_matmul_preferred_workspace_bytes, X.device)
        _check_matmul(lib().spin32_beaver_matmul(n, batch, M, N, K, _dev32(X, "X"), _dev32(Y, "Y"), _dev32(A, "A"),
                                                 _dev32(B, "B"), _dev32(C, "C"), _dev32_out(out, "Z", C.numel()), path,
                                                 _workspace_ptr(workspace), workspace.numel() * workspace.element_size(),
                                                 _stream()),
                      ring32.beaver_matmul_workspace_bytes, n, batch, M, N, K, path)
        return out

    @staticmethod
    def beaver_mul(x, y, a, b, c, out=None):
        n = x.shape[0]
        _same_words(x, y, a, b, c)
        if out is None:
            out = torch.empty_like(x)
        _check(lib().spin32_beaver_mul(n, x.numel() // (n or 1), _dev32(x, "x"), _dev32(y, "y"), _dev32(a, "a"),
                                       _dev32(b, "b"), _dev32(c, "c"), _dev32_out(out, "z", x.numel()), _stream()))
        return out

    @staticmethod
    def trunc(x, r, r_top, r_msb, f, out=None):
        n = x.shape[0]
        _same_words(x, r, r_top, r_msb)
        if out is None:
            out = torch.empty_like(x)
        _check(lib().spin32_trunc(n, x.numel() // (n or 1), f, _dev32(x, "x"), _dev32(r, "r"), _dev32(r_top, "r_top"),
                                  _dev32(r_msb, "r_msb"), _dev32_out(out, "out", x.numel()), _stream()))
        return out


KERNELS = {"random": 0, "share": 1, "open": 2, "beaver_mul": 3, "trunc": 4, "pack": 5, "gemm_limb": 6,
           "gemm_valu": 7, "lincomb": 8, "binary": 9, "cast": 10, "probe": 11, "beaver_mul_trunc": 12,
           "gemm_residue": 13, "combine": 14, "gemm_direct": 15}


def probe_mfma(operands, blocks, iters, sink=None):
    """Register-only int8 MFMA loop on the 24 operand fragments in `operands` ([24*128] int64); returns sink."""
    if operands.numel() != 24 * 128:
        raise SpinError("operands must hold 24 fragments of 128 words")
    if sink is None:
        sink = torch.empty(blocks * 256, dtype=torch.int64, device=operands.device)
    _check(lib().spin_probe_mfma(_dev(operands, "operands"), blocks, iters, _dev_out(sink, "sink", blocks * 256), _stream()))
    return sink


PROBE_OPS_PER_WAVE_ITERATION = 72 * 65536      # 72 MFMAs of 32x32x32 multiply-adds, two operations each


# Kernels by name (spin_bench.h): what a matmul would take, and a matmul by the one that is named, for tests and measurements.
WAYS = {"direct": 0, "rows": 1, "full": 2, "half": 3, "quarter": 4, "residues": 5, "separate": 6}
_WAY_NAMES = {v: k for k, v in WAYS.items()}


def matmul_way(n, batch, M, N, K, bits=64):
    """(name, parts) of the kernel among the digit kernels and the direct one; needs no GPU."""
    way = _MatmulWay()
    _check(lib().spin_matmul_way_of(bits, n, batch, M, N, K, ctypes.byref(way)))
    return _WAY_NAMES[way.kernel], way.parts


def matmul_grouped_way(n, shapes):
    """The name of the kernel that a grouped call takes; shapes: (batch, M, N, K) or (batch, M, N, K, y_transposed).  Needs no GPU."""
    desc = (_MatmulGroup * len(shapes))()
    for d, s in zip(desc, shapes):
        d.batch, d.M, d.N, d.K = s[:4]
        d.y_transposed = 1 if len(s) > 4 and s[4] else 0
    way = _MatmulWay()
    _check(lib().spin_matmul_grouped_way_of(n, len(shapes), desc, ctypes.byref(way)))
    return _WAY_NAMES[way.kernel]


def beaver_matmul_by(name, parts, X, Y, A, B, C, out=None, workspace=None, y_transposed=False):
    """beaver_matmul (or, of int32 tensors, ring32.beaver_matmul) by the named kernel."""
    n, batch, M, K = X.shape
    N = C.shape[3]
    if tuple(Y.shape) != ((n, batch, N, K) if y_transposed else (n, batch, K, N)) or A.shape != X.shape or B.shape != Y.shape \
            or tuple(C.shape) != (n, batch, M, N):
        raise SpinError("inconsistent operand shapes")
    bits, dev, dev_out = (64, _dev, _dev_out) if X.dtype == torch.int64 else (32, _dev32, _dev32_out)
    if out is None:
        out = torch.empty_like(C)
    if workspace is None:
        need = (beaver_matmul_workspace_bytes if bits == 64 else ring32.beaver_matmul_workspace_bytes)(n, batch, M, N, K)
        workspace = torch.empty(need, dtype=torch.uint8, device=X.device)
    _check(lib().spin_matmul_by(_MatmulWay(WAYS[name], parts), bits, n, batch, M, N, K, dev(X, "X"), dev(Y, "Y"), dev(A, "A"), dev(B, "B"),
                                dev(C, "C"), dev_out(out, "Z", C.numel()), 1 if y_transposed else 0, _workspace_ptr(workspace),
                                workspace.numel() * workspace.element_size(), _stream()))
    return out


def beaver_matmul_grouped_by(name, groups, workspace=None):
    """beaver_matmul_grouped with all products by the named kernel: rows, full or half tiles."""
    n, desc, outs = _descriptors(groups)
    if workspace is None:
        need = int(lib().spin_beaver_matmul_grouped_workspace_bytes(n, len(groups), desc, LIMB_MFMA))
        workspace = torch.empty(need, dtype=torch.uint8, device=outs[0].device)
    _check(lib().spin_matmul_grouped_by(_MatmulWay(WAYS[name], 1), n, len(groups), desc, _workspace_ptr(workspace),
                                        workspace.numel() * workspace.element_size(), _stream()))
    return outs


def profile_enable(on=True):
    lib().spin_profile_enable(1 if on else 0)


def profile_reset():
    lib().spin_profile_reset()


def profile_read(kernel):
    """(total milliseconds, launches) of one kernel class since the last reset; waits for the events."""
    ms, cnt = ctypes.c_double(0.0), ctypes.c_uint(0)
    _check(lib().spin_profile_read(KERNELS[kernel], ctypes.byref(ms), ctypes.byref(cnt)))
    return ms.value, cnt.value


# Fixed-point encoding of Section 4.1 (host-side convenience for the harness; not part of the C ABI).
def encode(x, f):
    """float64 tensor -> ring tensor holding floor(x * 2^f)."""
    return torch.floor(torch.ldexp(x.to(torch.float64), torch.tensor(f))).to(torch.int64)


def decode(u, f):
    return torch.ldexp(u.to(torch.float64), torch.tensor(-f))
