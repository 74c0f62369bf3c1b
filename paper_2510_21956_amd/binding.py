"""ctypes binding with the same names as the C ABI in include/la.h.

Argument marshalling only; for calls on plain tensors without a trace it is done in native code
(csrc/la_bind.cpp, _marshal.so), by the same rules.  There is no CPU fallback: if libla.so has not been
built, loading fails with an error that says how to build it.
"""
import ctypes
import importlib.util
import os
import sys
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libla.so")
_MARSHAL_PATH = os.path.join(_HERE, "_marshal.so")
_lib = None
_native = None  # the module of _marshal.so once the library is loaded

LA_F32 = 0
LA_BF16 = 1

LA_MAX_TRACE = 8

EXPORTS = ("la_version", "la_status_string", "la_workspace_bytes", "la_forward", "la_backward",
           "la_forward_traced", "la_backward_traced", "la_saved_state_bytes", "la_forward_save",
           "la_backward_saved", "la_debug_override", "la_forward_static", "la_decode_state_bytes",
           "la_decode_step", "la_decode_prefill", "la_backward_ab", "la_forward_qknorm",
           "la_backward_qknorm", "la_forward_qknorm_save", "la_backward_qknorm_saved")


class la_trace(ctypes.Structure):
    """struct la_trace of include/la.h."""
    _fields_ = [("events", ctypes.POINTER(ctypes.c_void_p)),
                ("capacity", ctypes.c_int),
                ("recorded", ctypes.c_int),
                ("names", ctypes.c_char_p * LA_MAX_TRACE)]


class LaError(RuntimeError):
    def __init__(self, code, where):
        self.code = int(code)
        super().__init__("%s failed: %s" % (where, la_status_string(code)))


def library_path():
    return _LIB_PATH


def load_library():
    """Load libla.so (built by paper_2510_21956_amd/build.py).  Raises if absent."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError(
            "HIP library %s not found; build it with "
            "`python -c 'import __graft_entry__ as g; g.build()'` "
            "(or python paper_2510_21956_amd/build.py).  There is no CPU fallback." % _LIB_PATH)
    lib = ctypes.CDLL(_LIB_PATH)
    vp, sz, i, f = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_float
    lib.la_version.restype = i
    lib.la_version.argtypes = []
    lib.la_status_string.restype = ctypes.c_char_p
    lib.la_status_string.argtypes = [i]
    lib.la_workspace_bytes.restype = sz
    lib.la_workspace_bytes.argtypes = [i, i, i, i, i, i, i]
    lib.la_forward.restype = i
    lib.la_forward.argtypes = [vp, vp, vp, vp, vp, i, i, i, i, f, f, i, i, vp, sz, vp]
    lib.la_backward.restype = i
    lib.la_backward.argtypes = [vp] * 9 + [i, i, i, i, f, f, i, i, vp, sz, vp]
    tp = ctypes.POINTER(la_trace)
    lib.la_forward_traced.restype = i
    lib.la_forward_traced.argtypes = lib.la_forward.argtypes + [tp]
    lib.la_backward_traced.restype = i
    lib.la_backward_traced.argtypes = lib.la_backward.argtypes + [tp]
    lib.la_saved_state_bytes.restype = sz
    lib.la_saved_state_bytes.argtypes = [i, i, i, i, i, i]
    lib.la_forward_save.restype = i
    lib.la_forward_save.argtypes = lib.la_forward.argtypes[:-1] + [vp, sz, vp, tp]
    lib.la_backward_saved.restype = i
    lib.la_backward_saved.argtypes = lib.la_backward.argtypes[:-1] + [vp, sz, vp, tp]
    lib.la_forward_static.restype = i
    lib.la_forward_static.argtypes = lib.la_forward.argtypes[:-3] + [vp]
    lib.la_decode_state_bytes.restype = sz
    lib.la_decode_state_bytes.argtypes = [i, i, i]
    lib.la_decode_step.restype = i
    lib.la_decode_step.argtypes = [vp, vp, vp, vp, vp, vp, sz, i, i, i, i, f, f, i, vp]
    lib.la_decode_prefill.restype = i
    lib.la_decode_prefill.argtypes = [vp, vp, vp, sz, i, i, i, i, i, i, vp, sz, vp]
    lib.la_forward_qknorm.restype = i
    lib.la_forward_qknorm.argtypes = lib.la_forward_traced.argtypes
    lib.la_backward_qknorm.restype = i
    lib.la_backward_qknorm.argtypes = lib.la_backward_traced.argtypes
    lib.la_forward_qknorm_save.restype = i
    lib.la_forward_qknorm_save.argtypes = lib.la_forward_save.argtypes
    lib.la_backward_qknorm_saved.restype = i
    lib.la_backward_qknorm_saved.argtypes = lib.la_backward_saved.argtypes
    lib.la_backward_ab.restype = i
    lib.la_backward_ab.argtypes = [vp] * 7 + [i, i, i, i, f, f, i, i, vp, sz, vp]
    lib.la_debug_override.restype = None
    lib.la_debug_override.argtypes = [i, i]
    _lib = lib
    _load_native(lib)
    return lib


def _load_native(lib):
    """The native marshalling, if there is one that fits; a file that does not load, or that was built for
    another torch or Python (whose tensors it would misread), is reported and left out: the Python functions
    below do all of it."""
    global _native
    if not os.path.exists(_MARSHAL_PATH):
        return
    try:
        _native = _open_native(lib)
    except Exception as e:
        warnings.warn("%s is not used, calls take a few microseconds longer: %s" % (_MARSHAL_PATH, e),
                      RuntimeWarning, stacklevel=3)


def _open_native(lib):
    spec = importlib.util.spec_from_file_location("_marshal", _MARSHAL_PATH)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    here = "torch %s, Python %d.%d" % (torch.__version__, *sys.version_info[:2])
    if getattr(module, "built_for", None) != here:
        raise ImportError("built for %s, not for %s" % (getattr(module, "built_for", "another version"), here))
    from . import autograd  # imports this module; by the first call both are there
    module.init(autograd.python_backward, _device_stream, *(ctypes.cast(f, ctypes.c_void_p).value for f in (
        lib.la_forward_traced, lib.la_forward_qknorm, lib.la_forward_save, lib.la_forward_qknorm_save,
        lib.la_backward_traced, lib.la_backward_qknorm, lib.la_backward_saved,
        lib.la_backward_qknorm_saved, lib.la_decode_step, lib.la_decode_prefill, lib.la_workspace_bytes,
        lib.la_saved_state_bytes)))
    return module


def la_version():
    return int(load_library().la_version())


def la_status_string(code):
    return load_library().la_status_string(int(code)).decode()


def la_debug_override(seg_len=0, force_generic=0):
    """la_debug_override of include/la.h (test / profiling hook; 0, 0 = automatic)."""
    load_library().la_debug_override(int(seg_len), int(bool(force_generic)))


def _dtype_code(t):
    if t.dtype == torch.float32:
        return LA_F32
    if t.dtype == torch.bfloat16:
        return LA_BF16
    raise TypeError("Q/K/V must be float32 or bfloat16, got %s" % t.dtype)


def la_workspace_bytes(B, H, N, D, dt, causal, is_backward):
    """is_backward: 0 forward, 1 backward, 2 backward that recomputes O / G (given as None)."""
    return int(load_library().la_workspace_bytes(B, H, N, D, dt, int(bool(causal)),
                                                 int(is_backward)))


def la_saved_state_bytes(B, H, N, D, dt, causal):
    return int(load_library().la_saved_state_bytes(B, H, N, D, dt, int(bool(causal))))


# A small call (a decode step, a toy layer) cost more in this file than on the GPU: a decode step of 128
# slices at D = 128, whose kernel takes 4.6 us, 7.4 us with the functions below and 4.8 us with the native
# ones, which return None for what they leave to these (other objects than tensors, a missing tensor, whatever
# is to be refused).
# What is done per tensor and per call is kept to integers: device indices, raw stream handles and
# addresses, which ctypes converts by the declared argument types.

def _check_tensors(ref, *ts):
    """Every tensor of a call, the first one included, is packed and on ref's device: the
    kernels read B*H*N*D elements from its address, whatever its strides say."""
    dev = ref.get_device()
    if not ref.is_cuda or not ref.is_contiguous():
        raise ValueError("tensors must be contiguous device tensors")
    for t in ts:
        if t is None:
            continue
        if not t.is_cuda or not t.is_contiguous():
            raise ValueError("tensors must be contiguous device tensors")
        if t.get_device() != dev:
            raise ValueError("tensors must live on one device")


_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _device_stream(index):
    """hipStream_t of the current stream of device ``index``."""
    if _raw_stream is not None:
        return _raw_stream(index)
    return torch.cuda.current_stream(index).cuda_stream


def _stream_ptr(stream, ref):
    """hipStream_t of ``stream``, or of the current stream of ref's device."""
    if stream is not None:
        return stream.cuda_stream
    return _device_stream(ref.get_device())


def _ptr(t):
    return None if t is None else t.data_ptr()


def la_forward(Q, K, V, O, G, a, b, causal, workspace, stream=None):
    """la_forward of include/la.h on torch device tensors.

    Q, K, V, O: [B, H, N, D] float32 or bfloat16; G: [B, H, N] float32;
    workspace: uint8 device tensor of at least la_workspace_bytes(..., 0) bytes."""
    la_forward_traced(Q, K, V, O, G, a, b, causal, workspace, stream, None)


LA_STATIC_SCRATCH_BYTES = 32 << 20


def la_forward_static(Q, K, V, O, G, a, b, causal, stream=None):
    """la_forward_static of include/la.h: la_forward with the library's own static scratch."""
    if Q.dim() != 4:
        raise ValueError("Q must be [B, H, N, D]")
    B, H, N, D = Q.shape
    _check_tensors(Q, K, V, O, G)
    if K.shape != Q.shape or V.shape != Q.shape or O.shape != Q.shape:
        raise ValueError("shape mismatch")
    if not (K.dtype == V.dtype == O.dtype == Q.dtype):
        raise TypeError("dtype mismatch")
    if G is not None and (G.shape != Q.shape[:3] or G.dtype != torch.float32):
        raise ValueError("G must be [B, H, N] float32 (or None)")
    rc = load_library().la_forward_static(_ptr(Q), _ptr(K), _ptr(V), _ptr(O), _ptr(G), B, H, N, D,
                                          float(a), float(b), int(bool(causal)), _dtype_code(Q),
                                          _stream_ptr(stream, Q))
    if rc != 0:
        raise LaError(rc, "la_forward_static")


def la_forward_traced(Q, K, V, O, G, a, b, causal, workspace, stream=None, trace=None):
    """la_forward_traced of include/la.h; ``trace`` is a la_trace structure or None."""
    _forward(Q, K, V, O, G, a, b, causal, workspace, None, stream, trace, False)


def la_forward_save(Q, K, V, O, G, a, b, causal, workspace, saved, stream=None, trace=None):
    """la_forward_save of include/la.h; ``saved`` is a uint8 device tensor of at least
    la_saved_state_bytes(...) bytes (None when that is 0)."""
    _forward(Q, K, V, O, G, a, b, causal, workspace, saved, stream, trace, True)


def _saved_args(saved, ref):
    if saved is None:
        return None, 0
    _check_tensors(ref, saved)
    return _ptr(saved), saved.numel() * saved.element_size()


_KIND = {False: 0, True: 1, "qknorm": 2, "qknorm_save": 3}


def _forward(Q, K, V, O, G, a, b, causal, workspace, saved, stream, trace, save):
    if _native is not None and trace is None:
        rc = _native.forward(_KIND[save], Q, K, V, O, G, a, b, causal, workspace, saved, stream)
        if rc == 0:
            return
        if rc is not None:
            raise LaError(rc, "la_forward_save" if save else "la_forward")
    if Q.dim() != 4:
        raise ValueError("Q must be [B, H, N, D]")
    shape = Q.shape
    B, H, N, D = shape
    _check_tensors(Q, K, V, O, G, workspace)
    if K.shape != shape or V.shape != shape or O.shape != shape:
        raise ValueError("shape mismatch")
    if not (K.dtype == V.dtype == O.dtype == Q.dtype):
        raise TypeError("dtype mismatch")
    if G is not None and (G.shape != Q.shape[:3] or G.dtype != torch.float32):
        raise ValueError("G must be [B, H, N] float32 (or None)")
    lib = load_library()
    head = (_ptr(Q), _ptr(K), _ptr(V), _ptr(O), _ptr(G), B, H, N, D, float(a), float(b),
            int(bool(causal)), _dtype_code(Q), _ptr(workspace),
            workspace.numel() * workspace.element_size())
    tr = ctypes.byref(trace) if trace is not None else None
    if save == "qknorm":
        rc = lib.la_forward_qknorm(*head, _stream_ptr(stream, Q), tr)
    elif save == "qknorm_save":
        sp, sb = _saved_args(saved, Q)
        rc = lib.la_forward_qknorm_save(*head, sp, sb, _stream_ptr(stream, Q), tr)
    elif save:
        sp, sb = _saved_args(saved, Q)
        rc = lib.la_forward_save(*head, sp, sb, _stream_ptr(stream, Q), tr)
    else:
        rc = lib.la_forward_traced(*head, _stream_ptr(stream, Q), tr)
    if rc != 0:
        raise LaError(rc, "la_forward_save" if save else "la_forward")


def la_backward(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, stream=None):
    """la_backward of include/la.h on torch device tensors (see la_forward)."""
    la_backward_traced(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, stream, None)


def la_backward_traced(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, stream=None,
                       trace=None):
    """la_backward_traced of include/la.h; ``trace`` is a la_trace structure or None."""
    _backward(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, None, stream, trace, False)


def la_backward_saved(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, saved, stream=None,
                      trace=None):
    """la_backward_saved of include/la.h; ``saved`` as filled by la_forward_save."""
    _backward(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, saved, stream, trace, True)


def _backward(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, saved, stream, trace,
              use_saved):
    if _native is not None and trace is None:
        rc = _native.backward(_KIND[use_saved], Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace,
                              saved, stream)
        if rc == 0:
            return
        if rc is not None:
            raise LaError(rc, "la_backward_saved" if use_saved else "la_backward")
    if Q.dim() != 4:
        raise ValueError("Q must be [B, H, N, D]")
    B, H, N, D = Q.shape
    _check_tensors(Q, K, V, O, G, dO, dQ, dK, dV, workspace)
    for name, t in (("K", K), ("V", V), ("O", O), ("dO", dO), ("dQ", dQ), ("dK", dK), ("dV", dV)):
        if t is None:
            if name == "O":
                continue  # recomputed inside the call
            raise ValueError("%s is required" % name)
        if t.shape != Q.shape:
            raise ValueError("shape mismatch")
        if t.dtype != Q.dtype:
            raise TypeError("dtype mismatch")
    if G is not None and (G.shape != Q.shape[:3] or G.dtype != torch.float32):
        raise ValueError("G must be [B, H, N] float32 (or None)")
    lib = load_library()
    head = (_ptr(Q), _ptr(K), _ptr(V), _ptr(O), _ptr(G), _ptr(dO), _ptr(dQ), _ptr(dK), _ptr(dV),
            B, H, N, D, float(a), float(b), int(bool(causal)), _dtype_code(Q), _ptr(workspace),
            workspace.numel() * workspace.element_size())
    tr = ctypes.byref(trace) if trace is not None else None
    if use_saved == "qknorm":
        rc = lib.la_backward_qknorm(*head, _stream_ptr(stream, Q), tr)
    elif use_saved == "qknorm_save":
        sp, sb = _saved_args(saved, Q)
        rc = lib.la_backward_qknorm_saved(*head, sp, sb, _stream_ptr(stream, Q), tr)
    elif use_saved:
        sp, sb = _saved_args(saved, Q)
        rc = lib.la_backward_saved(*head, sp, sb, _stream_ptr(stream, Q), tr)
    else:
        rc = lib.la_backward_traced(*head, _stream_ptr(stream, Q), tr)
    if rc != 0:
        raise LaError(rc, "la_backward_saved" if use_saved else "la_backward")


def attention(Q, K, V, a, b, causal, normalize):
    """O of linear_attention (autograd.py) through the autograd node in native code; None where that is left to
    the Python one."""
    if _native is None:
        load_library()
        if _native is None:
            return None
    O = _native.attention(Q, K, V, a, b, causal, normalize)
    if type(O) is int:
        raise LaError(O, "la_forward_save")
    return O


def la_decode_state_bytes(B, H, D):
    return int(load_library().la_decode_state_bytes(B, H, D))


def la_decode_step(q, k, v, o, g, state, a, b, stream=None):
    """la_decode_step of include/la.h: q, k, v, o [B, H, T, D]; g [B, H, T] float32 or None;
    state: float32 device tensor of la_decode_state_bytes(B, H, D) bytes, updated in place."""
    if _native is not None:
        rc = _native.decode_step(q, k, v, o, g, state, a, b, stream)
        if rc == 0:
            return
        if rc is not None:
            raise LaError(rc, "la_decode_step")
    if q.dim() != 4:
        raise ValueError("q must be [B, H, T, D]")
    shape = q.shape
    B, H, T, D = shape
    _check_tensors(q, k, v, o, g, state)
    if k.shape != shape or v.shape != shape or o.shape != shape:
        raise ValueError("shape mismatch")
    if not (k.dtype == v.dtype == o.dtype == q.dtype) or state.dtype != torch.float32:
        raise TypeError("dtype mismatch")
    if g is not None and (g.shape != q.shape[:3] or g.dtype != torch.float32):
        raise ValueError("g must be [B, H, T] float32 (or None)")
    rc = load_library().la_decode_step(_ptr(q), _ptr(k), _ptr(v), _ptr(o), _ptr(g), _ptr(state),
                                       state.numel() * 4, B, H, T, D, float(a), float(b),
                                       _dtype_code(q), _stream_ptr(stream, q))
    if rc != 0:
        raise LaError(rc, "la_decode_step")


def la_decode_prefill(K, V, state, accumulate, workspace, stream=None):
    """la_decode_prefill of include/la.h: K, V [B, H, N, D]."""
    if _native is not None:
        rc = _native.decode_prefill(K, V, state, accumulate, workspace, stream)
        if rc == 0:
            return
        if rc is not None:
            raise LaError(rc, "la_decode_prefill")
    if K.dim() != 4:
        raise ValueError("K must be [B, H, N, D]")
    B, H, N, D = K.shape
    _check_tensors(K, V, state, workspace)
    if V.shape != K.shape or V.dtype != K.dtype or state.dtype != torch.float32:
        raise ValueError("shape or dtype mismatch")
    rc = load_library().la_decode_prefill(_ptr(K), _ptr(V), _ptr(state), state.numel() * 4, B, H,
                                          N, D, _dtype_code(K), int(bool(accumulate)),
                                          _ptr(workspace),
                                          workspace.numel() * workspace.element_size(),
                                          _stream_ptr(stream, K))
    if rc != 0:
        raise LaError(rc, "la_decode_prefill")


def la_backward_ab(Q, K, V, O, G, dO, dab, a, b, causal, workspace, stream=None):
    """la_backward_ab of include/la.h; ``dab``: float32 device tensor of two elements."""
    if Q.dim() != 4:
        raise ValueError("Q must be [B, H, N, D]")
    B, H, N, D = Q.shape
    _check_tensors(Q, K, V, O, G, dO, dab, workspace)
    for t in (K, V, O, dO):
        if t.shape != Q.shape or t.dtype != Q.dtype:
            raise ValueError("shape or dtype mismatch")
    if G.shape != Q.shape[:3] or G.dtype != torch.float32:
        raise ValueError("G must be [B, H, N] float32")
    if dab.dtype != torch.float32 or dab.numel() < 2:
        raise ValueError("dab must hold two float32")
    rc = load_library().la_backward_ab(_ptr(Q), _ptr(K), _ptr(V), _ptr(O), _ptr(G), _ptr(dO),
                                       _ptr(dab), B, H, N, D, float(a), float(b),
                                       int(bool(causal)), _dtype_code(Q), _ptr(workspace),
                                       workspace.numel() * workspace.element_size(),
                                       _stream_ptr(stream, Q))
    if rc != 0:
        raise LaError(rc, "la_backward_ab")


def la_forward_qknorm(Q, K, V, O, G, a, b, causal, workspace, stream=None, trace=None):
    """la_forward_qknorm of include/la.h: la_forward on raw Q, K, normalised row by row inside."""
    _forward(Q, K, V, O, G, a, b, causal, workspace, None, stream, trace, "qknorm")


def la_backward_qknorm(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, stream=None,
                       trace=None):
    """la_backward_qknorm of include/la.h: gradients for the raw Q, K."""
    _backward(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, None, stream, trace,
              "qknorm")


def la_forward_qknorm_save(Q, K, V, O, G, a, b, causal, workspace, saved, stream=None, trace=None):
    """la_forward_qknorm_save of include/la.h (``saved`` as for la_forward_save)."""
    _forward(Q, K, V, O, G, a, b, causal, workspace, saved, stream, trace, "qknorm_save")


def la_backward_qknorm_saved(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, saved,
                             stream=None, trace=None):
    """la_backward_qknorm_saved of include/la.h; ``saved`` as filled by la_forward_qknorm_save."""
    _backward(Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, saved, stream, trace,
              "qknorm_save")
