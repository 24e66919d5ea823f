"""MI355X (gfx950) quadratic-neuron layers -- Python binding of ``libqlayer.so``.

The layer is the quadratic neuron of QuadraLib (arXiv 2204.01701, section 3.1,
eq:2ndneuron3): Y = (W_a*X + b_a) o (W_b*X + b_b) + (W_c*X + b_c), applied as a
2-D convolution and as a fully-connected layer, with the backward pass of
section 4.3 (eq:SD).  All arithmetic runs in the HIP kernels of the C
library; this module only marshals arguments through ctypes: torch tensors
become device pointers, the current HIP stream becomes the stream argument,
and workspaces are allocated with torch when the caller passes none.

Function names, argument order and layouts match ``include/qlayer.h``:
activations NHWC, conv weights OHWI, dense X B x I and W O x I, biases and
weight/bias gradients float32.  Every function raises ``QLError`` on a
non-zero status.  There is no fallback: if the library is not built, the
import of the first function call fails loudly.
"""
from __future__ import annotations

import ctypes
import os
import struct

__all__ = [
    "QL_F32", "QL_BF16", "QL_NEURON_QUADRA", "QL_NEURON_T4", "QL_NEURON_T4_IDENTITY", "QL_NEURON_T3",
    "QL_NEURON_T2", "QL_NEURON_T24", "NEURON_TERMS", "QLError", "ConvDesc", "LinearDesc", "conv_desc", "linear_desc", "lib",
    "qlayer_version", "qlayer_status_string",
    "qlayer_conv2d_fwd_workspace_size", "qlayer_conv2d_fwd",
    "qlayer_conv2d_bwd_data_workspace_size", "qlayer_conv2d_bwd_data", "qlayer_conv2d_bwd_data_ex",
    "qlayer_conv2d_bwd_weight_workspace_size", "qlayer_conv2d_bwd_weight", "qlayer_conv2d_bwd_weight_noalloc",
    "NOALLOC_SCRATCH_BYTES",
    "qlayer_linear_fwd_workspace_size", "qlayer_linear_fwd",
    "qlayer_linear_bwd_workspace_size", "qlayer_linear_bwd",
    "qlayer_conv2d_bwd_relu_workspace_size", "qlayer_conv2d_bwd_relu",
    "qlayer_linear_bwd_relu_workspace_size", "qlayer_linear_bwd_relu",
]

QL_F32 = 0
QL_BF16 = 1
# neuron types (qlayer.h ql_neuron): the proposed one and the earlier designs of Table 1
QL_NEURON_QUADRA, QL_NEURON_T4, QL_NEURON_T4_IDENTITY, QL_NEURON_T3, QL_NEURON_T2 = 0, 1, 2, 3, 4
QL_NEURON_T24 = 5  # T2&4: T_a o T_b + W_c (X o X) + b_c
NEURON_TERMS = {0: 3, 1: 2, 2: 2, 3: 1, 4: 1, 5: 3}  # first-order terms (weights) per type

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libqlayer.so")


class QLError(RuntimeError):
    def __init__(self, func, status):
        self.status = status
        super().__init__(f"{func} failed: status {status} ({qlayer_status_string(status)})")


class ConvDesc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in
                ("n", "c", "h", "w", "o", "kh", "kw", "stride_h", "stride_w", "pad_h", "pad_w", "dtype", "neuron",
                 "groups")]

    @property
    def ho(self):
        return (self.h + 2 * self.pad_h - self.kh) // self.stride_h + 1

    @property
    def wo(self):
        return (self.w + 2 * self.pad_w - self.kw) // self.stride_w + 1


class LinearDesc(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int), ("in_", ctypes.c_int), ("out", ctypes.c_int), ("dtype", ctypes.c_int),
                ("neuron", ctypes.c_int)]


class NetShape(ctypes.Structure):
    """qnet_shape: an NHWC tensor shape."""
    _fields_ = [(n, ctypes.c_int) for n in ("n", "h", "w", "c")]


def net_shape(t_or_dims) -> NetShape:
    """NetShape of an (N, H, W, C) tensor or tuple."""
    n, h, w, c = tuple(t_or_dims.shape) if hasattr(t_or_dims, "shape") else tuple(t_or_dims)
    return NetShape(n, h, w, c)


class Epilogue(ctypes.Structure):
    """ql_epilogue: y' = relu(scale * Y + shift) per output channel, and the
    per-channel sum / sum of squares of the stored y' (every member optional)."""
    _fields_ = [("scale", ctypes.c_void_p), ("shift", ctypes.c_void_p), ("relu", ctypes.c_int),
                ("sum", ctypes.c_void_p), ("sumsq", ctypes.c_void_p)]


def epilogue(scale=None, shift=None, relu=False, stat_sum=None, stat_sumsq=None) -> Epilogue:
    """An Epilogue over float32 device tensors of O values (or None); the tensors must outlive the call."""
    e = Epilogue(_ptr(scale), _ptr(shift), int(bool(relu)), _ptr(stat_sum), _ptr(stat_sumsq))
    e.tensors = (scale, shift, stat_sum, stat_sumsq)  # (_EPILOGUE: checked with the operands of a call)
    return e


def conv_desc(n, c, h, w, o, kh, kw, stride=1, pad=0, dtype=QL_BF16, neuron=QL_NEURON_QUADRA,
              groups=1) -> ConvDesc:
    """groups = c (with o == c) makes the layer depthwise: weights (c, kh, kw, 1)."""
    sh, sw = (stride, stride) if isinstance(stride, int) else stride
    ph, pw = (pad, pad) if isinstance(pad, int) else pad
    return ConvDesc(n, c, h, w, o, kh, kw, sh, sw, ph, pw, dtype, neuron, groups)


def linear_desc(batch, inp, out, dtype=QL_BF16, neuron=QL_NEURON_QUADRA) -> LinearDesc:
    return LinearDesc(batch, inp, out, dtype, neuron)


_lib = None
_vp = ctypes.c_void_p
_sz = ctypes.c_size_t


def lib():
    """The loaded C library (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise ImportError(f"{LIB_PATH} is missing: build it with `python -m paper_2204_01701_amd.build`")
    L = ctypes.CDLL(LIB_PATH)
    cd, ld = ctypes.POINTER(ConvDesc), ctypes.POINTER(LinearDesc)
    L.qlayer_status_string.argtypes = [ctypes.c_int]
    L.qlayer_status_string.restype = ctypes.c_char_p
    L.qlayer_version.restype = ctypes.c_int
    for name, d in (("conv2d_fwd", cd), ("conv2d_bwd_data", cd), ("conv2d_bwd_weight", cd),
                    ("linear_fwd", ld), ("linear_bwd", ld)):
        f = getattr(L, f"qlayer_{name}_workspace_size")
        f.argtypes = [d]
        f.restype = _sz
    L.qlayer_conv2d_fwd.argtypes = [cd] + [_vp] * 10 + [_vp, _sz, _vp]
    L.qlayer_conv2d_bwd_data.argtypes = [cd] + [_vp] * 7 + [_vp, _sz, _vp]
    L.qlayer_conv2d_bwd_data_ex.argtypes = [cd] + [_vp] * 8 + [_vp, _sz, _vp]
    L.qlayer_conv2d_bwd_data_ex.restype = ctypes.c_int
    L.qlayer_conv2d_bwd_weight.argtypes = [cd] + [_vp] * 10 + [_vp, _sz, _vp]
    L.qlayer_conv2d_bwd_weight_noalloc.argtypes = [cd] + [_vp] * 10 + [_vp]
    L.qlayer_conv2d_bwd_weight_noalloc.restype = ctypes.c_int
    L.qlayer_linear_fwd.argtypes = [ld] + [_vp] * 10 + [_vp, _sz, _vp]
    L.qlayer_linear_bwd.argtypes = [ld] + [_vp] * 14 + [_vp, _sz, _vp]
    for name, d in (("conv2d_bwd_relu", cd), ("linear_bwd_relu", ld)):
        f = getattr(L, f"qlayer_{name}_workspace_size")
        f.argtypes = [d]
        f.restype = _sz
        getattr(L, f"qlayer_{name}").argtypes = [d] + [_vp] * 15 + [_vp, _sz, _vp]
        getattr(L, f"qlayer_{name}").restype = ctypes.c_int
    ep = ctypes.POINTER(Epilogue)
    for name, d in (("conv2d_fwd_ex", cd), ("linear_fwd_ex", ld)):
        f = getattr(L, f"qlayer_{name}_workspace_size")
        f.argtypes = [d, ep]
        f.restype = _sz
        getattr(L, f"qlayer_{name}").argtypes = [d] + [_vp] * 10 + [ep, _vp, _sz, _vp]
        getattr(L, f"qlayer_{name}").restype = ctypes.c_int
    for name in ("conv2d_fwd", "conv2d_bwd_data", "conv2d_bwd_weight", "linear_fwd", "linear_bwd"):
        getattr(L, f"qlayer_{name}").restype = ctypes.c_int
    # the network glue (include/qnet.h)
    sp = ctypes.POINTER(NetShape)
    L.qnet_bn_act_fwd.argtypes = [sp, ctypes.c_int, _vp, _vp, _vp, ctypes.c_float, _vp, sp, ctypes.c_int, _vp, _vp,
                                  _vp, _vp]
    L.qnet_bn_act_bwd_workspace_size.argtypes = [sp]
    L.qnet_bn_act_bwd_workspace_size.restype = _sz
    L.qnet_bn_act_bwd.argtypes = [sp, ctypes.c_int, _vp, _vp, ctypes.c_int, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
    L.qnet_residual_bwd.argtypes = [sp, ctypes.c_int, _vp, _vp, sp, _vp, _vp]
    L.qnet_gap_fwd.argtypes = [sp, ctypes.c_int, _vp, _vp, _vp]
    L.qnet_gap_bwd.argtypes = [sp, ctypes.c_int, _vp, _vp, _vp]
    for name in ("bn_act_fwd", "bn_act_bwd", "residual_bwd", "gap_fwd", "gap_bwd"):
        getattr(L, f"qnet_{name}").restype = ctypes.c_int
    _lib = L
    return L


def qlayer_version() -> int:
    return lib().qlayer_version()


def qlayer_status_string(status: int) -> str:
    try:
        return lib().qlayer_status_string(int(status)).decode()
    except ImportError:
        return "unknown"


# --- marshalling -------------------------------------------------------------

def _ptr(t):
    """Device pointer of a tensor (None -> NULL).  Plain ints pass through (tests)."""
    if t is None:
        return None
    if isinstance(t, int):
        return t
    if not t.is_contiguous():
        raise ValueError("tensors passed to qlayer must be contiguous")
    return t.data_ptr()


def _device(*tensors):
    for t in tensors:
        if t is not None and not isinstance(t, int):
            return t.device
    return None


def _stream(stream, device):
    if stream is not None:
        return stream if isinstance(stream, int) else stream.cuda_stream
    if device is None or device.type != "cuda":
        return None
    import torch
    return torch.cuda.current_stream(device).cuda_stream


def _workspace(workspace, need, device, stream=None):
    """(pointer, bytes) of the workspace; allocates one with torch when none is given.

    The allocation is made on the current stream.  When the call runs on
    another stream, the block is recorded on that stream, so that the caching
    allocator does not hand it out again while the kernels there still use it;
    a raw stream handle (an int) cannot be recorded and needs an explicit
    workspace."""
    if workspace is not None:
        if isinstance(workspace, tuple):
            return workspace
        return workspace.data_ptr(), workspace.numel() * workspace.element_size()
    if need == 0:
        return None, 0
    import torch
    if isinstance(stream, int):
        raise ValueError("a raw stream handle needs an explicit workspace (the allocator cannot track its use)")
    ws = torch.empty(need, dtype=torch.uint8, device=device)
    if stream is not None and stream != torch.cuda.current_stream(device):
        ws.record_stream(stream)
    _workspace.keep = ws  # keep alive until the next allocation; the stream orders reuse
    return ws.data_ptr(), need


# --- tensor operands: checks and pointers --------------------------------------
# The C ABI sees bare pointers, so a tensor of the wrong size, dtype or device
# would make the kernels read or write out of bounds.  Every tensor argument is
# checked against the descriptor before the call: a contiguous CUDA tensor on
# the device of the others, with the element count and dtype that its role in
# _OPERANDS requires.
#
# A small layer's pass is a few microseconds of GPU work, so the host's share
# of a call counts: _pointers checks in one loop with a few attribute reads
# per tensor.  On anything it does not accept (a wrong tensor, raw pointers, an
# unknown dtype) the call goes on in _checked_pointers, which holds the same
# operands against the same requirements and raises what is to be raised.

# The tensor operands of an entry point in the order of its arguments, as
# name:role, kept as a tuple of names and one of roles; the roles are those of _needs.
_OPERANDS = {name: tuple(zip(*(o.split(":") for o in ops.split()))) for name, ops in {
    "qlayer_conv2d_fwd": "x:x wa:w wb:w wc:w ba:b bb:b bc:b y:y ta:y tb:y",
    "qlayer_conv2d_fwd_ex": "x:x wa:w wb:w wc:w ba:b bb:b bc:b y:y ta:y tb:y",
    "qlayer_conv2d_bwd_data": "gy:y ta:t tb:y wa:w wb:w wc:w dx:x",
    "qlayer_conv2d_bwd_data_ex": "gy:y ta:t tb:y x:x wa:w wb:w wc:w dx:x",
    "qlayer_conv2d_bwd_weight": "x:x gy:y ta:y tb:y dwa:g dwb:g dwc:g dba:b dbb:b dbc:b",
    "qlayer_conv2d_bwd_weight_noalloc": "x:x gy:y ta:y tb:y dwa:g dwb:g dwc:g dba:b dbb:b dbc:b",
    "qlayer_conv2d_bwd_relu": "x:x gy:y y_out:y ta:y tb:y wa:w wb:w wc:w dx:x dwa:g dwb:g dwc:g dba:b dbb:b dbc:b",
    "qlayer_linear_fwd": "x:x wa:w wb:w wc:w ba:b bb:b bc:b y:y ta:y tb:y",
    "qlayer_linear_fwd_ex": "x:x wa:w wb:w wc:w ba:b bb:b bc:b y:y ta:y tb:y",
    "qlayer_linear_bwd": "x:x gy:y ta:y tb:y wa:w wb:w wc:w dx:x dwa:g dwb:g dwc:g dba:b dbb:b dbc:b",
    "qlayer_linear_bwd_relu": "x:x gy:y y_out:y ta:y tb:y wa:w wb:w wc:w dx:x dwa:g dwb:g dwc:g dba:b dbb:b dbc:b",
}.items()}

_EPILOGUE = ("epi.scale", "epi.shift", "epi.sum", "epi.sumsq"), ("b", "b", "b", "b")

_CONV_FIELDS = struct.Struct("14i")  # ConvDesc
_LINEAR_FIELDS = struct.Struct("5i")  # LinearDesc
_dtypes = {}  # (filled on the first call: importing this module does not import torch)


def _needs(nx, nw, ny, no, code, t2=False):
    """Element count and dtype per role: "x" shaped like X, "w" a weight, "y" an
    output-side map, "t" the map T_a (X for the T2 neuron), "b" float32 of O, "g" a
    float32 weight gradient.  dtype None: a code the library rejects itself."""
    if not _dtypes:
        import torch
        _dtypes.update({QL_F32: torch.float32, QL_BF16: torch.bfloat16})
    dt, f32 = _dtypes.get(code), _dtypes[QL_F32]
    x, y = (nx, dt), (ny, dt)
    return {"x": x, "w": (nw, dt), "y": y, "t": x if t2 else y, "b": (no, f32), "g": (nw, f32)}


def _conv_needs(d):
    n, c, h, w, o, kh, kw, sh, sw, ph, pw, code, neuron, groups = _CONV_FIELDS.unpack_from(d)
    ny = n * ((h + 2 * ph - kh) // sh + 1) * ((w + 2 * pw - kw) // sw + 1) * o
    nw = o * kh * kw * (1 if groups == c and c > 1 else c)
    return _needs(n * h * w * c, nw, ny, o, code, neuron == QL_NEURON_T2)


def _linear_needs(d):
    b, i, o, code, _ = _LINEAR_FIELDS.unpack_from(d)
    return _needs(b * i, o * i, b * o, o, code)


def _expect(name, t, numel, dtype, device):
    if t is None or isinstance(t, int):
        return
    if t.device.type != "cuda":
        raise ValueError(f"{name}: a CUDA device tensor is required, got one on {t.device}")
    if device is not None and t.device != device:
        raise ValueError(f"{name}: on {t.device}, the other tensors on {device}")
    if t.numel() != numel:
        raise ValueError(f"{name}: {t.numel()} elements, the descriptor needs {numel}")
    if dtype is not None and t.dtype != dtype:
        raise ValueError(f"{name}: dtype {t.dtype}, expected {dtype}")


def _checked_pointers(needs, names, roles, tensors):
    """The pointers of `tensors` (raw pointers pass through) and their torch device."""
    dev = _device(*tensors)
    for name, role, t in zip(names, roles, tensors):
        _expect(name, t, *needs[role], dev)
    return [_ptr(t) for t in tensors], dev


def _pointers(needs, roles, tensors):
    """The data pointers of `tensors` (None: NULL) and their device index, or None."""
    out, dev = [], -1
    try:
        for role, t in zip(roles, tensors):
            if t is None:
                out.append(None)
                continue
            n, d = needs[role]
            if t.numel() != n or t.dtype is not d or not t.is_cuda or not t.is_contiguous():
                return None
            i = t.get_device()
            if i != dev:
                if dev >= 0:
                    return None
                dev = i
            out.append(t.data_ptr())
    except AttributeError:  # a raw pointer (asking each operand for its type costs as much as a check)
        return None
    return (out, dev) if dev >= 0 else None


def _check(func, status):
    if status != 0:
        raise QLError(func, status)


def _current_stream(dev):
    """Handle of the current stream of device `dev`."""
    import torch
    # the handle itself, without building a torch.cuda.Stream, where torch has it
    raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
    return raw(dev) if raw is not None else torch.cuda.current_stream(dev).cuda_stream


def _run(name, desc, needs, tensors, workspace, stream, epi=None):
    """The entry point `name` on its operands: checks, workspace, stream, call.

    epi: the epilogue of an _ex forward (a one-element tuple, its value None or an
    Epilogue, whose tensors are checked with the others)."""
    names, roles = _OPERANDS[name]
    n = len(tensors)
    if epi is not None and epi[0] is not None:
        extra = getattr(epi[0], "tensors", None)
        if extra is not None:
            names, roles = names + _EPILOGUE[0], roles + _EPILOGUE[1]
            tensors += extra
    got = _pointers(needs, roles, tensors)
    L = lib()
    ref = ctypes.byref(desc)
    args = () if epi is None else (_epi_ref(epi[0]),)
    if got is not None:
        ptrs, dev = got
        if stream is None:
            st = _current_stream(dev)
        else:
            st = stream if isinstance(stream, int) else stream.cuda_stream
    else:
        ptrs, dev = _checked_pointers(needs, names, roles, tensors)
        st = _stream(stream, dev)
    del ptrs[n:]
    if workspace is _NO_WORKSPACE:
        _check(name, getattr(L, name)(ref, *ptrs, st))
        return
    if workspace is None:
        # (both input gradients share one query; the epilogue's sums need room too)
        query = _QUERIES.get(name, name + "_workspace_size")
        need = getattr(L, query)(ref, *args)
        if got is not None and need:
            import torch
            dev = torch.device("cuda", dev)
        wp, wn = _workspace(None, need, dev, stream)
    else:
        wp, wn = _workspace(workspace, 0, dev)
    _check(name, getattr(L, name)(ref, *ptrs, *args, wp, wn, st))


_NO_WORKSPACE = object()
_QUERIES = {"qlayer_conv2d_bwd_data_ex": "qlayer_conv2d_bwd_data_workspace_size"}


# --- the C ABI, one Python function per entry point -------------------------

def qlayer_conv2d_fwd_workspace_size(desc: ConvDesc) -> int:
    return lib().qlayer_conv2d_fwd_workspace_size(ctypes.byref(desc))


def qlayer_conv2d_fwd(desc, x, wa, wb, wc, ba=None, bb=None, bc=None, y=None, ta=None, tb=None,
                      workspace=None, stream=None):
    _run("qlayer_conv2d_fwd", desc, _conv_needs(desc),
         (x, wa, wb, wc, ba, bb, bc, y, ta, tb), workspace, stream)


def qlayer_conv2d_bwd_data_workspace_size(desc: ConvDesc) -> int:
    return lib().qlayer_conv2d_bwd_data_workspace_size(ctypes.byref(desc))


def qlayer_conv2d_bwd_data(desc, gy, ta, tb, wa, wb, wc, dx, workspace=None, stream=None):
    _run("qlayer_conv2d_bwd_data", desc, _conv_needs(desc),
         (gy, ta, tb, wa, wb, wc, dx), workspace, stream)


def qlayer_conv2d_bwd_data_ex(desc, gy, ta, tb, x, wa, wb, wc, dx, workspace=None, stream=None):
    """qlayer_conv2d_bwd_data with the layer input X (T2&4 needs it; T2 may take it in place of `ta`)."""
    _run("qlayer_conv2d_bwd_data_ex", desc, _conv_needs(desc),
         (gy, ta, tb, x, wa, wb, wc, dx), workspace, stream)


def qlayer_conv2d_bwd_weight_workspace_size(desc: ConvDesc) -> int:
    return lib().qlayer_conv2d_bwd_weight_workspace_size(ctypes.byref(desc))


def qlayer_conv2d_bwd_weight(desc, x, gy, ta, tb, dwa, dwb, dwc, dba=None, dbb=None, dbc=None,
                             workspace=None, stream=None):
    _run("qlayer_conv2d_bwd_weight", desc, _conv_needs(desc),
         (x, gy, ta, tb, dwa, dwb, dwc, dba, dbb, dbc), workspace, stream)


NOALLOC_SCRATCH_BYTES = 32 << 20  # QLAYER_NOALLOC_SCRATCH_BYTES of qlayer.h


def qlayer_conv2d_bwd_weight_noalloc(desc, x, gy, ta, tb, dwa, dwb, dwc, dba=None, dbb=None, dbc=None,
                                     stream=None):
    """qlayer_conv2d_bwd_weight with the library's own scratch array in place of a
    workspace: allocates nothing (for graph capture and other callers that cannot)."""
    _run("qlayer_conv2d_bwd_weight_noalloc", desc, _conv_needs(desc),
         (x, gy, ta, tb, dwa, dwb, dwc, dba, dbb, dbc), _NO_WORKSPACE, stream)


def qlayer_linear_fwd_workspace_size(desc: LinearDesc) -> int:
    return lib().qlayer_linear_fwd_workspace_size(ctypes.byref(desc))


def qlayer_linear_fwd(desc, x, wa, wb, wc, ba=None, bb=None, bc=None, y=None, ta=None, tb=None,
                      workspace=None, stream=None):
    _run("qlayer_linear_fwd", desc, _linear_needs(desc),
         (x, wa, wb, wc, ba, bb, bc, y, ta, tb), workspace, stream)


def _epi_ref(epi):
    return ctypes.byref(epi) if epi is not None else None


def qlayer_conv2d_fwd_ex_workspace_size(desc: ConvDesc, epi=None) -> int:
    return lib().qlayer_conv2d_fwd_ex_workspace_size(ctypes.byref(desc), _epi_ref(epi))


def qlayer_conv2d_fwd_ex(desc, x, wa, wb, wc, ba=None, bb=None, bc=None, y=None, ta=None, tb=None, epi=None,
                         workspace=None, stream=None):
    """qlayer_conv2d_fwd with a fused epilogue (an Epilogue, see epilogue())."""
    _run("qlayer_conv2d_fwd_ex", desc, _conv_needs(desc),
         (x, wa, wb, wc, ba, bb, bc, y, ta, tb), workspace, stream, (epi,))


def qlayer_linear_fwd_ex_workspace_size(desc: LinearDesc, epi=None) -> int:
    return lib().qlayer_linear_fwd_ex_workspace_size(ctypes.byref(desc), _epi_ref(epi))


def qlayer_linear_fwd_ex(desc, x, wa, wb, wc, ba=None, bb=None, bc=None, y=None, ta=None, tb=None, epi=None,
                         workspace=None, stream=None):
    """qlayer_linear_fwd with a fused epilogue (an Epilogue, see epilogue())."""
    _run("qlayer_linear_fwd_ex", desc, _linear_needs(desc),
         (x, wa, wb, wc, ba, bb, bc, y, ta, tb), workspace, stream, (epi,))


def qlayer_linear_bwd_workspace_size(desc: LinearDesc) -> int:
    return lib().qlayer_linear_bwd_workspace_size(ctypes.byref(desc))


def qlayer_linear_bwd(desc, x, gy, ta, tb, wa, wb, wc, dx=None, dwa=None, dwb=None, dwc=None,
                      dba=None, dbb=None, dbc=None, workspace=None, stream=None):
    _run("qlayer_linear_bwd", desc, _linear_needs(desc),
         (x, gy, ta, tb, wa, wb, wc, dx, dwa, dwb, dwc, dba, dbb, dbc), workspace, stream)


def qlayer_conv2d_bwd_relu_workspace_size(desc: ConvDesc) -> int:
    return lib().qlayer_conv2d_bwd_relu_workspace_size(ctypes.byref(desc))


def qlayer_conv2d_bwd_relu(desc, x, gy, y_out, ta, tb, wa, wb, wc, dx=None, dwa=None, dwb=None, dwc=None,
                           dba=None, dbb=None, dbc=None, workspace=None, stream=None):
    """The layer's backward behind the fused ReLU: G = gy o [y_out > 0], then dX and/or dW_t, db_t from G."""
    _run("qlayer_conv2d_bwd_relu", desc, _conv_needs(desc),
         (x, gy, y_out, ta, tb, wa, wb, wc, dx, dwa, dwb, dwc, dba, dbb, dbc), workspace, stream)


def qlayer_linear_bwd_relu_workspace_size(desc: LinearDesc) -> int:
    return lib().qlayer_linear_bwd_relu_workspace_size(ctypes.byref(desc))


def qlayer_linear_bwd_relu(desc, x, gy, y_out, ta, tb, wa, wb, wc, dx=None, dwa=None, dwb=None, dwc=None,
                           dba=None, dbb=None, dbc=None, workspace=None, stream=None):
    """The dense layer's backward behind the fused ReLU (as qlayer_conv2d_bwd_relu)."""
    _run("qlayer_linear_bwd_relu", desc, _linear_needs(desc),
         (x, gy, y_out, ta, tb, wa, wb, wc, dx, dwa, dwb, dwc, dba, dbb, dbc), workspace, stream)


# --- the network glue (include/qnet.h) ----------------------------------------

def _net_dtype(t):
    import torch
    return QL_BF16 if t.dtype == torch.bfloat16 else QL_F32


def _net_expect(name, t, shape, dtype, device):
    _expect(name, t, int(shape[0]) * int(shape[1]) * int(shape[2]) * int(shape[3]) if len(shape) == 4
            else int(shape[0]) * int(shape[1]), dtype, device)


def qnet_bn_act_fwd(y, ssum, ssq, out, mean, rstd, eps=1e-5, res=None, relu=True, stream=None):
    """out = relu((y - mean) rstd + shortcut(res)); y, out, res NHWC device tensors."""
    import torch
    dev = y.device
    s = net_shape(y)
    dt = _net_dtype(y)
    _net_expect("out", out, y.shape, y.dtype, dev)
    for n, t in (("sum", ssum), ("sumsq", ssq), ("mean", mean), ("rstd", rstd)):
        _expect(n, t, s.c, torch.float32, dev)
    rs = net_shape(res) if res is not None else None
    if res is not None:
        _expect("res", res, rs.n * rs.h * rs.w * rs.c, y.dtype, dev)
    _check("qnet_bn_act_fwd", lib().qnet_bn_act_fwd(
        ctypes.byref(s), dt, _ptr(y), _ptr(ssum), _ptr(ssq), ctypes.c_float(eps), _ptr(res),
        ctypes.byref(rs) if rs is not None else None, int(bool(relu)), _ptr(out), _ptr(mean), _ptr(rstd),
        _stream(stream, dev)))


def qnet_bn_act_bwd_workspace_size(shape) -> int:
    return lib().qnet_bn_act_bwd_workspace_size(ctypes.byref(net_shape(shape)))


def qnet_bn_act_bwd(dout, out, y, mean, rstd, dy, relu=True, workspace=None, stream=None):
    """dy = the gradient at y of out = relu(bn(y) [+ r]) given dout."""
    import torch
    dev = y.device
    s = net_shape(y)
    for n, t in (("dout", dout), ("out", out), ("dy", dy)):
        _net_expect(n, t, y.shape, y.dtype, dev)
    for n, t in (("mean", mean), ("rstd", rstd)):
        _expect(n, t, s.c, torch.float32, dev)
    wp, wn = _workspace(workspace, qnet_bn_act_bwd_workspace_size(y.shape), dev, stream)
    _check("qnet_bn_act_bwd", lib().qnet_bn_act_bwd(
        ctypes.byref(s), _net_dtype(y), _ptr(dout), _ptr(out), int(bool(relu)), _ptr(y), _ptr(mean), _ptr(rstd),
        _ptr(dy), wp, wn, _stream(stream, dev)))


def qnet_residual_bwd(dout, out, dx, stream=None):
    """dx (the block input's gradient) += the shortcut's share of dout [out > 0]."""
    dev = dx.device
    _net_expect("out", out, dout.shape, dout.dtype, dev)
    _check("qnet_residual_bwd", lib().qnet_residual_bwd(
        ctypes.byref(net_shape(dout)), _net_dtype(dout), _ptr(dout), _ptr(out), ctypes.byref(net_shape(dx)),
        _ptr(dx), _stream(stream, dev)))


def qnet_gap_fwd(x, y, stream=None):
    dev = x.device
    _expect("y", y, x.shape[0] * x.shape[3], x.dtype, dev)
    _check("qnet_gap_fwd", lib().qnet_gap_fwd(ctypes.byref(net_shape(x)), _net_dtype(x), _ptr(x), _ptr(y),
                                              _stream(stream, dev)))


def qnet_gap_bwd(dy, dx, stream=None):
    dev = dx.device
    _expect("dy", dy, dx.shape[0] * dx.shape[3], dx.dtype, dev)
    _check("qnet_gap_bwd", lib().qnet_gap_bwd(ctypes.byref(net_shape(dx)), _net_dtype(dx), _ptr(dy), _ptr(dx),
                                              _stream(stream, dev)))
