"""ctypes binding of libhetumoe.so (argument marshalling only).

The functions named like the C ABI (moe_gate, moe_dispatch, ...) take torch
tensors that already live on the GPU, check dtype / device / contiguity and
that each holds the elements the call's sizes need, and forward raw device
pointers plus torch's current HIP stream.  The convenience
wrappers (gate, dispatch, ...) additionally allocate the outputs with
torch.empty; every value is computed by the library's HIP kernels.  There is no
fallback: if the library is missing or fails to load, every call raises.
"""

import ctypes
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
# HETUMOE_LIBRARY names another build of the library (for instance one made with
# `python -m paper_2203_14685_amd.build --out ... -D HETUMOE_ROUTE_VALU_ONLY` to
# time the vector-ALU projection); by default the in-tree build is loaded.
LIB_PATH = os.environ.get("HETUMOE_LIBRARY") or os.path.join(_PKG, "libhetumoe.so")

MOE_OK, MOE_ERR_INVALID_ARG, MOE_ERR_UNSUPPORTED, MOE_ERR_WORKSPACE, MOE_ERR_HIP, MOE_ERR_NOT_CONVERGED = range(6)
MOE_F32, MOE_BF16 = 0, 1
MOE_GATE_TOPK, MOE_GATE_KTOP1, MOE_GATE_HASH, MOE_GATE_HTOPK = 0, 1, 2, 3

EXPORTED = (
    "moe_gate_workspace_size", "moe_gate", "moe_gate_noalloc", "moe_dispatch", "moe_combine",
    "moe_dispatch_bwd", "moe_combine_bwd", "moe_gate_bwd_workspace_size", "moe_gate_bwd",
    "moe_hash_balanced_table", "moe_base_gate_workspace_size", "moe_base_gate",
    "moe_base_gate_async", "moe_status_string", "moe_last_error", "moe_abi_version",
)


class MoeError(RuntimeError):
    def __init__(self, status, message):
        super().__init__(f"{message} [status {status}]")
        self.status = status


class GateParams(ctypes.Structure):
    _fields_ = [
        ("S", ctypes.c_int32), ("d", ctypes.c_int32), ("E", ctypes.c_int32),
        ("k", ctypes.c_int32), ("capacity", ctypes.c_int32), ("kind", ctypes.c_int32),
        ("normalize", ctypes.c_int32), ("logits_in", ctypes.c_int32),
        ("dtype", ctypes.c_int32), ("groups", ctypes.c_int32),
        ("hash_seed", ctypes.c_uint64), ("temperature", ctypes.c_float), ("hash_vocab", ctypes.c_int32),
    ]


class Layout(ctypes.Structure):
    _fields_ = [
        ("S", ctypes.c_int32), ("d", ctypes.c_int32), ("E", ctypes.c_int32),
        ("k", ctypes.c_int32), ("capacity", ctypes.c_int32), ("dtype", ctypes.c_int32),
    ]


class GateBwdParams(ctypes.Structure):
    _fields_ = [
        ("S", ctypes.c_int32), ("d", ctypes.c_int32), ("E", ctypes.c_int32),
        ("k", ctypes.c_int32), ("kind", ctypes.c_int32), ("normalize", ctypes.c_int32),
        ("dtype", ctypes.c_int32), ("accumulate_dx", ctypes.c_int32),
        ("aux_coef", ctypes.c_float), ("temperature", ctypes.c_float),
    ]


class BaseParams(ctypes.Structure):
    _fields_ = [
        ("S", ctypes.c_int32), ("d", ctypes.c_int32), ("E", ctypes.c_int32), ("capacity", ctypes.c_int32),
        ("logits_in", ctypes.c_int32), ("dtype", ctypes.c_int32), ("max_rounds", ctypes.c_int32),
    ]


class BaseInfo(ctypes.Structure):
    _fields_ = [("phases", ctypes.c_int32), ("rounds", ctypes.c_int32), ("eps", ctypes.c_double)]


# moe_base_status, which moe_base_gate_async writes to device memory: 24 bytes,
# read back as int32 [6] (phases, rounds, eps as two words, status, pad)
BASE_STATUS_BYTES = 24
MOE_BASE_MAX_LAUNCH_ROUNDS = 16384


_lib = None


def load():
    """Load the in-tree libhetumoe.so (raises if it is missing)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2203_14685_amd.build`")
    lib = ctypes.CDLL(LIB_PATH)
    vp, i32p, f32p = ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p
    lib.moe_gate_workspace_size.argtypes = [ctypes.POINTER(GateParams), ctypes.POINTER(ctypes.c_size_t)]
    lib.moe_gate.argtypes = [ctypes.POINTER(GateParams), vp, vp, f32p, i32p, f32p, i32p, f32p, i32p, i32p,
                             f32p, i32p, i32p, i32p, vp, ctypes.c_size_t, vp]
    lib.moe_gate_noalloc.argtypes = [ctypes.POINTER(GateParams), vp, vp, f32p, i32p, f32p, i32p, f32p, i32p, i32p,
                                     f32p, i32p, i32p, i32p, vp]
    lib.moe_hash_balanced_table.argtypes = [vp, ctypes.c_int32, ctypes.c_int32, vp]
    lib.moe_dispatch.argtypes = [ctypes.POINTER(Layout), vp, i32p, i32p, i32p, vp, vp]
    lib.moe_combine.argtypes = [ctypes.POINTER(Layout), vp, i32p, i32p, f32p, vp, vp]
    lib.moe_dispatch_bwd.argtypes = [ctypes.POINTER(Layout), vp, i32p, i32p, vp, vp]
    lib.moe_combine_bwd.argtypes = [ctypes.POINTER(Layout), vp, vp, i32p, i32p, i32p, f32p, vp, f32p, vp]
    lib.moe_gate_bwd_workspace_size.argtypes = [ctypes.POINTER(GateBwdParams), ctypes.POINTER(ctypes.c_size_t)]
    lib.moe_gate_bwd.argtypes = [ctypes.POINTER(GateBwdParams), vp, vp, f32p, i32p, f32p, f32p, vp, f32p, f32p,
                                 f32p, vp, ctypes.c_size_t, vp]
    lib.moe_base_gate_workspace_size.argtypes = [ctypes.POINTER(BaseParams), ctypes.POINTER(ctypes.c_size_t)]
    lib.moe_base_gate.argtypes = [ctypes.POINTER(BaseParams), vp, vp, f32p, f32p, i32p, i32p, f32p, i32p, i32p,
                                  vp, vp, ctypes.c_size_t, ctypes.POINTER(BaseInfo), vp]
    lib.moe_base_gate_async.argtypes = [ctypes.POINTER(BaseParams), vp, vp, f32p, f32p, i32p, i32p, f32p, i32p,
                                        i32p, vp, vp, ctypes.c_size_t, ctypes.c_int32, vp, vp]
    for name in ("moe_gate_workspace_size", "moe_gate", "moe_dispatch", "moe_combine",
                 "moe_dispatch_bwd", "moe_combine_bwd", "moe_gate_bwd_workspace_size", "moe_gate_bwd",
                 "moe_hash_balanced_table", "moe_base_gate_workspace_size", "moe_base_gate",
                 "moe_base_gate_async"):
        getattr(lib, name).restype = ctypes.c_int
    lib.moe_status_string.argtypes = [ctypes.c_int]
    lib.moe_status_string.restype = ctypes.c_char_p
    lib.moe_last_error.argtypes = []
    lib.moe_last_error.restype = ctypes.c_char_p
    lib.moe_abi_version.argtypes = []
    lib.moe_abi_version.restype = ctypes.c_int32
    _lib = lib
    return lib


def _check(status):
    if status != MOE_OK:
        lib = load()
        raise MoeError(status, f"{lib.moe_status_string(status).decode()}: {lib.moe_last_error().decode()}")


def _dtype_code(t):
    if t.dtype == torch.float32:
        return MOE_F32
    if t.dtype == torch.bfloat16:
        return MOE_BF16
    raise TypeError(f"unsupported dtype {t.dtype}; float32 or bfloat16 expected")


_multi_gpu = None


def _ptr(t, dtype=None, name="tensor", n=0):
    """Device pointer of a contiguous GPU tensor (None -> NULL) holding at
    least n elements: a tensor smaller than the call's sizes would let a kernel
    run past its end, so it is refused here, before anything reaches the device."""
    global _multi_gpu
    if t is None:
        return None
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a torch.Tensor or None")
    numel = t.numel()
    if numel < n:
        raise ValueError(f"{name} holds {numel} elements; the call's sizes need {n}")
    if not t.is_cuda:
        raise ValueError(f"{name} must be on the GPU, found {t.device}")
    if _multi_gpu is None:
        _multi_gpu = torch.cuda.device_count() > 1
    if _multi_gpu and t.device.index is not None and t.device.index != torch.cuda.current_device():
        raise ValueError(f"{name} is on {t.device}, but the library launches on cuda:{torch.cuda.current_device()}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if dtype is not None and t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, found {t.dtype}")
    return t.data_ptr() if numel > 0 else None


# The current stream's handle without a torch.cuda.Stream object around it, which
# takes 3.0 us to make (0.2 us this way; a call of few tokens is bound by the
# host: gate, dispatch and combine of 32 tokens 49.1 -> 37.7 us).
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
_raw_device = getattr(torch._C, "_cuda_getDevice", None)


def _stream(stream):
    if stream is None:
        if _raw_stream is None or _raw_device is None or not torch.cuda.is_initialized():
            return torch.cuda.current_stream().cuda_stream
        return _raw_stream(_raw_device())
    return getattr(stream, "cuda_stream", stream)


def gate_params(S, d, E, k, capacity, kind, normalize=0, logits_in=0, dtype=MOE_F32, hash_seed=0, groups=0,
                temperature=0.0, hash_vocab=0):
    return GateParams(S, d, E, k, capacity, kind, normalize, logits_in, dtype, groups, hash_seed, temperature,
                      hash_vocab)


def moe_gate_workspace_size(params):
    n = ctypes.c_size_t(0)
    _check(load().moe_gate_workspace_size(ctypes.byref(params), ctypes.byref(n)))
    return n.value


def moe_gate(params, x, wg, bias, token_ids, noise, hash_table, logits, ids, slots, weights, counts, demand,
             slot_src, workspace, stream=None):
    lib = load()
    f32, i32 = torch.float32, torch.int32
    xdt = torch.bfloat16 if params.dtype == MOE_BF16 else torch.float32
    S, d, E, k, C = params.S, params.d, params.E, params.k, params.capacity
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(lib.moe_gate(
        ctypes.byref(params), _ptr(x, xdt, "x", S * d), _ptr(wg, xdt, "wg", d * E), _ptr(bias, f32, "bias", E),
        _ptr(token_ids, i32, "token_ids", S), _ptr(noise, f32, "noise", S * E),
        _ptr(hash_table, i32, "hash_table", params.hash_vocab), _ptr(logits, f32, "logits", S * E),
        _ptr(ids, i32, "ids", S * k), _ptr(slots, i32, "slots", S * k), _ptr(weights, f32, "weights", S * k),
        _ptr(counts, i32, "counts", E), _ptr(demand, i32, "demand", E), _ptr(slot_src, i32, "slot_src", E * C),
        _ptr(workspace, None, "workspace"), ws_bytes, _stream(stream)))


def moe_gate_noalloc(params, x, wg, bias, token_ids, noise, hash_table, logits, ids, slots, weights, counts, demand,
                     slot_src, stream=None):
    """moe_gate without a workspace: the library's fixed scratch serves it."""
    lib = load()
    f32, i32 = torch.float32, torch.int32
    xdt = torch.bfloat16 if params.dtype == MOE_BF16 else torch.float32
    S, d, E, k, C = params.S, params.d, params.E, params.k, params.capacity
    _check(lib.moe_gate_noalloc(
        ctypes.byref(params), _ptr(x, xdt, "x", S * d), _ptr(wg, xdt, "wg", d * E), _ptr(bias, f32, "bias", E),
        _ptr(token_ids, i32, "token_ids", S), _ptr(noise, f32, "noise", S * E),
        _ptr(hash_table, i32, "hash_table", params.hash_vocab), _ptr(logits, f32, "logits", S * E),
        _ptr(ids, i32, "ids", S * k), _ptr(slots, i32, "slots", S * k), _ptr(weights, f32, "weights", S * k),
        _ptr(counts, i32, "counts", E), _ptr(demand, i32, "demand", E), _ptr(slot_src, i32, "slot_src", E * C),
        _stream(stream)))


def _layout(S, d, E, k, capacity, dtype):
    return Layout(S, d, E, k, capacity, dtype)


def _rows(layout):
    """Elements of a token-row buffer [S, d], an expert buffer [E, C, d], a
    per-choice array [S, k] and slot_src [E, C] for this layout."""
    S, d, E, k, C = layout.S, layout.d, layout.E, layout.k, layout.capacity
    return S * d, E * C * d, S * k, E * C


def moe_dispatch(layout, x, ids, slots, slot_src, xe, stream=None):
    dt = torch.bfloat16 if layout.dtype == MOE_BF16 else torch.float32
    i32 = torch.int32
    tok, exp, ch, src = _rows(layout)
    _check(load().moe_dispatch(ctypes.byref(layout), _ptr(x, dt, "x", tok), _ptr(ids, i32, "ids", ch),
                               _ptr(slots, i32, "slots", ch), _ptr(slot_src, i32, "slot_src", src),
                               _ptr(xe, dt, "xe", exp), _stream(stream)))


def moe_combine(layout, ye, ids, slots, weights, y, stream=None):
    dt = torch.bfloat16 if layout.dtype == MOE_BF16 else torch.float32
    tok, exp, ch, _ = _rows(layout)
    _check(load().moe_combine(ctypes.byref(layout), _ptr(ye, dt, "ye", exp), _ptr(ids, torch.int32, "ids", ch),
                              _ptr(slots, torch.int32, "slots", ch), _ptr(weights, torch.float32, "weights", ch),
                              _ptr(y, dt, "y", tok), _stream(stream)))


def moe_dispatch_bwd(layout, dxe, ids, slots, dx, stream=None):
    dt = torch.bfloat16 if layout.dtype == MOE_BF16 else torch.float32
    tok, exp, ch, _ = _rows(layout)
    _check(load().moe_dispatch_bwd(ctypes.byref(layout), _ptr(dxe, dt, "dxe", exp),
                                   _ptr(ids, torch.int32, "ids", ch), _ptr(slots, torch.int32, "slots", ch),
                                   _ptr(dx, dt, "dx", tok), _stream(stream)))


def moe_combine_bwd(layout, dy, ye, ids, slots, slot_src, weights, dye, dw, stream=None):
    dt = torch.bfloat16 if layout.dtype == MOE_BF16 else torch.float32
    i32 = torch.int32
    tok, exp, ch, src = _rows(layout)
    _check(load().moe_combine_bwd(ctypes.byref(layout), _ptr(dy, dt, "dy", tok), _ptr(ye, dt, "ye", exp),
                                  _ptr(ids, i32, "ids", ch), _ptr(slots, i32, "slots", ch),
                                  _ptr(slot_src, i32, "slot_src", src), _ptr(weights, torch.float32, "weights", ch),
                                  _ptr(dye, dt, "dye", exp), _ptr(dw, torch.float32, "dw", ch), _stream(stream)))


# ---------------------------------------------------------------- convenience wrappers

def gate(kind, k, E, capacity, *, x=None, wg=None, bias=None, token_ids=None, logits=None,
         logits_in=False, normalize=0, hash_seed=0, want_logits=False, want_demand=True, dtype=None,
         groups=0, noise=None, temperature=0.0, hash_table=None, stream=None):
    """Allocate the outputs and run moe_gate; returns a dict of device tensors."""
    if kind == MOE_GATE_HASH:
        S, d = int(token_ids.shape[0]), 0
        dcode = MOE_F32 if dtype is None else dtype
    elif logits_in:
        S, d = int(logits.shape[0]), 0
        dcode = MOE_F32 if dtype is None else dtype
    else:
        S, d = int(x.shape[0]), int(x.shape[1])
        dcode = _dtype_code(x)
    ref = logits if logits is not None else (x if x is not None else token_ids)
    dev = ref.device
    vocab = 0 if hash_table is None else int(hash_table.shape[0])
    params = gate_params(S, d, E, k, capacity, kind, normalize, int(bool(logits_in)), dcode, hash_seed, groups,
                         temperature, vocab)
    out = {
        "ids": torch.empty((S, k), dtype=torch.int32, device=dev),
        "slots": torch.empty((S, k), dtype=torch.int32, device=dev),
        "weights": torch.empty((S, k), dtype=torch.float32, device=dev),
        "counts": torch.empty((E,), dtype=torch.int32, device=dev),
        "demand": torch.empty((E,), dtype=torch.int32, device=dev) if want_demand else None,
        "slot_src": torch.empty((E, capacity), dtype=torch.int32, device=dev),
    }
    if not logits_in and want_logits:
        logits = torch.empty((S, E), dtype=torch.float32, device=dev)
    elif not logits_in:
        logits = None
    out["logits"] = logits
    ws = torch.empty((moe_gate_workspace_size(params),), dtype=torch.uint8, device=dev)
    moe_gate(params, x, wg, bias, token_ids, noise, hash_table, logits, out["ids"], out["slots"], out["weights"],
             out["counts"], out["demand"], out["slot_src"], ws, stream)
    return out


def moe_hash_balanced_table(freq, E):
    """Balanced token -> expert table of the Hash Layer gate, built on the host by
    the library (freq: host array of token frequencies).  Returns an int32 numpy array."""
    import numpy as np
    f = np.ascontiguousarray(freq, dtype=np.float64)
    table = np.empty(f.shape[0], dtype=np.int32)
    _check(load().moe_hash_balanced_table(f.ctypes.data, int(f.shape[0]), int(E), table.ctypes.data))
    return table


def base_params(S, d, E, capacity, logits_in=0, dtype=MOE_F32, max_rounds=0):
    return BaseParams(S, d, E, capacity, logits_in, dtype, max_rounds)


def moe_base_gate_workspace_size(params):
    n = ctypes.c_size_t(0)
    _check(load().moe_base_gate_workspace_size(ctypes.byref(params), ctypes.byref(n)))
    return n.value


def moe_base_gate(params, x, wg, bias, logits, ids, slots, weights, counts, slot_src, prices, workspace, info=None,
                  stream=None):
    """BASE-layer balanced assignment (synchronizes the stream).  `prices`: a
    float64 [E] device tensor for the final prices, or None; `info`: a BaseInfo
    filled with the auction's statistics, or None."""
    lib = load()
    f32, i32 = torch.float32, torch.int32
    xdt = torch.bfloat16 if params.dtype == MOE_BF16 else torch.float32
    S, d, E, C = params.S, params.d, params.E, params.capacity
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(lib.moe_base_gate(
        ctypes.byref(params), _ptr(x, xdt, "x", S * d), _ptr(wg, xdt, "wg", d * E), _ptr(bias, f32, "bias", E),
        _ptr(logits, f32, "logits", S * E), _ptr(ids, i32, "ids", S), _ptr(slots, i32, "slots", S),
        _ptr(weights, f32, "weights", S), _ptr(counts, i32, "counts", E), _ptr(slot_src, i32, "slot_src", E * C),
        _ptr(prices, torch.float64, "prices", E), _ptr(workspace, None, "workspace"), ws_bytes,
        None if info is None else ctypes.byref(info),
        _stream(stream)))


def moe_base_gate_async(params, x, wg, bias, logits, ids, slots, weights, counts, slot_src, prices, workspace,
                        launch_rounds, status, stream=None):
    """moe_base_gate with `launch_rounds` auction rounds enqueued and no host
    synchronization; `status`: a device tensor of at least 24 bytes, 8-byte
    aligned, that receives the moe_base_status (see base_status)."""
    lib = load()
    f32, i32 = torch.float32, torch.int32
    xdt = torch.bfloat16 if params.dtype == MOE_BF16 else torch.float32
    S, d, E, C = params.S, params.d, params.E, params.capacity
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    if status is not None and status.numel() * status.element_size() < BASE_STATUS_BYTES:
        raise ValueError("status must hold at least 24 bytes")
    _check(lib.moe_base_gate_async(
        ctypes.byref(params), _ptr(x, xdt, "x", S * d), _ptr(wg, xdt, "wg", d * E), _ptr(bias, f32, "bias", E),
        _ptr(logits, f32, "logits", S * E), _ptr(ids, i32, "ids", S), _ptr(slots, i32, "slots", S),
        _ptr(weights, f32, "weights", S), _ptr(counts, i32, "counts", E), _ptr(slot_src, i32, "slot_src", E * C),
        _ptr(prices, torch.float64, "prices", E), _ptr(workspace, None, "workspace"), ws_bytes,
        int(launch_rounds), _ptr(status, None, "status"), _stream(stream)))


def base_status(status):
    """Decode a moe_base_status tensor (device or host) into a dict."""
    import numpy as np
    raw = status.detach().reshape(-1).view(torch.uint8)[:BASE_STATUS_BYTES].cpu().numpy()
    w = raw.view(np.int32)
    return dict(phases=int(w[0]), rounds=int(w[1]), eps=float(raw[8:16].view(np.float64)[0]), status=int(w[4]))


def base_gate(E, capacity=None, *, x=None, wg=None, bias=None, logits=None, logits_in=False, want_logits=False,
              max_rounds=0, launch_rounds=None, stream=None):
    """Allocate the outputs and run moe_base_gate; returns a dict of device
    tensors (ids, slots, weights as [S, 1], the shape the layout calls take;
    prices [E] float64) plus "info" (phases, rounds, eps of the auction).
    With launch_rounds, moe_base_gate_async runs instead and "status" is the
    device moe_base_status (int64 [3]; decode it with base_status)."""
    if logits_in:
        S, d, dcode = int(logits.shape[0]), 0, MOE_F32
        dev = logits.device
    else:
        S, d, dcode = int(x.shape[0]), int(x.shape[1]), _dtype_code(x)
        dev = x.device
    C = S // E if capacity is None else capacity
    params = base_params(S, d, E, C, int(bool(logits_in)), dcode, max_rounds)
    out = {
        "ids": torch.empty((S, 1), dtype=torch.int32, device=dev),
        "slots": torch.empty((S, 1), dtype=torch.int32, device=dev),
        "weights": torch.empty((S, 1), dtype=torch.float32, device=dev),
        "counts": torch.empty((E,), dtype=torch.int32, device=dev),
        "slot_src": torch.empty((E, C), dtype=torch.int32, device=dev),
        "prices": torch.empty((E,), dtype=torch.float64, device=dev),
    }
    if not logits_in:
        logits = torch.empty((S, E), dtype=torch.float32, device=dev) if want_logits else None
    out["logits"] = logits
    ws = torch.empty((moe_base_gate_workspace_size(params),), dtype=torch.uint8, device=dev)
    if launch_rounds is not None:
        out["status"] = torch.empty((3,), dtype=torch.int64, device=dev)
        moe_base_gate_async(params, x, wg, bias, logits, out["ids"], out["slots"], out["weights"], out["counts"],
                            out["slot_src"], out["prices"], ws, launch_rounds, out["status"], stream)
        return out
    info = BaseInfo()
    moe_base_gate(params, x, wg, bias, logits, out["ids"], out["slots"], out["weights"], out["counts"],
                  out["slot_src"], out["prices"], ws, info, stream)
    out["info"] = dict(phases=info.phases, rounds=info.rounds, eps=info.eps)
    return out


def dispatch(x, ids, slots, slot_src, stream=None):
    S, d = x.shape
    k = ids.shape[1]
    E, C = slot_src.shape
    xe = torch.empty((E, C, d), dtype=x.dtype, device=x.device)
    moe_dispatch(_layout(S, d, E, k, C, _dtype_code(x)), x, ids, slots, slot_src, xe, stream)
    return xe


def combine(ye, ids, slots, weights, stream=None):
    E, C, d = ye.shape
    S, k = ids.shape
    y = torch.empty((S, d), dtype=ye.dtype, device=ye.device)
    moe_combine(_layout(S, d, E, k, C, _dtype_code(ye)), ye, ids, slots, weights, y, stream)
    return y


def dispatch_bwd(dxe, ids, slots, stream=None):
    E, C, d = dxe.shape
    S, k = ids.shape
    dx = torch.empty((S, d), dtype=dxe.dtype, device=dxe.device)
    moe_dispatch_bwd(_layout(S, d, E, k, C, _dtype_code(dxe)), dxe, ids, slots, dx, stream)
    return dx


def combine_bwd(dy, ids, slots, slot_src, weights, ye=None, want_dw=True, stream=None):
    S, d = dy.shape
    E, C = slot_src.shape
    k = weights.shape[1]
    dye = torch.empty((E, C, d), dtype=dy.dtype, device=dy.device)
    dw = torch.empty((S, k), dtype=torch.float32, device=dy.device) if want_dw else None
    moe_combine_bwd(_layout(S, d, E, k, C, _dtype_code(dy)), dy, ye if want_dw else None, ids, slots, slot_src,
                    weights, dye, dw, stream)
    return dye, dw


def gate_bwd_params(S, d, E, k, kind, normalize=0, dtype=MOE_F32, accumulate_dx=0, aux_coef=0.0, temperature=0.0):
    return GateBwdParams(S, d, E, k, kind, normalize, dtype, accumulate_dx, aux_coef, temperature)


def moe_gate_bwd_workspace_size(params):
    n = ctypes.c_size_t(0)
    _check(load().moe_gate_bwd_workspace_size(ctypes.byref(params), ctypes.byref(n)))
    return n.value


def moe_gate_bwd(params, x, wg, logits, ids, dw, dlogits, dx, dwg, dbias, aux_loss, workspace, stream=None):
    dt = torch.bfloat16 if params.dtype == MOE_BF16 else torch.float32
    f32, i32 = torch.float32, torch.int32
    S, d, E, k = params.S, params.d, params.E, params.k
    ws_bytes = workspace.numel() * workspace.element_size() if workspace is not None else 0
    _check(load().moe_gate_bwd(ctypes.byref(params), _ptr(x, dt, "x", S * d), _ptr(wg, dt, "wg", d * E),
                               _ptr(logits, f32, "logits", S * E), _ptr(ids, i32, "ids", S * k),
                               _ptr(dw, f32, "dw", S * k), _ptr(dlogits, f32, "dlogits", S * E),
                               _ptr(dx, dt, "dx", S * d), _ptr(dwg, f32, "dwg", d * E), _ptr(dbias, f32, "dbias", E),
                               _ptr(aux_loss, f32, "aux_loss", 1), _ptr(workspace, None, "workspace"), ws_bytes,
                               _stream(stream)))


def gate_bwd(kind, logits, ids, dw, *, x=None, wg=None, normalize=0, dx=None, accumulate_dx=False,
             want_dlogits=True, want_dwg=True, want_dbias=True, want_dx=True, aux_coef=0.0, temperature=0.0,
             stream=None):
    """Allocating wrapper of moe_gate_bwd.  Returns a dict with dlogits, dwg,
    dbias, dx and aux_loss (None where not requested).  With accumulate_dx the
    given dx is updated in place and returned."""
    S, E = logits.shape
    k = ids.shape[1]
    dev = logits.device
    src = x if x is not None else (wg if wg is not None else dx)
    dt = torch.float32 if src is None else src.dtype
    d = x.shape[1] if x is not None else (wg.shape[0] if wg is not None else 1)
    params = gate_bwd_params(S, d, E, k, kind, normalize, MOE_BF16 if dt == torch.bfloat16 else MOE_F32,
                             1 if accumulate_dx else 0, aux_coef, temperature)
    f32 = torch.float32
    out = {
        "dlogits": torch.empty((S, E), dtype=f32, device=dev) if want_dlogits else None,
        "dwg": torch.empty((d, E), dtype=f32, device=dev) if want_dwg else None,
        "dbias": torch.empty((E,), dtype=f32, device=dev) if want_dbias else None,
        "aux_loss": torch.empty((1,), dtype=f32, device=dev) if aux_coef != 0.0 else None,
    }
    if want_dx:
        out["dx"] = dx if accumulate_dx else torch.empty((S, d), dtype=dt, device=dev)
    else:
        out["dx"] = None
    ws = torch.empty((moe_gate_bwd_workspace_size(params),), dtype=torch.uint8, device=dev)
    moe_gate_bwd(params, x if want_dwg else None, wg if want_dx else None, logits, ids, dw, out["dlogits"],
                 out["dx"], out["dwg"], out["dbias"], out["aux_loss"], ws, stream)
    return out
