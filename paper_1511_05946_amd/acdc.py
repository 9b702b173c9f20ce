"""Python binding of the ACDC / AFDF cascade library.

Argument marshalling only: every step of the computation runs in the HIP
kernels of libacdc.so.  Tensors are torch tensors on a ROCm device; the work
is enqueued on the current torch stream of that device.

Layer (Sec. 4 of arXiv:1511.05946): y = x A C D C^{-1} on row vectors, C the
orthonormal DCT-II; the complex AFDF layer of Sec. 3 uses the DFT.  A cascade
chains K layers with optional fixed permutations and ReLU between them, and
optionally a bias b_k added to each layer's D-domain term (Sec. 6.2):
y = (x A C D + b) C^{-1}.
"""

from __future__ import annotations

import ctypes
import functools

import torch

from ._lib import lib, status_string

FLAG_PERM = 1
FLAG_RELU = 2
FLAG_COMPLEX = 4
FLAG_BIAS = 8
FLAG_ACCUMULATE = 16
FLAG_MULTIPASS = 32


class ACDCError(RuntimeError):
    pass


def _check(rc: int, what: str):
    if rc != 0:
        extra = ""
        if rc == -4:
            extra = f" (hipError {lib().acdc_last_hip_error()})"
        raise ACDCError(f"{what}: {status_string(rc)}{extra}")


def _flags(flags: int, x: torch.Tensor, bias=None) -> int:
    if x.is_complex():
        flags |= FLAG_COMPLEX
    if bias is not None:
        flags |= FLAG_BIAS
    return flags


def _ptr(t):
    if t is None:
        return None
    return t.data_ptr()


def _nbytes(t) -> int:
    return 0 if t is None else t.numel() * t.element_size()


def _dims(x: torch.Tensor, A: torch.Tensor):
    if x.dim() != 2 or A.dim() != 2:
        raise ValueError("x must be [batch, N] and A, D [K, N]")
    if A.shape[1] != x.shape[1]:
        raise ValueError(f"A is {tuple(A.shape)}: its rows must have x's width N = {x.shape[1]}")
    return x.shape[0], x.shape[1], A.shape[0]


def _check_shapes(shapes: dict, B: int, N: int, K: int):
    """Every tensor handed to the library must have exactly the shape its
    pointer is read or written with: rows [B, N], layer vectors [K, N]. The
    library takes raw pointers, so a mismatch here would be an out-of-bounds
    device access there; this runs before any device or dtype check."""
    want = {"row": (B, N), "layer": (K, N)}
    for name, (t, kind) in shapes.items():
        if t is None:
            continue
        if tuple(t.shape) != want[kind]:
            raise ValueError(f"{name} is {tuple(t.shape)}, expected {want[kind]}")


def _validate(tensors, complex_: bool, device):
    for name, t in tensors.items():
        if t is None:
            continue
        if t.device != device:
            raise ValueError(f"{name} is on {t.device}, expected {device}")
        if not t.is_contiguous():
            raise ValueError(f"{name} must be contiguous")
        if name == "perm":
            if t.dtype != torch.int32:
                raise ValueError("perm must be int32")
        elif name == "workspace":
            pass
        elif complex_ and t.dtype != torch.complex64:
            raise ValueError(f"{name} must be complex64")
        elif not complex_ and t.dtype != torch.float32:
            raise ValueError(f"{name} must be float32")


def _stream(device):
    return torch.cuda.current_stream(device).cuda_stream


# A small cascade's kernels take tens of microseconds, about what the binding
# itself did, so its common path is short: one pass of plain comparisons per
# tensor (only a tensor that fails one goes through the checks above, which
# say what is wrong), the buffer sizes of a shape remembered, and no device
# switch where the tensors' device is the current one.  One layer N = 2048,
# 128 rows, forward and backward: 37 us before, 33 after
# (the calls themselves 18 and 23 us, and 14 and 18 us).

def _fits(shape, tensors) -> bool:
    for t in tensors:
        if t is not None and t.shape != shape:
            return False
    return True


def _plain(dtype, device, tensors) -> bool:
    for t in tensors:
        if t is not None and not (t.dtype is dtype and t.device == device and t.is_contiguous()):
            return False
    return True


@functools.lru_cache(maxsize=512)
def _sizes(B: int, N: int, K: int, flags: int):
    """Bytes of the saved buffer, the forward workspace and the backward
    workspace without and with the saved buffer: fixed by the shape alone."""
    L = lib()
    return (L.acdc_saved_bytes(B, N, K, flags), L.acdc_forward_workspace_size(B, N, K, flags),
            L.acdc_backward_workspace_size(B, N, K, flags, 0), L.acdc_backward_workspace_size(B, N, K, flags, 1))


def _call(fn, device, *args):
    """fn(*args, stream) on `device`."""
    if device.type == "cuda" and torch._C._cuda_getDevice() == device.index:
        return fn(*args, torch._C._cuda_getCurrentRawStream(device.index))
    with torch.cuda.device(device):
        return fn(*args, _stream(device))


def supported(N: int, flags: int = 0) -> bool:
    return bool(lib().acdc_supported(int(N), int(flags)))


def prepare(N: int, flags: int = 0, device=None):
    with torch.cuda.device(device if device is not None else torch.cuda.current_device()):
        _check(lib().acdc_prepare(int(N), int(flags)), "acdc_prepare")


def sync_timeouts(device=None, clear: bool = False) -> int:
    """Backward row syncs on `device` whose bounded wait ran out (0 when healthy).

    Synchronises the device first; with clear=True the count restarts at 0."""
    with torch.cuda.device(device if device is not None else torch.cuda.current_device()):
        torch.cuda.synchronize()
        n = ctypes.c_int64(0)
        _check(lib().acdc_sync_timeouts(ctypes.byref(n), int(bool(clear))), "acdc_sync_timeouts")
        return int(n.value)


def saved_numel(x: torch.Tensor, K: int, flags: int = 0) -> int:
    """Elements (of x's dtype) of the buffer acdc_forward fills for
    acdc_backward: the layer inputs u_1..u_{K-1}, preceded by u_0 (x gathered
    through perm[0]) with FLAG_PERM."""
    flags = _flags(flags, x)
    nbytes = lib().acdc_saved_bytes(x.shape[0], x.shape[1], K, flags)
    return nbytes // x.element_size()


def alloc_saved(x: torch.Tensor, K: int, flags: int = 0) -> torch.Tensor:
    return torch.empty(saved_numel(x, K, flags), dtype=x.dtype, device=x.device)


def saved_layer_inputs(saved: torch.Tensor, x: torch.Tensor, K: int, flags: int = 0) -> torch.Tensor:
    """View of the layer inputs inside a saved buffer, [slots, batch, N]:
    u_1..u_{K-1} in slots 0..K-2, and with FLAG_PERM u_0 (x gathered through
    perm[0]) in slot K-1."""
    B, N = x.shape
    L = K - 1 + (1 if flags & FLAG_PERM else 0)
    return saved[: L * B * N].view(L, B, N)


def forward_workspace_bytes(x, K: int, flags: int = 0, bias=None) -> int:
    """Bytes of the caller-owned workspace acdc_forward takes for x [B, N]."""
    flags = _flags(flags, x, bias)
    return int(lib().acdc_forward_workspace_size(x.shape[0], x.shape[1], K, flags))


def backward_workspace_bytes(x, K: int, flags: int = 0, have_saved: bool = True, bias=None) -> int:
    """Bytes of the caller-owned workspace acdc_backward takes for x [B, N]
    (more without the forward's saved layer inputs: the stash is rebuilt in
    it)."""
    flags = _flags(flags, x, bias)
    return int(lib().acdc_backward_workspace_size(x.shape[0], x.shape[1], K, flags, 1 if have_saved else 0))


def _workspace(ws, need: int, device):
    if ws is None:
        return torch.empty(max(need, 1), dtype=torch.uint8, device=device)
    if ws.dtype != torch.uint8 or ws.dim() != 1 or ws.numel() < need:
        raise ValueError(f"workspace must be a uint8 vector of at least {need} bytes")
    return ws


def forward(x, A, D, perm=None, flags: int = 0, save: bool = False, out=None, saved=None, bias=None,
            workspace=None):
    """y = cascade(x), with the D-domain biases ``bias`` [K, N] if given.
    Returns (y, saved) where saved holds the layer inputs u_1..u_{K-1} for
    acdc_backward when ``save`` (or a preallocated ``saved``) is given.
    ``workspace``: a uint8 device vector of forward_workspace_bytes() bytes
    (allocated here when not given)."""
    flags = _flags(flags, x, bias)
    cplx = bool(flags & FLAG_COMPLEX)
    B, N, K = _dims(x, A)
    perm = perm if flags & FLAG_PERM else None
    if not (_fits((K, N), (D, bias, perm)) and _fits((B, N), (out,))):
        _check_shapes({"D": (D, "layer"), "bias": (bias, "layer"), "y": (out, "row"), "perm": (perm, "layer")}, B, N, K)
    saved_bytes, ws_bytes, _, _ = _sizes(B, N, K, flags)
    if saved is not None and saved.numel() < saved_bytes // x.element_size():
        raise ValueError(f"saved holds {saved.numel()} elements, needs {saved_numel(x, K, flags)}")
    if out is None:
        out = torch.empty_like(x)
    if save and saved is None:
        saved = torch.empty(saved_bytes // x.element_size(), dtype=x.dtype, device=x.device)
    device = x.device
    if not (_plain(torch.complex64 if cplx else torch.float32, device, (x, A, D, bias, out, saved))
            and _plain(torch.int32, device, (perm,))):
        _validate({"x": x, "A": A, "D": D, "bias": bias, "y": out, "saved": saved, "perm": perm}, cplx, device)
    ws = _workspace(workspace, ws_bytes, device)
    if workspace is not None:
        _validate({"workspace": ws}, cplx, device)
    rc = _call(lib().acdc_forward, device, x.data_ptr(), out.data_ptr(), A.data_ptr(), _ptr(D), _ptr(bias),
               _ptr(perm), B, N, K, flags, saved.data_ptr() if (saved is not None and saved.numel() > 0) else None,
               _nbytes(saved), ws.data_ptr(), ws_bytes)
    _check(rc, "acdc_forward")
    return out, saved


def backward(x, grad_y, A, D, perm=None, flags: int = 0, saved=None, bias=None, grads=None, out=None,
             workspace=None):
    """(grad_x, grad_A, grad_D), plus grad_bias when ``bias`` is given; the
    parameter gradients are summed over the batch.  Without ``saved`` (from
    ``forward(..., save=True)`` on the same inputs) the forward is recomputed
    inside the call.  ``grads`` = (grad_A, grad_D[, grad_bias]) tensors to
    write into; with FLAG_ACCUMULATE in ``flags`` the sums are added to them.
    ``out``: a tensor to write grad_x into.  ``workspace``: a uint8 device
    vector of backward_workspace_bytes() bytes (allocated when not given)."""
    flags = _flags(flags, x, bias)
    cplx = bool(flags & FLAG_COMPLEX)
    B, N, K = _dims(x, A)
    if grads is None and flags & FLAG_ACCUMULATE:
        raise ValueError("FLAG_ACCUMULATE needs the gradient tensors to add into (grads=...)")
    if grads is not None and len(grads) != (3 if bias is not None else 2):
        raise ValueError("grads must be (grad_A, grad_D) or, with bias, (grad_A, grad_D, grad_bias)")
    perm = perm if flags & FLAG_PERM else None
    gA, gD = grads[:2] if grads is not None else (None, None)
    gB = grads[2] if grads is not None and bias is not None else None
    if not (_fits((B, N), (grad_y, out)) and _fits((K, N), (D, bias, perm, gA, gD, gB))):
        _check_shapes({"grad_y": (grad_y, "row"), "grad_x": (out, "row"), "D": (D, "layer"), "bias": (bias, "layer"),
                       "perm": (perm, "layer"), "grad_A": (gA, "layer"), "grad_D": (gD, "layer"),
                       "grad_bias": (gB, "layer")}, B, N, K)
    saved_bytes, _, ws_recompute, ws_saved = _sizes(B, N, K, flags)
    use_saved = saved is not None and saved.numel() > 0
    if use_saved and saved.numel() < saved_bytes // x.element_size():
        raise ValueError(f"saved holds {saved.numel()} elements, needs {saved_numel(x, K, flags)}")
    gx = torch.empty_like(x) if out is None else out
    if grads is None:
        gA, gD = torch.empty_like(A), torch.empty_like(D)
        gB = torch.empty_like(bias) if bias is not None else None
    device = x.device
    if not (_plain(torch.complex64 if cplx else torch.float32, device,
                   (x, grad_y, gx, A, D, bias, saved, gA, gD, gB)) and _plain(torch.int32, device, (perm,))):
        _validate({"x": x, "grad_y": grad_y, "grad_x": gx, "A": A, "D": D, "bias": bias, "saved": saved,
                   "grad_A": gA, "grad_D": gD, "grad_bias": gB, "perm": perm}, cplx, device)
    ws_bytes = ws_saved if use_saved or saved_bytes < x.element_size() else ws_recompute
    ws = _workspace(workspace, ws_bytes, device)
    if workspace is not None:
        _validate({"workspace": ws}, cplx, device)
    rc = _call(lib().acdc_backward, device, x.data_ptr(), _ptr(grad_y), A.data_ptr(), _ptr(D), _ptr(bias),
               _ptr(perm), saved.data_ptr() if use_saved else None, _nbytes(saved), gx.data_ptr(), _ptr(gA),
               _ptr(gD), _ptr(gB), B, N, K, flags, ws.data_ptr(), ws_bytes)
    _check(rc, "acdc_backward")
    return (gx, gA, gD, gB) if bias is not None else (gx, gA, gD)


class ACDCCascade(torch.autograd.Function):
    """autograd wrapper: stores the layer inputs in the forward pass."""

    @staticmethod
    def forward(ctx, x, A, D, perm, flags, bias=None):
        # the backward gets exactly the (contiguous) tensors the forward used
        x, A, D = x.contiguous(), A.contiguous(), D.contiguous()
        perm = perm.contiguous() if perm is not None else None
        bias = bias.contiguous() if bias is not None else None
        y, saved = forward(x, A, D, perm, flags, save=True, bias=bias)
        ctx.save_for_backward(x, A, D, perm, bias, saved)
        ctx.flags = flags
        return y

    @staticmethod
    def backward(ctx, gy):
        x, A, D, perm, bias, saved = ctx.saved_tensors
        out = backward(x, gy.contiguous(), A, D, perm, ctx.flags, saved, bias=bias)
        return out[0], out[1], out[2], None, None, out[3] if bias is not None else None


def acdc_cascade(x, A, D, perm=None, flags: int = 0, bias=None):
    return ACDCCascade.apply(x, A, D, perm, flags, bias)
