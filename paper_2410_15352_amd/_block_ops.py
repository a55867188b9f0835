"""Autograd functions over the block kernels of libcompact.so (csrc/block_ops.hip):
RMSNorm with its residual, SwiGLU and the mean cross-entropy.

They take dense bf16 tensors on the current GPU; `usable` says whether a call may
go that way.  Everything else (CPU, other types and strides, autocast, tracing,
functorch, forward-mode AD) takes the torch expressions beside each function, and so does a
backward that is itself recorded (create_graph=True) or batched (is_grads_batched=True), or that
gets its saved tensors back from a hook in another type, layout or place."""
from __future__ import annotations

import ctypes

import torch

from . import _lib, bwd_workspace_bytes, compact_bwd

_vp, _i64, _i32, _f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_float
RMSNORM_MAX_D = 4096
MAX_ROWS = 1 << 24  # one workgroup of 256 threads per row at most: a launch has under 2^32 threads
MAX_CHUNKS = (1 << 32) - 256  # of 8 elements, one per thread
IGNORE = -100  # F.cross_entropy's default ignore_index


class _NormArgs(ctypes.Structure):
    _fields_ = [("x", _vp), ("add", _vp), ("g", _vp), ("sum", _vp), ("y", _vp), ("rstd", _vp), ("rows", _i64),
                ("d", _i32), ("eps", _f32)]


class _NormGradArgs(ctypes.Structure):
    _fields_ = [("x", _vp), ("dy", _vp), ("dres", _vp), ("g", _vp), ("rstd", _vp), ("dx", _vp), ("part", _vp),
                ("dg", _vp), ("rows", _i64), ("d", _i32)]


class _CeArgs(ctypes.Structure):
    _fields_ = [("x", _vp), ("target", _vp), ("lse", _vp), ("loss_row", _vp), ("loss", _vp), ("count", _vp), ("valid", _vp),
                ("rows", _i64), ("V", _i64), ("ignore_index", _i64)]


class _CeGradArgs(ctypes.Structure):
    _fields_ = [("x", _vp), ("target", _vp), ("lse", _vp), ("count", _vp), ("dloss", _vp), ("dx", _vp), ("rows", _i64),
                ("V", _i64), ("ignore_index", _i64)]


_SIGNATURES = {
    "compact_block_rmsnorm_fwd": [ctypes.POINTER(_NormArgs), _vp],
    "compact_block_rmsnorm_parts": [_i64],
    "compact_block_rmsnorm_bwd": [ctypes.POINTER(_NormGradArgs), _vp],
    "compact_block_swiglu_fwd": [_vp, _vp, _vp, _i64, _i64, _vp],
    "compact_block_swiglu_bwd": [_vp, _vp, _vp, _vp, _i64, _i64, _vp],
    "compact_block_join3": [_vp, _vp, _vp, _vp, _i64, _i64, _vp],
    "compact_block_ce_fwd": [ctypes.POINTER(_CeArgs), _vp],
    "compact_block_ce_bwd": [ctypes.POINTER(_CeGradArgs), _vp],
}
_fns = {}


def _call(name, *args):
    fn = _fns.get(name)
    if fn is None:
        fn = getattr(_lib.load(), name)
        fn.restype, fn.argtypes = ctypes.c_int, _SIGNATURES[name]
        _fns[name] = fn
    rc = fn(*args)
    if rc < 0:
        raise RuntimeError(f"{name}: status {rc}")
    return rc


def _stream(t):
    return torch._C._cuda_getCurrentRawStream(t.get_device())


_TYPES = (torch.Tensor, torch.nn.Parameter)
_is_compiling, _is_tracing, _autocast = torch.compiler.is_compiling, torch._C._is_tracing, torch.is_autocast_enabled
_dispatch_modes, _functorch_level = torch._C._len_torch_dispatch_stack, torch._C._functorch.peek_interpreter_stack
_forward_ad = torch.autograd.forward_ad


def _plain(t):
    """A tensor of its own storage: no subclass, no functorch wrapper, none of the batched
    tensors that is_grads_batched hands to a backward (in the engine's thread, where no
    functorch level is seen).  Tensors that wrap another have no pointer to ask for."""
    if type(t) not in _TYPES:
        return False
    try:
        t.data_ptr()
    except RuntimeError:
        return False
    return True


def _eager():
    """Outside autocast and every kind of tracing.  Asked before any size is looked at:
    under a tracer a comparison of sizes would be traced, or guarded, too."""
    return not (_is_compiling() or _is_tracing() or _dispatch_modes() > 0 or _autocast()  # (the GPU's)
                or _functorch_level() is not None or _forward_ad._current_level >= 0)


def _kernel_tensors(*tensors):
    """Dense bf16 tensors on the current device."""
    dev = None
    for t in tensors:
        if type(t) not in _TYPES:
            return False
        try:
            p = t.data_ptr()  # 0: no elements
        except RuntimeError:  # (as in _plain)
            return False
        at = t.get_device()  # -1: the CPU
        if p == 0 or p % 16 != 0 or at < 0 or t.dtype != torch.bfloat16 or not t.is_contiguous():
            return False
        if at != dev:
            if dev is not None or at != torch._C._cuda_getDevice():
                return False
            dev = at
    return True


def usable(*tensors):
    """Dense bf16 tensors on the current device, outside autocast and every kind of
    tracing."""
    return _eager() and _kernel_tensors(*tensors)


def norm_usable(x, g, *rest):
    """Rows of x with one gain per element (other gains broadcast or are refused by torch)."""
    if not _eager():
        return False
    if x.dim() < 1 or x.shape[-1] % 8 != 0 or not 8 <= x.shape[-1] <= RMSNORM_MAX_D or g.shape != x.shape[-1:]:
        return False
    return x.numel() // x.shape[-1] < MAX_ROWS and _kernel_tensors(x, g, *rest)


def _grads(saved, *grads):
    """The gradients (None stays None) as a backward's kernel takes them, or None
    where that kernel must not run: a backward that is recorded, or batched
    (is_grads_batched), or whose saved tensors came back from a saved-tensor hook in
    another type, layout or place."""
    if torch.is_grad_enabled() or not _eager():
        return None
    given = [t for t in grads if t is not None]
    if _kernel_tensors(*saved, *given):
        return grads
    if not _kernel_tensors(*saved) or not all(map(_plain, given)):
        return None
    out = []
    for t in grads:
        if t is not None:
            t = t.to(torch.bfloat16).contiguous()
            t = t if t.data_ptr() % 16 == 0 else t.clone()
        out.append(t)
    return out if _kernel_tensors(*(t for t in out if t is not None)) else None


def _companion(t, dtype, count):
    """A saved tensor beside the bf16 ones is still what the forward's kernel wrote or read."""
    return (t.dtype == dtype and t.numel() == count and _plain(t) and t.is_cuda and t.is_contiguous()
            and t.get_device() == torch._C._cuda_getDevice())


def _torch_grad(fn, x, dy):
    """The gradient of the torch expression fn(x), itself differentiable where the
    backward is recorded."""
    recorded = torch.is_grad_enabled()
    with torch.enable_grad():
        x = x if recorded and x.requires_grad else x.detach().requires_grad_(True)
        return torch.autograd.grad(fn(x), x, dy, create_graph=recorded)[0]


# ------------------------------- RMSNorm -----------------------------------

def rmsnorm_reference_grad(x, rstd, g, dy, eps):
    if torch.is_grad_enabled():  # recorded: the saved 1 / rms is a constant, its own derivative is needed too
        rstd = torch.rsqrt(x.float().square().mean(-1) + eps)
    xhat = x.float() * rstd.unsqueeze(-1)
    dyf = dy.float()
    gdy = dyf * g.float()
    dx = rstd.unsqueeze(-1) * (gdy - xhat * (gdy * xhat).mean(-1, keepdim=True))
    dg = (dyf * xhat).reshape(-1, x.shape[-1]).sum(0)
    return dx.to(x.dtype), dg.to(g.dtype)


class _NormFn(torch.autograd.Function):
    """(x, y) with y = x / rms(x) * g, or with `add` (x + add, its norm): the first
    result carries the residual, so that its gradient and the norm's meet in one
    kernel.  Saves the normalised tensor and 1 / rms only."""

    @staticmethod
    def forward(ctx, x, add, g, eps):
        d = x.shape[-1]
        rows = x.numel() // d
        y = torch.empty_like(x)
        rstd = torch.empty(x.shape[:-1], dtype=torch.float32, device=x.device)
        total = torch.empty_like(x) if add is not None else None
        _call("compact_block_rmsnorm_fwd",
              ctypes.byref(_NormArgs(x.data_ptr(), None if add is None else add.data_ptr(), g.data_ptr(),
                                     None if add is None else total.data_ptr(), y.data_ptr(), rstd.data_ptr(), rows, d,
                                     eps)), _stream(x))
        ctx.set_materialize_grads(False)
        ctx.added, ctx.eps, ctx.size = add is not None, eps, (rows, d)
        ctx.save_for_backward(x if add is None else total, rstd, g)
        return (x if add is None else total), y

    @staticmethod
    def backward(ctx, dres, dy):
        x, rstd, g = ctx.saved_tensors
        if dy is None:
            return dres, dres if ctx.added else None, None, None
        rows, d = ctx.size
        grads = None
        if x.numel() == rows * d and x.size(-1) == d == g.numel() and _companion(rstd, torch.float32, rows):
            grads = _grads((x, g), dy, dres)
        if grads is None:
            dx, dg = rmsnorm_reference_grad(x, rstd, g, dy, ctx.eps)
            dx = dx if dres is None else dx + dres
            return dx, dx if ctx.added else None, dg, None
        dy, dres = grads
        need = ctx.needs_input_grad[0] or ctx.needs_input_grad[1]
        dx = torch.empty_like(dy) if need else None
        dg = torch.empty_like(g)
        part = torch.empty(_call("compact_block_rmsnorm_parts", rows), d, dtype=torch.float32, device=x.device)
        _call("compact_block_rmsnorm_bwd",
              ctypes.byref(_NormGradArgs(x.data_ptr(), dy.data_ptr(), None if dres is None else dres.data_ptr(),
                                         g.data_ptr(), rstd.data_ptr(), None if dx is None else dx.data_ptr(),
                                         part.data_ptr(), dg.data_ptr(), rows, d)), _stream(x))
        return dx, dx if ctx.added else None, dg, None


def rmsnorm(x, g, eps):
    """y alone."""
    return _NormFn.apply(x, None, g, eps)[1]


def rmsnorm_residual(x, g, eps):
    """(x, y): use the returned x for the residual."""
    return _NormFn.apply(x, None, g, eps)


def add_rmsnorm(x, add, g, eps):
    """(x + add, its norm)."""
    return _NormFn.apply(x, add, g, eps)


# -------------------------------- SwiGLU -----------------------------------

class _SwigluFn(torch.autograd.Function):
    """silu(gate) * up of gu = [gate | up]; keeps gu and silu(gate)."""

    @staticmethod
    def forward(ctx, gu):
        rows, f = gu.shape[0], gu.shape[1] // 2
        s = torch.empty(rows, f, dtype=gu.dtype, device=gu.device)
        act = torch.empty_like(s)
        _call("compact_block_swiglu_fwd", gu.data_ptr(), s.data_ptr(), act.data_ptr(), rows, f, _stream(gu))
        ctx.save_for_backward(gu, s)
        return act

    @staticmethod
    def backward(ctx, dact):
        gu, s = ctx.saved_tensors
        rows, f = dact.shape
        grads = _grads((gu, s), dact) if gu.numel() == 2 * rows * f and gu.size(-1) == 2 * f and s.numel() == rows * f else None
        if grads is None:
            return _torch_grad(lambda t: _swiglu_torch(t, f), gu, dact)
        (dact,) = grads
        dgu = torch.empty_like(gu)
        _call("compact_block_swiglu_bwd", gu.data_ptr(), s.data_ptr(), dact.data_ptr(), dgu.data_ptr(), rows, f,
              _stream(gu))
        return dgu


def _swiglu_torch(gu, f):
    return torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]


def swiglu(gu, f):
    """silu(gu[:, :f]) * gu[:, f:]."""
    if (_eager() and gu.dim() == 2 and gu.shape[1] == 2 * f and f % 8 == 0 and gu.numel() // 16 <= MAX_CHUNKS
            and _kernel_tensors(gu)):
        return _SwigluFn.apply(gu)
    return _swiglu_torch(gu, f)


# ------------------------- uncompressed layers -------------------------------

class _DenseFn(torch.autograd.Function):
    """x W with the weight's gradient x^T dy by the split-K kernel of the compressed
    gradients (z = x, r = n), rounded once from its fp32 sum."""

    @staticmethod
    def forward(ctx, x, W):
        ctx.save_for_backward(x, W)
        return x @ W

    @staticmethod
    def backward(ctx, dy):
        x, W = ctx.saved_tensors
        dx = dy @ W.t() if ctx.needs_input_grad[0] else None
        if not ctx.needs_input_grad[1]:
            return dx, None
        if torch.is_grad_enabled() or not usable(x, dy) or x.dim() != 2 or x.shape[0] != dy.shape[0]:
            return dx, x.t() @ dy
        T, n = x.shape
        m = dy.shape[1]
        G = torch.empty(n, m, dtype=torch.float32, device=x.device)
        ws = torch.empty(bwd_workspace_bytes(T, n, m, n), dtype=torch.uint8, device=x.device)
        compact_bwd(dy, None, x, None, G, ws=ws)
        return dx, G.to(W.dtype)


DENSE_TILE = 256 * 256


def dense_split(tokens, n, m):
    """The split-K kernel forms x^T dy of an (n, m) weight.  The library's GEMM gives it
    a few CUs and takes as long for 512 x 512 as for 1024 x 1024; split-K, with its
    partial sums and the rounding to bf16, is the faster one from some thousand tokens
    on (library -> split-K, us, MI355X):
      1024 x 1024   4096 tokens 32 -> 38, 5700 45 -> 38, 8192 57 -> 44, 65536 314 -> 148
      768 x 3072    4608 tokens 52 -> 48, 5700 68 -> 52, 8192 82 -> 61
      2048 x 2048   4096 tokens 47 -> 59, 6144 68 -> 71, 8192 87 -> 83, 9000 101 -> 88
      64 x 8192     4096 tokens 30 -> 22, 8192 54 -> 35, 65536 285 -> 195
    Narrower weights than 64 and wider ones than 8192 are the library's: 4096 x 8 over
    4096 tokens 20 -> 30, 8 x 524288 741 -> 987."""
    if n % 8 != 0 or m % 8 != 0 or min(n, m) < 64 or max(n, m) > 8192 or n * m > 64 * DENSE_TILE:
        return False
    least = 4096 if min(n, m) == 64 else 5632 if n * m <= 36 * DENSE_TILE else 8704
    return tokens >= least


def dense(x, W):
    """x W for 2-D x; where split-K forms the weight's gradient, through _DenseFn."""
    if (_eager() and x.dim() == 2 and W.dim() == 2 and dense_split(x.shape[0], *W.shape)
            and (x.requires_grad or W.requires_grad) and _kernel_tensors(x, W)):
        return _DenseFn.apply(x, W)
    return x @ W


# ------------------------------ q, k, v -------------------------------------

class _SplitQkvFn(torch.autograd.Function):
    """q, k, v (b, heads, l, hd) as views of qkv (b, l, 3, heads, hd); the backward
    joins their gradients in one pass when each is dense as (b, l, heads, hd), the
    layout attention's backward gives them."""

    @staticmethod
    def forward(ctx, qkv):
        ctx.shape = qkv.shape
        ctx.set_materialize_grads(False)
        return tuple(t.transpose(1, 2) for t in qkv.unbind(2))

    @staticmethod
    def backward(ctx, *grads):
        b, l, _, heads, hd = ctx.shape
        if any(g is None for g in grads):
            some = next((g for g in grads if g is not None), None)
            if some is None:
                return None
            grads = [torch.zeros_like(some) if g is None else g for g in grads]
        grads = [g.transpose(1, 2) for g in grads]
        d = heads * hd
        if torch.is_grad_enabled() or d % 8 != 0 or b * l * d // 8 > MAX_CHUNKS or not usable(*grads):
            return torch.stack(grads, 2)
        out = torch.empty(ctx.shape, dtype=grads[0].dtype, device=grads[0].device)
        _call("compact_block_join3", *(g.data_ptr() for g in grads), out.data_ptr(), b * l, d, _stream(out))
        return out


def split_qkv(qkv):
    """q, k, v (b, heads, l, hd) of qkv (b, l, 3, heads, hd)."""
    if usable(qkv):
        return _SplitQkvFn.apply(qkv)
    return tuple(t.transpose(1, 2) for t in qkv.unbind(2))


# ----------------------------- cross-entropy --------------------------------

class _CrossEntropyFn(torch.autograd.Function):
    """Mean cross-entropy of bf16 logits (rows, V), in fp32; keeps the logits and
    one log-sum-exp per row."""

    @staticmethod
    def forward(ctx, logits, targets):
        rows, V = logits.shape
        lse = torch.empty(rows + 1, dtype=torch.float32, device=logits.device)  # and the count
        loss_row = torch.empty(rows, dtype=torch.float32, device=logits.device)
        loss = torch.empty((), dtype=torch.float32, device=logits.device)
        valid = torch.empty((), dtype=torch.float32, device=logits.device)
        _call("compact_block_ce_fwd",
              ctypes.byref(_CeArgs(logits.data_ptr(), targets.data_ptr(), lse.data_ptr(), loss_row.data_ptr(),
                                   loss.data_ptr(), lse.data_ptr() + 4 * rows, valid.data_ptr(), rows, V, IGNORE)),
              _stream(logits))
        # on the GPU, as torch's own cross-entropy checks its targets; where that check
        # is compiled out, the loss and the row's gradient are NaN
        torch._assert_async(valid, "cross_entropy: a target is neither a class nor ignore_index")
        ctx.size = rows, V
        ctx.save_for_backward(logits, targets, lse)
        return loss

    @staticmethod
    def backward(ctx, dloss):
        logits, targets, lse = ctx.saved_tensors
        rows, V = ctx.size
        if (torch.is_grad_enabled() or not _plain(dloss) or not usable(logits) or logits.numel() != rows * V or logits.size(-1) != V
                or not _companion(lse, torch.float32, rows + 1)
                or not _companion(targets, torch.int64, rows)):
            return _torch_grad(lambda t: _cross_entropy_torch(t, targets), logits, dloss), None
        dloss = dloss.float().contiguous()
        dx = torch.empty_like(logits)
        _call("compact_block_ce_bwd",
              ctypes.byref(_CeGradArgs(logits.data_ptr(), targets.data_ptr(), lse.data_ptr(),
                                       lse.data_ptr() + 4 * rows, dloss.data_ptr(), dx.data_ptr(), rows, V, IGNORE)), _stream(logits))
        return dx, None


def _cross_entropy_torch(logits, targets):
    return torch.nn.functional.cross_entropy(logits.float(), targets)


def cross_entropy(logits, targets):
    """F.cross_entropy(logits.float(), targets) for 2-D logits and class targets."""
    if (_eager() and logits.dim() == 2 and _plain(targets) and targets.dtype == torch.int64 and targets.dim() == 1
            and targets.shape[0] == logits.shape[0] < MAX_ROWS and targets.device == logits.device
            and _kernel_tensors(logits)):
        return _CrossEntropyFn.apply(logits, targets.contiguous())
    return _cross_entropy_torch(logits, targets)
