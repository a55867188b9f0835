"""Which backwards of the block kernels' autograd functions may hand raw pointers to
the library.  On the CPU, with the library's calls replaced: the forwards' kernels by
numpy or by nothing, the backwards' by a failure.  Saved tensors that come back from
a hook in another type, layout or place, and batched gradients, must take the torch
expressions, whose values are compared with autograd through the plain operations."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
ops = pytest.importorskip("paper_2410_15352_amd._block_ops")

BF16_U = 2.0 ** -8  # one bf16 rounding, relative


def _bf16_at(ptr, count):
    u = np.ctypeslib.as_array((ctypes.c_uint16 * count).from_address(ptr)).astype(np.uint32) << 16
    return u.view(np.float32)


def _fake_call(name, *args):
    """The forwards as far as a torch backward depends on them: 1 / rms."""
    if name == "compact_block_rmsnorm_fwd":
        a = args[0]._obj
        x = _bf16_at(a.x, a.rows * a.d).reshape(a.rows, a.d).astype(np.float64)
        rstd = np.ctypeslib.as_array((ctypes.c_float * a.rows).from_address(a.rstd))
        rstd[:] = 1.0 / np.sqrt((x * x).mean(1) + a.eps)
        return 0
    assert name.endswith("_fwd"), f"{name} was given raw pointers"
    return 0


@pytest.fixture
def no_gpu(monkeypatch):
    monkeypatch.setattr(ops, "_call", _fake_call)
    monkeypatch.setattr(ops, "_stream", lambda t: 0)


def _bf16(*shape, seed=0, scale=1.0):
    return (scale * torch.randn(shape, generator=torch.Generator().manual_seed(seed))).to(torch.bfloat16)


def _norm(x, g):
    return ops.rmsnorm(x, g, 1e-6), x.float() * torch.rsqrt(x.float().square().mean(-1, keepdim=True) + 1e-6) * g.float()


def _swiglu(gu, _):
    f = gu.shape[1] // 2
    return ops._SwigluFn.apply(gu), torch.nn.functional.silu(gu[:, :f].float()) * gu[:, f:].float()


def _ce(x, _):
    t = torch.arange(x.shape[0]) % x.shape[1]
    t[1] = ops.IGNORE
    return ops._CrossEntropyFn.apply(x, t), torch.nn.functional.cross_entropy(x.float(), t)


HOOKS = {
    "fp32": (lambda t: t.float() if t.is_floating_point() else t, lambda t: t),
    "strided": (lambda t: t, lambda t: torch.stack([t, t], -1)[..., 0] if t.dim() > 1 else t),
    "as they were": (lambda t: t, lambda t: t),
}


@pytest.mark.parametrize("hook", list(HOOKS))
@pytest.mark.parametrize("fn,tol", [(_norm, 2 * BF16_U), (_swiglu, 4 * BF16_U), (_ce, 2 * BF16_U)])
def test_saved_tensors_from_hooks(no_gpu, fn, tol, hook):
    x, g = _bf16(6, 32).requires_grad_(True), (1 + 0.1 * _bf16(32, seed=1)).requires_grad_(True)
    with torch.autograd.graph.saved_tensors_hooks(*HOOKS[hook]):
        out, ref = fn(x, g)
    dy = _bf16(*out.shape, seed=2) if out.dim() else torch.tensor(1.5)
    ins = [x, g] if fn is _norm else [x]
    own = torch.autograd.grad(out, ins, dy.to(out.dtype))
    for a, b in zip(own, torch.autograd.grad(ref, ins, dy.float())):
        assert (a.double() - b.double()).norm() <= tol * b.double().norm()


@pytest.mark.parametrize("fn", [_norm, _swiglu, _ce])
def test_batched_gradients(no_gpu, fn):
    x, g = _bf16(6, 32).requires_grad_(True), 1 + 0.1 * _bf16(32, seed=1)
    out, ref = fn(x, g)
    dys = torch.stack([_bf16(*out.shape, seed=s).to(out.dtype) for s in (3, 4, 5)])
    (own,) = torch.autograd.grad(out, x, dys, is_grads_batched=True)
    (want,) = torch.autograd.grad(ref, x, dys.to(ref.dtype), is_grads_batched=True)
    assert own.shape == (3, 6, 32) and (own.double() - want.double()).norm() <= 4 * BF16_U * want.double().norm()


@pytest.mark.parametrize("hook", list(HOOKS))
def test_norm_with_residual_and_saved_tensors_from_hooks(no_gpu, hook):
    """Both results used: the gradients of x and of its norm meet."""
    x, g = _bf16(6, 32).requires_grad_(True), 1 + 0.1 * _bf16(32, seed=1)
    dres, dy = _bf16(6, 32, seed=2), _bf16(6, 32, seed=3)
    with torch.autograd.graph.saved_tensors_hooks(*HOOKS[hook]):
        res, y = ops.rmsnorm_residual(x, g, 1e-6)
    (own,) = torch.autograd.grad([res, y], x, [dres, dy])
    (want,) = torch.autograd.grad([x.float(), _norm(x, g)[1]], x, [dres.float(), dy.float()])
    assert (own.double() - want.double()).norm() <= 2 * BF16_U * want.double().norm()
