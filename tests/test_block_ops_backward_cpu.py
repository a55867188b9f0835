"""Which backwards of the block kernels' autograd functions may hand raw pointers to
the library, and the second derivatives.  On the CPU, with the library's calls replaced:
the forwards' kernels by torch or by nothing, the backwards' by a failure.  Saved tensors that come back from
a hook in another type, layout or place, and batched gradients, must take the torch
expressions, whose values are compared with autograd through the plain operations."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
ops = pytest.importorskip("paper_2410_15352_amd._block_ops")

BF16_U = 2.0 ** -8  # one bf16 rounding, relative


def _at(ptr, rows, d, dtype, word):
    return torch.frombuffer((word * (rows * d)).from_address(ptr), dtype=dtype).view(rows, d)


def _fake_call(name, *args):
    """The norm's forward; nothing for the others, whose torch backwards need no result of theirs."""
    if name == "compact_block_rmsnorm_fwd":
        a = args[0]._obj
        mat = lambda p: _at(p, a.rows, a.d, torch.bfloat16, ctypes.c_uint16)
        x = mat(a.x)
        if a.add:
            x = mat(a.sum).copy_(x + mat(a.add))
        rstd = _at(a.rstd, a.rows, 1, torch.float32, ctypes.c_float)
        rstd.copy_(torch.rsqrt(x.double().square().mean(-1, keepdim=True) + a.eps))
        mat(a.y).copy_(x.float() * rstd * _at(a.g, 1, a.d, torch.bfloat16, ctypes.c_uint16).float())
        return 0
    assert name.endswith("_fwd"), f"{name} was given raw pointers"
    return 0


@pytest.fixture
def no_gpu(monkeypatch):
    monkeypatch.setattr(ops, "_call", _fake_call)
    monkeypatch.setattr(ops, "_stream", lambda t: 0)
    monkeypatch.setattr(torch, "_assert_async", lambda t, msg: None)


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


def test_wrapped_tensors_are_not_plain():
    """Tensors without a storage of their own are known by themselves, whatever the thread."""
    seen = []

    class Look(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x):
            return x * 1

        @staticmethod
        def backward(ctx, dy):
            seen.append(ops._plain(dy))
            return dy

    x = torch.randn(3, requires_grad=True)
    torch.autograd.grad(Look.apply(x), x, torch.randn(2, 3), is_grads_batched=True)
    torch.func.vmap(lambda v: (seen.append(ops._plain(v)), v)[1])(torch.randn(2, 3))
    torch.func.grad(lambda v: (seen.append(ops._plain(v)), v.sum())[1])(torch.randn(3))
    assert seen == [False] * 3 and ops._plain(x) and ops._plain(torch.nn.Parameter(x.detach()))


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


def _second(fn, ins, dys, weights):
    """The gradient, over all inputs, of the weighted sum of the first gradients."""
    first = torch.autograd.grad(fn(*ins), ins, dys, create_graph=True)
    return torch.autograd.grad(sum((w * f.to(w.dtype)).sum() for w, f in zip(weights, first)), ins, allow_unused=True)


def _double(fn, ins, dys, weights):
    return _second(fn, [t.detach().double().requires_grad_(True) for t in ins], [d.double() for d in dys],
                   [w.double() for w in weights])


def _close(got, want, tol):
    for a, b in zip(got, want):
        assert (a.double() - b).norm() <= tol * b.norm()


def _norm64(x, g, eps=1e-6):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


def test_second_derivative_of_the_norm():
    """A recorded backward: 1 / rms depends on x as well.  In fp32, where the module
    takes its torch expressions."""
    blk = pytest.importorskip("paper_2410_15352_amd.block")
    norm = blk.RMSNorm(32, device="cpu").float()
    with torch.no_grad():
        norm.weight.copy_(1 + 0.1 * _bf16(32, seed=1).float())
    x, dy = _bf16(6, 32).float().requires_grad_(True), [_bf16(6, 32, seed=2).float()]
    w = [_bf16(6, 32, seed=3).float(), _bf16(32, seed=4).float()]
    got = _second(lambda x, g: [blk._RMSNormFn.apply(x, g, norm.eps)], [x, norm.weight], dy, w)
    _close(got, _double(lambda x, g: [_norm64(x, g)], [x, norm.weight], dy, w), 32 * 2.0 ** -24)


def test_second_derivatives_of_the_block_kernels(no_gpu):
    """The same through the functions whose forward is a kernel: bf16 results, so some
    bf16 roundings of terms that do not cancel."""
    x, o = (_bf16(6, 32, seed=s).requires_grad_(True) for s in (0, 1))
    g = (1 + 0.1 * _bf16(32, seed=2)).requires_grad_(True)
    dres, dy, w = _bf16(6, 32, seed=3), _bf16(6, 32, seed=4), [_bf16(6, 32, seed=5), _bf16(32, seed=6)]
    got = _second(lambda x, g: list(ops.rmsnorm_residual(x, g, 1e-6)), [x, g], [dres, dy], w)
    _close(got, _double(lambda x, g: [x * 1, _norm64(x, g)], [x, g], [dres, dy], w), 4 * BF16_U)
    w = [w[0], _bf16(6, 32, seed=7), w[1]]
    got = _second(lambda x, o, g: list(ops.add_rmsnorm(x, o, g, 1e-6)), [x, o, g], [dres, dy], w)
    s = (x + o).detach().double()  # the norm sees the rounded sum
    fix = lambda x, o: x + o + (s - (x + o).detach())
    _close(got, _double(lambda x, o, g: [fix(x, o), _norm64(fix(x, o), g)], [x, o, g], [dres, dy], w), 4 * BF16_U)
    gu, z, t = _bf16(6, 48).requires_grad_(True), _bf16(6, 32).requires_grad_(True), torch.arange(6)
    _close(_second(lambda v: [ops._SwigluFn.apply(v)], [gu], [_bf16(6, 24, seed=8)], [_bf16(6, 48, seed=9)]),
           _double(lambda v: [torch.nn.functional.silu(v[:, :24]) * v[:, 24:]], [gu], [_bf16(6, 24, seed=8)],
                   [_bf16(6, 48, seed=9)]), 4 * BF16_U)
    _close(_second(lambda v: [ops._CrossEntropyFn.apply(v, t)], [z], [torch.tensor(2.0)], [_bf16(6, 32, seed=9)]),
           _double(lambda v: [torch.nn.functional.cross_entropy(v, t)], [z], [torch.tensor(2.0)],
                   [_bf16(6, 32, seed=9)]), 4 * BF16_U)


def test_cross_entropy_asserts_that_its_targets_are_classes(no_gpu, monkeypatch):
    """Every forward checks its targets on the device, without waiting for it."""
    seen = []
    monkeypatch.setattr(torch, "_assert_async", lambda t, msg: seen.append((t.numel(), msg)))
    ops._CrossEntropyFn.apply(_bf16(3, 32), torch.tensor([0, 32, 1]))
    assert [n for n, _ in seen] == [1]
