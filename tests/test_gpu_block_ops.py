"""The block kernels (RMSNorm with its residual, SwiGLU, cross-entropy) against
float64, at the edges of their rows and 16-byte chunks, and next to the torch
expressions they stand in for.

Tolerances: a bf16 result is within one rounding (2^-8 of the value, with the fp32
arithmetic's few 2^-22 on top); sums over rows (dg) add sqrt(rows) fp32 roundings of
the terms; the loss is an fp32 value of fp32 exponentials (2^-20 of the logits'
range)."""
import pytest

from gpu_util import BF16_U, LAM, U32, dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ops = pytest.importorskip("paper_2410_15352_amd._block_ops")
blk = pytest.importorskip("paper_2410_15352_amd.block")


def _rand(*shape, scale=1.0, seed=0):
    g = torch.Generator(device=dev()).manual_seed(seed + sum(shape))
    return (scale * torch.randn(*shape, generator=g, device=dev())).to(torch.bfloat16)


def _close(a, ref, mag=None, extra=0.0):
    tol = (BF16_U + 8 * U32) * ref.abs() + extra * (ref.abs() if mag is None else mag) + 1e-30
    assert a.shape == ref.shape and bool(((a.double() - ref).abs() <= tol).all())


@pytest.mark.parametrize("rows,d", [(1, 8), (5, 512), (3, 520), (130, 1024), (4097, 1032), (33, 2736), (17, 4096),
                                    (9, 4104), (7, 12)])  # the last two take the torch expressions
@pytest.mark.parametrize("add", [False, True])
def test_rmsnorm(rows, d, add):
    norm = blk.RMSNorm(d)
    with torch.no_grad():
        norm.weight.copy_(1 + 0.1 * _rand(d))
    x, o = (_rand(rows, d, seed=s).requires_grad_(True) for s in (1, 2))
    dh, dr = _rand(rows, d, seed=3), _rand(rows, d, seed=4)
    assert ops.norm_usable(x, norm.weight) == (d % 8 == 0 and d <= 4096)
    s, h = norm.add(x, o) if add else norm.with_residual(x)
    torch.autograd.backward([s, h], [dr, dh])
    # float64, from the bf16 sum the norm sees
    xs = (x + o if add else x).detach()
    assert torch.equal(s, xs)
    X, g = xs.double(), norm.weight.detach().double()
    rstd = torch.rsqrt(X.square().mean(-1, keepdim=True) + norm.eps)
    _close(h, X * rstd * g, extra=8 * U32)
    gd, xh = dh.double() * g, X * rstd
    mean = (gd * xh).mean(-1, keepdim=True)
    dx = rstd * (gd - xh * mean) + dr.double()
    mag = rstd * (gd.abs() + xh.abs() * (gd * xh).abs().mean(-1, keepdim=True)) + dr.double().abs()
    # (the torch expressions round the norm's gradient before the residual's is added)
    _close(x.grad, dx, mag, extra=16 * U32 if ops.norm_usable(x, norm.weight) else BF16_U)
    assert not add or torch.equal(o.grad, x.grad)
    t = dh.double() * xh
    _close(norm.weight.grad, t.sum(0), t.abs().sum(0), extra=LAM * U32 * (8 + rows ** 0.5))
    y = norm(xs)
    assert torch.equal(y, h)
    # deterministic
    g1 = norm.weight.grad.clone()
    norm.weight.grad = None
    s2, h2 = norm.add(x, o) if add else norm.with_residual(x)
    torch.autograd.backward([s2, h2], [dr, dh])
    assert torch.equal(g1, norm.weight.grad)


def test_rmsnorm_gradient_routes():
    """x without a gradient, only one of the results used, a recorded backward."""
    norm, x = blk.RMSNorm(64), _rand(10, 64)
    _, h = norm.with_residual(x)
    h.sum().backward()
    assert norm.weight.grad is not None and x.grad is None
    x.requires_grad_(True)
    s, _ = norm.with_residual(x)
    s.sum().backward()
    assert torch.equal(x.grad, torch.ones_like(x))
    x.grad, w = None, _rand(10, 64, seed=5)
    (gx,) = torch.autograd.grad(norm(x), x, w, create_graph=True)
    gx.backward(w)
    # float64: the second derivative goes through 1 / rms too
    X = x.detach().double().requires_grad_(True)
    Y = X * torch.rsqrt(X.square().mean(-1, keepdim=True) + norm.eps) * norm.weight.detach().double()
    (GX,) = torch.autograd.grad(Y, X, w.double(), create_graph=True)
    GX.backward(w.double())
    assert (x.grad.double() - X.grad).norm() <= 4 * BF16_U * X.grad.norm()


@pytest.mark.parametrize("rows,f", [(1, 8), (3, 24), (257, 1376), (1000, 2736), (5, 12)])  # the last one: torch
def test_swiglu(rows, f):
    gu = _rand(rows, 2 * f, scale=2.0).requires_grad_(True)
    with torch.no_grad():
        gu[0, :4] = torch.tensor([0.0, 88.0, -100.0, float("inf")])
    da = _rand(rows, f, seed=9)
    act = ops.swiglu(gu, f)
    act.backward(da)
    g, u, d = gu.detach()[:, :f].double(), gu.detach()[:, f:].double(), da.double()
    s, sg = (g / (1 + torch.exp(-g))), 1 / (1 + torch.exp(-g))
    ok = torch.isfinite(g)
    _close(torch.where(ok, act, 0), torch.where(ok, s * u, 0), extra=2 * BF16_U)
    _close(torch.where(ok, gu.grad[:, f:], 0), torch.where(ok, d * s, 0), extra=2 * BF16_U)
    ref, mag = d * u * sg * (1 + g * (1 - sg)), (d * u * sg).abs() * (1 + (g * (1 - sg)).abs())
    _close(torch.where(ok, gu.grad[:, :f], 0), torch.where(ok, ref, 0), torch.where(ok, mag, 0), extra=2 * BF16_U)
    if f % 8 == 0:  # bitwise what the separate operations give, infinities and NaN included
        assert torch.equal(act.view(torch.int16), (torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]).view(torch.int16))


@pytest.mark.parametrize("rows,V", [(1, 1), (2, 7), (3, 1003), (64, 1000), (130, 32000), (1025, 2049), (5, 4104), (5, 12301)])
def test_cross_entropy(rows, V):
    x = _rand(rows, V, scale=3.0).requires_grad_(True)
    t = torch.randint(V, (rows,), device=dev())
    if rows > 2:
        t[1] = ops.IGNORE
        with torch.no_grad():
            x[0, 0], x[2, V // 2] = float("-inf"), -3.3895e38  # bf16's lowest value
        t[0], t[2] = V - 1, 0
    loss = ops.cross_entropy(x, t)
    assert loss.dtype == torch.float32 and loss.dim() == 0
    (2.0 * loss).backward()
    X = x.detach().double().requires_grad_(True)
    ref = torch.nn.functional.cross_entropy(X, t)
    (2.0 * ref).backward()
    assert abs(loss.item() - ref.item()) <= 2.0 ** -18 * max(1.0, abs(ref.item()))
    _close(x.grad, X.grad, 2.0 * torch.softmax(X.detach(), -1) / max(rows - 1, 1), extra=2.0 ** -17)


def test_cross_entropy_not_finite_and_empty_mean():
    t = torch.tensor([0, 1, 2], device=dev())
    for bad in (float("nan"), float("inf")):
        x = _rand(3, 40)
        x[1, 5] = bad
        assert torch.isnan(ops.cross_entropy(x, t)) and torch.isnan(torch.nn.functional.cross_entropy(x.float(), t))
    x = _rand(3, 40)
    x[1] = float("-inf")
    assert torch.isnan(ops.cross_entropy(x, t))
    x = _rand(3, 40).requires_grad_(True)
    loss = ops.cross_entropy(x, torch.full_like(t, ops.IGNORE))
    loss.backward()
    assert torch.isnan(loss) and torch.equal(x.grad, torch.zeros_like(x))
    x = _rand(3, 40).requires_grad_(True)
    (g,) = torch.autograd.grad(ops.cross_entropy(x, t), x, create_graph=True)
    (g1,) = torch.autograd.grad(ops.cross_entropy(x, t), x)
    _close(g.detach(), g1.double(), extra=BF16_U)
    g.float().square().sum().backward()
    X = x.detach().double().requires_grad_(True)
    (G,) = torch.autograd.grad(torch.nn.functional.cross_entropy(X, t), X, create_graph=True)
    G.square().sum().backward()
    assert (x.grad.double() - X.grad).norm() <= 4 * BF16_U * X.grad.norm()


@pytest.mark.parametrize("b,l,heads,hd", [(1, 1, 1, 8), (2, 33, 3, 24), (3, 65, 4, 64), (2, 9, 3, 4)])
def test_split_qkv(b, l, heads, hd):
    qkv = _rand(b, l, 3, heads, hd).requires_grad_(True)
    parts = ops.split_qkv(qkv)
    for i, t in enumerate(parts):
        assert torch.equal(t, qkv.detach()[:, :, i].transpose(1, 2))
    dense = [_rand(b, l, heads, hd, seed=i).transpose(1, 2) for i in (1, 2, 3)]  # as attention gives them
    other = [g.contiguous() for g in dense]                                      # another layout: the same result
    for grads in (dense, other):
        qkv.grad = None
        torch.autograd.backward(ops.split_qkv(qkv), grads)
        assert torch.equal(qkv.grad, torch.stack([g.transpose(1, 2) for g in dense], 2))
    qkv.grad = None
    ops.split_qkv(qkv)[1].backward(dense[1])  # only k is used
    assert torch.equal(qkv.grad[:, :, 1], dense[1].transpose(1, 2)) and not qkv.grad[:, :, 0::2].any()


@pytest.mark.parametrize("rows,n,m", [(4096, 64, 72), (4097, 2048, 64), (5632, 512, 520), (6003, 1024, 1024),
                                      (8705, 2048, 2048), (5700, 8192, 256), (4095, 64, 64), (5631, 512, 512),
                                      (8703, 2048, 2048), (9000, 2048, 2056), (9000, 56, 64), (9000, 64, 8200),
                                      (6000, 68, 64)])  # the last seven: the library
def test_dense_weight_gradient(rows, n, m):
    x, W, dy = _rand(rows, n).requires_grad_(True), _rand(n, m, seed=1), _rand(rows, m, seed=2)
    W = torch.nn.Parameter(W)
    y = ops.dense(x, W)
    assert torch.equal(y, x.detach() @ W.detach())
    own = (rows, n, m) in [(4096, 64, 72), (4097, 2048, 64), (5632, 512, 520), (6003, 1024, 1024), (8705, 2048, 2048),
                           (5700, 8192, 256)]
    assert ops.dense_split(rows, n, m) == own
    assert (type(y.grad_fn).__name__ == "_DenseFnBackward") == own
    y.backward(dy)
    assert torch.equal(x.grad, dy @ W.detach().t())
    # fp32 sums over the rows: LAM sqrt(rows) roundings of the terms' sum, then one to bf16
    X, D = x.detach().double(), dy.double()
    _close(W.grad, X.t().contiguous() @ D, X.abs().t().contiguous() @ D.abs(), extra=LAM * U32 * rows ** 0.5)
    W.grad = None
    ops.dense(x.detach(), W).backward(dy[:1].expand(rows, m))  # a gradient that is not dense: the library
    _close(W.grad, X.sum(0)[:, None] * D[:1], X.abs().sum(0)[:, None] * D[:1].abs(), extra=LAM * U32 * rows ** 0.5)


def test_routes_that_stay_torch():
    """A norm of another width is refused as before, autocast decides the types."""
    norm, x = blk.RMSNorm(64), _rand(10, 128)
    for call in (norm, norm.with_residual, lambda v: norm.add(v, v)):
        with pytest.raises(RuntimeError):
            call(x)
    W = _rand(64, 64, seed=1)
    x = _rand(4096, 64).requires_grad_(True)
    with torch.autocast("cuda", dtype=torch.float16):
        assert not ops.usable(x) and ops.dense(x, W).dtype == torch.float16


@pytest.mark.parametrize("bad", [-1, 40, 1 << 40, None])
def test_cross_entropy_checks_its_targets(monkeypatch, bad):
    """The flag that the forward's assertion looks at (the assertion itself ends the
    process, so it is left out here); behind it the loss and the row's gradient are NaN."""
    seen = []
    monkeypatch.setattr(torch, "_assert_async", lambda t, msg: seen.append(t))
    t = torch.arange(1500, device=dev()) % 40
    t[7] = ops.IGNORE
    if bad is not None:
        t[1200] = bad
    z = _rand(1500, 40).requires_grad_(True)
    loss = ops.cross_entropy(z, t)
    loss.backward()
    assert [v.item() for v in seen] == [1.0 if bad is None else 0.0]
    nan = torch.isnan(z.grad).any(1)
    assert bool(torch.isnan(loss)) == (bad is not None) and nan[1200] == (bad is not None) and nan.sum() <= 1


@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
def test_cross_entropy_ignored_row_that_is_not_finite(value):
    """NaN where torch's gradient is NaN, zero elsewhere in the row, the other rows as usual."""
    t = torch.tensor([3, ops.IGNORE, 5, ops.IGNORE], device=dev())
    x = _rand(4, 41)
    x[1, 7] = value
    x[3] = value if value == float("-inf") else x[3]
    x.requires_grad_(True)
    (g,) = torch.autograd.grad(ops.cross_entropy(x, t), x)
    (w,) = torch.autograd.grad(torch.nn.functional.cross_entropy(x.float(), t), x)
    assert torch.equal(torch.isnan(g), torch.isnan(w)) and not torch.nan_to_num(g)[1::2].any()
    _close(g[0::2], w[0::2].double(), extra=2 * BF16_U)


def _calls():
    norm, x, gu, z = blk.RMSNorm(64), _rand(10, 64), _rand(10, 48, scale=2.0), _rand(10, 40)
    t = torch.arange(10, device=dev())
    return [(norm, x), (lambda v: ops.swiglu(v, 24), gu), (lambda v: ops.cross_entropy(v, t), z)]


@pytest.mark.parametrize("i", range(3))
def test_saved_tensors_from_hooks_and_batched_gradients(i):
    """What a hook gives back in another type or layout, and batched gradients, take the
    torch expressions; offloading to the host and back keeps the kernels, bit for bit."""
    fn, x = _calls()[i]
    x.requires_grad_(True)
    out = fn(x)
    dy = (0.5 + torch.rand_like(out.float())).to(out.dtype)
    (want,) = torch.autograd.grad(out, x, dy, retain_graph=True)
    with torch.autograd.graph.save_on_cpu():
        off = fn(x)
    assert torch.equal(torch.autograd.grad(off, x, dy)[0], want)
    for pack in (lambda v: v.float() if v.is_floating_point() else v, lambda v: v.t().contiguous().t() if v.dim() == 2 else v):
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda v: v):
            y = fn(x)
        g = torch.autograd.grad(y, x, dy)[0].double()
        assert (g - want.double()).norm() <= 8 * BF16_U * want.double().norm()
    (b,) = torch.autograd.grad(out, x, torch.stack([dy, 2 * dy]), is_grads_batched=True)
    assert (b[0].double() - want.double()).norm() <= 8 * BF16_U * want.double().norm()
    assert (b[1].double() - 2 * want.double()).norm() <= 16 * BF16_U * want.double().norm()


def test_under_graph_capture():
    """Norm, SwiGLU, the split-K weight gradient and the cross-entropy with its check,
    forward and backward, recorded once and replayed on new inputs beside eager work."""
    T = 5700
    norm, W = blk.RMSNorm(128), torch.nn.Parameter(_rand(128, 80, scale=0.1))
    x, t = _rand(T, 128).requires_grad_(True), torch.randint(40, (T,), device=dev())

    def step():
        loss = ops.cross_entropy(ops.swiglu(ops.dense(norm(x), W), 40), t)
        return [loss.detach(), *torch.autograd.grad(loss, [x, norm.weight, W])]

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(2):
            step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = step()
    for i in range(4):
        with torch.no_grad():
            x.copy_(_rand(T, 128, seed=10 + i))
            t.copy_(torch.randint(40, (T,), device=dev()))
            W.copy_(_rand(128, 80, scale=0.1, seed=20 + i))
        want = step()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a, b)
