"""Which calls the block kernels take: the rules that do not ask for a GPU."""
import pytest

torch = pytest.importorskip("torch")
ops = pytest.importorskip("paper_2410_15352_amd._block_ops")
blk = pytest.importorskip("paper_2410_15352_amd.block")


@pytest.mark.parametrize("width,gains,takes", [(64, 64, True), (64, 128, False), (128, 64, False), (64, 1, False),
                                               (12, 12, False), (4096, 4096, True), (4104, 4104, False)])
def test_norm_takes_one_gain_per_element(monkeypatch, width, gains, takes):
    """The kernel reads `width` gains: any other number must not reach it."""
    monkeypatch.setattr(ops, "_kernel_tensors", lambda *t: True)
    x, g = torch.empty(3, width, dtype=torch.bfloat16), torch.ones(gains, dtype=torch.bfloat16)
    assert ops.norm_usable(x, g) == takes
    assert not ops.norm_usable(x, g.expand(2, gains))


def test_norm_of_another_width_is_refused():
    with pytest.raises(RuntimeError):
        blk.RMSNorm(64)(torch.randn(3, 128).to(torch.bfloat16))


def _block_on_cpu():
    torch.manual_seed(0)
    return blk.LlamaBlock(64, 1, 64, rank=None, device="cpu"), torch.randn(2, 8, 64).to(torch.bfloat16)


def test_block_runs_its_norms_as_modules():
    """Hooks on a block's norms run, and what a hook returns counts."""
    b, x = _block_on_cpu()
    calls, x = [], x.requires_grad_(True)
    for norm in (b.norm1, b.norm2):
        norm.register_forward_pre_hook(lambda m, a: calls.append("pre"))
        norm.register_forward_hook(lambda m, a, out: calls.append("forward"))
        norm.register_full_backward_hook(lambda m, gi, go: calls.append("backward"))
    b(x).float().sum().backward()
    assert calls.count("pre") == calls.count("forward") == calls.count("backward") == 2
    b, x = _block_on_cpu()
    y = b(x)
    b.norm2.register_forward_hook(lambda m, a, out: 0 * out)  # no MLP
    assert not torch.equal(b(x), y)
    b.norm2._forward_hooks.clear()
    assert torch.equal(b(x), y)


@pytest.mark.parametrize("make", [torch.nn.Identity, lambda: torch.nn.LayerNorm(64, dtype=torch.bfloat16),
                                  lambda: type("Sub", (blk.RMSNorm,), {"forward": lambda self, x: -x})(64, device="cpu")])
def test_block_takes_replaced_norms(make):
    b, x = _block_on_cpu()
    b.norm1, b.norm2 = make(), make()
    assert torch.isfinite(b(x)).all()


def test_fused_norms_only_where_the_module_is_plain(monkeypatch):
    """The kernels that join a norm with its residual take a norm without hooks."""
    fused = []
    monkeypatch.setattr(ops, "norm_usable", lambda *t: True)
    monkeypatch.setattr(ops, "rmsnorm", lambda x, g, eps: blk._RMSNormFn.apply(x, g, eps))
    monkeypatch.setattr(ops, "rmsnorm_residual", lambda x, g, eps: (fused.append(1), (x, blk._RMSNormFn.apply(x, g, eps)))[1])
    monkeypatch.setattr(ops, "add_rmsnorm", lambda x, o, g, eps: (fused.append(2), (x + o, blk._RMSNormFn.apply(x + o, g, eps)))[1])

    def routes(change, undo=lambda b: None):
        b, x = _block_on_cpu()
        change(b)
        fused.clear()
        try:
            b(x)
        finally:
            undo(b)
        return list(fused)

    hook = lambda *a: None
    handle = []
    assert routes(lambda b: None) == [1, 2]
    assert routes(lambda b: b.norm1.register_forward_hook(hook)) == [2]
    assert routes(lambda b: b.norm2.register_forward_pre_hook(hook)) == [1]
    assert routes(lambda b: b.norm2.register_full_backward_hook(hook)) == [1]
    assert routes(lambda b: b.norm1.register_full_backward_pre_hook(hook)) == [2]
    assert routes(lambda b: setattr(b.norm1, "forward", lambda x: x)) == [2]
    assert routes(lambda b: handle.append(torch.nn.modules.module.register_module_forward_hook(hook)),
                  lambda b: handle.pop().remove()) == []
    monkeypatch.setattr(blk.RMSNorm, "forward", lambda self, x: x)
    assert routes(lambda b: None) == []


@pytest.mark.parametrize("tokens,n,m,takes", [(4096, 1024, 1024, False), (8192, 1024, 1024, True), (8192, 512, 512, True),
                                              (4096, 2048, 2048, False), (8192, 2048, 2048, False), (16384, 2048, 2048, True),
                                              (8192, 4096, 8, False), (8192, 8, 524288, False), (65536, 16, 8, False),
                                              (4096, 64, 8192, True), (1 << 20, 1024, 1028, False)])
def test_weight_gradients_that_split_k_takes(tokens, n, m, takes):
    """Where the measurements beside the rule have it the faster one."""
    assert ops.dense_split(tokens, n, m) == takes


@pytest.mark.parametrize("rows,takes", [((1 << 32) - 256, True), ((1 << 32) - 255, False), (1 << 33, False)])
def test_swiglu_launches_have_less_than_2_32_threads(monkeypatch, rows, takes):
    """One thread per 8 elements of the result: more than a launch can have stay torch's."""
    seen = []
    monkeypatch.setattr(ops, "_kernel_tensors", lambda *t: True)
    monkeypatch.setattr(ops._SwigluFn, "apply", lambda gu: seen.append(True))
    monkeypatch.setattr(ops, "_swiglu_torch", lambda gu, f: seen.append(False))
    ops.swiglu(torch.empty(1, 16, dtype=torch.bfloat16).expand(rows, 16), 8)
    assert seen == [takes]


def test_no_size_is_compared_under_a_tracer(recwarn):
    """A traced block has no more of the sizes' comparisons in it than the shapes it unpacks."""
    b, x = _block_on_cpu()
    y = b(x)
    t = torch.jit.trace(b, (x,))
    assert torch.equal(t(x), y)
    assert not [w for w in recwarn if "_block_ops" in str(w.filename) or "norm_usable" in str(w.message)]


def test_block_compiles_in_one_graph():
    b, x = _block_on_cpu()
    for rows in (2, 3):  # another size: guards and recompilation
        z = torch.compile(b, backend="eager", fullgraph=True, dynamic=True)(x[:1].expand(rows, 8, 64))
        assert torch.equal(z, b(x[:1].expand(rows, 8, 64)))
