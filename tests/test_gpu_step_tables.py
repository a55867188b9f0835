"""The batched optimizer step at the edges of its layer tables (by shape: 84 layers
per Adam launch, 180 per decompression launch, 8 distinct shapes in either; with each
layer's own sizes: 8, or 70 and 112): bitwise compact_step of each layer, whose single-layer
tables the oracle tests cover; and the number of launches."""
import pytest

from gpu_util import dev, workspace

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
cp = pytest.importorskip("paper_2410_15352_amd")


def _layers(shapes, w_dtype, seed):
    g = torch.Generator(device=dev()).manual_seed(seed)
    out = []
    for i, (n, m, r) in enumerate(shapes):
        ldw = -(-m // 8) * 8
        W = (0.02 * torch.randn(n, ldw, generator=g, device=dev())).to(w_dtype)[:, :m]
        G, M = (torch.randn(r, m, generator=g, device=dev()) for _ in range(2))
        V = torch.rand(r, m, generator=g, device=dev())
        out.append(dict(W=W, G=G, M=M, V=V, seed=((i + 1) << 32) | 5, alpha=0.25 + 0.001 * i))
    return out


@pytest.mark.parametrize("count,distinct", [(1, 1), (84, 3), (85, 2), (168, 8), (169, 3), (180, 1), (181, 1), (9, 9),
                                            (17, 17), (100, 11), (70, 70), (71, 71), (84, 9), (112, 1), (113, 113), (155, 3), (8, 8)])
@pytest.mark.parametrize("w_dtype,proj", [(torch.bfloat16, "gaussian"), (torch.float32, "sparse-jl")])
def test_layer_tables(count, distinct, w_dtype, proj):
    # widths around the 128 x 128 tiles, ragged last columns; the shapes alternate
    kinds = [(96 + 17 * k, 120 + 5 * k, 8 + 3 * k) for k in range(distinct)]
    shapes = [kinds[i % distinct] for i in range(count)]
    a, b = _layers(shapes, w_dtype, count), _layers(shapes, w_dtype, count)
    cp.compact_step_batched(a, 3, 1e-3, proj=proj, ws=workspace(cp.step_batched_workspace_bytes(a)))
    for L in b:
        (n, m), r = L["W"].shape, L["G"].shape[0]
        cp.compact_step(L["W"], L["G"], L["M"], L["V"], L["seed"], 3, 1e-3, alpha=L["alpha"], proj=proj,
                        dtype="bf16",
                        ws=workspace(cp.step_workspace_bytes(n, m, r)))
    for x, y in zip(a, b):
        for k in "WMV":
            assert torch.equal(x[k], y[k]), (k, x["W"].shape)


@pytest.mark.parametrize("count,distinct,adam,dec", [(1, 1, 1, 1), (70, 70, 1, 1), (84, 8, 1, 1), (84, 9, 2, 1),
                                                     (112, 112, 2, 1), (168, 3, 2, 1), (168, 9, 3, 2),
                                                     (168, 168, 3, 2), (181, 2, 3, 2)])
def test_launches(count, distinct, adam, dec):
    """However many shapes the layers have, a launch takes at least 70 (Adam) and 112
    (decompression) of them, or what is left."""
    kinds = [(16 + 4 * k, 24, 4) for k in range(distinct)]
    layers = cp.prepare_layers(_layers([kinds[i % distinct] for i in range(count)], torch.bfloat16, 1))
    ws = workspace(cp.step_batched_workspace_bytes(layers))
    cp.compact_step_batched(layers, 3, 1e-3, ws=ws)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        cp.compact_step_batched(layers, 3, 1e-3, ws=ws)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    assert [sum(k in n for n in names) for k in ("k_adam_pt_batched", "k_dec_w4")] == [adam, dec], names
