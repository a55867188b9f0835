"""G^ of few tokens (one launch, 64 x 64 tiles, the waves splitting the tokens)
against float64, at the edges of its tiles and 32-token K tiles, for groups and in
accumulate mode; operands are column slices whose padding and neighbours hold NaN.
The bound is an fp32 sum over the tokens of exact products (acc_bound)."""
import numpy as np
import pytest

from gpu_util import U32, acc_bound, dev, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
cp = pytest.importorskip("paper_2410_15352_amd")


def _slice(rows, cols, seed, scale):
    g = torch.Generator(device=dev()).manual_seed(seed)
    buf = torch.full((rows, (cols + 7) // 8 * 8 + 16), float("nan"), dtype=torch.bfloat16, device=dev())
    v = buf[:, 8:8 + cols]
    v.copy_((scale * torch.randn(rows, cols, generator=g, device=dev())).to(torch.bfloat16))
    return v


@pytest.mark.parametrize("T,ms,rs", [
    (1, [8], [8]), (31, [64], [64]), (33, [65], [63]), (127, [1], [1]), (129, [200, 33], [72, 65]),
    (1000, [1376, 1376], [128, 128]), (1025, [520] * 7 + [513], [40] * 8), (2047, [1030], [342]),
    (300, [5461], [512]), (3001, [1376], [128]), (4096, [700], [330]), (1536, [2752], [500]),
])
def test_ghat_direct(T, ms, rs):
    n = max(64, *rs)
    dy, z = _slice(T, sum(ms), T, 0.01), _slice(T, sum(rs), T + 1, 2.0)
    ws = torch.empty(cp.bwd_group_workspace_bytes(T, n, ms, rs), dtype=torch.uint8, device=dev())
    G = [torch.empty(r, m, device=dev()) for r, m in zip(rs, ms)]
    cp.compact_bwd_group(dy, None, z, None, G, ms, rs, ws=ws)
    G2 = [torch.randn(r, m, device=dev()) for r, m in zip(rs, ms)]
    ref2 = [a + b for a, b in zip(G2, G)]
    cp.compact_bwd_group(dy, None, z, None, G2, ms, rs, ws=ws, accumulate=True)
    for a, b in zip(G2, ref2):
        assert torch.equal(a, b)
    D, Z, mo, ro = to_np(dy), to_np(z), 0, 0
    for g, m, r in zip(G, ms, rs):
        zt, d = Z[:, ro:ro + r].T, D[:, mo:mo + m]
        ref = zt @ d
        err = np.abs(g.cpu().numpy().astype(np.float64) - ref)
        assert (err <= acc_bound(T) * (np.abs(zt) @ np.abs(d)) + U32 * np.abs(ref)).all()
        mo, ro = mo + m, ro + r


@pytest.mark.parametrize("T,m,r,direct", [(1, 64, 16, True), (1000, 1376, 128, True), (64, 5461, 512, True),
                                          (4096, 2752, 256, True), (3000, 5461, 512, False), (16, 3000, 1500, False),
                                          (64, 5461, 2048, False), (1024, 3000, 1500, False), (8192, 1376, 128, False)])
def test_rule(T, m, r, direct):
    """The direct kernel where it was measured faster by more than a few percent."""
    dy, z = _slice(T, m, T, 0.01), _slice(T, r, T + 1, 2.0)
    ws = torch.empty(cp.bwd_workspace_bytes(T, r, m, r), dtype=torch.uint8, device=dev())
    G = torch.empty(r, m, device=dev())
    cp.compact_bwd(dy, None, z, None, G, ws=ws)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        cp.compact_bwd(dy, None, z, None, G, ws=ws)
        torch.cuda.synchronize()
    names = " ".join(e.name for e in prof.events())
    assert ("k_ghat_direct" in names) == direct and ("k_ghat_w4" in names) != direct, names


def test_precision():
    """The sums of a wave are folded every 4 K tiles.  With c = 2.4e-8, the rms rounding
    error of an fp32 addition, and two roundings per 16-deep MFMA step, 4096 tokens in four
    waves of 8 chunks give sqrt(8 + 4.5 + 2.25) c = 9.2e-8 (chunks, folds, waves); one chain
    per wave gives 8 c = 1.9e-7."""
    T, m, r = 4096, 1376, 128
    g = torch.Generator(device=dev()).manual_seed(7)
    dy, z = (torch.randn(T, c, generator=g, device=dev()).to(torch.bfloat16) for c in (m, r))
    G = torch.empty(r, m, device=dev())
    ws = torch.empty(cp.bwd_workspace_bytes(T, r, m, r), dtype=torch.uint8, device=dev())
    cp.compact_bwd(dy, None, z, None, G, ws=ws)
    ref = z.double().t().contiguous() @ dy.double()
    assert (G.double() - ref).norm() / ref.norm() <= 1.2 * 9.2e-8
