"""The fp32 MFMA GEMMs (32 x 32 tiles whose waves split K, 64 x 64, 128 x 32,
32 x 128 and 32 x 256 tiles): forward, backward and the update against float64 at
the edges of their tiles and of the 32-deep K steps.  Operands are column slices
whose row padding and neighbours hold NaN, outputs slices whose neighbours must
stay as they are.

Tolerance per element: an fp32 dot product of K terms in any order is within
8 sqrt(K) 2^-24 sum|terms| (gpu_util's bound), P adds one rounding and W' the one
of the subtraction."""
import numpy as np
import pytest

from oracle.pstream import projection
from gpu_util import U32, acc_bound, dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
cp = pytest.importorskip("paper_2410_15352_amd")


def _slice(a, ld=None):
    """The matrix as a slice, 4 columns in, of a NaN-filled wider buffer."""
    rows, cols = a.shape
    buf = torch.full((rows, ld or (cols + 3) // 4 * 4 + 8), float("nan"), device=dev())
    v = buf[:, 4:4 + cols]
    v.copy_(torch.from_numpy(a))
    return v


def _check(gpu, ref, absprod, K, extra=0.0):
    g = gpu.cpu().numpy().astype(np.float64)
    assert (np.abs(g - ref) <= (acc_bound(K) + extra) * absprod + U32 * np.abs(ref) + 1e-37).all()


def _neighbours_untouched(v):
    buf = v.as_strided((v.shape[0], v.stride(0)), (v.stride(0), 1), v.storage_offset() - 4)
    assert torch.isnan(buf[:, :4]).all() and torch.isnan(buf[:, 4 + v.shape[1]:]).all()


# (T, n, m, r): one WG per 32 x 32 tile; just past tile edges; 64 x 64 tiles with a
# small and a large G^; K just past, on and short of a K step
CASES = [(1, 1, 1, 1), (31, 33, 65, 5), (33, 64, 32, 32), (257, 127, 129, 63), (700, 96, 480, 40),
         (1025, 513, 1001, 65), (2047, 260, 1030, 130), (130, 1024, 3071, 512),
         (64, 700, 2001, 30)]  # the last two: the update's tiles of 384 and 256 columns


@pytest.mark.parametrize("proj", ["gaussian", "sparse-jl"])
@pytest.mark.parametrize("T,n,m,r", CASES)
def test_f32_layer(T, n, m, r, proj):
    g = np.random.default_rng(T + n)
    x, W = g.standard_normal((T, n), np.float32), np.float32(0.02) * g.standard_normal((n, m), np.float32)
    dy, G0 = g.standard_normal((T, m), np.float32), g.standard_normal((r, m), np.float32)
    seed = 77 << 32
    P = torch.empty(n, r, device=dev())
    cp.compact_projection(seed, P, proj)
    P = P.cpu().numpy().astype(np.float64) / np.sqrt(r if proj == "gaussian" else 8)
    xd, Wd, dyd = _slice(x), _slice(W), _slice(dy)
    y, z, dx = (_slice(np.zeros(s, np.float32)) for s in ((T, m), (T, r), (T, n)))
    cp.compact_fwd(xd, Wd, y, z, seed, proj=proj)
    G = torch.from_numpy(G0).to(dev())
    cp.compact_bwd_group(dyd, Wd, z, dx, [G], [m], [r], accumulate=True)
    x, W, dy = (a.astype(np.float64) for a in (x, W, dy))
    _check(y, x @ W, np.abs(x) @ np.abs(W), n)
    _check(z, x @ P, np.abs(x) @ np.abs(P), n, extra=2 * U32)
    _check(dx, dy @ W.T, np.abs(dy) @ np.abs(W.T), m)
    zh = z.cpu().numpy().astype(np.float64)
    ref = zh.T @ dy
    _check(G, G0 + ref, np.abs(zh.T) @ np.abs(dy) + np.abs(G0) + np.abs(ref), T, extra=U32)
    # the update on its own: M = 0, V = 0, beta = 0 give N = G / (|G| + eps)
    M, V = torch.zeros(r, m, device=dev()), torch.zeros(r, m, device=dev())
    ws = torch.empty(cp.step_workspace_bytes(n, m, r, cp.F32), dtype=torch.uint8, device=dev())
    Gh = G.cpu().numpy().astype(np.float64)
    cp.compact_step(Wd, G, M, V, seed, 1, 0.01, beta1=0.0, beta2=0.0, eps=1.0, proj=proj, ws=ws)
    N = Gh / (np.abs(Gh) + 1.0)
    U = 0.01 * (P @ N)
    _check(Wd, W - U, 0.01 * (np.abs(P) @ np.abs(N)) + np.abs(W), r, extra=8 * U32)
    for v in (y, z, dx, Wd):
        _neighbours_untouched(v)


def test_f32_wide_leading_dimension():
    """Rows of 16 MB and more take the plain kernel: the same bounds hold."""
    T, n, m, r = 5, 40, 36, 8
    g = np.random.default_rng(3)
    x, W = g.standard_normal((T, n), np.float32), g.standard_normal((n, m), np.float32)
    y, z = (_slice(np.zeros(s, np.float32)) for s in ((T, m), (T, r)))
    cp.compact_fwd(_slice(x, 1 << 22), _slice(W), y, z, 5)
    x, W = x.astype(np.float64), W.astype(np.float64)
    _check(y, x @ W, np.abs(x) @ np.abs(W), n)
    P = np.asarray(projection(5, n, r), np.float64)
    _check(z, x @ P, np.abs(x) @ np.abs(P), n, extra=4 * U32)


def test_f32_wide_leading_dimension_backward():
    """dL/dx and G^, overwritten and accumulated, by the plain kernel: dL/do in rows of 16 MB."""
    T, n, m, r = 5, 40, 36, 8
    g = np.random.default_rng(4)
    W, dy = g.standard_normal((n, m), np.float32), g.standard_normal((T, m), np.float32)
    z, G0 = g.standard_normal((T, r), np.float32), g.standard_normal((r, m), np.float32)
    dx, dyd, Wd, zd = _slice(np.zeros((T, n), np.float32)), _slice(dy, 1 << 22), _slice(W), _slice(z)
    G, G2 = torch.empty(r, m, device=dev()), torch.from_numpy(G0).to(dev())
    cp.compact_bwd(dyd, Wd, zd, dx, G)
    cp.compact_bwd_group(dyd, Wd, zd, None, [G2], [m], [r], accumulate=True)
    W, dy, zt = W.astype(np.float64), dy.astype(np.float64), z.T.astype(np.float64)
    _check(dx, dy @ W.T, np.abs(dy) @ np.abs(W.T), m)
    _check(G, zt @ dy, np.abs(zt) @ np.abs(dy), T)
    _check(G2, G0 + zt @ dy, np.abs(zt) @ np.abs(dy) + np.abs(G0), T, extra=U32)
    _neighbours_untouched(dx)


def test_f32_wide_update():
    """m of 2^22 and a ragged rest: N's rows are too long for the MFMA kernel's offsets."""
    n, m, r, seed = 3, (1 << 22) + 5, 2, 9 << 32
    W = _slice(0.02 * np.random.default_rng(5).standard_normal((n, m)).astype(np.float32))
    W0 = W.clone().double()
    gen = torch.Generator(device=dev()).manual_seed(6)
    G = torch.randn(r, m, generator=gen, device=dev())
    M, V = torch.zeros(r, m, device=dev()), torch.zeros(r, m, device=dev())
    ws = torch.empty(cp.step_workspace_bytes(n, m, r, cp.F32), dtype=torch.uint8, device=dev())
    cp.compact_step(W, G, M, V, seed, 1, 0.01, beta1=0.0, beta2=0.0, eps=1.0, ws=ws)
    P = torch.empty(n, r, device=dev())
    cp.compact_projection(seed, P)
    P, N = P.double() / r ** 0.5, G.double() / (G.double().abs() + 1.0)
    U, mag = 0.01 * (P @ N), 0.01 * (P.abs() @ N.abs())
    assert bool(((W.double() - (W0 - U)).abs() <= (acc_bound(r) + 8 * U32) * mag + U32 * (W0.abs() + U.abs())).all())
    _neighbours_untouched(W)
