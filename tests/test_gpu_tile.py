"""The tile GEMMs (one workgroup per 256 x 128, 128 x 128, 64 x 128 or 64 x 64
output tile), which take the bf16 forward and dL/dx where the persistent kernel
would leave CUs without a tile.  Row t of y, z and dL/dx depends on row t of the
input alone and every bf16 GEMM sums K in the same order, so the first T rows
computed alone are bitwise the first T rows of a long call (the persistent
kernel); the long call itself is checked against the oracle elsewhere.  The
shapes put T, the output widths and K on, one past and one short of the tile
edges; operands are column slices whose padding and neighbours hold NaN."""
import numpy as np
import pytest

from gpu_util import assert_elementwise, dev, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
cp = pytest.importorskip("paper_2410_15352_amd")


def _slice(rows, cols, g, scale):
    """A (rows, cols) view inside a NaN-filled wider buffer."""
    buf = torch.full((rows, (cols + 7) // 8 * 8 + 16), float("nan"), dtype=torch.bfloat16, device=dev())
    v = buf[:, 8:8 + cols]
    v.copy_((scale * torch.randn(rows, cols, generator=g, device=dev())).to(torch.bfloat16))
    return v


def _bits(t):
    return t.contiguous().view(torch.int16)


# (T, n, m, r): K = n forward, K = m backward
CASES = [
    (1, 512, 256, 32), (63, 1024, 257, 31), (65, 505, 512, 129),       # 64 x 64
    (257, 392, 1376, 64), (1000, 512, 1381, 128),                      # 64 x 64, 64 x 128
    (1025, 509, 1536, 384), (2047, 2736, 1023, 342),                   # 64 x 128
    (4097, 1021, 1000, 128), (3333, 1461, 701, 200),                   # 128 x 128
    (8191, 3072, 1030, 250), (8192, 1024, 3075, 128),                  # 256 x 128
    (200, 40, 24, 8), (129, 265, 129, 65), (77, 8, 5472, 4),           # K below the persistent kernel's least
]
LONG = 36864


@pytest.mark.parametrize("T,n,m,r", CASES)
def test_tile_rows_equal_long_call(T, n, m, r):
    g = torch.Generator(device=dev()).manual_seed(T * 7 + n)
    long = max(LONG, T)
    x, W = _slice(long, n, g, 1.0), _slice(n, m, g, 0.02)
    dy = _slice(long, m, g, 0.01)
    fws = torch.empty(cp.fwd_workspace_bytes(n, m, r), dtype=torch.uint8, device=dev())
    bws = torch.empty(cp.bwd_workspace_bytes(long, n, m, r), dtype=torch.uint8, device=dev())
    out = []
    for rows in (long, T):
        y, z, dx = (_slice(rows, c, g, 0.0) for c in (m, r, n))
        cp.compact_fwd(x[:rows], W, y, z, 9 << 32, ws=fws)
        cp.compact_bwd(dy[:rows], W, None, dx, None, ws=bws)
        out.append((y, z, dx))
    torch.cuda.synchronize()
    for a, b in zip(*out):
        assert torch.equal(_bits(a[:T]), _bits(b))
    # and without a workspace (P generated in LDS, W read as it is)
    y, z, dx = (_slice(T, c, g, 0.0) for c in (m, r, n))
    cp.compact_fwd(x[:T], W, y, z, 9 << 32)
    cp.compact_bwd(dy[:T], W, None, dx, None)
    torch.cuda.synchronize()
    for a, b in zip(out[1], (y, z, dx)):
        assert torch.equal(_bits(a), _bits(b))
    # a sample of rows against float64
    rows = np.unique(np.linspace(0, T - 1, 24).astype(int))
    Wn = to_np(W)
    for gpu, op, B, K in ((out[1][0], x, Wn, n), (out[1][2], dy, Wn.T, m)):
        A = to_np(op[torch.as_tensor(rows, device=dev())])
        assert_elementwise(to_np(gpu[torch.as_tensor(rows, device=dev())]), A @ B, np.abs(A) @ np.abs(B), K)
