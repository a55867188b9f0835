"""The tile GEMMs (one workgroup per 256 x 128, 128 x 128, 64 x 128 or 64 x 64
output tile), which take the bf16 forward and dL/dx where the persistent kernel
would leave CUs without a tile.  Row t of y, z and dL/dx depends on row t of the
input alone and every bf16 GEMM sums K in the same order, so the first T rows
computed alone are bitwise the first T rows of a call long enough for another
kernel: the persistent one (the eight-wave one for K < 320), where there is a length
from which it is the faster one; the long call itself is checked against the oracle
elsewhere.  The forward without a workspace is a third kernel (P generated in LDS);
dL/dx without one reads W as it lies, by a tile kernel again.  A sample of rows is
compared with float64.  Which kernel takes each side is written beside the cases
(tests/test_tile_rules.py checks it on the CPU).  The shapes put T, the output widths
and K on, one past and one short of the tile edges; operands are column slices whose
padding and neighbours hold NaN."""
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


# (T, n, m, r): K = n forward, K = m backward; the kernels of the forward and of dL/dx,
# and the rows of the long call, 0 in the place of a kernel that no length brings
T256, T128, T64W, T64, PERS = range(5)  # 256 x 128, 128 x 128, 64 x 128, 64 x 64, persistent or eight-wave
CASES = [
    ((1, 512, 256, 32), T64, T64, 65536, 65536), ((63, 1024, 257, 31), T64, T64, 0, 36864),
    ((65, 505, 512, 129), T64, T64, 49152, 49152), ((257, 392, 1376, 64), T64, T64, 36864, 36864),
    ((1000, 512, 1381, 128), T64W, T64, 36864, 36864), ((1025, 509, 1536, 384), T64W, T64, 36864, 36864),
    ((2047, 2736, 1023, 342), T128, T256, 36864, 36864), ((3333, 1461, 701, 200), T128, T256, 36864, 36864),
    ((4097, 1021, 1000, 128), T256, T256, 36864, 36864), ((8191, 3072, 1030, 250), PERS, T256, 36864, 36864),
    ((8192, 1024, 3075, 128), PERS, T256, 36864, 36864),
    # K below the persistent kernel's least
    ((200, 40, 24, 8), T64, T64, 49152, 49152), ((129, 265, 129, 65), T64, T64, 36864, 36864),
    ((77, 8, 5472, 4), T64, T64, 36864, 0),
]


@pytest.mark.parametrize("shape,_f,_d,long_f,long_d", CASES)
def test_tile_rows_equal_long_call(shape, _f, _d, long_f, long_d):
    T, n, m, r = shape
    g = torch.Generator(device=dev()).manual_seed(T * 7 + n)
    long = max(long_f, long_d)
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
