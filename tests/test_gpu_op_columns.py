"""op_apply for one to six columns in one call: every column is that of a call of its
own, bit for bit, and the oracle's A x within the rounding of its nine operations
(16 eps |A| |x| per cell), at sizes around the kernel's tiles of 64 x 16 cells.
"""
import numpy as np
import pytest

from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(16, 16), (63, 33), (64, 16), (65, 17), (127, 31), (130, 18)]


@pytest.mark.parametrize("bc", [(1, 1, 0, 0), (0, 0, 1, 0), (0, 0, 0, 0)], ids=str)
@pytest.mark.parametrize("size", SIZES, ids=lambda c: f"{c[0]}x{c[1]}")
def test_op_columns(size, bc):
    nx, ny = size
    print(f"op_apply {nx}x{ny} bc {bc}", flush=True)
    dev = torch.device("cuda:0")
    n = nx * ny
    rng = np.random.Generator(np.random.PCG64(71))
    K = np.exp(rng.standard_normal(n))
    x = rng.standard_normal((6, n))
    ctx = B.Context(B.Config(nx, ny, bc, 16, 16, 0, 10.0, 0, 0, 2, 1, 0),
                    torch.tensor(K, device=dev))
    xd = torch.tensor(x, device=dev)
    one = torch.full_like(xd, np.nan)
    for k in range(6):
        ctx.op(xd[k], one[k])
    for k in range(1, 7):
        y = torch.full_like(xd, np.nan)
        ctx.op(xd[:k].contiguous(), y[:k])
        assert torch.equal(y[:k], one[:k])
        assert torch.isnan(y[k:]).all()
    mr = MRCM(K, nx=nx, ny=ny, bc=bc, sx=16, sy=16, oversample=0, alpha=10.0, beta_len="H",
              sweeps=0, overlap=2, degree=1)
    bound = 16 * np.finfo(np.float64).eps * (abs(mr.A) @ np.abs(x).T).T
    assert (np.abs(one.cpu().numpy() - (mr.A @ x.T).T) <= bound).all()
    ctx.close()
