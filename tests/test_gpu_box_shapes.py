"""Box solves at the edges of their shapes: boxes of one, two and three rows
(no row on one or both sides of the middle row of a two-ended factor), of odd
and even heights, much taller than wide and much wider than tall, and every
column width class at its narrowest and widest; T against the oracle in the
three precisions (gates of tests/_gates.py), and multi-column and
multi-context applications equal to the one-column ones bit for bit.
"""
import numpy as np
import pytest

from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B
from tests._gates import t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# nx, ny, sx, sy, l, overlap, bc
SHAPES = [
    (23, 1, 8, 1, 0, 0, (1, 1, 0, 0)),     # one row
    (24, 2, 8, 2, 2, 1, (0, 1, 0, 0)),     # two rows
    (24, 6, 8, 2, 1, 1, (1, 1, 0, 0)),     # boxes of three and four rows
    (26, 5, 26, 5, 0, 2, (0, 0, 0, 0)),    # one pinned box
    (9, 90, 3, 45, 2, 2, (1, 0, 0, 0)),    # narrow and tall
    (120, 9, 60, 3, 2, 2, (0, 0, 1, 0)),   # 62 columns, 7 rows
    (34, 33, 17, 11, 0, 0, (1, 1, 0, 0)),  # 17 and 20-column class
    (57, 40, 19, 20, 1, 1, (1, 1, 0, 0)),  # 21 columns
    (75, 50, 25, 25, 4, 2, (0, 0, 0, 0)),  # 32-column class, 33 columns
    (96, 70, 32, 35, 2, 2, (1, 1, 0, 1)),  # 36 columns, odd heights
    (88, 45, 44, 15, 4, 2, (1, 1, 0, 0)),  # 48-column class
]


def _field(n, seed):
    return np.exp(1.5 * np.random.Generator(np.random.PCG64(seed)).standard_normal(n))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:5])))
@pytest.mark.parametrize("precision", (0, 1, 2))
def test_box_shapes(shape, precision):
    nx, ny, sx, sy, l, overlap, bc = shape
    print(f"box shapes {shape} precision {precision}", flush=True)
    dev = torch.device("cuda:0")
    n = nx * ny
    K = _field(n, 11)
    r = np.random.Generator(np.random.PCG64(12)).standard_normal((3, n))
    if not any(bc):
        r -= r.mean(axis=1, keepdims=True)
    ctx = B.Context(B.Config(nx, ny, bc, sx, sy, l, 10.0, 0, 1, overlap, 1, precision),
                    torch.tensor(K, device=dev))
    rd = torch.tensor(r, device=dev)
    z = torch.full_like(rd, np.nan)
    ctx.apply(rd, z)
    one = torch.full((n,), np.nan, dtype=torch.float64, device=dev)
    for k in range(3):
        ctx.apply(rd[k].contiguous(), one)
        assert torch.equal(one, z[k])
    many = torch.full_like(rd, np.nan)
    B.apply_many([ctx], [rd], [many])
    torch.cuda.synchronize()
    assert torch.equal(many, z)
    if precision:
        ctx.close()
        return
    mr = MRCM(K, nx=nx, ny=ny, bc=bc, sx=sx, sy=sy, oversample=l, alpha=10.0, beta_len="H",
              sweeps=1, overlap=overlap, degree=1)
    gate = t_gate(mr)
    for k in range(3):
        ref = mr.apply(r[k])
        err = np.linalg.norm(z[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
        assert err <= gate
    ctx.close()
