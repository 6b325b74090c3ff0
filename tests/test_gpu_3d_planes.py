"""Plane products of the 3-D box solves at the edges of their tiling: planes of
one cell, of one cell less and more than a multiple of 16, odd and even numbers
of tile rows, the largest plane (256 cells), boxes of one plane, and boxes of
different plane sizes in one launch; T in both precisions against the oracle
(gates of tests/_gates.py) and repeated, bit for bit.
"""
import numpy as np
import pytest

from oracle import mrcm3d as M3
from paper_2606_08883_amd import binding as B
from tests._gates import mixed_t_gate3, t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# nx, ny, nz, (sx, sy, sz), l, overlap: plane sizes of the oversampled boxes
SHAPES = [
    (1, 1, 6, (1, 1, 3), 0, 0),        # 1
    (5, 3, 4, (5, 3, 2), 0, 0),        # 15
    (4, 4, 4, (4, 4, 2), 0, 0),        # 16
    (17, 2, 1, (17, 1, 1), 0, 0),      # 17, one plane
    (16, 6, 4, (8, 3, 2), 0, 1),       # 24; patches 36
    (22, 7, 3, (11, 3, 3), 0, 1),      # 33 and 44
    (21, 21, 6, (7, 6, 3), 2, 1),      # 63 to 110, ragged
    (32, 31, 8, (16, 16, 4), 0, 0),    # 240, 256
    (24, 24, 10, (12, 12, 5), 2, 2),   # 196
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:3] + s[3])))
@pytest.mark.parametrize("precision", (0, 2))
def test_plane_shapes(shape, precision):
    nx, ny, nz, s, l, overlap = shape
    print(f"plane shapes {shape} precision {precision}", flush=True)
    dev = torch.device("cuda:0")
    bc = (1, 0, 0, 0, 0, 1)
    cfg = B.Config3(nx, ny, nz, bc, *s, l, 10.0, 0, 1, overlap, 1, precision)
    rng = np.random.Generator(np.random.PCG64(21))
    K = np.exp(1.5 * rng.standard_normal(cfg.n))
    r = rng.standard_normal(cfg.n)
    ctx = B.Context3(cfg, torch.tensor(K, device=dev))
    rd = torch.tensor(r, device=dev)
    z, again = torch.full_like(rd, np.nan), torch.full_like(rd, np.nan)
    ctx.apply(rd, z)
    ctx.apply(rd, again)
    torch.cuda.synchronize()
    assert torch.equal(z, again)
    mr = M3.MRCM3D(K, nx, ny, nz, bc, *s, l, 10.0, "H", 1, overlap, 1)
    ref = mr.apply(r)
    gate = t_gate(mr) + (mixed_t_gate3(mr) if precision else 0.0)
    err = np.linalg.norm(z.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
    assert err <= gate
    ctx.close()
