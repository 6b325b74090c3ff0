"""T in the three precisions against the oracle, over the column width classes of the
box kernels: one column, three, and through a launch over several contexts.  The field is
smooth, so that the gate on the rounding of the factors (mixed_t_gate) bounds T.
"""
import numpy as np
import pytest

from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B
from tests._gates import mixed_t_gate, t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# nx, ny, sx, sy, l, overlap: widest boxes
SHAPES = [
    (37, 20, 18, 10, 0, 0),  # 18 columns beside a last subdomain of one
] + [
    # every column width class at its narrowest and widest, boxes of nine and five rows
    (2 * w + 3, 14, w, 9, 0, 0) for w in (2, 16, 17, 20, 21, 24, 25, 32, 33, 36, 37, 40, 41, 48, 49,
                                          64)
] + [
    (70, 42, 16, 13, 2, 2),  # oversampled boxes of 20 columns, patches of 20
    (99, 84, 30, 26, 5, 3),  # 40 and 36
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("precision", (0, 1, 2))
def test_box_modes(shape, precision):
    nx, ny, sx, sy, l, overlap = shape
    print(f"box modes {shape} precision {precision}", flush=True)
    dev = torch.device("cuda:0")
    n = nx * ny
    x, y = np.meshgrid(np.arange(nx), np.arange(ny))
    K = np.exp(np.sin(x / 5.0) + np.cos(y / 7.0)).reshape(-1)
    r = np.random.Generator(np.random.PCG64(41)).standard_normal((3, n))
    ctx = B.Context(B.Config(nx, ny, (1, 1, 0, 0), sx, sy, l, 10.0, 0, 1, overlap, 1, precision),
                    torch.tensor(K, device=dev))
    rd = torch.tensor(r, device=dev)
    z = torch.full_like(rd, np.nan)
    ctx.apply(rd, z)
    one = torch.full_like(rd[0], np.nan)
    many = torch.full_like(rd, np.nan)
    B.apply_many([ctx], [rd], [many])
    for k in range(3):
        ctx.apply(rd[k].contiguous(), one)
        assert torch.equal(one, z[k])
    torch.cuda.synchronize()
    assert torch.equal(many, z)
    mr = MRCM(K, nx=nx, ny=ny, bc=(1, 1, 0, 0), sx=sx, sy=sy, oversample=l, alpha=10.0,
              beta_len="H", sweeps=1, overlap=overlap, degree=1)
    gate = t_gate(mr) + (mixed_t_gate(mr) if precision else 0.0)
    for k in range(3):
        ref = mr.apply(r[k])
        err = np.linalg.norm(z[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
        assert err <= gate
    ctx.close()
