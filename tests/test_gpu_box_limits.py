"""The largest boxes that the box kernels accept: a box counts with one vector slot of
whole lane groups, its couplings and its cells in 64 KB of LDS, although a launch of it
may take more; T of the largest ones against the oracle (gates of tests/_gates.py), one
column and three, and the next larger box refused.
"""
import numpy as np
import pytest

from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B
from tests._gates import mixed_t_gate, t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# precision, sx, sy, box (2 x 2 subdomains, each grown by 2 cells inwards)
LARGEST = [
    (0, 61, 61, (63, 63)),
    (0, 60, 62, (62, 64)),
    (0, 54, 69, (56, 71)),
    (0, 14, 252, (16, 254)),
    (2, 14, 337, (16, 339)),
    (1, 14, 508, (16, 510)),
]


def _config(sx, sy, precision):
    return B.Config(2 * sx, 2 * sy, (1, 1, 0, 0), sx, sy, 2, 10.0, 0, 1, 2, 1, precision)


def _field(nx, ny):
    x, y = np.meshgrid(np.arange(nx), np.arange(ny))
    return np.exp(np.sin(x / 5.0) + np.cos(y / 7.0)).reshape(-1)


@pytest.mark.parametrize("case", LARGEST, ids=lambda c: f"mode{c[0]}-{c[3][0]}x{c[3][1]}")
def test_largest_boxes(case):
    precision, sx, sy, box = case
    nx, ny = 2 * sx, 2 * sy
    print(f"largest boxes {box} precision {precision}", flush=True)
    dev = torch.device("cuda:0")
    K = _field(nx, ny)
    r = np.random.Generator(np.random.PCG64(21)).standard_normal((3, nx * ny))
    ctx = B.Context(_config(sx, sy, precision), torch.tensor(K, device=dev))
    rd = torch.tensor(r, device=dev)
    z = torch.full_like(rd, np.nan)
    ctx.apply(rd, z)
    one = torch.full_like(rd[0], np.nan)
    ctx.apply(rd[0].contiguous(), one)
    many = torch.full_like(rd, np.nan)
    B.apply_many([ctx], [rd], [many])
    torch.cuda.synchronize()
    assert torch.equal(one, z[0])
    assert torch.equal(many, z)
    mr = MRCM(K, nx=nx, ny=ny, bc=(1, 1, 0, 0), sx=sx, sy=sy, oversample=2, alpha=10.0,
              beta_len="H", sweeps=1, overlap=2, degree=1)
    gate = t_gate(mr) + (mixed_t_gate(mr) if precision else 0.0)
    for k in range(3):
        ref = mr.apply(r[k])
        err = np.linalg.norm(z[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
        assert err <= gate
    ctx.close()


@pytest.mark.parametrize("precision, sx, sy", [(0, 62, 62), (0, 14, 253), (2, 14, 339),
                                               (1, 14, 510)])
def test_larger_boxes_are_refused(precision, sx, sy):
    K = torch.ones(4 * sx * sy, dtype=torch.float64, device="cuda:0")
    with pytest.raises(B.MrcmError) as e:
        B.Context(_config(sx, sy, precision), K)
    assert e.value.code == B.MRCM_EINVAL
