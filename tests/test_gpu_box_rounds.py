"""Trace moments where the subdomains of a workgroup need different numbers of rounds over
their faces (two FP64 boxes of 128 threads each; 34-wide subdomains: 136 faces inside,
102 and 68 at the edges of the grid), and a single subdomain, which has none: T against the
oracle, one column, three, and through a launch over several contexts.
"""
import numpy as np
import pytest

from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B
from tests._gates import t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx, ny, s, degree", [(136, 102, 34, 1), (102, 170, 34, 8),
                                               (34, 34, 34, 1)])
def test_rounds(nx, ny, s, degree):
    print(f"rounds {nx}x{ny} s {s} degree {degree}", flush=True)
    dev = torch.device("cuda:0")
    n = nx * ny
    x, y = np.meshgrid(np.arange(nx), np.arange(ny))
    K = np.exp(np.sin(x / 5.0) + np.cos(y / 7.0)).reshape(-1)
    r = np.random.Generator(np.random.PCG64(31)).standard_normal((3, n))
    ctx = B.Context(B.Config(nx, ny, (1, 1, 0, 0), s, s, 1, 10.0, 0, 1, 1, degree, 0),
                    torch.tensor(K, device=dev))
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
    mr = MRCM(K, nx=nx, ny=ny, bc=(1, 1, 0, 0), sx=s, sy=s, oversample=1, alpha=10.0,
              beta_len="H", sweeps=1, overlap=1, degree=degree)
    gate = t_gate(mr)
    for k in range(3):
        ref = mr.apply(r[k])
        err = np.linalg.norm(z[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
        assert err <= gate
    ctx.close()
