"""The Arnoldi step for one right-hand side, for several in one launch per phase
(at different steps of their cycles), and through the batched solver, which are
the same bit for bit; the iterate against the oracle's GMRES at the same step
(gate of tests/_gates.py for FP64 solutions at the same step), within a cycle
and past a restart, on vectors of one and of several workgroups.
"""
import numpy as np
import pytest

from oracle.gmres import gmres
from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B
from tests._gates import t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# nx, ny, restart, steps
CASES = [(31, 33, 5, 7), (32, 32, 1, 3), (41, 25, 10, 13), (48, 40, 20, 23), (125, 131, 10, 12),
         (128, 128, 10, 11), (129, 128, 10, 11), (384, 320, 10, 12)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}-m{c[2]}")
def test_arnoldi_step_forms(case):
    nx, ny, restart, steps = case
    print(f"GMRES({restart}) on {nx}x{ny}, {steps} steps", flush=True)
    dev = torch.device("cuda:0")
    n = nx * ny
    rng = np.random.Generator(np.random.PCG64(31))
    K = np.exp(rng.standard_normal(n))
    b = rng.standard_normal((3, n))
    ctx = B.Context(B.Config(nx, ny, (1, 1, 0, 0), 16, 16, 0, 10.0, 0, 0, 2, 1, 0),
                    torch.tensor(K, device=dev))
    bd = torch.tensor(b, device=dev)
    one = torch.full((n,), np.nan, dtype=torch.float64, device=dev)
    st = ctx.gmres(bd[0].contiguous(), one, rtol=0.0, restart=restart, maxit=steps,
                   raise_on_noconv=False)
    several = torch.full_like(bd, np.nan)
    ctx.gmres(bd, several, rtol=0.0, restart=restart, maxit=steps, raise_on_noconv=False)
    batched = torch.full_like(bd, np.nan)
    batch = B.Batch(restart)
    tag = batch.add(ctx, bd, batched, rtol=0.0, maxit=steps)
    while batch.tick():
        pass
    batch.remove(tag)
    batch.close()
    torch.cuda.synchronize()
    assert st.iterations == steps
    assert torch.equal(one, several[0]) and torch.equal(several, batched)
    mr = MRCM(K, nx=nx, ny=ny, bc=(1, 1, 0, 0), sx=16, sy=16, oversample=0, alpha=10.0,
              beta_len="H", sweeps=0, overlap=2, degree=1)
    ref = gmres(lambda x: mr.A @ x, mr.apply, b[0], rtol=0.0, restart=restart, maxit=steps,
                atol=0.0)
    err = np.linalg.norm(one.cpu().numpy() - ref.p) / np.linalg.norm(ref.p)
    gate = t_gate(mr)
    print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
    assert err <= gate
    ctx.close()
