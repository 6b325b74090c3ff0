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


# a quiet NaN, and the signalling NaN that marks a scalar as not yet written
NANS = {"quiet": 0x7FF8000000000000, "unset-mark": 0x7FF4A5C3E1D2B697}


@pytest.mark.parametrize("kind", NANS)
def test_nan_right_hand_sides_end(kind):
    """A right-hand side of NaN runs its steps and ends unconverged: no scalar the host
    waits for looks as if it had not arrived."""
    print(f"NaN right-hand side ({kind})", flush=True)
    dev = torch.device("cuda:0")

    def rhs(k, n):
        return torch.tensor(np.full((k, n), NANS[kind], dtype=np.uint64).view(np.int64),
                            device=dev).view(torch.float64)

    ctx = B.Context(B.Config(36, 32, (1, 1, 0, 0), 16, 16, 2, 10.0, 0, 1, 2, 1, 0),
                    torch.ones(36 * 32, dtype=torch.float64, device=dev))
    for k in (1, 3):
        b = rhs(k, ctx.n)
        p = torch.zeros_like(b)
        st = ctx.gmres(b, p, rtol=1e-8, restart=2, maxit=3, raise_on_noconv=False)
        assert not st.converged and st.iterations == 3 * k
        batch = B.Batch(2)
        tag = batch.add(ctx, b, p, rtol=1e-8, maxit=3)
        ticks = 0
        while batch.tick():
            ticks += 1
            assert ticks < 20
        batch.remove(tag)
        batch.close()
    ctx.close()
    ctx3 = B.Context3(B.Config3(12, 12, 8, (1, 1, 0, 0, 0, 0), 4, 4, 4, 1, 10.0, 0, 1, 1, 1, 0),
                      torch.ones(12 * 12 * 8, dtype=torch.float64, device=dev))
    b = rhs(1, ctx3.n)[0]
    st = ctx3.gmres(b, torch.zeros_like(b), rtol=1e-8, restart=2, maxit=3, raise_on_noconv=False)
    assert not st.converged and st.iterations == 3
    ctx3.close()
