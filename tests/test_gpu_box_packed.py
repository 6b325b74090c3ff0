"""Many boxes: launches of more than 2048 waves of boxes up to 16 columns wide, and of more
than 3072 boxes up to 20 wide, run several boxes to a wave, and FP64 boxes of 37 to 48
columns past 1024 waves run on kernels of their own.  Boxes of different heights and widths,
down to a row or a column, share a wave; T of one, seven and eight columns and through a
launch over several contexts is the same bit for bit, and the oracle's within the gates.
"""
import numpy as np
import pytest

from oracle.mrcm import MRCM
from paper_2606_08883_amd import binding as B
from tests._gates import mixed_t_gate, t_gate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# nx, ny, sx, sy, l, overlap, degree, precisions: FP64 packs past 1024 boxes, FP32 storage past
# 2048, a launch over several contexts by the boxes of all its columns
SHAPES = [
    (168, 101, 5, 3, 1, 1, 1, (0,)),      # 1156 boxes of 2 to 7 rows and columns
    (462, 63, 14, 2, 0, 1, 1, (0,)),      # 1056, patches of 16 columns, last row of boxes one high
    (66, 320, 2, 10, 0, 3, 1, (0,)),      # 1056, patches 8 x 16
    (231, 33, 6, 1, 0, 0, 8, (0,)),       # 1287 single rows, last column three wide
    (205, 156, 4, 3, 0, 1, 1, (1, 2)),    # 2704, last column of boxes one wide
    (171, 165, 4, 3, 1, 2, 1, (1, 2)),    # 2365
    (130, 122, 5, 4, 1, 1, 1, (0, 1, 2)),  # 806: one column on its own waves, eight packed
    (545, 190, 17, 2, 0, 1, 1, (0, 1)),    # 3135 boxes, patches 19 x 4, last column one wide
    (576, 98, 18, 1, 0, 1, 1, (2,)),       # 3136, patches 20 x 3
    (400, 104, 40, 2, 1, 1, 1, (0,)),      # 520 of 42 x 4: FP64 at two waves per SIMD
    (360, 156, 36, 3, 1, 2, 1, (0,)),      # 520 of 38 x 5 and 40 x 7
]
CASES = [(s, p) for s in SHAPES for p in s[-1]]


@pytest.mark.parametrize("shape, precision", CASES,
                         ids=lambda v: f"mode{v}" if isinstance(v, int)
                         else "x".join(map(str, v[:6])))
def test_packed_boxes(shape, precision):
    nx, ny, sx, sy, l, overlap, degree, _ = shape
    print(f"packed boxes {shape} precision {precision}", flush=True)
    dev = torch.device("cuda:0")
    n = nx * ny
    x, y = np.meshgrid(np.arange(nx), np.arange(ny))
    K = np.exp(np.sin(x / 5.0) + np.cos(y / 7.0)).reshape(-1)
    r = np.random.Generator(np.random.PCG64(51)).standard_normal((8, n))
    ctx = B.Context(B.Config(nx, ny, (1, 1, 0, 0), sx, sy, l, 10.0, 0, 1, overlap, degree,
                             precision), torch.tensor(K, device=dev))
    rd = torch.tensor(r, device=dev)
    z = torch.full_like(rd, np.nan)
    ctx.apply(rd, z)
    one = torch.full_like(rd[0], np.nan)
    for k in (0, 6, 7):
        ctx.apply(rd[k].contiguous(), one)
        assert torch.equal(one, z[k])
    for cols in (7, 8):
        out = torch.full_like(rd[:cols], np.nan)
        ctx.apply(rd[:cols].contiguous(), out)
        assert torch.equal(out, z[:cols])
        out.fill_(np.nan)
        B.apply_many([ctx], [rd[:cols].contiguous()], [out])
        torch.cuda.synchronize()
        assert torch.equal(out, z[:cols])
    mr = MRCM(K, nx=nx, ny=ny, bc=(1, 1, 0, 0), sx=sx, sy=sy, oversample=l, alpha=10.0,
              beta_len="H", sweeps=1, overlap=overlap, degree=degree)
    gate = t_gate(mr) + (mixed_t_gate(mr) if precision else 0.0)
    for k in (0, 7):
        ref = mr.apply(r[k])
        err = np.linalg.norm(z[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  rel L2 {err:.2e} gate {gate:.2e}", flush=True)
        assert err <= gate
    ctx.close()
