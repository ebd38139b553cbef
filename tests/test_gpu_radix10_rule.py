"""Last axes of radix-10 lengths on both sides of the rule that chooses between
the radix-10 and the generic kernel (periodic or Neumann, float64 or float32,
2D workgroups below and above half a wavefront, 3D, small and large grids),
against the oracle's solve (the bars of the solves: float64 1e-11, float32
5e-5, defect correction 1e-10 relative L2)."""
import numpy as np
import pytest

from oracle import Grid, poisson
from tests.helpers import rel_l2, to_np

pytestmark = pytest.mark.gpu

NE, P = "neumann", "periodic"
CASES = [
    ((400, 400), (P, NE)), ((128, 400), (NE, P)), ((1000, 400), (NE, NE)), ((2000, 400), (P, NE)),
    ((2000, 200), (NE, NE)), ((4096, 200), (NE, NE)), ((4096, 200), (NE, P)),
    ((200, 1000), (NE, P)), ((200, 1000), (P, NE)), ((64, 2000), (NE, P)), ((10, 2000), (P, NE)),
    ((32, 32, 200), (NE, P, NE)), ((32, 32, 200), (P, NE, P)), ((48, 32, 400), (NE, NE, P)),
    ((8, 12, 1000), (NE, NE, P)), ((64, 64, 400), (P, NE, P)),
]


@pytest.fixture(scope="module")
def pc():
    from paper_2304_14690_amd import pcorr
    return pcorr


@pytest.mark.parametrize("n,bc", CASES,
                         ids=["x".join(map(str, n)) + "-" + "".join(c[0] for c in bc)
                              for n, bc in CASES])
def test_last_axis_of_radix_10_lengths(pc, n, bc):
    import torch
    d = len(n)
    h = (1.0 / n[0],) * d
    grid = Grid(d, n, h, bc)
    plan = pc.Plan(d, n, h, bc=bc)
    b = np.random.Generator(np.random.PCG64(sum(n))).normal(size=grid.G) + 0.2
    ref, bm_ref = poisson.solve(grid, b)
    bt = torch.from_numpy(b).cuda()
    bm = torch.zeros(1, dtype=torch.float64, device="cuda")
    for mode, dt, tol in ((pc.PC_F64, torch.float64, 1e-11), (pc.PC_F32, torch.float32, 5e-5),
                          (pc.PC_MIXED, torch.float64, 1e-10)):
        x = bt.to(dt)
        phi = torch.empty_like(x)
        ws = pc.Workspace(plan, None, mode)
        pc.poisson_fft_solve(plan, x, phi, mode, bmean=bm, ws=ws)
        torch.cuda.synchronize()
        assert rel_l2(to_np(phi), ref) <= tol
        assert abs(bm.item() - bm_ref) <= (1e-5 if dt == torch.float32 else 1e-12)
