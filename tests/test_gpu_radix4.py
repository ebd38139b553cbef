"""The register transforms on both sides of the rules that choose their plan: the
fused last axis and the middle axis of grids of 2^20 points (radix 4) and
above (radix 8), and long x rows, as cosine and real Fourier transforms in
every precision, against the oracle's solve (the bars of the solves: float64
1e-11, float32 5e-5, defect correction 1e-10 relative L2)."""
import numpy as np
import pytest

from oracle import Grid, poisson
from tests.helpers import rel_l2, to_np

pytestmark = pytest.mark.gpu

NE, P = "neumann", "periodic"
CASES = [
    ((1024, 1024), (NE, P)), ((2048, 1024), (P, NE)), ((4096, 512), (NE, P)),
    ((4096, 258), (NE, NE)), ((1024, 1026), (P, NE)),
    ((64, 512, 32), (NE, P, NE)), ((128, 512, 32), (P, NE, P)), ((512, 256, 64), (NE, NE, P)),
    ((64, 64, 512), (P, P, NE)), ((256, 32, 32), (P, P, P)),
    # more than 2048 x rows of a large 2D grid, 3D grids above 2^24 points
    ((1024, 4096), (NE, P)), ((512, 2048), (P, NE)), ((512, 512, 128), (NE, NE, P)),
    # radix 10: last axes of 200 and 400 points on both sides of their rule
    ((4096, 400), (NE, P)), ((64, 128, 200), (P, NE, P)), ((64, 128, 200), (NE, P, NE)),
    ((400, 400), (P, P)), ((200, 200), (NE, NE)), ((200, 200), (P, P)),
]


@pytest.fixture(scope="module")
def pc():
    from paper_2304_14690_amd import pcorr
    return pcorr


@pytest.mark.parametrize("n,bc", CASES, ids=["x".join(map(str, n)) + "-" + "".join(c[0] for c in bc) for n, bc in CASES])
def test_solve_on_both_sides_of_the_rule(pc, n, bc):
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
