"""The generic line transforms where a prime factor takes a direct sum per
output (11, 17, 19, 23, 37, 1009), with and without their twiddles in LDS
(lines of up to 512 points and longer), the radix-7 butterfly, tiles that end
inside the grid and lines shorter than a wavefront, on Neumann, periodic and
vertex axes in every position and precision, against the oracle's solve
(float64 1e-11, float32 5e-5, defect correction 1e-10 relative L2)."""
import numpy as np
import pytest

from oracle import Grid, poisson
from tests.helpers import rel_l2, to_np

pytestmark = pytest.mark.gpu

N, P = "neumann", "periodic"
CASES = [
    ((22, 14), (N, N), False), ((22, 34), (P, P), False), ((506, 518), (N, P), False),
    ((528, 516), (P, N), False), ((1998, 34), (N, N), False), ((38, 1998), (P, P), False),
    ((2018, 10), (P, N), False), ((10, 2018), (N, N), False), ((98, 686), (N, N), False),
    ((26, 22, 38), (N, P, N), False), ((46, 28, 34), (P, N, P), False),
    ((14, 574, 10), (N, N, N), False),
    ((24, 562), (N, N), True), ((562, 12), (N, N), True), ((15, 24, 12), (N, N, N), True),
]


@pytest.fixture(scope="module")
def pc():
    from paper_2304_14690_amd import pcorr
    return pcorr


@pytest.mark.parametrize("n,bc,vertex", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_generic_lines(pc, n, bc, vertex):
    import torch
    d = len(n)
    h = (1.0 / n[0],) * d
    grid = Grid(d, n, h, bc, vertex=vertex)
    plan = pc.Plan(d, n, h, bc=bc, grid="vertex" if vertex else "cell")
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
