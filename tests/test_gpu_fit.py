"""WLS rows evaluated from positions instead of read from stored
coefficients, against the oracle's rows: node targets (pc_stencil.h's tensor
fit) on every block shape, axis condition and placement it is chosen for, at
the walls, across periodic faces, for nodes outside the box, with a support
radius below the block's, and on anisotropic grids."""
import numpy as np
import pytest

from oracle import Grid
from oracle import projection as P
from paper_2304_14690_amd import inputs
from tests.helpers import rel_l2, to_np

pytestmark = pytest.mark.gpu

N, PER = "neumann", "periodic"
# d, n, h, bc, vertex, k_node, support, outside
NODE = {
    "2d_m4": (2, (16, 22), (1.0, 1.0), (N, N), False, 16, 3.0, False),
    "2d_m3_per": (2, (18, 14), (0.1, 0.1), (PER, N), False, 9, 3.0, False),
    "2d_m4_aniso_per": (2, (20, 12), (0.05, 0.125), (N, PER), False, 16, 3.0, False),
    "2d_m4_small_support": (2, (16, 16), (0.1, 0.1), (PER, PER), False, 16, 0.5, False),
    "2d_m4_vertex": (2, (17, 13), (0.25, 0.25), (N, N), True, 16, 3.0, False),
    "2d_m4_outside": (2, (16, 16), (0.1, 0.1), (N, N), False, 16, 3.0, True),
    "3d_m3": (3, (10, 12, 8), (0.5, 0.5, 0.5), (N, N, N), False, 27, 3.0, False),
    "3d_m3_per": (3, (8, 10, 12), (0.1, 0.2, 0.15), (PER, N, PER), False, 27, 3.0, False),
    "3d_m4": (3, (8, 10, 8), (0.1, 0.1, 0.1), (PER, PER, PER), False, 64, 1.0, False),
    "3d_m3_vertex": (3, (9, 11, 10), (0.1, 0.1, 0.1), (N, N, N), True, 27, 3.0, False),
}


@pytest.fixture(scope="module")
def pc():
    from paper_2304_14690_amd import pcorr
    return pcorr


@pytest.mark.parametrize("name", list(NODE))
def test_node_rows(pc, name):
    import torch
    d, n, h, bc, vertex, kn, support, outside = NODE[name]
    grid = Grid(d, n, h, bc, vertex=vertex)
    cells = n if not vertex else tuple(v - 1 for v in n)
    x = inputs.jittered_lattice(cells, h, 5, 0.45)
    if outside:
        x = (x - 0.5) * 1.08 + 0.5  # up to 0.6 spacings beyond every wall
    kind = np.zeros(x.shape[1], np.uint8)
    kind[::7] = inputs.KIND_B
    kg = 16 if d == 2 else 27
    st = P.build_stencils(grid, x.T.copy(), kind, kg, kn, support=support)
    plan = pc.Plan(d, n, h, bc=bc, grid="vertex" if vertex else "cell")
    geom = pc.wls_build(plan, torch.from_numpy(x.copy()).cuda(), torch.from_numpy(kind).cuda(),
                        kg, kn, support=support, want_f32=True)
    M = x.shape[1]
    coef = torch.empty((d, kn, M), dtype=torch.float64, device="cuda")
    base = torch.empty(M, dtype=torch.int32, device="cuda")
    pc.geom_export(geom, node_base=base, node_coef=coef)
    stride = np.cumprod([1] + list(n[:-1]))
    wrapped = np.mod(st.node_base, np.asarray(n))
    np.testing.assert_array_equal(to_np(base), wrapped @ stride)
    # the exported rows, applied to a field, and the transfer itself
    rng = np.random.Generator(np.random.PCG64(3))
    phi = rng.standard_normal(grid.G)
    ref = P.grad_to_nodes(st, phi).T
    m = round(kn ** (1.0 / d))
    o = np.arange(kn)
    off = np.stack([(o // m ** a) % m for a in range(d)], 1)
    idx = np.mod(wrapped[:, None, :] + off[None], np.asarray(n)) @ stride
    assert rel_l2(np.einsum("akm,mk->am", to_np(coef), phi[idx]), ref) <= 1e-12
    pt = torch.from_numpy(phi).cuda()
    g = torch.empty((d, M), dtype=torch.float64, device="cuda")
    pc.grad_to_nodes(geom, pt, g)
    gi = torch.empty((d, geom.n_ib), dtype=torch.float64, device="cuda")
    pc.grad_to_nodes(geom, pt, gi, pc.PC_IB)
    assert rel_l2(to_np(g), ref) <= 1e-12
    np.testing.assert_allclose(to_np(gi), to_np(g)[:, kind != 0], rtol=0,
                               atol=1e-13 * np.abs(ref).max())
    # float32 fields: float64 rows and sums, one rounding of the result
    p32 = pt.float()
    g32 = torch.empty((d, M), dtype=torch.float32, device="cuda")
    pc.grad_to_nodes(geom, p32, g32)
    ref32 = P.grad_to_nodes(st, to_np(p32).astype(np.float64)).T
    assert rel_l2(to_np(g32), ref32) <= 2.0 ** -24


def test_degenerate_weight_is_refused(pc):
    """A weight so narrow that the block's outer lines vanish under it makes
    every node's normal matrix singular (Sec. 2.2: the ratio of its pivots)."""
    import torch
    n, h = (16, 16), (1.0 / 16,) * 2
    x = inputs.jittered_lattice(n, h, 5)
    plan = pc.Plan(2, n, h)
    for eps in (300.0, 3000.0, 3.0e5):
        with pytest.raises(pc.PcError) as e:
            pc.wls_build(plan, torch.from_numpy(x).cuda(),
                         torch.zeros(x.shape[1], dtype=torch.uint8, device="cuda"), 16, 16,
                         eps=eps)
        assert e.value.code == pc.PC_ERR_SINGULAR_STENCIL
