"""The divergence from rows and tile node lists where its dispatch changes: a
shape parameter beyond the range of the unclamped weight, the tile shapes of
thin and short grids, and clouds refined in places, whose dense tiles hold more
nodes than a list and keep coefficients."""
import numpy as np
import pytest

from oracle import Grid
from oracle import projection as P
from paper_2304_14690_amd import inputs
from tests.helpers import rel_l2, stored_order, to_np

pytestmark = pytest.mark.gpu

N, PER = "neumann", "periodic"


@pytest.fixture(scope="module")
def pc():
    from paper_2304_14690_amd import pcorr
    return pcorr


def check_divergence(pc, n, h, bc, x, kind, kg, tol=1e-12, tol32=2.0 ** -24, near=True, **opts):
    """div_to_grid of the whole grid and of the near-IB subset, float64 and
    float32, and the exported stencils against the oracle's; the geometry."""
    import torch
    d = len(n)
    grid = Grid(d, n, (h,) * d, bc)
    st = P.build_stencils(grid, x.T.copy(), kind, kg, 16 if d == 2 else 27, **opts)
    assert not st.singular_grid.any()
    plan = pc.Plan(d, n, (h,) * d, bc=bc)
    geom = pc.wls_build(plan, torch.from_numpy(x.copy()).cuda(), torch.from_numpy(kind).cuda(),
                        kg, 16 if d == 2 else 27, want_f32=True, **opts)
    G = grid.G
    gi = torch.empty((kg, G), dtype=torch.int32, device="cuda")
    gc = torch.empty((d, kg, G), dtype=torch.float64, device="cuda")
    pc.geom_export(geom, gi, gc)
    order = stored_order(grid, x.T, st.grid_idx)
    np.testing.assert_array_equal(to_np(gi).T, np.take_along_axis(st.grid_idx, order, 1))
    ref_c = np.take_along_axis(st.grid_coef, order[:, None, :], 2)
    assert rel_l2(np.transpose(to_np(gc), (2, 0, 1)), ref_c) <= tol
    u = np.random.Generator(np.random.PCG64(4)).standard_normal(x.shape)
    ib = np.flatnonzero(kind)
    for dt, lim in ((torch.float64, tol), (torch.float32, tol32)):
        ut = torch.from_numpy(u).to(dt).cuda()
        uh = to_np(ut).astype(np.float64)
        b = torch.full((G,), 7.0, dtype=dt, device="cuda")
        pc.div_to_grid(geom, ut, b)
        assert rel_l2(to_np(b), P.div_to_grid(st, uh.T)) <= lim
        if near:
            bn = torch.zeros(G, dtype=dt, device="cuda")
            pc.div_to_grid(geom, ut[:, ib].contiguous(), bn, pc.PC_NEAR_IB)
            refn = P.div_to_grid(st, np.where(kind != 0, uh, 0.0).T)
            # float32: rounded coefficients and 32 float32 sums of random values
            assert rel_l2(to_np(bn), refn) <= (tol if dt == torch.float64 else 32 * 2.0 ** -24)
    return geom


def lattice(n, h, seed, ratio=1):
    x = inputs.jittered_lattice(tuple(v * ratio for v in n), (h / ratio,) * len(n), seed, 0.3)
    kind = np.zeros(x.shape[1], np.uint8)
    kind[::11] = inputs.KIND_B
    return x, kind


@pytest.mark.parametrize("n,bc,kg,eps,support", [
    ((34, 18), (N, PER), 16, 700.0, 31.6), ((34, 18), (N, N), 12, 2500.0, 60.0),
    ((18, 10, 8), (N, N, PER), 27, 700.0, 31.6), ((18, 10, 8), (N, N, N), 20, 2500.0, 60.0),
], ids=["2d", "2d_2500", "3d", "3d_2500"])
def test_large_shape_parameter(pc, n, bc, kg, eps, support):
    """eps above 690, with a support that keeps the weights ordinary (Eq. 17:
    eps / support^2 = 0.7)."""
    x, kind = lattice(n, 0.125, 8)
    check_divergence(pc, n, 0.125, bc, x, kind, kg, eps=eps, support=support)


@pytest.mark.parametrize("n,bc", [
    ((8, 70), (N, PER)), ((16, 34), (N, N)), ((40, 34), (PER, N)), ((70, 12), (N, N)),
    ((72, 64), (N, N)), ((8, 10, 12), (N, N, PER)), ((8, 12, 16), (N, N, N)),
    ((16, 10, 8), (N, PER, N)), ((18, 8, 10), (N, N, N)), ((32, 10, 12), (PER, N, N)),
    ((32, 12, 10), (N, N, N)), ((24, 16, 12), (N, N, N)),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v[0], int) else "")
def test_tile_shapes(pc, n, bc):
    """Grids that end inside a tile or take another tile shape than 32 x 8 and
    16 x 4 x 4."""
    x, kind = lattice(n, 0.125, 8)
    check_divergence(pc, n, 0.125, bc, x, kind, 16 if len(n) == 2 else 27)


@pytest.mark.parametrize("n,bc,kg", [((34, 10, 8), (N, N, PER), 27), ((32, 12, 10), (N, N, N), 27),
                                     ((16, 10, 12), (PER, N, N), 20), ((8, 10, 12), (N, N, N), 16)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple)
                         and isinstance(v[0], int) else None)
def test_tile_shapes_of_fine_clouds(pc, n, bc, kg):
    """Clouds of eight nodes a cell keep stored coefficients in tiles of their
    own shapes (float32: rounded coefficients and k float32 sums)."""
    h = 0.125
    x, kind = lattice(n, h, 8, 2)
    check_divergence(pc, n, h, bc, x, kind, kg, tol32=3 * kg * 2.0 ** -24, delta=h / 2)


@pytest.mark.parametrize("n,m", [((8, 64), (64, 8)), ((16, 128), (128, 16)),
                                 ((8, 32, 32), (32, 32, 8))],
                         ids=["8x64", "16x128", "8x32x32"])
def test_thin_grids_hold_no_padding(pc, n, m):
    """A thin grid's geometry is as large as that of the same grid laid flat:
    no tile reaches beyond it."""
    size = []
    for g in (n, m):
        plan = pc.Plan(len(n), g, (0.125,) * len(n))
        kn = 16 if len(n) == 2 else 27
        size.append(pc.geom_footprint(plan, int(np.prod(n)), 0, 0, 16, kn)[0])
    assert size[0] == size[1]


def tile_nodes(n, idx, shape):
    """Distinct nodes of every tile of `shape` points (idx [G, k], x fastest)."""
    c = np.stack(np.unravel_index(np.arange(idx.shape[0]), n[::-1])[::-1], 1) // np.asarray(shape)
    tile = np.zeros(idx.shape[0], np.int64)
    for a in reversed(range(len(n))):
        tile = tile * (-(-n[a] // shape[a])) + c[:, a]
    key = np.unique(tile[:, None] * (idx.max() + 1) + idx)
    return np.bincount(key // (idx.max() + 1))


def refined(n, h, sparse):
    """A cloud of ordinary density, or sparse nodes, refined in one corner."""
    d = len(n)
    e = 1.5 if sparse else 1.0
    x = inputs.jittered_lattice(tuple(int(v / e) for v in n), tuple(
        v * h / int(v / e) for v in n), 8, 0.3)
    fine = inputs.jittered_lattice((32 * 4, 8 * 4) if d == 2 else (32, 12, 12),
                                   (h / (4 if d == 2 else 2),) * d, 9, 0.3)
    corner = np.array([32, 8] if d == 2 else [16, 6, 6])[:, None] * h
    return np.concatenate([x[:, ~(x < corner).all(0)], fine], axis=1)


@pytest.mark.parametrize("n,bc,kg,sparse", [
    ((64, 24), (PER, N), 32, False), ((64, 24), (N, N), 27, False),
    ((16, 16, 16), (N, PER, N), 27, False), ((32, 16, 16), (N, N, N), 20, False),
    ((128, 48), (N, PER), 16, True), ((128, 48), (N, N), 32, True),
    ((24, 16, 16), (PER, N, N), 27, True), ((24, 16, 16), (N, N, N), 32, True),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) and isinstance(v[0], int) else None)
def test_tiles_without_a_list(pc, n, bc, kg, sparse):
    """The refined tiles hold more nodes than the longest list (2048 or 1365).
    With fewer nodes than grid points in all (sparse) nothing is allowed for
    their coefficients and their entries are gathered."""
    d, h = len(n), 1.0 / n[0]
    grid = Grid(d, n, (h,) * d, bc)
    x = refined(n, h, sparse)
    G, M = grid.G, x.shape[1]
    assert M <= (5 if d == 2 else 2) * G  # rows are kept
    kind = np.zeros(M, np.uint8)
    kind[::11] = inputs.KIND_B
    st = P.build_stencils(grid, x.T.copy(), kind, kg, 16 if d == 2 else 27)
    nodes = tile_nodes(n, st.grid_idx, (32, 8) if d == 2 else (16, 4, 4))
    assert nodes.max() > (2048 if d == 2 else 1365) and nodes.min() < 853
    allowed = max(0, M - G) // 1024 if d == 2 else max(0, M - G - G // 32) // 213
    assert (allowed == 0) == sparse
    # nodes a quarter or half a spacing apart under a support of three: the
    # normal matrices' rounding is about (3 / 0.8)^4 = 200 times the usual
    geom = check_divergence(pc, n, h, bc, x, kind, kg, tol=1e-11)
    plan = pc.Plan(d, n, (h,) * d, bc=bc)
    held = pc.geom_footprint(plan, M, geom.n_ib, geom.n_near, kg, 16 if d == 2 else 27,
                             want_f32=True)[0]
    assert geom.bytes <= held


def test_dense_tiles_of_a_large_grid(pc):
    """More than 2048 3D tiles, few of them with more than 853 nodes: these keep
    coefficients, as the geometry's size shows, and the divergence is that of
    the exported coefficients."""
    import torch
    n, h, k = (144, 64, 64), 1.0 / 64, 27
    G = int(np.prod(n))
    x = inputs.jittered_lattice(n, (h,) * 3, 8, 0.3)
    fine = inputs.jittered_lattice((24, 12, 12), (h * 2 / 3,) * 3, 9, 0.3)
    corner = np.array([16, 8, 8])[:, None] * h
    x = np.concatenate([x[:, ~(x < corner).all(0)], fine], axis=1)
    M = x.shape[1]
    kind = np.zeros(M, np.uint8)
    plan = pc.Plan(3, n, (h,) * 3)
    geom = pc.wls_build(plan, torch.from_numpy(x).cuda(), torch.from_numpy(kind).cuda(), k, 27)
    gi = torch.empty((k, G), dtype=torch.int32, device="cuda")
    gc = torch.empty((3, k, G), dtype=torch.float64, device="cuda")
    pc.geom_export(geom, gi, gc)
    nodes = tile_nodes(n, to_np(gi).T.astype(np.int64), (16, 4, 4))
    dense, allowed = int((nodes > 853).sum()), (M - G) // 64
    assert nodes.size > 2048 and 0 < dense <= min(allowed, nodes.size // 16)
    assert nodes.max() <= 1365
    held = pc.geom_footprint(plan, M, 0, 0, k, 27)[0]
    assert held - geom.bytes == (allowed - dense) * 3 * k * 256 * 8
    u = torch.randn(3, M, dtype=torch.float64, device="cuda")
    b = torch.empty(G, dtype=torch.float64, device="cuda")
    pc.div_to_grid(geom, u, b)
    ref = (gc * u[:, gi.long()]).sum((0, 1))
    assert rel_l2(to_np(b), to_np(ref)) <= 1e-14


@pytest.mark.parametrize("n,bc,kg", [((4000, 8), (PER, N), 16), ((4000, 8), (N, N), 16),
                                     ((4000, 8), (PER, PER), 20), ((4000, 8), (PER, N), 12),
                                     ((2000, 8, 8), (PER, N, N), 27), ((2000, 8, 8), (N, N, N), 20)],
                         ids=["2d_per", "2d", "2d_k20_per", "2d_k12_per", "3d_per", "3d_k20"])
def test_offsets_are_those_of_the_rows(pc, n, bc, kg):
    """Far from the origin the offset of a node from a grid point keeps the
    rounding of the grid point's position that the rows were built with.  An
    offset with that product unrounded is off by up to half an ulp of the box,
    2e-13 of a spacing at 4000 points (no power of two: its points are rounded),
    and takes the divergence as far; the rest of either side's rounding is a
    tenth of that."""
    x, kind = lattice(n, 1.0 / n[0], 8)
    d, h = len(n), 1.0 / n[0]
    import torch
    grid = Grid(d, n, (h,) * d, bc)
    st = P.build_stencils(grid, x.T.copy(), kind, kg, 16 if d == 2 else 27)
    plan = pc.Plan(d, n, (h,) * d, bc=bc)
    geom = pc.wls_build(plan, torch.from_numpy(x.copy()).cuda(), torch.from_numpy(kind).cuda(),
                        kg, 16 if d == 2 else 27)
    u = np.random.Generator(np.random.PCG64(4)).standard_normal(x.shape)
    b = torch.empty(plan.G, dtype=torch.float64, device="cuda")
    pc.div_to_grid(geom, torch.from_numpy(u).cuda(), b)
    e = rel_l2(to_np(b), P.div_to_grid(st, u.T))
    print("relative difference", e)
    assert e <= 1e-13
