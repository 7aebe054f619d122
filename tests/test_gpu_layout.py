"""Layout kernels at the edges of their work division: the caller-order <->
tile-lane moves take 16 rows of an 8x8 tile per workgroup and wrap columns
shorter than 16 cells their own way; assembly takes one row of 64 cells.  A
vector through PC_NONE's apply comes back bit for bit; the assembled matrix is
checked through the product (per entry <= 1e-12 (|A||x|): at most 21 products
and sums in another order)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1602_05901_amd import inputs as I  # noqa: E402
import oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1602_05901_amd import rsv
    c = rsv.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("ordering", [0, 1])
@pytest.mark.parametrize("dims", [(1, 1, 1), (8, 8, 1), (7, 9, 2), (8, 8, 15), (9, 8, 16), (8, 17, 17), (23, 8, 31),
                                  (16, 16, 32), (5, 25, 33), (33, 41, 47)])
def test_moves_and_assembly(ctx, dims, ordering):
    from paper_1602_05901_amd import rsv
    print("layout", dims, ordering, flush=True)
    cfg = I.GenConfig(*dims, I.LNK_IID, 1.0, 0.0, 2.0, 0, 1e3, 1.0, 7)
    B = I.blocks(cfg)
    nx, ny, nz = dims
    x = I.test_vector(11, 3 * cfg.ncell)
    # top-down rows: the same system with the layers in reverse
    flip = (lambda v: np.ascontiguousarray(v.reshape(nz, -1)[::-1]).reshape(v.shape)) if ordering else (lambda v: v)
    g = rsv.Grid(ctx, nx, ny, nz, ordering)
    A = rsv.Matrix(g, torch.from_numpy(flip(B)).cuda())
    M = rsv.Precond(A, type=rsv.PC_NONE)
    xd = torch.from_numpy(flip(x)).cuda()
    z = torch.full_like(xd, -3.0)
    M.apply(xd, z)
    assert torch.equal(z, xd)
    y0 = I.test_vector(12, 3 * cfg.ncell)
    y = torch.from_numpy(flip(y0)).cuda()
    A.spmv(xd, y, alpha=-0.75, beta=2.0)
    ref = -0.75 * O.BCSR.from_stencil(nx, ny, nz, B).spmv(x) + 2.0 * y0
    scale = 0.75 * O.BCSR.from_stencil(nx, ny, nz, np.abs(B)).spmv(np.abs(x)) + 2.0 * np.abs(y0)
    assert np.all(np.abs(flip(y.cpu().numpy()) - ref) <= 1e-12 * scale)
    M.close(); A.close(); g.close()


@pytest.mark.parametrize("ordering", [0, 1])
@pytest.mark.parametrize("dims", [
    (430, 413, 1), (300, 401, 2), (283, 170, 5),      # whole tiles, several to a workgroup
    (97, 131, 16), (113, 98, 15),                     # whole tiles, few workgroups
    (60, 61, 47), (1, 1, 3000), (41, 3, 700),         # chunks of rows, few workgroups
    (161, 90, 33), (3000, 3, 17)])                    # chunks of rows
def test_moves_by_runs(ctx, dims, ordering):
    """The moves of grids above 2^22 / 24 padded cells, which go by x-runs."""
    from paper_1602_05901_amd import rsv
    nx, ny, nz = dims
    assert ((nx + 7) // 8) * ((ny + 7) // 8) * nz * 64 > 2 ** 22 // 24
    test_moves_and_assembly(ctx, dims, ordering)


def test_flat_grid_products_cost_like_a_cubes(ctx):
    """The product of a one-layer grid moves the bytes of a cube's of as many
    cells (less: no vertical neighbours): its time, layout moves
    included, stays below 1.8 times the cube's."""
    import time
    from paper_1602_05901_amd import rsv

    def spmv_time(dims):
        n = dims[0] * dims[1] * dims[2]
        B = torch.zeros((n, 7, 3, 3), device="cuda", dtype=torch.float64)
        B[:, 3] = torch.eye(3, device="cuda", dtype=torch.float64)
        g = rsv.Grid(ctx, *dims)
        A = rsv.Matrix(g, B)
        del B
        x = torch.randn(3 * n, device="cuda", dtype=torch.float64)
        y = torch.zeros_like(x)
        best = 1e9
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            A.spmv(x, y)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        assert torch.equal(x, y)
        A.close(); g.close()
        return best

    flat, cube = spmv_time((2048, 2048, 1)), spmv_time((128, 256, 128))
    print("product us: flat %.0f, cube %.0f" % (flat * 1e6, cube * 1e6), flush=True)
    assert flat <= 1.8 * cube
