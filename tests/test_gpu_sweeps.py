"""Pipelined block sweeps at the edges of their steps and tiles: columns shorter
and longer than the ring of operands and than a tile's diagonals, grids of more
tiles than workgroups (a workgroup then goes from tile to tile), ragged tiles,
and 2^21 slots (factors loaded without keeping them in the caches).
Against the sweep by hyperplanes: FP64 runs the same operations in the same
order, so the bits are the same; FP32 lies within 4e-6 of the largest entry
(each is allowed 2e-6 against the FP32 oracle)."""
import pytest

torch = pytest.importorskip("torch")

from paper_1602_05901_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1602_05901_amd import rsv
    c = rsv.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("dims", [(1, 1, 1), (8, 8, 1), (9, 17, 2), (16, 16, 9), (8, 24, 10), (17, 9, 13), (25, 16, 14),
                                  (16, 31, 15), (24, 24, 16), (9, 9, 29), (139, 128, 1), (136, 133, 3), (200, 130, 12),
                                  (131, 270, 21), (128, 128, 128)])
def test_steps_and_tiles(ctx, dims, fp32):
    from paper_1602_05901_amd import rsv
    print("sweeps", dims, fp32, flush=True)
    cfg = I.GenConfig(*dims, I.LNK_IID, 1.0, 0.0, 2.0, 0, 1e3, 1.0, 5)
    g = rsv.Grid(ctx, *dims)
    A = rsv.Matrix(g, torch.from_numpy(I.blocks(cfg)).cuda())
    kw = dict(type=rsv.PC_BILU0, precision=rsv.FP32 if fp32 else rsv.FP64)
    M0, M1 = rsv.Precond(A, pipelined=0, **kw), rsv.Precond(A, pipelined=1, **kw)
    r = torch.from_numpy(I.test_vector(9, 3 * cfg.ncell)).cuda()
    z0 = torch.full_like(r, float("nan"))
    M0.apply(r, z0)
    for _ in range(3):
        z1 = torch.full_like(r, float("nan"))
        M1.apply(r, z1)
        if fp32:
            assert bool(((z1 - z0).abs() <= 4e-6 * z0.abs().max()).all())
        else:
            assert torch.equal(z1, z0)
    M1.close(); M0.close(); A.close(); g.close()


@pytest.mark.parametrize("dims", [(100, 9, 2), (65, 130, 1), (9, 200, 3), (250, 3, 1), (41, 33, 12), (1, 1, 40),
                                  (120, 120, 5), (17, 90, 30)])
def test_planes_of_wide_grids(ctx, dims):
    """Hyperplanes that meet some of the grid's diagonals of tiles, and all of
    them: the factors and the sweeps by hyperplanes against the oracle's, and
    the pipelined sweeps on the same factors.  Entries to 1e-12 of the largest:
    at most 21 products and one 3x3 inverse per cell, in another order, of
    factors whose rows are diagonally dominant."""
    import numpy as np
    import oracle as O
    from paper_1602_05901_amd import rsv
    print("planes", dims, flush=True)
    cfg = I.GenConfig(*dims, I.LNK_IID, 1.0, 0.0, 2.0, 0, 1e3, 1.0, 6)
    B = I.blocks(cfg)
    g = rsv.Grid(ctx, *dims)
    A = rsv.Matrix(g, torch.from_numpy(B).cuda())
    r = I.test_vector(10, 3 * cfg.ncell)
    ref = O.ILU(O.BCSR.from_stencil(*dims, B)).apply(r)
    rd = torch.from_numpy(r).cuda()
    for pipelined in (0, 1):
        M = rsv.Precond(A, type=rsv.PC_BILU0, pipelined=pipelined)
        z = torch.full_like(rd, float("nan"))
        M.apply(rd, z)
        assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
        M.close()
    A.close(); g.close()
