"""Where the CGS2 kernels change over from summing the last kernel's partials
themselves to a reduction of its own: padded vectors of 65472 entries (256
blocks, the most one block sums) and of 65664 (257), with 1, 9 and 30 basis
vectors, plain and flexible, against the oracle's CGS2 GMRES: the histories of
the first 20 steps to 1e-8, as for the other unpreconditioned solves."""
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


@pytest.mark.parametrize("restart", [1, 9, 30])
@pytest.mark.parametrize("dims", [(88, 8, 31), (72, 8, 38)])
def test_fold_boundary(ctx, dims, restart):
    from paper_1602_05901_amd import rsv
    print("cgs2", dims, restart, flush=True)
    cfg = I.GenConfig(*dims, I.LNK_IID, 1.0, 0.0, 2.0, 0, 1e3, 1.0, 3)
    B = I.blocks(cfg)
    g = rsv.Grid(ctx, *dims)
    A = rsv.Matrix(g, torch.from_numpy(B).cuda())
    bo = I.test_vector(4, 3 * cfg.ncell)
    b = torch.from_numpy(bo).cuda()
    ref = O.gmres(O.BCSR.from_stencil(*dims, B), bo, pc=None, m=restart, tol=1e-30, maxit=20, hist=True)
    for method in (rsv.GMRES, rsv.FGMRES):
        x = torch.zeros_like(b)
        M = rsv.Precond(A, type=rsv.PC_NONE) if method == rsv.FGMRES else None
        st = rsv.solve(A, M, b, x, method=method, restart=restart, tol=1e-30, maxit=20, record_history=1)
        assert st["its"] == 20
        assert np.allclose(st["hist"][:21], ref["hist"][:21], rtol=1e-8, atol=0)
        if M is not None:
            M.close()
    A.close(); g.close()
