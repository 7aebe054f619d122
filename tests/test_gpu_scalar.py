"""GPU parity of the scalar (one unknown per cell) path -- the paper's Poisson
Equation example, GMRES(30) with RAS (overlap one, ILU(0) per subdomain) --
against the oracle's scalar routines, through the C ABI.  Bars as for the
block path: the product per entry within 1e-12 of |A||x|; ILU(0) and RAS
applies per entry within 1e-12 of the largest entry; solves reach a
recomputed relative residual <= 1e-8, agree with the oracle's solution to
1e-6 and its first ten residual estimates to 1e-8."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1602_05901_amd import inputs as I  # noqa: E402
import oracle as O  # noqa: E402
from oracle import scalar as S  # noqa: E402

pytestmark = pytest.mark.gpu


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def rsv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_05901_amd import rsv as R
    R.lib()
    return R


@pytest.fixture(scope="module")
def ctx(rsv):
    c = rsv.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def system(dims, sigma=0.0, seed=0):
    cfg = I.GenConfig(*dims, I.LNK_IID, sigma, 0.0, 0.0, 0, 1e3, 1.0, seed)
    C = I.poisson(cfg, I.lnk(cfg) if sigma > 0 else None)
    return cfg, C, S.CSR(*dims, C)


class Sys:
    def __init__(self, rsv, ctx, dims, sigma=0.0, seed=0):
        self.cfg, self.C, self.Ao = system(dims, sigma, seed)
        self.g = rsv.Grid(ctx, *dims)
        self.A = rsv.Matrix(self.g, dev(self.C), scalar=True)
        self.n = self.cfg.ncell

    def close(self):
        self.A.close()
        self.g.close()


GRIDS = [(8, 8, 8), (13, 9, 5), (1, 1, 7), (7, 1, 1), (17, 3, 19), (32, 32, 16), (3, 2, 2)]


@pytest.mark.parametrize("dims", GRIDS)
@pytest.mark.parametrize("sigma", [0.0, 2.0])
def test_scalar_spmv_per_entry(rsv, ctx, dims, sigma):
    T = Sys(rsv, ctx, dims, sigma, 1)
    x = I.test_vector(2, T.n)
    y0 = I.test_vector(3, T.n)
    y = dev(y0)
    T.A.spmv(dev(x), y, alpha=0.5, beta=-2.0)
    ref = 0.5 * T.Ao.spmv(x) - 2.0 * y0
    scale = 0.5 * S.CSR(*dims, np.abs(T.C)).spmv(np.abs(x)) + 2.0 * np.abs(y0)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 1e-12 * scale)
    ynn = torch.zeros_like(y)
    T.A.spmv_noalloc(dev(x), ynn)
    assert np.all(np.abs(ynn.cpu().numpy() - T.Ao.spmv(x)) <= 1e-12 * scale / 0.5)
    T.close()


@pytest.mark.parametrize("dims,parts", [((6, 5, 4), (2, 2, 2)), ((37, 9, 6), (2, 1, 2))])
def test_scalar_top_down_numbering(rsv, ctx, dims, parts):
    # the second grid puts several 8-cell x-chunks in a row of every subdomain
    nx, ny, nz = dims
    cfg, C, Ao = system(dims, 1.0, 3)
    c = np.arange(cfg.ncell)
    perm = ((nz - 1 - c // (nx * ny)) * ny + (c // nx) % ny) * nx + c % nx
    # a row's coefficients toward -z and +z swap roles in top-down numbering? no: slots follow the
    # cell's directions, so the rows are only permuted
    Ct = np.empty_like(C)
    Ct[perm] = C
    g = rsv.Grid(ctx, *dims, rsv.TOP_DOWN)
    A = rsv.Matrix(g, dev(Ct), scalar=True)
    x = I.test_vector(9, cfg.ncell)
    xt = np.empty_like(x)
    xt[perm] = x
    y = torch.zeros(cfg.ncell, dtype=torch.float64, device="cuda")
    A.spmv(dev(xt), y)
    assert np.allclose(y.cpu().numpy()[perm], Ao.spmv(x), rtol=1e-13, atol=1e-13)
    M = rsv.Precond(A, type=rsv.PC_RAS, ras_px=parts[0], ras_py=parts[1], ras_pz=parts[2], ras_overlap=1)
    r = I.test_vector(10, cfg.ncell)
    rt = np.empty_like(r)
    rt[perm] = r
    z = torch.zeros_like(y)
    M.apply(dev(rt), z)
    ref = S.RAS(Ao, dims, parts, 1).apply(r)
    assert np.max(np.abs(z.cpu().numpy()[perm] - ref)) <= 1e-12 * np.max(np.abs(ref))
    M.close(); A.close(); g.close()


@pytest.mark.parametrize("dims", GRIDS)
def test_scalar_ilu0_apply(rsv, ctx, dims):
    T = Sys(rsv, ctx, dims, 1.5, 4)
    M = rsv.Precond(T.A, type=rsv.PC_BILU0)
    r = I.test_vector(5, T.n)
    z = torch.zeros(T.n, dtype=torch.float64, device="cuda")
    M.apply(dev(r), z)
    ref = S.ILU(T.Ao).apply(r)
    assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    M.close(); T.close()


@pytest.mark.parametrize("dims,parts,ov", [((20, 20, 10), (2, 2, 2), 1), ((13, 9, 5), (3, 2, 1), 1),
                                           ((16, 16, 8), (4, 4, 4), 1), ((12, 10, 6), (2, 2, 2), 2),
                                           ((12, 10, 6), (2, 3, 1), 0), ((10, 1, 1), (3, 1, 1), 1),
                                           ((33, 29, 11), (4, 3, 2), 1), ((9, 9, 9), (9, 9, 9), 0)])
@pytest.mark.parametrize("sigma", [0.0, 2.0])
def test_scalar_ras_apply(rsv, ctx, dims, parts, ov, sigma):
    T = Sys(rsv, ctx, dims, sigma, 6)
    M = rsv.Precond(T.A, type=rsv.PC_RAS, ras_px=parts[0], ras_py=parts[1], ras_pz=parts[2], ras_overlap=ov)
    r = I.test_vector(7, T.n)
    z = torch.zeros(T.n, dtype=torch.float64, device="cuda")
    M.apply(dev(r), z)
    ref = S.RAS(T.Ao, dims, parts, ov).apply(r)
    assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    M.close(); T.close()


def run(rsv, T, pc_kw, oracle_pc, method="gmres", restart=30, tol=1e-8, maxit=3000):
    xt = I.x_true_scalar(T.cfg)
    bo = T.Ao.spmv(xt)
    b = dev(bo)
    M = rsv.Precond(T.A, **pc_kw) if pc_kw else None
    x = torch.zeros_like(b)
    st = rsv.solve(T.A, M, b, x, method=(rsv.GMRES if method == "gmres" else rsv.BICGSTAB), restart=restart,
                   tol=tol, maxit=maxit, record_history=1)
    xg = x.cpu().numpy()
    relres = np.linalg.norm(bo - T.Ao.spmv(xg)) / np.linalg.norm(bo)
    if method == "gmres":
        ref = S.gmres(T.Ao, bo, pc=oracle_pc, m=restart, tol=tol, maxit=maxit, hist=True)
    else:
        ref = S.bicgstab(T.Ao, bo, pc=oracle_pc, tol=tol, maxit=maxit, hist=True)
    if M is not None:
        M.close()
    return st, ref, xg, xt, relres


@pytest.mark.parametrize("dims,parts", [((32, 32, 32), (2, 2, 2)), ((24, 20, 16), (3, 2, 2)), ((20, 20, 10), (1, 1, 1))])
@pytest.mark.parametrize("sigma", [0.0, 2.0])
def test_scalar_gmres_ras_against_oracle(rsv, ctx, dims, parts, sigma):
    T = Sys(rsv, ctx, dims, sigma, 8)
    st, ref, xg, xt, relres = run(rsv, T, dict(type=rsv.PC_RAS, ras_px=parts[0], ras_py=parts[1], ras_pz=parts[2],
                                               ras_overlap=1), S.RAS(T.Ao, dims, parts, 1))
    log("scalar gmres", dims, parts, sigma, "its", st["its"], ref["its"], "relres", relres)
    assert st["status"] == 0 and ref["rc"] == 0 and relres <= 1e-8
    assert abs(st["final_relres"] - relres) <= 1e-3 * relres + 1e-15
    assert rel(xg, ref["x"]) <= 1e-6
    assert abs(st["its"] - ref["its"]) <= max(2, 0.05 * ref["its"])
    k = min(10, len(st["hist"]), len(ref["hist"]))
    assert np.allclose(st["hist"][:k], ref["hist"][:k], rtol=1e-8, atol=0)
    T.close()


def test_scalar_bicgstab_and_unpreconditioned(rsv, ctx):
    dims = (24, 20, 16)
    T = Sys(rsv, ctx, dims, 1.0, 9)
    st, ref, xg, xt, relres = run(rsv, T, dict(type=rsv.PC_RAS, ras_px=2, ras_py=2, ras_pz=2, ras_overlap=1),
                                  S.RAS(T.Ao, dims, (2, 2, 2), 1), method="bicgstab")
    assert st["status"] == 0 and relres <= 1e-8 and rel(xg, ref["x"]) <= 1e-6
    k = min(6, len(st["hist"]), len(ref["hist"]))
    assert np.allclose(st["hist"][:k], ref["hist"][:k], rtol=1e-8, atol=0)
    st, ref, xg, xt, relres = run(rsv, T, None, None, maxit=5000)
    assert st["status"] == 0 and relres <= 1e-8 and rel(xg, ref["x"]) <= 1e-6
    T.close()


def test_scalar_errors(rsv, ctx):
    dims = (5, 4, 3)
    cfg, C, _ = system(dims)
    g = rsv.Grid(ctx, *dims)
    bad = C.copy()
    bad[0, 2] = -1.0                      # toward a missing -x neighbour
    with pytest.raises(rsv.RsvError) as e:
        rsv.Matrix(g, dev(bad), scalar=True)
    assert e.value.status == rsv.ERR_PATTERN
    bad = C.copy()
    bad[7, 3] = np.inf
    with pytest.raises(rsv.RsvError) as e:
        rsv.Matrix(g, dev(bad), scalar=True)
    assert e.value.status == rsv.ERR_NAN
    zp = C.copy()
    zp[0, 3] = 0.0
    A = rsv.Matrix(g, dev(zp), scalar=True)
    with pytest.raises(rsv.RsvError) as e:
        rsv.Precond(A, type=rsv.PC_BILU0)
    assert e.value.status == rsv.ERR_ZERO_PIVOT and e.value.bad_cell == 0
    A.close()
    A = rsv.Matrix(g, dev(C), scalar=True)
    for kw in (dict(type=rsv.PC_BILU0, precision=rsv.FP32), dict(type=rsv.PC_RAS, ras_px=9),
               dict(type=rsv.PC_LEARNED)):
        with pytest.raises(rsv.RsvError):
            rsv.Precond(A, **kw)
    A.close(); g.close()


@pytest.mark.parametrize("pipelined", [1, 0])   # tile columns; one workgroup per subdomain
@pytest.mark.parametrize("dims,parts,ov,ordering", [
    ((16, 16, 1), (2, 2, 1), 1, 0),      # one layer: shorter than the diagonal ramp and the load lead
    ((24, 17, 3), (1, 1, 1), 0, 1), ((40, 33, 15), (2, 2, 1), 3, 0), ((33, 47, 16), (2, 3, 1), 1, 1),
    ((64, 9, 70), (3, 1, 2), 2, 0), ((50, 50, 50), (3, 3, 3), 1, 1),
    ((70, 20, 20), (2, 2, 2), 25, 0),    # an overlap wider than a box's neighbour
    ((12, 12, 12), (6, 6, 6), 1, 0), ((9, 8, 7), (9, 8, 7), 1, 0)])    # boxes far below a tile
def test_scalar_ras_tile_columns(rsv, ctx, dims, parts, ov, ordering, pipelined):
    """The tile-column sweeps at the edges of their work division, in both
    numberings, twice on the same buffers (the face words' epochs move on)."""
    log("tile columns", dims, parts, ov, ordering, pipelined)
    nx, ny, nz = dims
    cfg, C, Ao = system(dims, 2.0, 12)
    c = np.arange(cfg.ncell)
    perm = ((nz - 1 - c // (nx * ny)) * ny + (c // nx) % ny) * nx + c % nx if ordering else c
    Ct = np.empty_like(C)
    Ct[perm] = C
    g = rsv.Grid(ctx, *dims, ordering)
    A = rsv.Matrix(g, dev(Ct), scalar=True)
    M = rsv.Precond(A, type=rsv.PC_RAS, ras_px=parts[0], ras_py=parts[1], ras_pz=parts[2], ras_overlap=ov,
                    pipelined=pipelined)
    R = S.RAS(Ao, dims, parts, ov)
    for q in range(2):
        r = I.test_vector(20 + q, cfg.ncell)
        rt = np.empty_like(r)
        rt[perm] = r
        z = torch.full((cfg.ncell,), 9.0, dtype=torch.float64, device="cuda")
        M.apply(dev(rt), z)
        ref = R.apply(r)
        assert np.max(np.abs(z.cpu().numpy()[perm] - ref)) <= 1e-12 * np.max(np.abs(ref))
    M.close(); A.close(); g.close()


def test_scalar_wait_limit_reports_timeout_and_recovers(rsv, ctx):
    """A wait bound of 0.1 us, set from the host, makes the tile columns' waits
    give up: the apply says so and the next one is right."""
    T = Sys(rsv, ctx, (64, 64, 64), 1.0, 13)
    M = rsv.Precond(T.A, type=rsv.PC_RAS, ras_px=1, ras_py=1, ras_pz=1, ras_overlap=0)
    r = I.test_vector(22, T.n)
    z = torch.zeros(T.n, dtype=torch.float64, device="cuda")
    ctx.set_wait_limit(1e-7)
    try:
        with pytest.raises(rsv.RsvError) as e:
            M.apply(dev(r), z)
        assert e.value.status == rsv.ERR_TIMEOUT
    finally:
        ctx.set_wait_limit(2.0)
    M.apply(dev(r), z)
    ref = S.ILU(T.Ao).apply(r)
    assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    M.close(); T.close()


@pytest.mark.parametrize("dims,parts,ov,ordering", [
    ((200, 150, 1), (1, 1, 1), 0, 0), ((150, 140, 2), (2, 1, 1), 2, 0),      # planes over some diagonals of tiles
    ((60, 60, 40), (1, 1, 1), 0, 1), ((100, 90, 9), (2, 2, 1), 1, 1),        # over all tiles of a box
    ((32, 32, 7), (1, 1, 1), 0, 1), ((70, 66, 6), (2, 2, 1), 1, 0), ((1, 1, 300), (1, 1, 3), 2, 0)])   # one workgroup per box
def test_scalar_factor_planes(rsv, ctx, dims, parts, ov, ordering):
    """The factorisation's launches at the shapes of their rules."""
    test_scalar_ras_tile_columns(rsv, ctx, dims, parts, ov, ordering, 1)


def test_scalar_set_up_of_wide_grids(rsv, ctx):
    """Set-up of the tile columns on one wide layer takes at most twice that of
    the form with one workgroup per subdomain."""
    import time
    n = 4096
    C = torch.full((n * n, 7), -1.0, device="cuda", dtype=torch.float64)
    C[:, 3] = 6.0
    C[:, 0] = C[:, 6] = 0.0
    C = C.view(n, n, 7)
    C[0, :, 1] = C[-1, :, 5] = 0.0
    C[:, 0, 2] = C[:, -1, 4] = 0.0
    g = rsv.Grid(ctx, n, n, 1)
    A = rsv.Matrix(g, C.view(-1, 7), scalar=True)

    def set_up(pipelined):
        best = 1e9
        for _ in range(3):
            t0 = time.perf_counter()
            M = rsv.Precond(A, type=rsv.PC_RAS, ras_px=4, ras_py=4, ras_pz=1, ras_overlap=1, pipelined=pipelined)
            best = min(best, time.perf_counter() - t0)
            M.close()
        return best

    tiles, chunks = set_up(1), set_up(0)
    log("set-up ms: tile columns %.1f, one workgroup per subdomain %.1f" % (tiles * 1e3, chunks * 1e3))
    assert tiles <= 2 * chunks
    A.close(); g.close()


@pytest.mark.parametrize("dims,parts", [((20000, 8, 1), (1, 1, 1)), ((100000, 1, 1), (64, 1, 1)), ((64, 64, 64), (4, 4, 4))])
def test_scalar_apply_of_thin_boxes(rsv, ctx, dims, parts):
    """The default form's apply takes at most 1.5 times that of one workgroup
    per subdomain, also on boxes a layer thin and long in x."""
    import time
    T = Sys(rsv, ctx, dims, 0.0, 14)
    r = dev(I.test_vector(23, T.n))
    z = torch.zeros_like(r)

    def apply_time(pipelined):
        M = rsv.Precond(T.A, type=rsv.PC_RAS, ras_px=parts[0], ras_py=parts[1], ras_pz=parts[2], ras_overlap=1,
                        pipelined=pipelined)
        best = 1e9
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            M.apply(r, z)
            best = min(best, time.perf_counter() - t0)
        M.close()
        return best

    default, chunks = apply_time(1), apply_time(0)
    log("thin boxes", dims, parts, "us: default %.0f, one workgroup per subdomain %.0f" % (default * 1e6, chunks * 1e6))
    assert default <= 1.5 * chunks
    T.close()


def test_scalar_wait_that_gave_up_is_remembered(rsv, ctx):
    """After one wait has given up the sweeps go on without waiting: with a
    bound of 0.1 us an apply comes back with its error sooner than an ordinary
    apply with its result, whose tiles wait for one another's faces."""
    import time
    T = Sys(rsv, ctx, (128, 128, 128), 0.0, 15)
    M = rsv.Precond(T.A, type=rsv.PC_BILU0)
    r = dev(I.test_vector(24, T.n))
    z = torch.zeros_like(r)

    def apply_time(status):
        best = 1e9
        for _ in range(8):
            got = 0
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            try:
                M.apply(r, z)
            except rsv.RsvError as e:
                got = e.status
            best = min(best, time.perf_counter() - t0)
            assert got == status
        return best

    whole = apply_time(0)
    ctx.set_wait_limit(1e-7)
    try:
        error = apply_time(rsv.ERR_TIMEOUT)
    finally:
        ctx.set_wait_limit(2.0)
    log("us: apply %.0f, to the error %.0f" % (whole * 1e6, error * 1e6))
    assert error <= 0.8 * whole
    assert apply_time(0) < 1e9
    M.close(); T.close()
