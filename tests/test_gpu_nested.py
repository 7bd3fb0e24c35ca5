"""GPU: nested-dissection factors and solves against the FP64 oracle.

Small grids just above the size where the block factorisation hands over
(33 x 33; 96 x 33, as wide as that may be), odd and long rectangles in both directions (ring sides missing on one, two
and three sides; separators of 16k, 16k + 1 and 32k + 1 nodes; leaves of every
shape), one and 19 right-hand sides, forward and adjoint, in both precisions.
Solutions are held to 1e-9 per column, the bound of the other parity tests
(their conditioning is the same); residuals to the tolerance asked for.  A
batch, a forced partial pivoting in every tile, a plain complex128 solve and
the allocation-free solve are checked on the same grids.
"""
import numpy as np
import pytest

import oracle
from tests.parity import assert_cols

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = [(33, 33), (96, 33), (65, 65), (67, 77), (130, 51), (41, 140), (401, 37), (97, 129)]


@pytest.fixture(scope="module")
def helm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_10762_amd import helm as h
    h.lib()
    yield h
    h.set_tile_pivoting(False)


def _system(nx, nz, S, ppw=9.0):
    rng = np.random.default_rng(nx * 1000 + nz + S)
    h = 0.025
    m = 1.0 / (1.5 + 3.0 * rng.random(nx * nz)) ** 2
    B = rng.standard_normal((S, nx * nz)) + 1j * rng.standard_normal((S, nx * nz))
    return m, 2 * np.pi * 1.5 / (ppw * h), B, h


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("nx,nz", GRIDS)
def test_nested_matches_oracle(helm, nx, nz, precision):
    for S in (1, 19):
        print(f"{nx}x{nz}, {S} columns, {precision}", flush=True)
        m, w, B, h = _system(nx, nz, S)
        G, Bd = helm.Grid(nx, nz, h, 0.9 * h), torch.as_tensor(B, device="cuda")
        Fo = oracle.Factor(oracle.Grid(nx, nz, h, 0.9 * h), m, w)
        Xo, Lo = Fo.solve(B), Fo.adjoint_solve(B)
        Fo.close()
        F = helm.factor(G, m, w, precision)
        X, info = F.solve(Bd, tol=1e-10)
        L, ainfo = F.adjoint_solve(Bd, tol=1e-10)
        assert info.max_relres <= 1e-10 and ainfo.max_relres <= 1e-10
        assert_cols(X.cpu().numpy(), Xo, 1e-9, what="forward")
        assert_cols(L.cpu().numpy(), Lo, 1e-9, what="adjoint")
        Xn = torch.full_like(Bd, complex(np.nan, np.nan))
        helm.solve_noalloc(F, Bd, Xn, tol=1e-10)
        assert torch.equal(Xn, X)
        Xp, _ = F.solve(Bd)
        assert_cols(Xp.cpu().numpy(), Xo, 1e-9, what="no tolerance")
        F.close()
        # with a second frequency and another block of columns in the batch: bitwise the same
        Fs = helm.factor_batch([G, G], [m, m], [w, 0.7 * w], precision)
        Xb, _ = helm.solve_batch(Fs, [Bd, Bd[:1].repeat(3, 1)], tol=1e-10)
        assert torch.equal(Xb[0], X)
        for F in Fs:
            F.close()


@pytest.mark.parametrize("nx,nz", [(65, 65), (41, 140)])
def test_nested_forced_tile_pivoting(helm, nx, nz):
    m, w, B, h = _system(nx, nz, 5)
    Fo = oracle.Factor(oracle.Grid(nx, nz, h, h), m, w)
    Xo = Fo.solve(B)
    Fo.close()
    helm.set_tile_pivoting(True)
    try:
        F = helm.factor(helm.Grid(nx, nz, h, h), m, w)
    finally:
        helm.set_tile_pivoting(False)
    X, info = F.solve(torch.as_tensor(B, device="cuda"), tol=1e-10)
    F.close()
    assert info.max_relres <= 1e-10
    assert_cols(X.cpu().numpy(), Xo, 1e-9, what="forced pivoting")


def _excess(helm, G, m, w, B, X, adjoint=False):
    """Largest column's ||b - A x|| over eps max(N^(1/4), 8) (||x|| + ||b|| / 4)."""
    n = helm.residual(G, m, w, B, X, adjoint=adjoint)[1].cpu().numpy()
    x = torch.linalg.vector_norm(X, dim=1).cpu().numpy()
    return float((np.sqrt(n[:, 0]) / (2.0 ** -52 * max(G.N ** 0.25, 8.0) * (x + 0.25 * np.sqrt(n[:, 1])))).max())


# Layered models at 8 to 20 points per wavelength, where boxes of the
# dissection come near resonance.  Block factors leave an excess of 0.8 to 1.2
# in complex128; solves to a tolerance may leave 1.25 or a residual of 2e-14, in
# either precision and direction, for sources and for smooth right-hand sides.
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("nx,nz", [(41, 77), (101, 101), (151, 97), (201, 201), (401, 37)])
def test_nested_as_accurate_as_blocks(helm, nx, nz, precision):
    from paper_2301_10762_amd import inputs as I
    G = helm.Grid(nx, nz, I.H_KM, I.H_KM)
    for seed in range(3):
        mh = (1.0 / I.layered_velocity(nx, nz, seed, I.H_KM) ** 2).reshape(-1)
        m = torch.as_tensor(mh, device="cuda")
        for ppw in (8.0, 9.5, 12.0, 20.0):
            w = I.omega_from_ppw(ppw, I.C_MIN, I.H_KM)
            F = helm.factor(G, m, w, precision)
            B = torch.zeros(3, G.N, dtype=torch.complex128, device="cuda")
            B[0, 2 * nx + nx // 3] = B[1, (nz // 2) * nx + nx // 2] = 1.0
            B[2] = F.solve(B[:1], tol=1e-10)[0][0] * m
            for adjoint in (False, True):
                X, info = (F.adjoint_solve if adjoint else F.solve)(B, tol=1e-10)
                ex = _excess(helm, G, m, w, B, X, adjoint)
                print(f"{nx}x{nz} {precision} seed {seed} ppw {ppw}: excess {ex:.2f}, {info.ir_iters} corrections",
                      flush=True)
                assert ex <= 1.25 or info.max_relres <= 2e-14
            F.close()


# The same without a tolerance in complex128, where the factor decides on
# corrections: twice what block factors leave.
@pytest.mark.parametrize("nx,nz", [(41, 77), (101, 101), (151, 97), (201, 201), (401, 37)])
def test_nested_plain_as_accurate_as_blocks(helm, nx, nz):
    from paper_2301_10762_amd import inputs as I
    G = helm.Grid(nx, nz, I.H_KM, I.H_KM)
    for seed in range(3):
        mh = (1.0 / I.layered_velocity(nx, nz, seed, I.H_KM) ** 2).reshape(-1)
        m = torch.as_tensor(mh, device="cuda")
        for ppw in (8.0, 9.5, 12.0, 20.0):
            w = I.omega_from_ppw(ppw, I.C_MIN, I.H_KM)
            F = helm.factor(G, m, w)
            B = torch.zeros(3, G.N, dtype=torch.complex128, device="cuda")
            B[0, 2 * nx + nx // 3] = B[1, (nz // 2) * nx + nx // 2] = 1.0
            B[2] = F.solve(B[:1])[0][0] * m
            for adjoint in (False, True):
                X, info = (F.adjoint_solve if adjoint else F.solve)(B)
                ex = _excess(helm, G, m, w, B, X, adjoint)
                print(f"{nx}x{nz} plain seed {seed} ppw {ppw}: excess {ex:.2f}, {info.ir_iters} corrections", flush=True)
                assert ex <= 2.0
            F.close()


def test_nested_plain_close_to_resonance(helm):
    """A model whose plain solves are off by 3e-7 before, and 5e-13 after one correction."""
    from paper_2301_10762_amd import inputs as I
    n = 301
    G = helm.Grid(n, n, I.H_KM, I.H_KM)
    m = torch.as_tensor((1.0 / I.layered_velocity(n, n, 0, I.H_KM) ** 2).reshape(-1), device="cuda")
    w = I.omega_from_ppw(9.53957342752774, I.C_MIN, I.H_KM)
    B = torch.zeros(3, G.N, dtype=torch.complex128, device="cuda")
    B[torch.arange(3), 2 * n + torch.tensor([20, 150, 270])] = 1.0
    F = helm.factor(G, m, w)
    X, info = F.solve(B)
    F.close()
    ex = _excess(helm, G, m, w, B, X)
    print(f"excess {ex:.2f}, {info.ir_iters} corrections", flush=True)
    assert ex <= 2.0


# The widest narrow fronts: boxes of 60 to 65 nodes a side with a ring on every
# side (tests/test_plan_host.py holds what their levels ask of a compute unit).
@pytest.mark.parametrize("nx,nz,precision", [(256, 256, "fp64"), (243, 251, "fp32_ir"), (122, 239, "fp64")])
def test_nested_widest_narrow_fronts(helm, nx, nz, precision):
    print(f"{nx}x{nz}, {precision}", flush=True)
    m, w, B, h = _system(nx, nz, 3)
    G, Bd = helm.Grid(nx, nz, h, h), torch.as_tensor(B, device="cuda")
    Fo = oracle.Factor(oracle.Grid(nx, nz, h, h), m, w)
    Xo, Lo = Fo.solve(B), Fo.adjoint_solve(B)
    Fo.close()
    F = helm.factor(G, m, w, precision)
    X, info = F.solve(Bd, tol=1e-10)
    L, ainfo = F.adjoint_solve(Bd, tol=1e-10)
    F.close()
    assert info.max_relres <= 1e-10 and ainfo.max_relres <= 1e-10
    assert_cols(X.cpu().numpy(), Xo, 1e-9, what="forward")
    assert_cols(L.cpu().numpy(), Lo, 1e-9, what="adjoint")
