"""GPU: block sweeps of narrow grids, one workgroup per front and 16 columns.

Widths at the edges of that path (one row tile; 64, 65 and 96 nodes, where
the contraction's split and the number of row tiles change; 97, the first
that takes a launch per step instead), few and many rows (one front, two of
unequal length), 1, 16 and 17 columns, forward and adjoint, both precisions,
against the FP64 oracle.  The bounds are those of the other parity tests:
1e-9 per column at a residual of 1e-10.  A batch with a wide grid in it and
the allocation-free solve give the same bits.
"""
import numpy as np
import pytest

import oracle
from tests.parity import assert_cols

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def helm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_10762_amd import helm as h
    return h


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("nx,nz", [(3, 40), (16, 3), (17, 4), (48, 33), (64, 5), (65, 2), (81, 6), (96, 9), (97, 5)])
def test_narrow_sweeps_match_oracle(helm, nx, nz, precision):
    h = 0.025
    rng = np.random.default_rng(100 * nx + nz)
    m = 1.0 / (1.5 + 3.0 * rng.random(nx * nz)) ** 2
    w = 2 * np.pi * 1.5 / (9.0 * h)
    G = helm.Grid(nx, nz, h, 0.9 * h)
    Fo = oracle.Factor(oracle.Grid(nx, nz, h, 0.9 * h), m, w)
    wide = helm.Grid(113, 4, h, h)
    mw = 1.0 / (1.5 + 3.0 * rng.random(wide.N)) ** 2
    F, Fw = helm.factor(G, m, w, precision), helm.factor(wide, mw, w, precision)
    Bw = torch.as_tensor(rng.standard_normal((3, wide.N)) + 0j, device="cuda")
    for S in (1, 16, 17):
        print(f"{nx}x{nz}, {S} columns, {precision}", flush=True)
        B = rng.standard_normal((S, nx * nz)) + 1j * rng.standard_normal((S, nx * nz))
        Bd = torch.as_tensor(B, device="cuda")
        X, info = F.solve(Bd, tol=1e-10)
        L, ainfo = F.adjoint_solve(Bd, tol=1e-10)
        assert info.max_relres <= 1e-10 and ainfo.max_relres <= 1e-10
        assert_cols(X.cpu().numpy(), Fo.solve(B), 1e-9, what="forward")
        assert_cols(L.cpu().numpy(), Fo.adjoint_solve(B), 1e-9, what="adjoint")
        Xb, _ = helm.solve_batch([Fw, F], [Bw, Bd], tol=1e-10)
        assert torch.equal(Xb[1], X)
        Xn = torch.empty_like(Bd)
        helm.solve_noalloc(F, Bd, Xn, tol=1e-10)
        assert torch.equal(Xn, X)
    Fo.close()
    F.close()
    Fw.close()


# Complex64 blocks lose no digits in the tile inverses: errors of one sweep over
# 24 layered models, geometric mean in units of 2^-24, within a tenth of what
# products added up by themselves give (28.5, 25.5, 191; 49.8, 47.0, 217 where
# each step was rounded at the size of the entry it is added to).
@pytest.mark.parametrize("nx,nz,bound", [(30, 60, 31.4), (33, 30, 28.0), (120, 38, 210.0)])
def test_complex64_blocks_lose_no_digits(helm, nx, nz, bound):
    from paper_2301_10762_amd import inputs as I
    G, logs = helm.Grid(nx, nz, I.H_KM, I.H_KM), []
    for seed in range(24):
        rng = np.random.default_rng(seed)
        m = torch.as_tensor((1.0 / I.layered_velocity(nx, nz, seed, I.H_KM) ** 2).reshape(-1), device="cuda")
        w = I.omega_from_ppw(rng.uniform(9, 30), I.C_MIN, I.H_KM)
        B = torch.zeros(8, G.N, dtype=torch.complex128, device="cuda")
        B[torch.arange(6), 2 * nx + torch.linspace(1, nx - 2, 6).long()] = 1.0
        B[6:] = torch.as_tensor(rng.standard_normal((2, G.N)) + 1j * rng.standard_normal((2, G.N)))
        F = helm.factor(G, m, w, "fp64")
        Y, _ = F.solve(B, tol=1e-14)
        F.close()
        F = helm.factor(G, m, w, "fp32_ir")
        X, info = F.solve(B, tol=1e-3)
        F.close()
        assert info.ir_iters == 0
        logs.append(float(torch.log((X - Y).norm() / Y.norm())))
    mean = float(np.exp(np.mean(logs))) * 2.0 ** 24
    print(f"{nx}x{nz}: {mean:.1f}", flush=True)
    assert mean <= bound
