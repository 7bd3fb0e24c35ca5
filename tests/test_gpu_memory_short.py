"""GPU: nested dissection when memory is short.

Factors and solves ask for less at a time and give the same bits: a system is
factored the same way whatever memory was free.  Failures are injected into
the calling thread's allocations (helm_fail_allocations); nothing is exhausted.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def helm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_10762_amd import helm as h
    h.lib()
    yield h
    h.lib().helm_fail_allocations(0, 0)


def _systems(n, nx, nz, S):
    rng = np.random.default_rng(n + nx)
    ms = [1.0 / (1.5 + 3.0 * rng.random(nx * nz)) ** 2 for _ in range(n)]
    B = torch.as_tensor(rng.standard_normal((S, nx * nz)) + 1j * rng.standard_normal((S, nx * nz)), device="cuda")
    return ms, [2 * np.pi * 1.5 / (p * 0.025) for p in np.linspace(8.0, 14.0, n)], B


# Five systems take two allocations each, then the working memory of the group
# is asked for: refused once (two and one at a time are tried) or until single
# systems are left.
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("skip,count", [(10, 1), (11, 1), (10, 2)])
def test_factor_in_smaller_groups(helm, skip, count, precision):
    G = helm.Grid(65, 77, 0.025, 0.025)
    ms, ws, B = _systems(5, 65, 77, 3)
    Fs = helm.factor_batch([G] * 5, ms, ws, precision)
    want, _ = helm.solve_batch(Fs, [B] * 5, tol=1e-10)
    for F in Fs:
        F.close()
    helm.lib().helm_fail_allocations(skip, count)
    Fs = helm.factor_batch([G] * 5, ms, ws, precision)
    helm.lib().helm_fail_allocations(0, 0)
    got, _ = helm.solve_batch(Fs, [B] * 5, tol=1e-10)
    for F, a, b in zip(Fs, got, want):
        assert torch.equal(a, b)
        F.close()


# A solve of 64 columns at 201 x 201 takes the fixed region (or the cache) in
# several pieces; refusing the fourth, and with it the first attempt, leaves
# fewer columns at a time.
@pytest.mark.parametrize("tol", [0.0, 1e-10])
@pytest.mark.parametrize("noalloc", [True, False])
def test_solve_in_fewer_columns(helm, noalloc, tol):
    G = helm.Grid(201, 201, 0.025, 0.025)
    ms, ws, B = _systems(1, 201, 201, 64)
    F = helm.factor(G, ms[0], ws[0])
    want, winfo = F.solve(B, tol=tol)
    X = torch.full_like(B, complex(np.nan, np.nan))
    helm.lib().helm_fail_allocations(4, 1)
    if noalloc:
        info = helm.solve_noalloc(F, B, X, tol=tol)
    else:
        X, info = F.solve(B, tol=tol)
    helm.lib().helm_fail_allocations(0, 0)
    assert torch.equal(X, want) and info.ir_iters == winfo.ir_iters
    F.close()
