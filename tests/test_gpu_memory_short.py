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
