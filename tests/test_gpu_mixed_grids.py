"""GPU: batches of different grids, whose groups run side by side.

Solutions have the bits of the same systems one by one; right-hand sides
written on the call's stream just before and solutions read on it just after
are in order; several threads and streams at once change nothing.
"""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = [(33, 40), (101, 77), (33, 40), (48, 61), (150, 40), (65, 65), (24, 24), (41, 140)]   # 24 x 24: by blocks


@pytest.fixture(scope="module")
def helm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_10762_amd import helm as h
    h.lib()
    return h


def _systems(helm):
    rng = np.random.default_rng(8)
    Gs = [helm.Grid(nx, nz, 0.025, 0.025) for nx, nz in GRIDS]
    ms = [torch.as_tensor(1.0 / (1.5 + 3.0 * rng.random(G.N)) ** 2, device="cuda") for G in Gs]
    ws = [2 * np.pi * 1.5 / (p * 0.025) for p in np.linspace(8.0, 14.0, len(Gs))]
    Bs = [torch.as_tensor(rng.standard_normal((3 + q, G.N)) + 1j * rng.standard_normal((3 + q, G.N)), device="cuda")
          for q, G in enumerate(Gs)]
    return Gs, ms, ws, Bs


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("tol", [0.0, 1e-10])
def test_batch_has_the_bits_of_single_calls(helm, precision, tol):
    Gs, ms, ws, Bs = _systems(helm)
    want = []
    for G, m, w, B in zip(Gs, ms, ws, Bs):
        F = helm.factor(G, m, w, precision)
        want.append((F.solve(B, tol=tol)[0], F.adjoint_solve(B, tol=tol)[0]))
        F.close()
    torch.cuda.synchronize()
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(3):
                Fs = helm.factor_batch(Gs, ms, ws, precision)
                for adjoint in (False, True):
                    late = [torch.full_like(B, complex(np.nan, 0.0)) for B in Bs]
                    torch.cuda._sleep(200_000)
                    for a, b in zip(late, Bs):
                        a.copy_(b)
                    Xs, _ = helm.solve_batch(Fs, late, adjoint=adjoint, tol=tol)
                    copies = [X.clone() for X in Xs]
                    for X in Xs:
                        X.fill_(0)
                    bad.extend((k, q, adjoint) for q, X in enumerate(copies) if not torch.equal(X, want[q][adjoint]))
                for F in Fs:
                    F.close()

    work(0)
    ts = [threading.Thread(target=work, args=(k,)) for k in (1, 2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
