"""GPU: plans of many grids (one per grid, kept while few and small).

More grids than are kept: solutions stay the oracle's and a grid that comes
back is factored again, from several threads too; and no call waits for work
that other streams have queued.
"""
import threading
import time

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
    h.lib()
    return h


GRIDS = [(nx, nz) for nx in range(33, 50) for nz in range(nx, 50)] + [(nx, nz) for nx in range(33, 46) for nz in range(52, 64)]


def _system(nx, nz):
    rng = np.random.default_rng(nx * 100 + nz)
    B = rng.standard_normal((2, nx * nz)) + 1j * rng.standard_normal((2, nx * nz))
    return 1.0 / (1.5 + 3.0 * rng.random(nx * nz)) ** 2, 2 * np.pi * 1.5 / (9.0 * 0.025), B


def _solve(helm, nx, nz, stream=None):
    m, w, B = _system(nx, nz)
    F = helm.factor(helm.Grid(nx, nz, 0.025, 0.025), m, w, stream=stream)
    X, _ = F.solve(B, tol=1e-10, stream=stream)
    if stream is not None:
        stream.synchronize()
    F.close()
    return X.cpu().numpy()


def test_more_grids_than_are_kept(helm):
    assert len(GRIDS) > 256
    first = {g: _solve(helm, *g) for g in GRIDS}
    for nx, nz in GRIDS[::40]:
        m, w, B = _system(nx, nz)
        Fo = oracle.Factor(oracle.Grid(nx, nz, 0.025, 0.025), m, w)
        assert_cols(first[nx, nz], Fo.solve(B), 1e-9, what=f"{nx}x{nz}")
        Fo.close()
        assert np.array_equal(_solve(helm, nx, nz), first[nx, nz])


def test_grids_from_several_threads(helm):
    want = {g: _solve(helm, *g) for g in GRIDS[:24]}
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for q in range(48):
                g = GRIDS[(7 * q + 5 * k) % 24 if q % 2 else 24 + (q * 4 + k) % 250]
                X = _solve(helm, *g)
                if g in want and not np.array_equal(X, want[g]):
                    bad.append(g)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_new_grids_wait_for_no_other_stream(helm):
    cycles = 1_000_000
    for _ in range(2):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        torch.cuda._sleep(cycles)
        torch.cuda.synchronize()
        each = time.perf_counter() - t0
    cycles = int(cycles * 5.0 / each)   # about five seconds of one busy wavefront
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    _solve(helm, 33, 33, stream=b)
    done = torch.cuda.Event()
    with torch.cuda.stream(a):
        torch.cuda._sleep(cycles)
        done.record()
    with torch.cuda.stream(b):
        torch.zeros(1, device="cuda").add_(1)
    b.synchronize()
    if done.query():
        pytest.skip("the two streams share a hardware queue")
    t0 = time.perf_counter()
    new = [(nx, nz) for nx in range(33, 46) for nz in range(64, 88)]
    for g in new:
        with torch.cuda.stream(b):
            m, w, B = _system(*g)
            F = helm.factor(helm.Grid(*g, 0.025, 0.025), m, w)
            F.close()
    took, waited = time.perf_counter() - t0, done.query()
    print(f"{len(new)} grids in {took:.2f} s", flush=True)
    torch.cuda.synchronize()
    assert not waited
