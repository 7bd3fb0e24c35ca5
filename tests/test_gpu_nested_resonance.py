"""GPU: nested dissection where boxes come near resonance.

The 55 x 55 grid divides into leaves of 6 x 6 nodes (three 16-row tiles, the
last of four nodes); with unit spacing the operator inside a leaf is the
five-point Laplacian less w^2 m, real, so a leaf is brought as near to
singular as wanted through w or through m at its nodes.  Near one, plain
solves take the corrections that the factor counted (w^2 m at a distance d
from the lowest mode: the leaf's inverse has a largest entry of 0.0737 / d, in
its middle tile, which has small pivots and waits for the last); at one the
system is factored row by row.  Solutions are held to 1e-9 per column against
the FP64 oracle, the bound of the other parity tests, residuals of plain solves
to twice what block factors leave: eps N^(1/4) (||x|| + ||b|| / 4).
"""
import math

import numpy as np
import pytest

import oracle
from tests.parity import assert_cols

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 55
LEAF = [(7 + i, 7 + j) for j in range(6) for i in range(6)]   # nodes of an interior leaf, in its order


@pytest.fixture(scope="module")
def helm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_10762_amd import helm as h
    return h


def _rhs(seed, S=5):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((S, N * N)) + 1j * rng.standard_normal((S, N * N))


def _oracle(m, w, B):
    F = oracle.Factor(oracle.Grid(N, N, 1.0, 1.0), m, w)
    out = F.solve(B), F.adjoint_solve(B)
    F.close()
    return out


def _check(helm, F, m, w, Bd, Xo, Lo):
    """Plain and refined solves both ways; returns the corrections of the plain ones."""
    G = helm.Grid(N, N, 1.0, 1.0)
    md = torch.as_tensor(m, device="cuda")
    its = []
    for adjoint, ref in ((False, Xo), (True, Lo)):
        for tol in (0.0, 1e-10):
            X, info = (F.adjoint_solve if adjoint else F.solve)(Bd, tol=tol)
            assert_cols(X.cpu().numpy(), ref, 1e-9, what=f"tol {tol}, adjoint {adjoint}")
            n = helm.residual(G, md, w, Bd, X, adjoint=adjoint)[1].cpu().numpy()
            x = torch.linalg.vector_norm(X, dim=1).cpu().numpy()
            ex = (np.sqrt(n[:, 0]) / (2.0 ** -52 * math.sqrt(N) * (x + 0.25 * np.sqrt(n[:, 1])))).max()
            print(f"tol {tol} adjoint {adjoint}: excess {ex:.2f}, {info.ir_iters} corrections", flush=True)
            if F.precision == 0 or tol > 0.0:
                assert ex <= 2.0 or np.sqrt(n[:, 0] / n[:, 1]).max() <= (2e-14 if F.precision == 0 else 1e-10)
            if tol == 0.0:
                its.append(info.ir_iters)
    return its


def _model(seed, w):
    return (0.2 + 0.15 * np.random.default_rng(seed).random(N * N)) / w ** 2


LOWEST = 4.0 * (1.0 - math.cos(math.pi / 7.0))   # of a 6 x 6 leaf's Laplacian


@pytest.mark.parametrize("d,want", [(1e-4, 1), (7e-6, 2), (7e-7, 3), (1.5e-7, 5), (1e-11, 0), (0.0, 0)])
def test_leaf_near_resonance(helm, d, want):
    """One leaf at a distance d from its lowest mode."""
    w = 0.7
    m, B = _model(7, w), _rhs(1)
    for i, j in LEAF:
        m[j * N + i] = (LOWEST - d) / w ** 2
    Xo, Lo = _oracle(m, w, B)
    F = helm.factor(helm.Grid(N, N, 1.0, 1.0), m, w)
    its = _check(helm, F, m, w, torch.as_tensor(B, device="cuda"), Xo, Lo)
    F.close()
    assert its == [want, want]


@pytest.mark.parametrize("d", [1e-4, 7e-6, 4.6e-7, 4.6e-8, 1e-11, 0.0])
def test_every_box_near_resonance(helm, d):
    """A homogeneous model: all leaves, and the boxes of 13 x 6, 13 x 13 and 27 x 27
    nodes above them, share the mode."""
    w = math.sqrt(LOWEST - d)
    m, B = np.ones(N * N), _rhs(1)
    Xo, Lo = _oracle(m, w, B)
    F = helm.factor(helm.Grid(N, N, 1.0, 1.0), m, w)
    _check(helm, F, m, w, torch.as_tensor(B, device="cuda"), Xo, Lo)
    F.close()


def _laplacian(nodes):
    """Dirichlet five-point Laplacian of some nodes."""
    A = 4.0 * np.eye(len(nodes))
    for a, (i, j) in enumerate(nodes):
        for b, (p, q) in enumerate(nodes):
            if abs(i - p) + abs(j - q) == 1:
                A[a, b] = -1.0
    return A


@pytest.mark.parametrize("tiles", [(0,), (1,), (0, 1), (1, 2), (0, 1, 2)])
def test_leaf_tiles_singular_by_themselves(helm, tiles):
    """Diagonal tiles of a leaf that are singular while the leaf is not: they wait for the others."""
    w = 0.7
    m, B = _model(3, w), _rhs(2)
    for t in tiles:
        part = LEAF[16 * t:16 * t + 16]
        lam = np.linalg.eigvalsh(_laplacian(part))[0]
        for i, j in part:
            m[j * N + i] = lam / w ** 2
    A = _laplacian(LEAF) - w ** 2 * np.diag([m[j * N + i] for i, j in LEAF])
    assert np.abs(np.linalg.eigvalsh(A)).min() > 1e-3
    Xo, Lo = _oracle(m, w, B)
    F = helm.factor(helm.Grid(N, N, 1.0, 1.0), m, w)
    _check(helm, F, m, w, torch.as_tensor(B, device="cuda"), Xo, Lo)
    F.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_singular_leaf_in_a_batch(helm, precision):
    """A leaf whose diagonal vanishes (the grid graph's adjacency, of which six
    eigenvalues are zero) sends its system to the blocks and no other."""
    w = 0.7
    G, B = helm.Grid(N, N, 1.0, 1.0), _rhs(4)
    Bd = torch.as_tensor(B, device="cuda")
    regular, singular = _model(5, w), _model(6, w)
    for i, j in LEAF:
        singular[j * N + i] = 4.0 / w ** 2
    F = helm.factor(G, regular, w, precision)
    alone, _ = F.solve(Bd, tol=1e-10)
    F.close()
    Fs = helm.factor_batch([G] * 3, [regular, singular, regular], [w, w, w], precision)
    Xs, infos = helm.solve_batch(Fs, [Bd] * 3, tol=1e-10)
    assert torch.equal(Xs[0], alone) and torch.equal(Xs[2], alone)
    Xo, Lo = _oracle(singular, w, B)
    its = _check(helm, Fs[1], singular, w, Bd, Xo, Lo)
    if precision == "fp64":
        assert its == [0, 0]
    for F in Fs:
        F.close()
