"""Gram-Schmidt, true residual, assembly and sensitivity kernels at the edges of
their tiles and dispatch rules, against NumPy and the oracle's operator.

Tolerances: complex128 sums of m terms of size one are off by about sqrt(m)
roundings of 1.1e-16, and no sum here has more than 5e6 terms, so 1e-12 of the
largest value; complex64 inputs and results round at 6e-8, and the second
Gram-Schmidt pass works on w rounded once: 1e-6."""
import numpy as np
import pytest

import synth
from oracle import Problem as OProblem
from tests.gpu_util import require_gpu, announce

pytestmark = pytest.mark.gpu


def _rc(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,S,k", [(3, 1, 1), (1023, 1, 7), (1025, 1, 8), (257, 2, 9), (300, 64, 17), (16383, 64, 2),
                                   (16384, 64, 3), (65536, 64, 2)])
def test_gram_schmidt_edges(n, S, k, dtype):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"gram-schmidt n={n} S={S} k={k} {dtype}")
    rng = np.random.default_rng(n + S + k)
    dt = np.complex128 if dtype == "c128" else np.complex64
    tol = 1e-12 if dtype == "c128" else 1e-6
    V = np.zeros((k + 1, n, S), dtype=dt)
    for r in range(S):
        q, _ = np.linalg.qr(_rc(rng, n, k))
        V[:k, :, r] = q.T
    w = _rc(rng, n, S).astype(dt)
    Vd, wd = torch.from_numpy(V).cuda(), torch.from_numpy(w).cuda()
    h = P.shk_orthogonalize(n, k, Vd, wd, S)
    v = Vd[k].cpu().numpy()
    for r in range(S):
        Q = V[:k, :, r].astype(np.complex128)
        x = w[:, r].astype(np.complex128)
        a = Q.conj() @ x
        x = x - Q.T @ a
        b = Q.conj() @ x
        x = x - Q.T @ b
        nx = np.linalg.norm(x)
        scale = np.linalg.norm(w[:, r])
        assert np.abs(h[r, :k] - (a + b)).max() <= tol * scale
        assert abs(h[r, k] - nx) <= tol * scale
        if nx > 1e-3 * scale:
            assert np.abs(v[:, r] - x / nx).max() <= tol * scale / nx


@pytest.mark.parametrize("shape", [(1, 1), (3, 65), (16, 64), (17, 63), (33, 257), (2, 300), (1, 1, 1), (4, 3, 65),
                                   (5, 17, 64), (9, 16, 63), (3, 33, 130)])
@pytest.mark.parametrize("nf", [1, 4, 5])
def test_true_residual_edges(shape, nf):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"residual {shape} nf={nf}")
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=94, idx=nf)
    op = OProblem.fv(K)
    gp = P.Problem.fv2d(K) if len(shape) == 2 else P.Problem.fv3d(K)
    rng = np.random.default_rng(7)
    sig = 1j * rng.uniform(0.01, 1.0, nf)
    X = _rc(rng, nf, op.n) * 1e4
    b = _rc(rng, op.n)
    rel = P.shk_true_residual(gp, sig, torch.from_numpy(b).cuda(), torch.from_numpy(X).cuda())
    for j in range(nf):
        want = np.linalg.norm(b - op.apply(sig[j], X[j])) / np.linalg.norm(b)
        assert abs(rel[j] - want) <= 1e-12 * want


@pytest.mark.parametrize("n,k,nf", [(1, 1, 1), (15, 3, 16), (16, 4, 17), (17, 5, 63), (33, 9, 64), (100, 2, 65),
                                    (49, 25, 200)])
@pytest.mark.parametrize("acc", [False, True])
def test_assemble_edges(n, k, nf, acc):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"assemble n={n} k={k} nf={nf} acc={acc}")
    rng = np.random.default_rng(n)
    Z, Y, X0 = _rc(rng, k, n), _rc(rng, nf, k), _rc(rng, nf, n)
    X = torch.from_numpy(X0.copy()).cuda()
    P.shk_assemble(n, k, nf, torch.from_numpy(Z).cuda(), torch.from_numpy(Y).cuda(), X, accumulate=acc)
    want = Y @ Z + (X0 if acc else 0)
    assert np.abs(X.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("shape", [(1, 1), (5, 7), (3, 257), (3, 4, 5)])
@pytest.mark.parametrize("ns,nr", [(1, 1), (4, 2), (5, 3)])
def test_sensitivity_edges(shape, ns, nr):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"sensitivity {shape} {ns}x{nr}")
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=95, idx=ns)
    gp = P.Problem.fv2d(K) if len(shape) == 2 else P.Problem.fv3d(K)
    rng = np.random.default_rng(ns + nr)
    nf, n = 2, K.size
    phi, psi = _rc(rng, ns, nf, *shape), _rc(rng, nr, nf, *shape)
    want = np.zeros((nf, ns, nr) + shape, dtype=np.complex128)
    for j in range(nf):
        for s in range(ns):
            for r in range(nr):
                f, g, o = phi[s, j], psi[r, j], want[j, s, r]
                for ax in range(len(shape)):
                    m = shape[ax]
                    at = lambda a, i: np.take(a, [i], ax)
                    for i in range(m - 1):
                        ka, kb = at(K, i), at(K, i + 1)
                        T = 2 * ka * kb / (ka + kb)
                        e = T * (at(f, i + 1) - at(f, i)) * (at(g, i + 1) - at(g, i))
                        sl = [slice(None)] * len(shape)
                        sl[ax] = slice(i, i + 1)
                        o[tuple(sl)] -= e * kb / (ka + kb)
                        sl[ax] = slice(i + 1, i + 2)
                        o[tuple(sl)] -= e * ka / (ka + kb)
                    for i in (0, m - 1):
                        sl = [slice(None)] * len(shape)
                        sl[ax] = slice(i, i + 1)
                        o[tuple(sl)] -= at(K, i) * at(f, i) * at(g, i)
    for dt, tol in ((torch.complex128, 1e-12), (torch.complex64, 1e-6)):
        J = torch.empty(nf * ns * nr * n, dtype=dt, device="cuda")
        P.shk_sensitivity(gp, torch.from_numpy(phi).cuda(), torch.from_numpy(psi).cuda(), J, nf, ns, nr)
        got = J.cpu().numpy().reshape(want.shape)
        assert np.abs(got - want).max() <= tol * np.abs(want).max()
