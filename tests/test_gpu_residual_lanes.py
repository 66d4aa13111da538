"""True residuals of several lanes on grids whose rows, segments and planes do not
fill the row-marching kernel's tiles, over its line of 4 Mi entries of X: as a
solve reports them and as its refinement uses them.

Tolerance: ||x|| <= ||b|| / (omega Ss) = 1.6e7 ||b|| for the longest period and
||K|| <= 12 exp(-11.5 + 3) = 2.4e-3, so an entry of b - (K + sigma M) x is a sum of
terms of 4e4 ||b|| at the very most; some ten roundings of 1.1e-16 leave a relative
residual right to 5e-11, whatever its own size."""
import numpy as np
import pytest

import synth
from oracle import Problem as OProblem
from tests.gpu_util import require_gpu, announce

pytestmark = pytest.mark.gpu

# (shape, shifts, right-hand sides): 2-D two segments and a bit, 3-D planes and rows
# with remainders; 3 lanes (4 of them), 5 (8) and 16, shifts not a multiple of eight
CASES = [((129, 250), 45, 3), ((141, 250), 25, 5), ((17, 33, 63), 27, 5), ((33, 250), 33, 16), ((9, 49, 62), 10, 16)]


def _case(shape, nf, nr):
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=97, idx=nf)
    assert K.size * nf * nr >= 4 << 20
    sig = synth.shifts_from_periods(synth.periods(nf, 10.0, 1000.0))
    rng = np.random.default_rng(nf)
    b = (rng.standard_normal((nr, K.size)) + 1j * rng.standard_normal((nr, K.size)))
    return K, OProblem.fv(K), sig, b


def _true(op, sig, b, X):
    return np.array([[np.linalg.norm(b[r] - op.apply(sig[j], X[r, j])) / np.linalg.norm(b[r])
                      for j in range(len(sig))] for r in range(b.shape[0])])


@pytest.mark.parametrize("shape,nf,nr", CASES)
def test_reported_residuals_of_ragged_grids(shape, nf, nr):
    """A basis of three columns: far from converged, so the residuals are large."""
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"reported residuals {shape} nf={nf} nr={nr}")
    K, op, sig, b = _case(shape, nf, nr)
    gp = P.Problem.fv2d(K) if len(shape) == 2 else P.Problem.fv3d(K)
    prm, keep = P.make_params(sig[[nf // 2]], m_restart=3, max_restarts=0, max_refine=0, tol=1e-12, eps_inner=1e-4,
                              inner_precond=P.SHK_PRECOND_MULTIGRID)
    x, st = P.fgmres_sh_solve(gp, prm, sig, torch.from_numpy(b).cuda())
    got, want = st["true_relres"], _true(op, sig, b, x.cpu().numpy())
    assert want.max() > 1e-3
    assert np.all(np.abs(got - want) <= 5e-11)


@pytest.mark.parametrize("shape,nf,nr,tol", [CASES[1] + (1e-6,), CASES[2] + (1e-7,)])
def test_refinement_on_ragged_grids(shape, nf, nr, tol):
    """A first pass in complex64 that misses its target: the sweeps project every
    shift's residual on the worst one's (the second form of the sums).  The targets
    are ones that the complex64 basis reaches for random right-hand sides."""
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"refinement {shape} nf={nf} nr={nr}")
    K, op, sig, b = _case(shape, nf, nr)
    gp = P.Problem.fv2d(K) if len(shape) == 2 else P.Problem.fv3d(K)
    prm, keep = P.make_params(sig[[0, nf // 2, nf - 1]], m_restart=50, max_restarts=20, max_refine=4, tol=tol,
                              eps_inner=1e-6, precision=P.SHK_MIXED, inner_precond=P.SHK_PRECOND_MULTIGRID)
    x, st = P.fgmres_sh_solve(gp, prm, sig, torch.from_numpy(b).cuda())
    assert st["refine_sweeps"].min() >= 1
    got, want = st["true_relres"], _true(op, sig, b, x.cpu().numpy())
    assert np.all(st["status"] == P.SHK_CONVERGED) and want.max() <= tol + 5e-11
    assert np.all(np.abs(got - want) <= 5e-11)
