"""The 2-D V-cycle tail that keeps its cells in registers, at the sizes where
its layout changes: one cell, the 32 x 32 base grid and one past it, the
64 x 64 top level and one past it, ragged and thin grids, one and many lanes.
complex128: iterates of the oracle; complex64: the bits of the LDS tail
(tail2d = 0), whose kernels the rest of the suite checks against the oracle."""
import numpy as np
import pytest

import synth
from oracle import Problem as OProblem
from oracle.mg import Hierarchy, mg_cocg
from tests.gpu_util import require_gpu, to_dev, announce

pytestmark = pytest.mark.gpu

CASES = [((1, 1), 1), ((1, 2), 2), ((2, 2), 1), ((3, 5), 4), ((5, 9), 1), ((32, 32), 1), ((32, 33), 2), ((33, 17), 1),
         ((34, 34), 4), ((64, 64), 1), ((64, 64), 8), ((64, 7), 2), ((65, 64), 1), ((67, 130), 4), ((129, 33), 16),
         ((40, 128), 64)]


@pytest.mark.parametrize("shape,S", CASES)
def test_register_tail(shape, S):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    from paper_1212_3660_amd import autotune
    announce(f"register tail {shape} S={S}")
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=93, idx=shape[0])
    op = OProblem.fv(K)
    gp = P.Problem.fv2d(K)
    tau = 2j * np.pi / 300.0
    rng = np.random.default_rng(3)
    V = rng.normal(size=(op.n, S)) + 1j * rng.normal(size=(op.n, S))

    def run(dtype, its):
        z = torch.zeros(op.n * S, dtype=torch.complex128, device="cuda")
        P.shk_inner_solve(gp, tau, to_dev(V.ravel(), dtype), z, fixed_iters=its, n_rhs=S,
                          precond=P.SHK_PRECOND_MULTIGRID)
        return z.cpu().numpy().reshape(op.n, S)

    its = 4 if op.n > 8 else 1
    Z = run("c128", its)
    H = Hierarchy.of(op)
    for r in range(min(S, 3)):
        xo, _, _, _ = mg_cocg(op, tau, V[:, r], 0.0, 100, H, fixed_iters=its)
        assert np.allclose(Z[:, r], xo, rtol=0, atol=1e-9 * np.abs(xo).max()), r
    new = run("c64", its)
    try:
        P.shk_tune_set(P.TUNE_ALL, "tail2d", 0)
        old = run("c64", its)
    finally:
        P.shk_tune_reset()
        autotune.load()
    assert np.array_equal(new, old)
