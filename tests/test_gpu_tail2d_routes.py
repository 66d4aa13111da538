"""Where the 2-D V-cycle's register tail starts: one level below the finest
because the LDS tail is given too little room to start there first, and with its
32 x 32 form alone (tail2d = 32).  complex128: iterates of the oracle;
complex64: the bits of the LDS tail (tail2d = 0) in the same setting."""
import numpy as np
import pytest

import synth
from oracle import Problem as OProblem
from oracle.mg import Hierarchy, mg_cocg
from tests.gpu_util import require_gpu, to_dev, announce

pytestmark = pytest.mark.gpu

CASES = [((33, 17), 1, {"tail_lds": 16384}), ((17, 33), 2, {"tail_lds": 16384}), ((33, 40), 1, {"tail_lds": 4096}),
         ((64, 64), 1, {"tail2d": 32}), ((64, 64), 8, {"tail2d": 32}), ((67, 130), 4, {"tail2d": 32}),
         ((129, 33), 16, {"tail2d": 32}), ((40, 128), 64, {"tail2d": 32})]


@pytest.mark.parametrize("shape,S,knobs", CASES)
def test_where_the_register_tail_starts(shape, S, knobs):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    from paper_1212_3660_amd import autotune
    announce(f"register tail {shape} S={S} {knobs}")
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=92, idx=shape[0])
    op = OProblem.fv(K)
    gp = P.Problem.fv2d(K)
    tau = 2j * np.pi / 300.0
    rng = np.random.default_rng(4)
    V = rng.normal(size=(op.n, S)) + 1j * rng.normal(size=(op.n, S))

    def run(dtype, **more):
        try:
            for k, v in {**knobs, **more}.items():
                P.shk_tune_set(P.TUNE_ALL, k, v)
            z = torch.zeros(op.n * S, dtype=torch.complex128, device="cuda")
            P.shk_inner_solve(gp, tau, to_dev(V.ravel(), dtype), z, fixed_iters=4, n_rhs=S,
                              precond=P.SHK_PRECOND_MULTIGRID)
            return z.cpu().numpy().reshape(op.n, S)
        finally:
            P.shk_tune_reset()
            autotune.load()

    Z = run("c128")
    H = Hierarchy.of(op)
    for r in range(min(S, 3)):
        xo, _, _, _ = mg_cocg(op, tau, V[:, r], 0.0, 100, H, fixed_iters=4)
        assert np.allclose(Z[:, r], xo, rtol=0, atol=1e-9 * np.abs(xo).max()), r
    assert np.array_equal(run("c64"), run("c64", tail2d=0))
