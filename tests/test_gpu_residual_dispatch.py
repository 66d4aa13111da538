"""True residuals of one lane on both sides of the rule that picks the kernel:
entries of X (3, 4 and 16 Mi), the part of the marching kernel's lanes and shifts
in use, thin grids and few shifts, the last round of blocks in 3-D, against the oracle's
operator.

Tolerance: FP64 sums of at most 400,000 terms without cancellation, off by at most
about 650 roundings of 1.1e-16: 1e-12 relative."""
import numpy as np
import pytest

import synth
from oracle import Problem as OProblem
from tests.gpu_util import require_gpu, announce

pytestmark = pytest.mark.gpu

CASES = [((129, 250), 97), ((129, 250), 98), ((129, 250), 128), ((129, 250), 131), ((129, 250), 133),     # 3 Mi is 97.5 shifts, 4 Mi 130.1
         ((655, 97), 64), ((655, 97), 68), ((655, 97), 133), ((655, 97), 141),   # 0.38 of the lanes in use, 4 Mi is 66.02
         ((1400, 600), 5), ((1400, 600), 8),                          # 0.49 and 0.78 in use, over 4 Mi
         ((65536, 1), 70), ((30000, 3), 50), ((400000, 2), 6),        # thin
         ((5, 17, 70), 2825), ((4, 16, 64), 4095), ((4, 16, 64), 4097), ((17, 33, 63), 476), ((3, 50, 130), 900),
         # 12 blocks for every four shifts: under 4 Mi, over it, 768 blocks, 780, 1020, 1032
         ((7, 33, 125), 145), ((7, 33, 125), 146), ((7, 33, 125), 256), ((7, 33, 125), 257), ((7, 33, 125), 340), ((7, 33, 125), 344),
         ((4, 16, 64), 1023), ((4, 16, 64), 1024), ((4, 16, 64), 3072), ((4, 16, 64), 3073)]


@pytest.mark.parametrize("shape,nf", CASES)
def test_residuals_either_way(shape, nf):
    torch = require_gpu()
    import paper_1212_3660_amd as P
    announce(f"residual dispatch {shape} nf={nf}")
    K = synth.cell_conductivity(shape, -11.5, 1.0, 5, cfg=98, idx=nf)
    op = OProblem.fv(K)
    gp = P.Problem.fv2d(K) if len(shape) == 2 else P.Problem.fv3d(K)
    rng = np.random.default_rng(nf)
    sig = 1j * rng.uniform(0.01, 1.0, nf)
    X = rng.standard_normal((nf, op.n, 2)).view(np.complex128)[..., 0] * 1e4
    b = rng.standard_normal(op.n) + 1j * rng.standard_normal(op.n)
    rel = P.shk_true_residual(gp, sig, torch.from_numpy(b).cuda(), torch.from_numpy(X).cuda())
    bn = np.linalg.norm(b)
    for j0 in range(0, nf, 256):
        s = sig[j0:j0 + 256]
        Y = b[:, None] - op.K @ X[j0:j0 + 256].T - (s * op.Mdiag[:, None]) * X[j0:j0 + 256].T
        want = np.linalg.norm(Y, axis=0) / bn
        assert np.all(np.abs(rel[j0:j0 + 256] - want) <= 1e-12 * want)
