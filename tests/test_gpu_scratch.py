"""Step-level calls share kept device scratch: repeated calls of growing and
shrinking sizes, from several threads on their own streams and across the
destruction of the last problem, give what a single call gives."""
import threading

import numpy as np
import pytest

import synth
from tests.gpu_util import require_gpu, announce

pytestmark = pytest.mark.gpu


def test_step_calls_reuse_scratch():
    torch = require_gpu()
    import paper_1212_3660_amd as P
    rng = np.random.default_rng(1)
    sizes = [(1500, 1, 3), (40, 2, 5), (9000, 4, 7), (700, 1, 2)]
    data = []
    for n, S, k in sizes:
        V = rng.standard_normal((k + 1, n, S)) + 1j * rng.standard_normal((k + 1, n, S))
        w = rng.standard_normal((n, S)) + 1j * rng.standard_normal((n, S))
        for r in range(S):
            q, _ = np.linalg.qr(V[:k, :, r].T)
            V[:k, :, r] = q.T
        K = synth.cell_conductivity((20 + k, 31), -11.5, 1.0, 5, cfg=96, idx=k)
        x = rng.standard_normal((4, K.size)) + 1j * rng.standard_normal((4, K.size))
        data.append((n, S, k, V, w, K, x))

    def work(d):
        n, S, k, V, w, K, x = d
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            Vd, wd, xd = (torch.from_numpy(a).cuda() for a in (V, w, x))
            h = P.shk_orthogonalize(n, k, Vd, wd, S)
            p = P.Problem.fv2d(K)
            rel = P.shk_true_residual(p, 1j * np.array([0.1, 0.2, 0.5, 1.0]), xd[0].contiguous(), xd)
            z = torch.zeros(K.size, dtype=torch.complex128, device="cuda")
            P.shk_inner_solve(p, 0.3j, xd[1].contiguous(), z, eps=1e-8, precond=P.SHK_PRECOND_MULTIGRID)
            st.synchronize()
            p.close()     # the last of them frees the scratch
            return h, Vd[k].cpu().numpy(), rel, z.cpu().numpy()

    announce("scratch: one call each")
    want = [work(d) for d in data]
    out, errs = {}, []

    def loop(t):
        try:
            for i in range(6):
                j = (t + i) % len(data)
                out[(t, i)] = (j, work(data[j]))
        except Exception as e:  # noqa: BLE001
            errs.append(e)

    announce("scratch: four threads")
    ts = [threading.Thread(target=loop, args=(t,)) for t in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs
    for j, got in out.values():
        for a, b in zip(got, want[j]):
            assert np.array_equal(a, b)
