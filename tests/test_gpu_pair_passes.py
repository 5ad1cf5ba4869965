"""Paired block products at the edges of their tiling: 1 .. 21 tiles of 16
unknowns (one to four wavefronts, equal and unequal shares), passes of 4, 8 and
16 columns in both precisions up to the sizes where 16 no longer fit, against
the FP64 oracle (1e-12 in FP64, 2e-5 in FP32, as for the other products).  A
column's bits do not depend on the pass that it shares."""
import numpy as np
import pytest

import workload as W
from oracle import coupling as C

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("n", [1, 16, 17, 33, 64, 65, 96, 97, 128, 129, 145, 177, 208, 273, 288, 289, 320, 321])
def test_passes_and_tiles(n):
    import paper_1911_04576_amd as E
    nx, ny = (3, 2) if n > 128 else (7, 5)
    B = W.random_blocks(nx, ny, n, seed=n)
    B = (B + B[::-1, ::-1].swapaxes(-1, -2)) / 2
    S, tm = W.random_types(1, n, seed=2), np.zeros((ny, nx), np.int32)
    plan = E.emsurf_plan_create(nx, ny, n, 1, 17, B, S, tm, recip=1)
    x = W.random_vectors(17, nx, ny, n, seed=11)
    yr = C.apply_T_direct(lambda dy, dx: B[dy + ny - 1, dx + nx - 1], x)
    for prec, dt, tol in ((E.EMSURF_FP64, np.complex128, 1e-12), (E.EMSURF_FP32, np.complex64, 2e-5)):
        xd = dev(x.astype(dt))
        first = None
        for nrhs in (17, 16, 9, 8, 5, 4, 1):
            y = torch.empty_like(xd[:nrhs])
            E.emsurf_apply_T(plan, prec, nrhs, xd[:nrhs], y)
            if first is None:
                first, yh = y, y.cpu().numpy()
                for r in range(nrhs):
                    assert np.linalg.norm(yh[r] - yr[r]) <= tol * np.linalg.norm(yr[r])
            assert torch.equal(y, first[:nrhs])
    plan.destroy()
