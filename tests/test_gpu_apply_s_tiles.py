"""The macromodel apply at the edges of its tiles: row blocks of 32 and 48,
k-tiles of 16, column blocks of 32, groups of 32 .. 256 elements with counts
just past them, odd n_eq (no 16-byte columns), few items and many, alone and
fused into x - S t, against the product in double precision (1e-12 in FP64;
2e-5 in FP32, as for the other applies)."""
import numpy as np
import pytest

import workload as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("nx,ny,n,counts,nrhs", [
    (1, 1, 1, (1,), 1), (1, 1, 33, (1,), 1), (7, 5, 15, (33, 2), 3), (8, 8, 16, (32, 31, 1), 1),
    (8, 8, 17, (64,), 5), (12, 12, 48, (129, 15), 2), (20, 20, 49, (257, 128, 15), 4), (20, 20, 96, (100,) * 4, 6),
    (24, 20, 150, (300, 179, 1), 2), (9, 9, 289, (80, 1), 2), (64, 64, 33, (4000, 96), 16), (64, 64, 64, (2048, 2048), 17)])
def test_tiles_groups_and_edges(nx, ny, n, counts, nrhs):
    import paper_1911_04576_amd as E
    T = len(counts)
    rng = np.random.default_rng(n)
    tm = rng.permutation(np.repeat(np.arange(T), counts)).reshape(ny, nx).astype(np.int32)
    S = W.random_types(T, n, seed=n)
    B = np.zeros((2 * ny - 1, 2 * nx - 1, n, n), complex)
    B[ny - 1, nx - 1] = np.eye(n)   # T x = x: A x = x - S x
    plan = E.emsurf_plan_create(nx, ny, n, T, nrhs, B, S, tm)
    x = W.random_vectors(nrhs, nx, ny, n, seed=11)
    sx = np.empty_like(x)
    for t in range(T):
        sx[:, tm == t] = x[:, tm == t] @ S[t].T
    for prec, dt, tol in ((E.EMSURF_FP64, np.complex128, 1e-12), (E.EMSURF_FP32, np.complex64, 2e-5)):
        xd = dev(x.astype(dt))
        y = torch.empty_like(xd)
        E.emsurf_apply_S(plan, prec, nrhs, xd, y)
        assert np.linalg.norm(y.cpu().numpy() - sx) <= tol * np.linalg.norm(sx)
        E.emsurf_apply_A(plan, prec, nrhs, xd, y)
        assert np.linalg.norm(y.cpu().numpy() - (x - sx)) <= tol * (np.linalg.norm(x) + np.linalg.norm(sx))
        one = torch.empty_like(xd[:1])
        E.emsurf_apply_A(plan, prec, 1, xd[-1:], one)
        if dt is np.complex128:
            assert torch.equal(one[0], y[-1])
    plan.destroy()
