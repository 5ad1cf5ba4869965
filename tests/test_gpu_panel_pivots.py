"""Macromodels of interiors without a dominant diagonal: every column of the
register panels exchanges rows.  Sizes at the edges of the panels (8-column
sub-blocks, 32-column panels, 512 and 1024 rows)."""
import numpy as np
import pytest

from oracle import macromodel_gen as MG

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def run(Z, n, Zself):
    import paper_1911_04576_amd as E
    T, N, _ = Z.shape
    out = torch.empty((2, T, n, n), dtype=torch.complex128, device="cuda")
    E.emsurf_macromodels(T, n, N - n, torch.from_numpy(Z).cuda(), torch.from_numpy(Zself).cuda(), out[0], out[1])
    torch.cuda.synchronize()
    return out[0].cpu().numpy(), out[1].cpu().numpy()


@pytest.mark.parametrize("T,n,m", [(3, 1, 2), (2, 5, 8), (2, 9, 17), (3, 30, 41), (2, 65, 63), (1, 40, 472), (1, 41, 472),
                                   (2, 256, 3), (1, 257, 40), (1, 24, 1000), (1, 25, 1000)])
def test_random_interiors(T, n, m):
    print(f"{T} x ({n} + {m})", flush=True)
    rng = np.random.default_rng(1000 * n + m)
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    Z = cn(T, n + m, n + m)
    Z[:, n:] *= 4.0 ** rng.integers(-6, 7, size=(T, m, 1))      # rows of very different size
    Zself = cn(n, n)
    S, Zt = run(Z, n, Zself)
    Zt_ref, S_ref = MG.macromodels(Z, n, Zself)
    N, eps = n + m, np.finfo(float).eps
    for t in range(T):
        # forward error of an elimination with partial pivoting: N eps times
        # the condition of the equilibrated interior (rows scale freely)
        r = Z[t, n:, n:] / np.linalg.norm(Z[t, n:, n:], axis=1)[:, None]
        size = np.linalg.norm(Z[t, :n, n:]) * np.linalg.norm(np.linalg.solve(Z[t, n:, n:], Z[t, n:, :n]))
        bz = N * eps * np.linalg.cond(r) * (size + np.linalg.norm(Z[t, :n, :n]))
        ez = np.linalg.norm(Zt[t] - Zt_ref[t])
        A = Zt_ref[t] + Zself
        bs = np.linalg.cond(A) * (bz / np.linalg.norm(A, 2) + N * eps) * np.linalg.norm(S_ref[t])
        es = np.linalg.norm(S[t] - S_ref[t])
        print(f"  type {t}: Z~ {ez:.1e} of {bz:.1e}, S {es:.1e} of {bs:.1e}", flush=True)
        assert ez <= bz and es <= bs


@pytest.mark.parametrize("m", [7, 33, 64, 130, 600])
def test_permutation_interior_is_exact(m):
    """Every pivot column has one non-zero entry: the elimination only moves rows."""
    print(f"m {m}", flush=True)
    rng = np.random.default_rng(m)
    n = 20
    Z = np.zeros((1, n + m, n + m), complex)
    perm = rng.permutation(m)
    Z[0, n + np.arange(m), n + perm] = 1.0
    Z[0, :n, n:] = rng.integers(-8, 9, (n, m))
    Z[0, n:, :n] = rng.integers(-8, 9, (m, n))
    Z[0, :n, :n] = rng.integers(-8, 9, (n, n)) + 1000 * np.eye(n)
    S, Zt = run(Z, n, np.zeros((n, n), complex))
    want = Z[0, :n, :n] - Z[0, :n, n:] @ (Z[0, n:, n:].T @ Z[0, n:, :n])
    assert np.array_equal(Zt[0], want)
