"""Arnoldi steps of every basis size class (2, 4, 8 held vectors, more read
twice) and chunk remainder, through solves whose iterations pass all of them,
against the oracle's GMRES iterates; and the same right-hand side alone and in
sessions whose slots sit at other basis sizes."""
import numpy as np
import pytest

import workload as W
from oracle import krylov as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# N = nx ny n: below a chunk of 1024 values, exactly one, ragged several, a
# breakdown at the first step (one element), more than 512 chunks
@pytest.mark.parametrize("nx,ny,n,nrhs", [(3, 2, 7, 2), (8, 8, 16, 1), (9, 7, 33, 3), (1, 1, 40, 5), (91, 61, 96, 1)])
@pytest.mark.parametrize("restart", [14, 3])
def test_iterates_match_the_oracle(nx, ny, n, nrhs, restart):
    import paper_1911_04576_amd as E
    steps = 14
    S, tm = W.random_types(2, n, seed=32), W.random_type_map(nx, ny, 2, seed=33)
    b = W.random_vectors(nrhs, nx, ny, n, seed=34)
    print(f"{nx}x{ny} n {n} rhs {nrhs} restart {restart}", flush=True)
    if n == 96:
        g = W.box_geometry(24)
        plan = E.emsurf_plan_create_green(nx, ny, 2, nrhs, E.Geometry(g.rho, g.area, g.tan, W.PITCH, W.K0), S, tm,
                                          store=1)
    else:   # strong coupling: many steps
        plan = E.emsurf_plan_create(nx, ny, n, 2, nrhs, 4.0 * W.random_blocks(nx, ny, n, seed=31), S, tm, store=1)
    x = torch.zeros(b.shape, dtype=torch.complex128, device="cuda")
    E.emsurf_solve(plan, E.solve_opts(E.EMSURF_FP64, tol=1e-30, restart=restart, max_iter=steps), nrhs, dev(b), x)

    def A(v):
        y, vd = torch.empty((1, ny, nx, n), dtype=torch.complex128, device="cuda"), dev(v.reshape(1, ny, nx, n))
        E.emsurf_apply_A(plan, E.EMSURF_FP64, 1, vd, y)
        torch.cuda.synchronize()
        return y.cpu().numpy().ravel()

    for r in range(nrhs):
        xr, _ = K.gmres(A, b[r], 1e-30, restart=restart, max_iter=steps)
        err = np.linalg.norm(x[r].cpu().numpy().ravel() - xr) / np.linalg.norm(xr)
        print(f"  rhs {r} err {err:.2e}", flush=True)
        # the same iterate: rounding (1e-15) times the condition of the
        # least-squares problem, below 1e3 here
        assert err <= 1e-12
    plan.destroy()


def test_slots_at_different_basis_sizes():
    """Requests joining at different steps are bitwise what they are alone."""
    import paper_1911_04576_amd as E
    nx, ny, n = 7, 5, 24
    B = 4.0 * W.random_blocks(nx, ny, n, seed=41)
    S, tm = W.random_types(2, n, seed=42), W.random_type_map(nx, ny, 2, seed=43)
    plan = E.emsurf_plan_create(nx, ny, n, 2, 6, B, S, tm, store=3)
    b = dev(W.random_vectors(6, nx, ny, n, seed=44))
    opts = E.solve_opts(E.EMSURF_FP64, tol=1e-11, restart=12)

    def run(joins):
        sess = E.emsurf_session_create(plan, 6, opts)
        out, step = {}, 0
        while len(out) < len(joins):
            for r, at in joins.items():
                if at == step:
                    E.emsurf_session_submit(sess, b[r], tag=r)
            E.emsurf_session_step(sess)
            for slot, tag in E.emsurf_session_finished(sess):
                x = torch.empty((ny, nx, n), dtype=torch.complex128, device="cuda")
                E.emsurf_session_collect(sess, slot, x)
                out[tag] = x.cpu()
            step += 1
            assert step < 400
        sess.destroy()
        return out

    mix = run({0: 0, 1: 1, 2: 3, 3: 5, 4: 9, 5: 10})
    for r in range(6):
        assert torch.equal(run({r: 0})[r], mix[r])
