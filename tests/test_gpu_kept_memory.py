"""Call workspaces and request memory that the library keeps between calls:
results do not depend on what an earlier or concurrent call left in them."""
import threading

import numpy as np
import pytest

import workload as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def macromodels(E, seed, n_types, n, n_int, stream=None):
    Z, Zs = W.cell_interiors(n_types, n, n_int, seed)
    z, zs = torch.from_numpy(Z).cuda(), torch.from_numpy(Zs).cuda()
    torch.cuda.synchronize()
    out = torch.empty((2, n_types, n, n), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    E.emsurf_macromodels(n_types, n, n_int, z, zs, out[0], out[1], stream=stream)
    return out


def test_concurrent_macromodels_equal_serial_ones():
    import paper_1911_04576_amd as E
    shapes = [(3, 40, 70), (5, 96, 33), (2, 17, 120), (4, 64, 64)]
    want = [macromodels(E, 50 + i, *s).cpu() for i, s in enumerate(shapes)]
    print("serial done", flush=True)
    got = [None] * len(shapes)

    def work(i):
        st = torch.cuda.Stream()
        for _ in range(3):
            got[i] = macromodels(E, 50 + i, *shapes[i], stream=st)
        st.synchronize()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(shapes))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for w, g in zip(want, got):
        assert torch.equal(w, g.cpu())


def test_far_field_after_larger_and_smaller_calls():
    import paper_1911_04576_amd as E
    g = W.box_geometry(24)
    geom = E.Geometry(g.rho, g.area, g.tan, W.PITCH, W.K0)

    def pattern(nx, ny, rhs, bins, seed):
        x = torch.from_numpy(W.random_vectors(rhs, nx, ny, 96, seed=seed)).cuda()
        D = torch.empty((rhs, 2, bins, bins), dtype=torch.float64, device="cuda")
        p = E.emsurf_directivity(geom, nx, ny, rhs, bins, bins, x, D)
        return D.cpu(), p

    first = pattern(5, 4, 2, 32, 1)
    pattern(12, 9, 3, 64, 2)          # a larger block, which the next call takes over
    again = pattern(5, 4, 2, 32, 1)
    assert torch.equal(first[0], again[0]) and np.array_equal(first[1], again[1])


def test_requests_beyond_the_pinned_memory():
    """Three requests of 453 MB in the queue: the third does not fit the pinned gigabyte and takes pageable memory."""
    import paper_1911_04576_amd as E
    n, rhs, nt = 96, 32, 2
    g = W.box_geometry(24)
    geom = E.Geometry(g.rho, g.area, g.tan, W.PITCH, W.K0)
    S, tm = W.random_types(nt, 96, seed=1), W.random_type_map(n, n, nt, seed=1)
    b = np.zeros((rhs, n, n, 96), dtype=np.complex128)
    b[5] = W.random_vectors(1, n, n, 96, seed=2)[0]
    srv = E.emsurf_server_create(64 << 30, rhs, E.solve_opts(E.EMSURF_FP32_IR, tol=1e-6, restart=8))
    ids = [E.emsurf_server_submit(srv, 7, n, n, nt, geom, S, tm, b, recip=1) for _ in range(3)]
    got = {}
    for _ in range(200):
        E.emsurf_server_step(srv)
        while (c := E.emsurf_server_next_completed(srv)) is not None:
            got[c[0]] = E.emsurf_server_fetch(srv, *c)
            print("fetched", c[0], flush=True)
        if len(got) == 3:
            break
    assert sorted(got) == sorted(ids)
    x0 = got[ids[0]][0]
    assert np.linalg.norm(x0[5]) > 0 and not np.any(x0[:5]) and not np.any(x0[6:])
    for i in ids:
        x, infos, _ = got[i]
        assert all(q["converged"] for q in infos) and np.array_equal(x, x0)
    srv.destroy()
