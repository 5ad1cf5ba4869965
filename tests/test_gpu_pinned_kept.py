"""Pinned memory of a server's requests, by the process's mappings of the card."""
import numpy as np
import pytest

import workload as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
MB = 1 << 20


def mapped():
    total = 0
    for line in open("/proc/self/maps"):
        if "renderD" in line:
            lo, hi = line.split()[0].split("-")
            total += int(hi, 16) - int(lo, 16)
    return total


def test_a_request_that_cannot_be_pinned_leaves_the_idle_blocks():
    """1.1 GB of right-hand sides take pageable memory; the 38 MB of an earlier request stay for the next."""
    import paper_1911_04576_amd as E
    g = W.box_geometry(24)
    geom = E.Geometry(g.rho, g.area, g.tan, W.PITCH, W.K0)
    S = W.random_types(2, 96, seed=1)
    srv = E.emsurf_server_create(64 << 30, 64, E.solve_opts(E.EMSURF_FP32_IR, tol=1e-6, restart=8))

    def submit(key, n, b):
        E.emsurf_server_submit(srv, key, n, n, 2, geom, S, W.random_type_map(n, n, 2, seed=1), b, recip=1)

    b = W.random_vectors(64, 20, 20, 96, seed=2)
    submit(1, 20, b)
    while (done := E.emsurf_server_next_completed(srv)) is None:
        E.emsurf_server_step(srv)
    E.emsurf_server_fetch(srv, *done)
    before = mapped()
    submit(2, 106, np.zeros((64, 106, 106, 96), np.complex128))
    kept = mapped() - before
    print(f"mapped {before // MB} MB, then {kept / MB:+.1f} MB", flush=True)
    assert before > b.nbytes and abs(kept) < 8 * MB
    # (and a small request takes none of them)
    submit(1, 20, b[:1])
    small = mapped() - before - kept
    assert 0 <= small < 8 * MB
    srv.destroy()
