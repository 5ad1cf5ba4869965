"""Device memory that the library keeps between calls, by the card's free bytes."""
import gc

import numpy as np
import pytest

import workload as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
MB = 1 << 20


def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def box(E, P=24):
    g = W.box_geometry(24)
    return E.Geometry(g.rho[:P], g.area[:P], g.tan[:P], W.PITCH, W.K0)


def nothing_kept(E):
    """The process's last plan gives everything back."""
    gc.collect()
    S, tm = np.zeros((1, 96, 96), complex), np.zeros((1, 1), np.int32)
    E.emsurf_plan_create_green(1, 1, 1, 1, box(E), S, tm, store=E.EMSURF_STORE_FP64).destroy()


class Macromodels:
    """Calls whose workspace is half a MB per cell type."""

    def __init__(self, E, types, n=64, m=64):
        self.E, self.args = E, (types, n, m)
        self.z = torch.eye(n + m, dtype=torch.complex128, device="cuda").repeat(types, 1, 1)
        self.out = torch.empty((types, n, n), dtype=torch.complex128, device="cuda")

    def __call__(self):
        self.E.emsurf_macromodels(*self.args, self.z, None, self.out)
        return free()


class Pattern:
    """Calls whose workspace is nrhs ny Lu / 1024 MB and a little more."""

    def __init__(self, E, nrhs, ny=16, Lu=64, P=16):
        self.E, self.args = E, (box(E, P), 4, ny, nrhs, Lu, 64)
        self.x = torch.ones((nrhs, ny, 4, 4 * P), dtype=torch.complex128, device="cuda")
        self.D = torch.empty((nrhs, 2, 64, Lu), dtype=torch.float64, device="cuda")

    def __call__(self):
        self.E.emsurf_directivity(*self.args, self.x, self.D)
        return free()


def test_a_small_request_does_not_take_a_large_block():
    """The pattern's workspace of 70 MB takes over the macromodels' 100 MB, which its geometry's 2 KB do not hold."""
    import paper_1911_04576_amd as E
    nothing_kept(E)
    macromodels, pattern = Macromodels(E, 200), Pattern(E, 64)
    before = macromodels()
    assert abs(before - pattern()) < 16 * MB
    assert abs(before - pattern()) < 16 * MB


def test_a_block_beyond_the_limit_leaves_the_others():
    """A workspace of 4.6 GB cannot be kept; the macromodels' 100 MB still are."""
    import paper_1911_04576_amd as E
    nothing_kept(E)
    macromodels, pattern = Macromodels(E, 200), Pattern(E, 64, ny=64, Lu=1024, P=18)
    before = macromodels()
    assert abs(before - pattern()) < 16 * MB


def test_kept_memory_is_released_on_request():
    """Without a plan nothing else gives it back."""
    import paper_1911_04576_amd as E
    nothing_kept(E)
    macromodels, pattern = Macromodels(E, 200), Pattern(E, 64)
    macromodels()
    E.emsurf_release_idle_memory()
    before = free()                       # (what the first calls load once is loaded)
    assert before - macromodels() > 90 * MB
    pattern()
    E.emsurf_release_idle_memory()
    assert abs(before - free()) < 16 * MB
    assert before - pattern() > 60 * MB   # and the calls work on


def test_a_server_keeps_within_its_budget():
    """Building the surface's plan takes 470 MB of workspace, which a budget of its own bytes does not leave."""
    import paper_1911_04576_amd as E
    nothing_kept(E)
    S, tm = W.random_types(2, 96, seed=1), W.random_type_map(20, 20, 2, seed=1)
    b = W.random_vectors(2, 20, 20, 96, seed=2)
    probe = E.emsurf_server_create(1 << 40, 4, E.solve_opts(E.EMSURF_FP32_IR, tol=1e-6))
    budget = (E.emsurf_server_entry_bytes(probe, 20, 20, 96, 2) + 4 * E.emsurf_server_slot_bytes(probe, 20, 20, 96, 2)
              + 32 * MB)
    probe.destroy()
    Pattern(E, 1)()
    E.emsurf_release_idle_memory()
    before = free()
    srv = E.emsurf_server_create(budget, 4, E.solve_opts(E.EMSURF_FP32_IR, tol=1e-6))
    E.emsurf_server_submit(srv, 1, 20, 20, 2, box(E), S, tm, b, recip=0)
    while (done := E.emsurf_server_next_completed(srv)) is None:
        E.emsurf_server_step(srv)
    x, infos, _ = E.emsurf_server_fetch(srv, *done)
    used = before - free()
    print(f"budget {budget // MB} MB, {used // MB} MB in use", flush=True)
    assert all(i["converged"] for i in infos) and used <= budget + 64 * MB
    srv.destroy()
