"""Far field and directivity at every bin count (the y transform runs in LDS,
one workgroup per x bin), patch counts that leave the last group of patches
ragged, and patches in an order whose y and z change from one to the next;
against the oracle at 1e-12."""
import numpy as np
import pytest

import workload as W
from oracle import far_field as FF

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("Lv", [2, 4, 8, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024])
def test_every_bin_count(Lv):
    import paper_1911_04576_amd as E
    rng = np.random.default_rng(Lv)
    P = 24 if Lv % 3 else 19
    g = W.box_geometry(24)
    keep = rng.permutation(24)[:P]
    rho = g.rho[keep] + rng.uniform(-0.02, 0.02, (P, 3)) * (rng.random((P, 1)) < 0.5)
    # tilted tangents
    q = np.linalg.qr(rng.standard_normal((P, 3, 3)))[0]
    area, tan = g.area[keep], np.ascontiguousarray(q[:, :2])
    nx, ny, nrhs, Lu = 3, min(Lv, 5), 2, 16
    print(f"Lv {Lv} patches {P}", flush=True)
    x = W.random_vectors(nrhs, nx, ny, 4 * P, seed=Lv)
    geom = E.Geometry(rho, area, tan, W.PITCH, W.K0)
    xd = torch.from_numpy(x).cuda()
    D = torch.empty((nrhs, 2, Lv, Lu), dtype=torch.float64, device="cuda")
    power = E.emsurf_directivity(geom, nx, ny, nrhs, Lu, Lv, xd, D)
    Dr, pr = FF.directivity(rho, area, tan, W.PITCH, W.K0, x, Lu, Lv)
    e = rel(D.cpu().numpy(), Dr), rel(power, pr)
    F = torch.empty((nrhs, Lv, Lu, 2), dtype=torch.complex128, device="cuda")
    E.emsurf_far_field(geom, nx, ny, nrhs, Lu, Lv, xd, F)
    u, v = FF.fft_bin_directions(Lu, Lv, W.PITCH, W.K0)
    vis = u * u + v * v < 1.0
    Fr = np.zeros((nrhs, Lv, Lu, 2), complex)
    Fr[:, vis] = FF.far_field(rho, area, tan, W.PITCH, W.K0, x, u[vis], v[vis])
    e += (rel(F.cpu().numpy(), Fr),)
    print(f"  directivity, power, field: {e}", flush=True)
    assert max(e) <= 1e-12
