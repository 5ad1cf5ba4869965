"""Far field and directivity on both sides of the rule between the fused
pattern kernel and the projection by single bins: few columns of many bins, and
many columns of few bins."""
import numpy as np
import pytest

import workload as W
from oracle import far_field as FF

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Lu,Lv,nrhs", [
    # at most 128 columns from 384 bins on (64 at 1024 for the directivity), one right-hand side more beyond
    (128, 384, 1), (64, 384, 3), (32, 512, 4), (32, 512, 5), (64, 768, 2), (64, 768, 3), (16, 1024, 4), (16, 1024, 5), (16, 1024, 9),
    # the far field from 192 bins on, and at 96
    (64, 192, 2), (64, 192, 3), (128, 256, 1), (32, 96, 4), (32, 96, 5), (32, 128, 4),
    # from 20 or 40 times the patches' count of columns on, up to 32 bins
    (128, 8, 1), (128, 8, 2), (256, 16, 1), (64, 24, 3), (64, 24, 4), (128, 32, 2), (128, 48, 2), (512, 2, 1)])
def test_either_side(Lu, Lv, nrhs):
    import paper_1911_04576_amd as E
    print(f"{Lu} x {Lv} bins, {nrhs} right-hand sides", flush=True)
    rng = np.random.default_rng(Lu + Lv)
    P, nx, ny = 5, 3, min(Lv, 2)
    g = W.box_geometry(24)
    keep = rng.permutation(24)[:P]
    rho, area = g.rho[keep] + rng.uniform(-0.02, 0.02, (P, 3)), g.area[keep]
    tan = np.ascontiguousarray(np.linalg.qr(rng.standard_normal((P, 3, 3)))[0][:, :2])
    x = W.random_vectors(nrhs, nx, ny, 4 * P, seed=Lv)
    geom = E.Geometry(rho, area, tan, W.PITCH, W.K0)
    xd = torch.from_numpy(x).cuda()
    D = torch.empty((nrhs, 2, Lv, Lu), dtype=torch.float64, device="cuda")
    power = E.emsurf_directivity(geom, nx, ny, nrhs, Lu, Lv, xd, D)
    F = torch.empty((nrhs, Lv, Lu, 2), dtype=torch.complex128, device="cuda")
    E.emsurf_far_field(geom, nx, ny, nrhs, Lu, Lv, xd, F)
    Dr, pr = FF.directivity(rho, area, tan, W.PITCH, W.K0, x, Lu, Lv)
    u, v = FF.fft_bin_directions(Lu, Lv, W.PITCH, W.K0)
    vis = u * u + v * v < 1.0
    Fr = FF.far_field(rho, area, tan, W.PITCH, W.K0, x, u[vis], v[vis])
    got = F.cpu().numpy()
    assert not np.any(got[:, ~vis]) and not np.any(D.cpu().numpy()[:, :, ~vis])
    rel = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)
    e = rel(D.cpu().numpy(), Dr), rel(power, pr), rel(got[:, vis], Fr)
    print(f"  directivity, power, field: {e}", flush=True)
    assert max(e) <= 1e-12
