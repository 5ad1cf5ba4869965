"""A directivity call that is refused (a right-hand side radiates no power)
leaves the caller's array alone; the powers of many right-hand sides."""
import numpy as np
import pytest

import workload as W
from oracle import far_field as FF

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def inputs(nrhs, nx=3, ny=4):
    import paper_1911_04576_amd as E
    g = W.box_geometry(24)
    return g, E.Geometry(g.rho, g.area, g.tan, W.PITCH, W.K0), W.random_vectors(nrhs, nx, ny, 96, seed=nrhs)


@pytest.mark.parametrize("nrhs", [1, 3, 6])
@pytest.mark.parametrize("bad", [0.0, np.nan, np.inf])
def test_refused_call_leaves_the_array(nrhs, bad):
    import paper_1911_04576_amd as E
    g, geom, x = inputs(nrhs)
    x[nrhs // 2] = bad
    D = torch.full((nrhs, 2, 16, 24), 7.0, dtype=torch.float64, device="cuda")
    with pytest.raises(E.EmsurfError, match="radiate no power"):
        E.emsurf_directivity(geom, 3, 4, nrhs, 24, 16, torch.from_numpy(x).cuda(), D)
    assert bool((D == 7.0).all())


@pytest.mark.parametrize("nrhs", [4, 5, 64])
def test_powers_of_many_right_hand_sides(nrhs):
    import paper_1911_04576_amd as E
    g, geom, x = inputs(nrhs)
    D = torch.empty((nrhs, 2, 16, 24), dtype=torch.float64, device="cuda")
    power = E.emsurf_directivity(geom, 3, 4, nrhs, 24, 16, torch.from_numpy(x).cuda(), D)
    Dr, pr = FF.directivity(g.rho, g.area, g.tan, W.PITCH, W.K0, x, 24, 16)
    assert np.linalg.norm(D.cpu().numpy() - Dr) <= 1e-12 * np.linalg.norm(Dr)
    assert np.max(np.abs(power - pr) / pr) <= 1e-12
