"""Rounding of the mixed transform lengths: an FP32 apply of the identity
operator is four transforms and nothing else."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# mixed lengths and the next power of two or three times one, which a longer axis pads to
PAIRS = ((20, 24), (36, 48), (40, 48), (60, 64), (72, 96), (80, 96), (100, 128), (120, 128), (144, 192), (160, 192),
         (180, 192), (200, 256), (225, 256), (240, 256), (288, 384))
N, NY, RHS = 16, 4, 4


def error(nx, x, axis, length):
    """Relative error of T x = x for x[rhs][point][other][u] on the first points of an axis of nx elements."""
    import paper_1911_04576_amd as E
    full = torch.zeros((RHS, nx, NY, N), dtype=torch.complex64, device="cuda")
    full[:, :x.shape[1]] = x
    shape = (NY, nx) if axis == 0 else (nx, NY)
    T = torch.zeros((2 * shape[0] - 1, 2 * shape[1] - 1, N, N), dtype=torch.complex128, device="cuda")
    T[shape[0] - 1, shape[1] - 1] = torch.eye(N, dtype=torch.complex128, device="cuda")
    p = E.emsurf_plan_create(shape[1], shape[0], N, 1, RHS, T, np.zeros((1, N, N), complex),
                             np.zeros(shape, np.int32), store=E.EMSURF_STORE_FP32)
    s = E.emsurf_plan_query(p)
    assert (s.Lx if axis == 0 else s.Ly) == length
    v = full.transpose(1, 2).contiguous() if axis == 0 else full
    y = torch.empty_like(v)
    E.emsurf_apply_T(p, E.EMSURF_FP32, RHS, v, y)
    y = (y.transpose(1, 2) if axis == 0 else y)[:, :x.shape[1]].to(torch.complex128)
    p.destroy()
    x = x.to(torch.complex128)
    return (torch.linalg.norm(y - x) / torch.linalg.norm(x)).item()


@pytest.mark.parametrize("axis", (0, 1))
def test_mixed_lengths_round_no_worse_than_the_longer_ones(axis):
    """A shorter transform has no more roundings than the longer one it stands for, so over the lengths its error
    is no larger; 5% for the radices' different operations."""
    ratios = []
    for short, long in PAIRS:
        g = torch.Generator(device="cuda").manual_seed(short)
        x = torch.randn((RHS, (short + 1) // 2, NY, N), dtype=torch.complex64, device="cuda", generator=g)
        a, b = error((short + 1) // 2, x, axis, short), error(long // 2, x, axis, long)
        print(f"axis {axis} {short} points {a:.3e}, {long} points {b:.3e}", flush=True)
        ratios.append(a / b)
    assert np.exp(np.mean(np.log(ratios))) <= 1.05
