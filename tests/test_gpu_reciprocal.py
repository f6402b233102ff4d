"""The float64 smoothers' reciprocal of the diagonal against what a division
gives: over the binades, random diagonals, and where the diagonal or its
reciprocal leaves the normal range."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")

# (nx, ny, nz), sweeps of the finest level: legs, half-sweeps, tiles of 62
# pairs, rows of one wave
FORMS = [((16, 16, 16), "auto"), ((32, 16, 16), "half"), ((32, 16, 16), "fused"), ((128, 96, 96), "auto")]


def _fields(shape, decades, seed=11):
    nx, ny, nz = shape
    rng = np.random.default_rng(seed)
    a = np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(10.0 ** decades))
    return a, rng.standard_normal(a.shape)


def _vcycle(a, v, sweep, h):
    s = gm.GMGPoisson(torch.tensor(a, device=DEV), h=h, precision="fp64", fine_sweep=sweep)
    return s.vcycle(torch.tensor(v, device=DEV))


@pytest.mark.parametrize("shape,sweep", FORMS)
def test_powers_of_two(shape, sweep):
    """A V-cycle of (a 2^s, v 2^s) is that of (a, v) to the bit: every operation
    commutes with a power of two, the reciprocal of the diagonal among them."""
    print(f"powers {shape} {sweep}", flush=True)
    a, v = _fields(shape, 2)
    ref = _vcycle(a, v, sweep, (1.0, 1.0, 1.0))
    for s in (-900, -500, -1, 3, 500, 900):
        assert torch.equal(_vcycle(np.ldexp(a, s), np.ldexp(v, s), sweep, (1.0, 1.0, 1.0)), ref), s


@pytest.mark.parametrize("shape,sweep", FORMS)
def test_relaxed_cells_satisfy_their_equation(shape, sweep):
    """Red cells, which the last half-sweep wrote: D z = v + sum_f w_f z_nb.
    With u = 2^-53: each w is a sum and a product (2 u), D and the right side are
    sums of six of them (5 and 6 u more), the reciprocal and its product 2 u:
    at most 16 u of the sum of absolute values."""
    print(f"relaxed {shape} {sweep}", flush=True)
    a, v = _fields(shape, 12)
    h = (1.0, 0.5, 2.0)
    z = _vcycle(a, v, sweep, h).cpu().numpy()
    D, off, size = np.zeros_like(a), v.copy(), np.abs(v)
    for axis, hd in ((2, h[0]), (1, h[1]), (0, h[2])):
        lo = [slice(None)] * 3
        hi = [slice(None)] * 3
        lo[axis], hi[axis] = slice(0, -1), slice(1, None)
        lo, hi = tuple(lo), tuple(hi)
        w = 0.5 * (a[lo] + a[hi]) / hd ** 2
        for p, q in ((lo, hi), (hi, lo)):
            D[p] += w
            off[p] += w * z[q]
            size[p] += w * np.abs(z[q])
    for k in (0, -1):  # through a plate: the mirrored ghost
        D[k] += 2.0 * a[k] / h[2] ** 2
    red = np.indices(a.shape).sum(0) % 2 == 0
    err = np.abs(D * z - off)[red]
    assert (err <= 16 * 2.0 ** -53 * (size + D * np.abs(z))[red]).all()


@pytest.mark.parametrize("shape,sweep", FORMS)
def test_subnormal_reciprocal(shape, sweep):
    """Diagonals between 2^1022 and 2^1024: a reciprocal of at least 51 bits, so
    the scaled cycle keeps 1e-12 of the unscaled one."""
    print(f"subnormal {shape} {sweep}", flush=True)
    a, v = _fields(shape, 0.2)
    h = (2.0 ** -10,) * 3  # faces a 2^20
    ref = _vcycle(a, v, sweep, h)
    z = _vcycle(np.ldexp(a, 1000), np.ldexp(v, 1000), sweep, h)
    assert ((z - ref).norm() / ref.norm()).item() < 1e-12


@pytest.mark.parametrize("shape,sweep", FORMS)
def test_overflowing_diagonal(shape, sweep):
    """Faces of 2^1022, whose sum overflows: the quotient by infinity is 0 in
    every cell of the finest level (the levels below are in range)."""
    print(f"overflow {shape} {sweep}", flush=True)
    nx, ny, nz = shape
    a = np.full((nz, ny, nx), 2.0 ** 1000)
    v = np.ldexp(_fields(shape, 0)[1], 1000)
    z = _vcycle(a, v, sweep, (2.0 ** -11,) * 3)
    assert (z == 0.0).all()
